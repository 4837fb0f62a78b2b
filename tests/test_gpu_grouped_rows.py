"""Grouped launches of the pipelined 256x256 tiles: a group's last tile row runs a loop of the height its rows need (a quarter,
half, three quarters or all of the tile).  Integer operands: bit for bit the once-rounded product, nothing outside C written."""
import pytest
import torch

from test_gpu_chained import BF16, E4M3, FP16, IN, SLAB, _padded

POISON = 12345.0


# rows at both sides of each height, alone and below whole tiles; slab counts around the turns of the ring; an empty group
ROWS = [1, 64, 65, 0, 128, 129, 192, 193, 255, 256, 300, 449, 321, 16]


def _check(shapes_of, dtype, bl, ragged, beta=0.0):
    """beta: C = 0.5 * A @ B + beta * C of a C of integers, else of one that holds a mark."""
    from paper_2512_04226_amd import binding as g
    gen = torch.Generator(device="cuda").manual_seed(4)
    per16, out_t = (16 if dtype == E4M3 else 8), torch.float16 if dtype == FP16 else torch.bfloat16
    shapes, dev, refs, olds = [], [], [], []
    for m, n, k in shapes_of:
        shapes.append((m, n, k))
        if m == 0:
            dev.append((None, None, None))
            refs.append(None)
            olds.append(None)
            continue
        A, B = (torch.randint(-3, 4, s, device="cuda", generator=gen).float() for s in ((m, k), (k, n)))
        old = torch.randint(-4, 5, (m, n), device="cuda", generator=gen).double() if beta else None
        refs.append((0.5 * (A.double() @ B.double()) + beta * old if beta else A.double() @ B.double()).to(out_t))
        A, B = (_padded(x, per16).to(IN[dtype]) for x in (A, B.t().contiguous() if bl else B))
        C = torch.full((m + 1, -(-n // 8) * 8 + 8), POISON, dtype=out_t, device="cuda")
        dev.append((A[:, :k], B[:, :k] if bl else B[:, :n], C[:m, :n]))
        olds.append(old)
    mark = torch.full((1,), POISON, dtype=out_t).item()
    probs = g.make_problems(shapes, bl, dev)
    for p, (A, B, C) in zip(probs, dev):
        if A is not None:
            p.lda, p.ldb, p.ldc = A.stride(0), B.stride(0), C.stride(0)
    seen = 0
    for vid in range(g.gemm_variant_count(dtype)):
        c = g.gemm_cfg_at_grouped(vid, probs, dtype, bl)
        if c is None or (c.block_m, c.block_n, c.block_k, c.stages, c.mfma) != (256, 256, SLAB[dtype], 2, 32 if dtype == E4M3 else 16):
            continue
        table, _ = g.gemm_grouped_plan(c, probs)
        assert g.gemm_launched_kernel(c, table) == ("pipelined ragged" if ragged else "pipelined", 2, 2, 7)
        if beta:
            c.alpha, c.beta = 0.5, beta
            for (_, _, C), old in zip(dev, olds):
                if C is not None:
                    C.copy_(old)
        g.gemm_run_grouped(c, table, g.table_to_device(table))
        torch.cuda.synchronize()
        for (m, n, k), (_, _, C), ref in zip(shapes, dev, refs):
            if m:
                whole = C._base
                assert torch.equal(C, ref), (c.describe(), m, n, k, int((C != ref).sum()))
                assert bool((whole[m:] == mark).all()) and bool((whole[:, n:] == mark).all()), (m, n)
                whole.fill_(POISON)
        seen += 1
    assert seen == 2


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [BF16, E4M3, FP16])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("ragged", [0, 1])
def test_short_tile_rows_are_exact(dtype, bl, ragged):
    _check([(m, 272 - 16 * (i % 3) - 5 * ragged, (20 + i) * SLAB[dtype] - (13 * ragged if i % 2 else 0)) for i, m in enumerate(ROWS)], dtype, bl, ragged)


# 32 slots of an XCD full and 3 (10, 16, 17) more: the tiles of the last round in quarters (halves, halves, whole), some of them short
@pytest.mark.gpu
@pytest.mark.parametrize("more", [3, 10, 16, 17])
@pytest.mark.parametrize("dtype,bl,ragged", [(BF16, 0, 0), (BF16, 1, 1), (E4M3, 1, 0), (E4M3, 0, 1), (FP16, 0, 1), (FP16, 1, 0)])
def test_the_last_round_shares_its_tiles(more, dtype, bl, ragged):
    rows = [x for x in ROWS if x] * 2
    _check([(8192, 2048, 24 * SLAB[dtype])] + [(rows[i + more % 7], 272 - 5 * ragged, 20 * SLAB[dtype] - 13 * ragged) for i in range(more)], dtype, bl, ragged)


# The store stage that reads the old C is another: staged as fp32, in rows dealt to the waves by MFMA row blocks
@pytest.mark.gpu
@pytest.mark.parametrize("more", [None, 3, 10])
@pytest.mark.parametrize("dtype,bl,ragged", [(BF16, 0, 0), (BF16, 1, 1), (E4M3, 1, 0), (E4M3, 0, 1), (FP16, 0, 1), (FP16, 1, 0)])
def test_short_and_shared_tiles_accumulate(more, dtype, bl, ragged):
    if more is None:
        shapes = [(m, 272 - 16 * (i % 3) - 5 * ragged, (20 + i) * SLAB[dtype] - (13 * ragged if i % 2 else 0)) for i, m in enumerate(ROWS)]
    else:
        rows = [x for x in ROWS if x] * 2
        shapes = [(8192, 2048, 24 * SLAB[dtype])] + [(rows[i + more % 7], 272 - 5 * ragged, 20 * SLAB[dtype] - 13 * ragged) for i in range(more)]
    _check(shapes, dtype, bl, ragged, beta=2.0)
