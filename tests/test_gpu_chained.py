"""The chained kernels: a workgroup computes several tiles and its requests for a tile's slabs run ahead of the tiles before
it.  Integer-valued operands, whose sums are exact in fp32 whatever their order: every result has to equal the once-rounded
product bit for bit (a plain fp64 product is the reference), and nothing outside C may be written."""
import pytest
import torch

BF16, E4M3, FP16 = 0, 1, 2
IN = {BF16: torch.bfloat16, E4M3: torch.float8_e4m3fn, FP16: torch.float16}
SLAB = {BF16: 64, E4M3: 128, FP16: 64}
SLOTS = {(256, 256): 256, (256, 128): 256, (128, 256): 256, (128, 128): 512, (128, 64): 768, (64, 128): 768, (64, 64): 1280}
POISON = 12345.0


def _padded(x, per16):
    """Rows padded with NaN to whole chunks and one more."""
    r, c = x.shape[-2:]
    out = torch.full(x.shape[:-1] + (-(-c // per16) * per16 + per16,), float("nan"), device="cuda")
    out[..., :c] = x
    return out


def _problem(batch, M, N, K, dtype, bl, seed=3, alpha=1.0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    A, B = (torch.randint(-3, 4, s, device="cuda", generator=gen).float() for s in ((batch, M, K), (batch, K, N)))
    ref = (alpha * torch.bmm(A.double(), B.double())).to(torch.float16 if dtype == FP16 else torch.bfloat16)
    per16 = 16 if dtype == E4M3 else 8
    B = B.transpose(1, 2).contiguous() if bl else B
    return _padded(A, per16).to(IN[dtype]), _padded(B, per16).to(IN[dtype]), ref


def _run(g, c, A, B, M, N, dtype):
    batch = A.shape[0]
    ldc = -(-N // 8) * 8 + 8
    C = torch.full((batch, M + 1, ldc), POISON, dtype=torch.float16 if dtype == FP16 else torch.bfloat16, device="cuda")
    mark = C[0, 0, 0].item()
    c.lda, c.ldb, c.ldc = A.stride(1), B.stride(1), ldc
    c.stride_a, c.stride_b, c.stride_c = A.stride(0), B.stride(0), C.stride(0)
    g.gemm_run(c, A, B, C)
    torch.cuda.synchronize()
    assert (C[:, M:] == mark).all() and (C[:, :, N:] == mark).all(), (c.describe(), "written outside C")
    return C[:, :M, :N]


def _per_tile_size(g, M, N, K, batch, dtype, bl):
    """One cfg per tile size of SLOTS (another variant of it in each call's order)."""
    seen = {}
    for i in range(0, g.gemm_cfg_count(dtype), 7):
        c = g.gemm_cfg_at_batched(i, M, N, K, batch, dtype, bl)
        if c is not None and (c.block_m, c.block_n) in SLOTS:
            seen.setdefault((c.block_m, c.block_n), c)
    return seen


def _unchained_256(dtype, bl, ragged, slabs):
    """The 256x256 tile has no ragged chained kernel, none for fp8 with row-major B, and in fp8 runs it up to four slabs."""
    return {(256, 256)} if ragged or dtype == E4M3 and (bl == 0 or slabs > 4) else set()


# (M, N): tiles with rows and columns missing at both ends; K: part of one slab, one slab, two, five and a rest -- with the
# ring of two or three stages fewer slabs per tile than stages, as many and more
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,bl", [(d, b) for d in (BF16, FP16, E4M3) for b in (0, 1)])
@pytest.mark.parametrize("slabs,short,ragged_n", [(1, 0, 0), (1, 24, 0), (2, 0, 0), (2, 32, 5), (5, 16, 0), (5, 13, 1), (1, 3, 3)])
def test_chained_bit_exact_on_a_batch(dtype, bl, slabs, short, ragged_n):
    from paper_2512_04226_amd import binding as g
    M, N, K = 200, 272 - ragged_n, slabs * SLAB[dtype] - short * (2 if dtype == E4M3 and short % 8 == 0 else 1)
    ragged = N % (16 if dtype == E4M3 else 8) or K % (16 if dtype == E4M3 else 8)
    chained = set()
    whole = None
    for size, slots in SLOTS.items():
        tiles = -(-M // size[0]) * -(-N // size[1])
        batch = -(-8 * slots // tiles) + 3          # eight rounds: every size and type chains
        c = _per_tile_size(g, M, N, K, batch, dtype, bl).get(size)
        if c is None:
            continue
        kind = g.gemm_launched_kernel(c)[0]
        if kind not in ("chained", "chained ragged"):
            continue
        assert (kind == "chained ragged") == bool(ragged)
        if whole is None or whole[0].shape[0] < batch:
            whole = _problem(batch, M, N, K, dtype, bl)
        A, B, ref = (x[:batch] for x in whole)
        out = _run(g, c, A, B, M, N, dtype)
        assert torch.equal(out, ref), (c.describe(), int((out != ref).sum()))
        chained.add(size)
    assert chained == set(SLOTS) - _unchained_256(dtype, bl, ragged, slabs)


# one problem: rounds from two to many (a last block of tiles of its own width), bands of both heights, no XCD
# renumbering; a tile count that no XCD count divides
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,group_m,remap", [(4100, 4208, 0, 1), (20011, 1104, 0, 1), (9000, 3008, 3, 1), (4100, 4208, 1, 0), (3333, 8896, 64, 1), (11700, 11296, 0, 1)])
@pytest.mark.parametrize("dtype,bl", [(BF16, 1), (FP16, 0), (E4M3, 1)])
def test_chained_walk_covers_every_tile_once(M, N, group_m, remap, dtype, bl):
    from paper_2512_04226_amd import binding as g
    K = SLAB[dtype] + 16
    A, B, ref = _problem(1, M, N, K, dtype, bl)
    chained = set()
    for c in _per_tile_size(g, M, N, K, 1, dtype, bl).values():
        if g.gemm_launched_kernel(c)[0] != "chained":
            continue
        if group_m:
            c.group_m = group_m
        c.xcd_remap = remap
        out = _run(g, c, A, B, M, N, dtype)
        assert torch.equal(out, ref), (c.describe(), int((out != ref).sum()))
        chained.add((c.block_m, c.block_n))
    expected = {(128, 64), (64, 128)}                      # two to four rounds; 64x64 3.4 to 5.8, fp8 from four on
    if dtype != E4M3 or M != 4100:
        expected.add((64, 64))
    if M == 11700:                                         # eight rounds of 256x256 tiles, 16 of their halves
        expected |= {(256, 128), (128, 256)} | ({(256, 256), (128, 128)} if dtype != E4M3 else set())
    assert chained == expected


# alpha: powers of two, so that the scaled sum has one rounding all the same
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,bl", [(d, b) for d in (BF16, FP16, E4M3) for b in (0, 1)])
@pytest.mark.parametrize("alpha,K,ragged_n", [(0.5, 64, 0), (-2.0, 80, 0), (0.25, 77, 3)])
def test_chained_scales_by_alpha(dtype, bl, alpha, K, ragged_n):
    from paper_2512_04226_amd import binding as g
    M, N = 200, 272 - ragged_n
    K = K * (2 if dtype == E4M3 and not ragged_n else 1)
    chained = set()
    for size, slots in SLOTS.items():
        batch = -(-8 * slots // (-(-M // size[0]) * -(-N // size[1]))) + 3
        c = _per_tile_size(g, M, N, K, batch, dtype, bl).get(size)
        if not g.gemm_launched_kernel(c)[0].startswith("chained"):
            continue
        A, B, ref = _problem(batch, M, N, K, dtype, bl, alpha=alpha)
        c.alpha = alpha
        out = _run(g, c, A, B, M, N, dtype)
        assert torch.equal(out, ref), (c.describe(), int((out != ref).sum()))
        chained.add(size)
    assert chained == set(SLOTS) - _unchained_256(dtype, bl, ragged_n, -(-K // SLAB[dtype]))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,bl", [(d, b) for d in (BF16, FP16, E4M3) for b in (0, 1)])
@pytest.mark.parametrize("ragged", [0, 1])
def test_chained_infinities_and_nan_stay_in_their_rows_and_columns(dtype, bl, ragged):
    """A NaN row and column, and (16-bit) infinities of both signs: what the plain product gives, and the tiles before and
    after in the same workgroup untouched by them."""
    from paper_2512_04226_amd import binding as g
    M, N, K = 200, 272 - 3 * ragged, 2 * SLAB[dtype] - 5 * ragged
    batch = -(-8 * 1280 // 20) + 3
    A, B, ref = _problem(batch, M, N, K, dtype, bl)
    nan, inf = float("nan"), float("nan") if dtype == E4M3 else float("inf")
    Af = A.float()
    Bf = B.float()
    k = (lambda b, kk, n: (b, n, kk)) if bl else (lambda b, kk, n: (b, kk, n))
    for b in (0, batch // 2, batch - 1):
        Af[b, 3, K - 1], Af[b, 130, 1], Af[b, M - 1, 5] = nan, inf, -inf
        Bf[k(b, 2, 65)], Bf[k(b, K - 1, N - 1)], Bf[k(b, 0, 0)] = nan, inf, -inf
        left, right = Af[b, :, :K].double(), Bf[b].double()
        right = right[:, :K].t() if bl else right[:, :N]
        ref[b] = (left.cpu() @ right.cpu()).to(ref.dtype)
    A, B = Af.to(A.dtype), Bf.to(B.dtype)
    sizes = _per_tile_size(g, M, N, K, batch, dtype, bl)
    for size in ((64, 64), (128, 64), (128, 128), (256, 128)):
        c = sizes[size]
        if not g.gemm_launched_kernel(c)[0].startswith("chained"):
            assert size in ((128, 128), (256, 128)), c.describe()        # (fewer than eight rounds of them here)
            continue
        out = _run(g, c, A, B, M, N, dtype)
        same = (out == ref) | (out.isnan() & ref.isnan())
        assert bool(same.all()), (c.describe(), int((~same).sum()))


def test_where_a_launch_is_chained():
    """beta = 0, one K slice, three rounds of tiles, few slabs; what it refuses runs the kernel it ran before."""
    from paper_2512_04226_amd import binding as g
    def cfg(M, N, K):
        return next(x for x in (g.gemm_cfg_at_ex(i, M, N, K, BF16, 1) for i in range(0, g.gemm_cfg_count(BF16), 7))
                    if x is not None and (x.block_m, x.block_n, x.block_k, x.mfma) == (256, 256, 64, 16))
    c = cfg(4096, 12288, 256)
    assert g.gemm_launched_kernel(c)[0] == "chained"
    d = c.copy(); d.beta = 0.5
    assert g.gemm_launched_kernel(d)[0] == "plain"
    for M, N, K, kind in ((4096, 12288 - 256, 256, "plain"), (4096, 12288, 9 * 64, "plain"), (4096, 12288, 20 * 64, "pipelined")):
        d = cfg(M, N, K)
        assert g.gemm_launched_kernel(d)[0] == kind, (M, N, K)


# What the chained kernel takes longer for: fp8 128x128 tiles of one problem; 128x128 tiles of one slab whose rows of C start
# inside a line, with more of them than the memory-side cache holds (1.2 to 1.5 times); a fp8 256x256 tile; 2.5 slabs of a tile
# that computes half slabs; the larger tiles from eight slabs on; two rounds of them.
@pytest.mark.parametrize("batch,M,N,K,dtype,bl", [
    (1, 15544, 10064, 32, E4M3, 0), (1, 30152, 10128, 16, E4M3, 1), (1, 22456, 5520, 32, BF16, 0), (1, 18936, 6256, 16, FP16, 1),
    (1, 11384, 22016, 848, E4M3, 1), (1, 5320, 10560, 160, FP16, 1), (1, 5272, 10320, 480, BF16, 0), (1, 2448, 14336, 112, BF16, 1)])
def test_launches_that_chaining_slows_are_not_chained(batch, M, N, K, dtype, bl):
    from paper_2512_04226_amd import binding as g
    c = g.gemm_select_batched(M, N, K, batch, dtype, bl)
    assert g.gemm_launched_kernel(c)[0] in ("plain", "ragged"), c.describe()


@pytest.mark.parametrize("batch,M,N,K,dtype,bl", [
    (32, 2048, 2048, 128, BF16, 1), (1, 65536, 2048, 128, BF16, 0), (142, 400, 1056, 64, BF16, 1), (1, 16408, 2960, 64, BF16, 1),
    (52, 808, 1720, 576, FP16, 0), (9, 4048, 3088, 352, FP16, 1)])
def test_launches_that_chaining_speeds_up_are_chained(batch, M, N, K, dtype, bl):
    from paper_2512_04226_amd import binding as g
    c = g.gemm_select_batched(M, N, K, batch, dtype, bl)
    assert g.gemm_launched_kernel(c)[0] == "chained", c.describe()
