"""The sliced kernel: four waves of a workgroup compute one 16x16 tile over a quarter of K each.  Integer operands, whose sums are
exact in fp32 whatever their order: bit for bit the once-rounded product, and nothing outside C is written."""
import pytest
import torch

from test_gpu_chained import BF16, E4M3, FP16, _problem, _run

SLAB = {BF16: 128, E4M3: 256, FP16: 128}


def _cfg(g, M, N, K, batch, dtype, bl, split=1):
    """A cfg that the sliced kernel replaces: 16x16 tiles in one piece, or K slices of 16x64 and 16x128 ones."""
    for i in range(g.gemm_cfg_count(dtype)):
        c = g.gemm_cfg_at_batched(i, M, N, K, batch, dtype, bl)
        if c is not None and not c.stream_k and c.split_k == split and (c.block_m, c.block_n) in (((16, 16),) if split == 1 else ((16, 64), (16, 128))):
            return c
    return None


# slabs: all slices full and alike; the last one a slab short; the fourth slice empty (three of three); many; with a K that ends
# inside a slab by whole chunks or (ragged) inside a chunk
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [BF16, E4M3, FP16])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("ragged", [0, 1])
@pytest.mark.parametrize("M,N,batch,slabs,short", [(1, 16, 1, 20, 0), (17, 40, 1, 23, 16), (33, 61, 1, 17, 0), (16, 250, 1, 32, 48),
                                                   (5, 33, 7, 21, 32), (100, 100, 1, 20, 80)])
def test_sliced_is_exact(M, N, batch, slabs, short, dtype, bl, ragged):
    from paper_2512_04226_amd import binding as g
    K = slabs * SLAB[dtype] - short - (13 if ragged else 0)
    N = N if ragged else -(-N // 16) * 16
    c = _cfg(g, M, N, K, batch, dtype, bl)
    assert c is not None and g.gemm_launched_kernel(c) == ("sliced ragged" if ragged else "sliced", 1, 1, 0), c and g.gemm_launched_kernel(c)
    assert g.gemm_launched_tile(c) == (16, 16, 1)
    A, B, ref = _problem(batch, M, N, K, dtype, bl)
    out = _run(g, c, A, B, M, N, dtype)
    assert torch.equal(out, ref), (c.describe(), int((out != ref).sum()))


# 9 slabs: three to a slice, the fourth without; K slices of the cfg that are not launched, beta in the only kernel
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,split,slabs", [(BF16, 16, 32), (BF16, 1, 9), (FP16, 8, 40), (E4M3, 1, 9), (E4M3, 32, 64)])
@pytest.mark.parametrize("ragged", [0, 1])
def test_sliced_in_place_of_k_slices_accumulates(dtype, split, slabs, ragged):
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    M, N, K = 19, 48 - 7 * ragged, slabs * SLAB[dtype] - 5 * ragged
    c = _cfg(g, M, N, K, 1, dtype, 1, split)
    c.alpha, c.beta = 0.5, 2.0
    assert g.gemm_launched_kernel(c)[0] == ("sliced ragged" if ragged else "sliced"), c.describe()
    workspace_for(c)
    A, B, _ = _problem(1, M, N, K, dtype, 1)
    C = torch.randint(-4, 5, (M, 56), device="cuda").to(torch.float16 if dtype == FP16 else torch.bfloat16)
    old = C.clone()
    ref = (0.5 * (A[0, :, :K].double() @ B[0, :, :K].double().t().contiguous()) + 2.0 * old[:, :N].double()).to(C.dtype)
    c.lda, c.ldb, c.ldc = A.stride(1), B.stride(1), 56
    g.gemm_run(c, A, B, C)
    torch.cuda.synchronize()
    assert torch.equal(C[:, :N], ref) and torch.equal(C[:, N:], old[:, N:])


# row-major B in place of K slices: 16 and 32 of them, the shortest and longest K, tiles of the last column half empty
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [BF16, FP16])
@pytest.mark.parametrize("split,M,N,slabs", [(16, 5, 208, 16), (16, 33, 72, 32), (32, 2, 24, 32), (32, 47, 80, 32)])
@pytest.mark.parametrize("ragged", [0, 1])
@pytest.mark.parametrize("beta", [0.0, 2.0])
def test_sliced_in_place_of_k_slices_of_row_major_weights(dtype, split, M, N, slabs, ragged, beta):
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    N, K = N - 3 * ragged, slabs * SLAB[dtype] - 5 * ragged
    c = _cfg(g, M, N, K, 1, dtype, 0, split)
    c.alpha, c.beta = 0.5, beta
    assert g.gemm_launched_kernel(c)[0] == ("sliced ragged" if ragged else "sliced"), c.describe()
    workspace_for(c)
    A, B, _ = _problem(1, M, N, K, dtype, 0)
    ldc = -(-N // 8) * 8 + 8
    C = torch.randint(-4, 5, (M + 1, ldc), device="cuda").to(torch.float16 if dtype == FP16 else torch.bfloat16)
    old = C.clone()
    ref = (0.5 * (A[0, :, :K].double() @ B[0, :K, :N].double()) + beta * old[:M, :N].double()).to(C.dtype)
    c.lda, c.ldb, c.ldc = A.stride(1), B.stride(1), ldc
    g.gemm_run(c, A, B, C)
    torch.cuda.synchronize()
    assert torch.equal(C[:M, :N], ref) and torch.equal(C[:, N:], old[:, N:]) and torch.equal(C[M], old[M])


def test_where_a_launch_is_sliced():
    """At most 256 tiles, small tiles or K slices, a K between the limits."""
    from paper_2512_04226_amd import binding as g
    def kind(M, N, K, dtype=BF16, bl=1, **more):
        return g.gemm_launched_kernel(_cfg(g, M, N, K, 1, dtype, bl, **more))[0]
    assert kind(40, 64, 896) == "sliced" and kind(40, 64, 880) == "plain"
    assert kind(256, 256, 2048) == "sliced" and kind(257, 256, 2048) == "plain"
    assert kind(40, 64, 12288, split=8) == "sliced" and kind(40, 64, 12416, split=8) == "plain" and kind(40, 64, 4096, split=2) == "plain"
    assert kind(16, 4096, 4096) == "plain" and kind(16, 2048, 4096) == "sliced"          # weights from memory on most CUs
    assert kind(100, 240, 4096, bl=0) == "sliced" and kind(100, 240, 4096, bl=0, split=8) == "plain" and kind(250, 240, 4096, bl=0) == "plain"
    # one tile row of many columns, row-major: only where the rows of B are whole KB apart
    assert kind(16, 2304, 2048, bl=0) == "plain" and kind(16, 2560, 2048, bl=0) == "sliced" and kind(16, 1776, 2048, bl=0) == "sliced"
    assert kind(64, 128, 2048, E4M3) == "sliced" and kind(64, 128, 1792, E4M3) == "plain" and kind(64, 128, 2048, E4M3, 0) == "plain"
