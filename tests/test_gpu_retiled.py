"""Launches whose cfg names one tile and that run a pipelined kernel of another (retile.hpp): which tile, K slices and slabs
they come to, and results that equal the once-rounded exact product bit for bit (integer operands, whose sums are exact in
fp32 whatever their order)."""
import os
import random
import re
import shutil
import subprocess

import pytest
import torch

from test_gpu_chained import BF16, E4M3, FP16, IN, SLAB, _problem, _run
from test_kernel_resources import CSRC, HIPCC

# (what runs; the cfg's tile and K slices; M, N, K slabs, batch): the ring's prologue alone and a turn of its period more,
# row and column counts that end inside a tile, one slice in place of several and fewer than the cfg's
LAUNCHES = [((64, 128, 1), (128, 128, 2), 18, 557, 9, 20), ((64, 128, 3), (128, 128, 4), 350, 685, 27, 1),
            ((64, 128, 3), (128, 256, 4), 19, 541, 27, 8), ((64, 256, 1), (256, 256, 2), 131, 701, 9, 20),
            ((128, 128, 1), (256, 128, 2), 65, 429, 9, 40), ((128, 256, 1), (128, 128, 1), 386, 157, 9, 40),
            ((128, 256, 3), (128, 256, 4), 333, 685, 30, 8), ((192, 128, 1), (256, 256, 1), 133, 411, 14, 40),
            ((256, 128, 1), (128, 256, 1), 962, 29, 9, 40),
            ((192, 256, 1), (256, 256, 1), 180, 253, 21, 240), ((256, 256, 1), (128, 256, 1), 229, 253, 20, 240)]


def _cfg(g, tile, M, N, K, batch, dtype, bl):
    for i in range(g.gemm_cfg_count(dtype)):
        c = g.gemm_cfg_at_batched(i, M, N, K, batch, dtype, bl)
        if c is not None and not c.stream_k and (c.block_m, c.block_n, c.split_k) == tile and c.block_k == SLAB[dtype]:
            return c
    return None


@pytest.mark.gpu
@pytest.mark.parametrize("runs,tile,M,N,slabs,batch", LAUNCHES)
@pytest.mark.parametrize("dtype", [BF16, E4M3, FP16])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("ragged", [0, 1])
def test_retiled_launch_is_exact(runs, tile, M, N, slabs, batch, dtype, bl, ragged):
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    N, K = (N, slabs * SLAB[dtype] - 3) if ragged else (N // 16 * 16, slabs * SLAB[dtype] - 16)
    c = _cfg(g, tile, M, N, K, batch, dtype, bl)
    assert c is not None and g.gemm_launched_tile(c) == runs, (c and c.describe(), c and g.gemm_launched_tile(c))
    assert g.gemm_launched_kernel(c) == ("pipelined ragged" if ragged else "pipelined", 2, 2, 7)
    workspace_for(c)
    A, B, ref = _problem(batch, M, N, K, dtype, bl)
    out = _run(g, c, A, B, M, N, dtype)
    assert torch.equal(out, ref), (c.describe(), int((out != ref).sum()))


@pytest.mark.gpu
@pytest.mark.parametrize("runs,tile,M,N,slabs,batch", [LAUNCHES[1], LAUNCHES[7]])
def test_retiled_launch_accumulates(runs, tile, M, N, slabs, batch):
    """beta reads the old C in the store stage, or in the summation of the slices."""
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    K = slabs * 64
    c = _cfg(g, tile, M, N, K, batch, BF16, 1)
    c.alpha, c.beta = 0.5, 2.0
    assert g.gemm_launched_tile(c) == runs
    workspace_for(c)
    A, B, _ = _problem(batch, M, N, K, BF16, 1)
    ldc = -(-N // 8) * 8
    C = torch.randint(-4, 5, (batch, M, ldc), device="cuda").to(torch.bfloat16)
    ref = (0.5 * torch.bmm(A[..., :K].double(), B[..., :K].double().transpose(1, 2).contiguous()) + 2.0 * C[..., :N].double()).bfloat16()
    c.lda, c.ldb, c.ldc, c.stride_a, c.stride_b, c.stride_c = A.stride(1), B.stride(1), ldc, A.stride(0), B.stride(0), C.stride(0)
    g.gemm_run(c, A, B, C)
    torch.cuda.synchronize()
    assert torch.equal(C[..., :N], ref)


@pytest.mark.gpu
@pytest.mark.parametrize("runs,tile,M,N,slabs,batch", [LAUNCHES[1], LAUNCHES[8]])
def test_own_tile_launches_the_cfgs_kernel(runs, tile, M, N, slabs, batch):
    """With own_tile the cfg's K slices, all of them, leave their sums in the workspace; the replacement uses fewer."""
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    K = slabs * 64
    c = _cfg(g, tile, M, N, K, batch, BF16, 1)
    assert g.gemm_launched_tile(c) == runs
    c.own_tile = 1
    assert g.gemm_launched_tile(c) == tile and g.gemm_launched_kernel(c)[1:3] == (c.waves_m, c.waves_n)
    ws = workspace_for(c)
    if ws is not None:
        ws.fill_(float("nan"))
    A, B, ref = _problem(batch, M, N, K, BF16, 1)
    assert torch.equal(_run(g, c, A, B, M, N, BF16), ref), c.describe()
    if ws is not None:
        need = g.gemm_workspace_bytes(c) // 4
        slices = ws[:need].view(batch * c.split_k, M, -1)[..., :N]
        assert not bool(torch.isnan(slices).any())


def test_a_retiled_launch_fits_what_the_cfg_was_checked_for():
    """Of drawn cfgs: no more K slices than the cfg has (its workspace holds their slabs), none of them empty, nine slabs or more
    each; small grids, small tiles and Stream-K run their own tile."""
    from paper_2512_04226_amd import binding as g
    rng, retiled = random.Random(3), 0
    for _ in range(4000):
        dtype = rng.choice((BF16, E4M3, FP16))
        M, N, K, batch = rng.randint(1, 6000), rng.randint(1, 6000), rng.randint(1, 12000), rng.choice((1, 1, 7, 50))
        c = g.gemm_cfg_at_batched(rng.randrange(g.gemm_cfg_count(dtype)), M, N, K, batch, dtype, rng.randrange(2))
        if c is None:
            continue
        bm, bn, split = g.gemm_launched_tile(c)
        if (bm, bn, split) == (c.block_m, c.block_n, c.split_k) or g.gemm_launched_kernel(c)[0].startswith("sliced"):
            continue
        retiled += 1
        slabs = -(-K // SLAB[dtype])
        per = -(-slabs // split)
        assert split <= c.split_k and per * (split - 1) < slabs and per >= 9
        assert (bm, bn) in {(m, n) for m in (64, 128, 192, 256) for n in (128, 256)}
        assert c.block_m * c.block_n >= 128 * 128 and not c.stream_k
        assert -(-M // c.block_m) * -(-N // c.block_n) * c.split_k * batch >= 64
    assert retiled > 100


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_largest_retiled_kernels_keep_no_scratch(tmp_path):
    """192x256: 192 accumulators per lane and the fragments of two k-steps on one wave per SIMD."""
    src = tmp_path / "k.hip"
    src.write_text('#include "gemm_kernel.hpp"\nnamespace g355 {\n' + "".join(
        "template __global__ void gemm_kernel<Tile<%d, 192, 256, %d, 2, 2, %d, 2, %d, 0, 7, %d, 3>>(const KernelArgs);\n" %
        (es, 128 // es, 16 if es == 2 else 32, bl, rg) for es in (1, 2) for bl in (0, 1) for rg in (0, 1)) + "}\n")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", "-I", CSRC, "-o", os.devnull, str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert scratch == [0] * 8, scratch


# One tile row of 129 to 256 rows over large weights (the threshold lowered, so that small ones count): K walked in a rotated order
# where the pitch is a power of two of 16 KiB and more, K slices that are halved, a last slab that ends inside the K range
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K_bytes,tile,runs", [(129, 384, 16384, (256, 128, 1), (192, 128, 1)), (192, 400, 16384, (256, 128, 2), (192, 128, 2)),
                                                   (193, 272, 18432, (256, 256, 2), (256, 128, 1)), (256, 144, 16384 - 96, (256, 256, 4), (256, 128, 2))])
@pytest.mark.parametrize("dtype", [BF16, E4M3, FP16])
@pytest.mark.parametrize("bl", [0, 1])
def test_streaming_launch_of_a_pipelined_tile_is_exact(M, N, K_bytes, tile, runs, dtype, bl):
    from gpu_util import workspace_for
    from paper_2512_04226_amd import binding as g
    K = K_bytes // (1 if dtype == E4M3 else 2)
    hw = g.gemm_hw_get()
    hw.mall_bytes = 1 << 20
    g.gemm_hw_set(hw)
    try:
        c = _cfg(g, tile, M, N, K, 1, dtype, bl)
        gen = torch.Generator(device="cuda").manual_seed(5)
        A, B = (torch.randint(-3, 4, s, device="cuda", generator=gen).float() for s in ((M, K), (K, N)))
        ref = (A.double() @ B.double()).to(torch.float16 if dtype == FP16 else torch.bfloat16)
        A, B = (x.to(IN[dtype]) for x in (A, B.t().contiguous() if bl else B))
        c.lda, c.ldb, c.ldc = A.stride(0), B.stride(0), N
        assert g.gemm_launched_kernel(c) == ("streaming", 2, 2, 7) and g.gemm_launched_tile(c) == runs
        workspace_for(c)
        C = torch.full((M + 1, N), 99.0, dtype=ref.dtype, device="cuda")
        g.gemm_run(c, A, B, C)
        torch.cuda.synchronize()
        assert torch.equal(C[:M], ref) and bool((C[M] == 99.0).all()), c.describe()
    finally:
        g.gemm_hw_reset()
