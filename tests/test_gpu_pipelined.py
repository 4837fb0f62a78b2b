"""The pipelined instantiations of the 256x256 tiles (K-loop form 7, from twenty K slabs per workgroup): slab counts around
the five-slab unroll and its tail, K ranges that end inside a slab, tiles over the edge of C, both storages of B, split-K,
Stream-K, a batch, a group and beta.  Integer-valued operands: bit for bit the oracle's."""
import numpy as np
import pytest
import torch

from paper_2512_04226_amd import workloads as wl

pytestmark = pytest.mark.gpu

BF16, E4M3, FP16 = 0, 1, 2
SLAB = {BF16: 64, FP16: 64, E4M3: 128}


def _operands(oracle, M, N, K, dtype):
    if dtype == E4M3:
        gen = np.random.default_rng([21, M, N, K])
        vals = np.arange(-4, 5).astype(np.float64)
        return oracle.encode_e4m3(vals[gen.integers(0, 9, size=(M, K))]), oracle.encode_e4m3(vals[gen.integers(0, 9, size=(K, N))])
    make = wl.integer_fp16 if dtype == FP16 else wl.integer_bf16
    return make(M, N, K, seed=21, case=M + 3 * N + 7 * K)


def _cfgs(g, M, N, K, dtype, bl):
    for idx in range(g.gemm_cfg_count(dtype)):
        c = g.gemm_cfg_at_ex(idx, M, N, K, dtype, bl)
        if c is not None and (c.block_m, c.block_n, c.block_k, c.stages, c.mfma) == (256, 256, SLAB[dtype], 2, 32 if dtype == E4M3 else 16):
            yield c


# (slabs, K elements short of the last whole slab): 20 = the first pipelined count, 23..28 every position in the unrolled
# ring (the loop runs whole fives of the slabs below slabs - 3), 41 for a split in two; an odd shortfall: the ragged form,
# with NaN patterns between K and the leading dimension
@pytest.mark.parametrize("slabs,short", [(20, 0), (20, 16), (23, 0), (24, 48), (25, 0), (26, 32), (27, 0), (28, 16), (41, 0), (21, 1), (25, 13),
                                         (41, 127)])
@pytest.mark.parametrize("dtype", [BF16, FP16, E4M3])
@pytest.mark.parametrize("bl", [0, 1])
def test_pipelined_bit_exact(oracle, slabs, short, dtype, bl):
    from gpu_util import run_cfg, to_dev
    from paper_2512_04226_amd import binding as g
    M, N, K = 300, 272, slabs * SLAB[dtype] - short
    A, B = _operands(oracle, M, N, K, dtype)
    ref16, _ = oracle.gemm(A, B, dtype)
    pad = lambda x: np.pad(x, ((0, 0), (0, -x.shape[1] % 16)), constant_values=0x7F if dtype == E4M3 else 0x7FC0 if dtype == BF16 else 0x7E00)
    dA, dB = to_dev(pad(A)), to_dev(pad(np.ascontiguousarray(B.T) if bl else B))
    modes = set()
    for c in _cfgs(g, M, N, K, dtype, bl):
        if c.split_k > 2:
            continue
        c.lda, c.ldb = dA.shape[1], dB.shape[1]
        if c.split_k == 1:
            assert g.gemm_launched_kernel(c) == ("pipelined ragged" if K % (16 if dtype == E4M3 else 8) else "pipelined", 2, 2, 7)
        out = run_cfg(c, dA, dB, M, N)
        assert np.array_equal(out, ref16), (c.describe(), int((out != ref16).sum()))
        modes.add((c.split_k, c.stream_k))
    assert (1, 0) in modes and (2, 0) in modes


def test_pipelined_stream_k_with_whole_tiles(oracle):
    """More tiles than workgroups: whole tiles and Stream-K segments in one launch."""
    from gpu_util import run_cfg, to_dev
    from paper_2512_04226_amd import binding as g
    M, N, K = 4097, 4352, 1288
    A, B = _operands(oracle, M, N, K, BF16)
    rows = np.unique(np.concatenate([np.arange(0, M, 131), [255, 256, 4095, 4096]]))
    ref16, _ = oracle.gemm_rows(A, B, rows, BF16)
    dA, dB = to_dev(A), to_dev(B)
    n = 0
    for c in _cfgs(g, M, N, K, BF16, 0):
        if c.stream_k:
            assert g.gemm_launched_kernel(c)[0] == "pipelined"
            assert np.array_equal(run_cfg(c, dA, dB, M, N)[rows], ref16), c.describe()
            n += 1
    assert n >= 1


@pytest.mark.parametrize("bl", [0, 1])
def test_pipelined_batch_group_and_beta(oracle, bl):
    from gpu_util import to_dev
    from paper_2512_04226_amd import binding as g
    M, N, K, batch = 40, 264, 1352, 3
    ops = [_operands(oracle, M + i, N, K, BF16) for i in range(batch)]
    Cin = wl.integer_bf16(M, N, 8, seed=22, case=1)[0][:, :1].repeat(N, axis=1)
    tr = (lambda b: np.ascontiguousarray(b.T)) if bl else (lambda b: b)
    dA, dB = to_dev(np.stack([a[:M] for a, _ in ops])), to_dev(np.stack([tr(b) for _, b in ops]))
    for idx in range(g.gemm_cfg_count(BF16)):
        c = g.gemm_cfg_at_batched(idx, M, N, K, batch, BF16, bl)
        if c is None or (c.block_m, c.block_n, c.block_k, c.stages, c.mfma, c.split_k) != (256, 256, 64, 2, 16, 1):
            continue
        c.alpha, c.beta = 0.5, 2.0
        dC = to_dev(np.stack([Cin] * batch))
        g.gemm_run(c, dA, dB, dC)
        torch.cuda.synchronize()
        out = dC.cpu().numpy().view(np.uint16)
        for i, (a, b) in enumerate(ops):
            ref16, _ = oracle.accumulate(oracle.gemm(a[:M], b, BF16, alpha=0.5)[1], 2.0, Cin)
            assert np.array_equal(out[i], ref16), (c.describe(), i)
    # a group of unequal M and K whose tiles walk twenty slabs or more on average
    shapes = [(300, 264, 1352), (0, 264, 64), (260, 520, 1280), (17, 264, 640)]
    gops = [_operands(oracle, max(m, 1), n, k, BF16) for m, n, k in shapes]
    dev = [(to_dev(a[:m]), to_dev(tr(b)), torch.full((m, n), 0x7FC0, dtype=torch.int16, device="cuda")) if m else (None, None, None)
           for (m, n, k), (a, b) in zip(shapes, gops)]
    probs = g.make_problems(shapes, bl, dev)
    n = 0
    for vid in range(g.gemm_variant_count(BF16)):
        c = g.gemm_cfg_at_grouped(vid, probs, BF16, bl)
        if c is None or (c.block_m, c.block_n, c.block_k, c.stages, c.mfma) != (256, 256, 64, 2, 16):
            continue
        table, _ = g.gemm_grouped_plan(c, probs)
        dtab = g.table_to_device(table)
        g.gemm_run_grouped(c, table, dtab)
        torch.cuda.synchronize()
        for (m, _, _), (a, b), (_, _, dC) in zip(shapes, gops, dev):
            if m:
                assert np.array_equal(dC.cpu().numpy().view(np.uint16), oracle.gemm(a[:m], b, BF16)[0]), (c.describe(), m)
                dC.fill_(0x7FC0)
        n += 1
    assert n >= 2


@pytest.mark.parametrize("M,N,K,batch,dtype,bl", [(4100, 4360, 72, 1, BF16, 0), (4100, 4360, 1288, 1, BF16, 1), (260, 264, 200, 141, BF16, 1),
                                                  (4100, 4360, 272, 1, E4M3, 1)])
def test_more_tiles_than_the_device_holds_workgroups(oracle, M, N, K, batch, dtype, bl):
    """306 tiles of 256x256, 1155 of 128x128; 564 to 1269 of a batch: every tile of every problem is written, bit for bit,
    whatever order the workgroups run in.  Sampled rows of the product against the oracle; every row against a second configuration."""
    from gpu_util import to_dev
    from paper_2512_04226_amd import binding as g
    A, B = _operands(oracle, batch * M, N, K, dtype)
    per16 = 16 if dtype == E4M3 else 8
    pad = lambda x: np.pad(x, ((0, 0), (0, -x.shape[1] % per16)))
    dA, dB = to_dev(pad(A)), to_dev(pad(np.ascontiguousarray(B.T) if bl else B))
    dBs = dB.repeat(batch, 1)
    rows = np.unique(np.concatenate([np.arange(0, batch * M, 997), [M - 1, batch * M - 1]]))
    ref16, _ = oracle.gemm_rows(A, B, rows, dtype)
    first, n = None, 0
    for idx in range(g.gemm_cfg_count(dtype)):
        c = g.gemm_cfg_at_batched(idx, M, N, K, batch, dtype, bl)
        if c is None or c.split_k > 1 or c.stream_k or c.block_m * c.block_n < 128 * 128:
            continue
        dC = torch.full((batch * M, c.ldc), 0x7FC0, dtype=torch.int16, device="cuda")
        c.stride_a, c.stride_b, c.stride_c = M * c.lda, dB.shape[0] * c.ldb, M * c.ldc
        g.gemm_run(c, dA, dBs, dC)
        torch.cuda.synchronize()
        out = dC.cpu().numpy().view(np.uint16)[:, :N]
        assert np.array_equal(out[rows], ref16), c.describe()
        first = out if first is None else first
        assert np.array_equal(out, first), c.describe()
        n += 1
    assert n >= 4


def _padded(x, dtype):
    """Rows of whole 16-byte chunks, NaN patterns between K (or N) and the pitch."""
    per16 = 16 if dtype == E4M3 else 8
    return np.pad(x, ((0, 0), (0, -x.shape[1] % per16)), constant_values=0x7F if dtype == E4M3 else 0x7FC0 if dtype == BF16 else 0x7E00)


def _old_c(M, N, dtype):
    make = wl.integer_fp16 if dtype == FP16 else wl.integer_bf16
    return make(M, N, 8, seed=23, case=1)[0][:, :1].repeat(N, axis=1)


@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("dtype", [BF16, FP16, E4M3])
@pytest.mark.parametrize("bl", [0, 1])
def test_pipelined_ragged_batch_with_splits_and_beta(oracle, dtype, bl, split):
    """Each problem's and each K slice's own last slab, an old C that is read and whose padding is not written."""
    from gpu_util import to_dev, workspace_for
    from paper_2512_04226_amd import binding as g
    M, N, K, batch = 70, 261, 40 * SLAB[dtype] - 13, 3
    ops = [_operands(oracle, M + i, N, K, dtype) for i in range(batch)]
    dA = to_dev(np.stack([_padded(a[:M], dtype) for a, _ in ops]))
    dB = to_dev(np.stack([_padded(np.ascontiguousarray(b.T) if bl else b, dtype) for _, b in ops]))
    Cin, n = _old_c(M, N, dtype), 0
    for idx in range(g.gemm_cfg_count(dtype)):
        c = g.gemm_cfg_at_batched(idx, M, N, K, batch, dtype, bl)
        if c is None or c.split_k != split or (c.block_m, c.block_n, c.block_k, c.stages, c.mfma) != (
                256, 256, SLAB[dtype], 2, 32 if dtype == E4M3 else 16):
            continue
        c.alpha, c.beta, c.lda, c.ldb, c.ldc = 0.5, 2.0, dA.shape[2], dB.shape[2], 272
        c.stride_a, c.stride_b, c.stride_c = dA[0].numel(), dB[0].numel(), M * 272
        assert g.gemm_launched_kernel(c)[0] == "pipelined ragged"
        workspace_for(c)
        dC = to_dev(np.stack([np.pad(Cin, ((0, 0), (0, 272 - N)), constant_values=0x7FC0)] * batch))
        g.gemm_run(c, dA, dB, dC)
        torch.cuda.synchronize()
        out = dC.cpu().numpy().view(np.uint16)
        for i, (a, b) in enumerate(ops):
            ref16, _ = oracle.accumulate(oracle.gemm(a[:M], b, dtype, alpha=0.5)[1], 2.0, Cin, dtype)
            assert np.array_equal(out[i][:, :N], ref16), (c.describe(), i)
        assert (out[:, :, N:] == 0x7FC0).all()
        n += 1
    assert n == 2


@pytest.mark.parametrize("bl", [0, 1])
def test_pipelined_stream_k_ragged_with_beta(oracle, bl):
    """200 tiles on 256 workers, every tile cut, twenty slabs a worker and a second segment for most: the ring is used twice in
    one workgroup, and the odd last slab is trimmed wherever a segment ends a tile."""
    from gpu_util import to_dev, workspace_for
    from paper_2512_04226_amd import binding as g
    M, N, K = 2047, 6397, 26 * 64 - 13
    A, B = _operands(oracle, M, N, K, BF16)
    rows = np.unique(np.concatenate([np.arange(0, M, 173), [255, 256, M - 1]]))
    Cin = _old_c(M, N, BF16)
    ref16, _ = oracle.accumulate(oracle.gemm_rows(A, B, rows, BF16)[1], 2.0, Cin[rows], BF16)
    dA, dB = to_dev(_padded(A, BF16)), to_dev(_padded(np.ascontiguousarray(B.T) if bl else B, BF16))
    n = 0
    for idx in range(g.gemm_cfg_count(BF16)):
        c = g.gemm_cfg_at_ex(idx, M, N, K, BF16, bl)
        if c is None or not c.stream_k or (c.block_m, c.block_n, c.block_k, c.stages, c.mfma) != (256, 256, 64, 2, 16):
            continue
        c.beta, c.lda, c.ldb = 2.0, dA.shape[1], dB.shape[1]
        assert g.gemm_launched_kernel(c)[0] == "pipelined ragged" and g.gemm_stream_k_plan(c)[2] == 0
        workspace_for(c)
        dC = to_dev(np.pad(Cin, ((0, 0), (0, c.ldc - N))))
        g.gemm_run(c, dA, dB, dC)
        torch.cuda.synchronize()
        assert np.array_equal(dC.cpu().numpy().view(np.uint16)[rows][:, :N], ref16), c.describe()
        n += 1
    assert n == 2
