"""The library's work in earnest, as measured cases: what its users have it do, through its public entry points.

A case is a plain dict.  `kind` says which entry points a program goes through:

  matmul    api.matmul(A, B): one product per call, the pick looked up and the result allocated by the call
            (`beta` != 0: accumulated into an `out` that the program keeps)
  run       a program that keeps its cfg and its output and calls gemm_run per step
  batched   gemm_select_batched once, then gemm_run per step on a strided batch
  grouped   gemm_select_grouped + gemm_grouped_plan once per routing, then gemm_run_grouped per projection

`dtype` bf16 | fp16 | fp8 (e4m3 with per-tensor scales, entering as alpha), `kc` True: B stored N x K (an nn.Linear
weight, the layout of the paper's runs), False: K x N.  Rows that are no whole number of 16-byte chunks are views of
tensors with padded rows, as the boundary asks; the padding holds ordinary values, not zeros.
"""
import math

import numpy as np
import torch

from paper_2512_04226_amd import api
from paper_2512_04226_amd import binding as g
from paper_2512_04226_amd import workloads as wl

_TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp8": torch.float8_e4m3fn}
_GEMM = {"bf16": g.GEMM_BF16, "fp16": g.GEMM_FP16, "fp8": g.GEMM_FP8_E4M3}
_LARGEST = 2.0 * 8192 ** 3      # flop of the largest listed case


def _case(kind, M, N, K, dtype, kc, beta=0.0, **more):
    return dict({"kind": kind, "M": M, "N": N, "K": K, "dtype": dtype, "kc": kc, "beta": beta}, **more)


def listed():
    return [
        # the smallest benchmark configuration: a call whose latency counts, not its rate
        dict(_case("matmul", 512, 512, 512, "bf16", False), name="square_512_bf16"),
        # one projection of a small model, a few sequences decoding: a program that keeps its cfg
        dict(_case("run", 8, 4096, 4096, "fp16", True), name="decode_m8_fp16_kc"),
        # decode of one token against a large Linear weight: every byte of the weight once
        dict(_case("matmul", 1, 28672, 8192, "bf16", True), name="decode_m1_bf16_kc"),
        # decode of 64 sequences, fp8 weights stored K x N, long reduction
        dict(_case("matmul", 64, 8192, 28672, "fp8", False), name="decode_m64_fp8"),
        # a short prefill chunk at the ridge between memory and matrix cores
        dict(_case("matmul", 256, 28672, 8192, "bf16", False), name="prefill_m256_bf16"),
        # the paper's precision and operand layout on a square
        dict(_case("matmul", 4096, 4096, 4096, "fp16", True), name="square_4096_fp16_kc"),
        # the headline benchmark shape
        dict(_case("matmul", 8192, 8192, 8192, "bf16", False), name="square_8192_bf16"),
        # the same in fp8 with per-tensor scales
        dict(_case("matmul", 8192, 8192, 8192, "fp8", False), name="square_8192_fp8"),
        # irregular shape with a long reduction (too few tiles for the chip), accumulated into a kept result
        dict(_case("matmul", 1152, 2240, 11696, "bf16", False, beta=0.5), name="irregular_accumulate_bf16"),
        # odd extents in every dimension: no row is a whole number of chunks
        dict(_case("matmul", 1501, 3003, 2005, "bf16", False), name="ragged_bf16"),
        # attention scores of 32 heads: short reduction, large output
        dict(_case("batched", 2048, 2048, 128, "bf16", True, batch=32), name="batched_scores_bf16_kc"),
        # tokens routed to 16 experts: uneven row counts against per-expert weights in one launch
        dict(_case("grouped", 16384, 4096, 4096, "bf16", False, groups=16, skew=1.0), name="grouped_experts_bf16"),
    ]


def _log(rng, lo, hi, step=1):
    return max(lo, min(hi, step * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)))


def draw(rng):
    """One more case: small calls, skinny products (decode to short prefill), irregular and large ones, ragged extents,
    strided batches and routed groups, over all types and both storages of B; at most the largest listed case's work."""
    while True:
        what = rng.choice(["small", "skinny", "skinny", "irregular", "irregular", "ragged", "ragged", "batched", "grouped"])
        dtype, kc = rng.choice(["bf16", "bf16", "fp16", "fp8"]), rng.random() < 0.5
        beta = 0.5 if rng.random() < 0.15 else 0.0
        if what == "small":
            c = _case("run" if rng.random() < 0.5 else "matmul", _log(rng, 16, 1024), _log(rng, 64, 1024, 8),
                      _log(rng, 64, 1024, 16), dtype, kc, beta)
        elif what == "skinny":
            c = _case("matmul", _log(rng, 1, 256), _log(rng, 2048, 28672, 128), _log(rng, 2048, 28672, 128), dtype, kc)
        elif what == "irregular":
            c = _case("matmul", _log(rng, 64, 16384, 16), _log(rng, 64, 16384, 16), _log(rng, 64, 16384, 16), dtype, kc, beta)
        elif what == "ragged":
            c = _case("matmul", _log(rng, 33, 6000), _log(rng, 33, 6000), _log(rng, 33, 6000), dtype, kc, beta)
        elif what == "batched":
            c = _case("batched", _log(rng, 64, 2048), _log(rng, 64, 2048, 8), _log(rng, 64, 2048, 16), dtype, kc,
                      batch=rng.randint(2, 64))
        else:
            c = _case("grouped", _log(rng, 256, 16384), _log(rng, 1024, 8192, 16), _log(rng, 1024, 8192, 16), dtype, kc,
                      groups=rng.randint(2, 32), skew=rng.choice([0.3, 1.0, 3.0]))
        if work(c)["flops"] <= _LARGEST and work(c)["bytes"] <= 1.5e9:
            return c


def _rows(case):
    return wl.routed_rows(case["groups"], case["M"], case["groups"] * 1000 + case["M"], skew=case["skew"])


def work(case):
    es = 1 if case["dtype"] == "fp8" else 2
    M, N, K = case["M"], case["N"], case["K"]
    if case["kind"] == "grouped":
        shapes = [(m, N, K) for m in _rows(case) if m]
    else:
        shapes = [(M, N, K)] * case.get("batch", 1)
    out = 4 if case["beta"] else 2      # an accumulated result is read as well
    return {"bytes": sum((m * k + k * n) * es + m * n * out for m, n, k in shapes),
            "flops": sum(2.0 * m * n * k for m, n, k in shapes)}


def tolerance(case):
    """The sums are 32-bit.  Taken in another order (other tiles, K splits) they differ by about 1e-6, which moves a few
    results across a rounding boundary of the 16-bit format: measured over the K splits of several tiles, rel 2e-5 (K = 512)
    to 6e-5 (K = 11696) and max 0.0076 (one last place) in bf16, 1.4e-5 and 0.00096 in fp16.  Stated: four times that,
    rel at the longest K of the range (28672, about 9e-5)."""
    return {"rel": 1e-4, "max": 4e-3} if case["dtype"] == "fp16" else {"rel": 4e-4, "max": 3.2e-2}


def _operand(gen, rows, cols, dtype, std):
    """(rows, cols) values N(0, std) of the dtype and their scale; rows start on 16-byte boundaries."""
    per16 = 16 if dtype == "fp8" else 8
    x = torch.randn((rows, -(-cols // per16) * per16), device="cuda", generator=gen).mul_(std)
    scale = 1.0
    if dtype == "fp8":
        scale = float(x.abs().max()) / 448.0
        x = (x / scale).clamp_(-448.0, 448.0)
    return x.to(_TORCH[dtype])[:, :cols], scale


def _product(gen, case, M):
    """Operands of one product: activations N(0, 1), weights N(0, 0.02) (scores: N(0, 1) both)."""
    N, K, dtype = case["N"], case["K"], case["dtype"]
    A, sa = _operand(gen, M, K, dtype, 1.0)
    B, sb = _operand(gen, *((N, K) if case["kc"] else (K, N)), dtype, 1.0 if case["kind"] == "batched" else 0.02)
    return A, B, sa * sb


def _out(M, N, dtype):
    t = torch.float16 if dtype == "fp16" else torch.bfloat16
    return torch.empty((M, -(-N // 8) * 8), dtype=t, device="cuda")[:, :N]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    M, N, K, dtype, kc, kind = (case[k] for k in ("M", "N", "K", "dtype", "kc", "kind"))
    layout = g.GEMM_B_K_CONTIGUOUS if kc else g.GEMM_B_ROW_MAJOR
    s = {"kind": kind, "kc": kc, "beta": case["beta"], "out": None, "ws": None}
    if kind in ("matmul", "run"):
        s["A"], s["B"], s["alpha"] = _product(gen, case, M)
        if case["beta"] or kind == "run":
            s["out"] = _out(M, N, dtype)
            s["out"].copy_(torch.randn((M, N), device="cuda", generator=gen))
        if kind == "run":
            s["cfg"] = g.gemm_select_ex(M, N, K, _GEMM[dtype], layout)
            s["cfg"].lda, s["cfg"].ldb, s["cfg"].ldc = s["A"].stride(0), s["B"].stride(0), s["out"].stride(0)
            s["cfg"].alpha, s["cfg"].beta = s["alpha"], case["beta"]
    elif kind == "batched":
        b = case["batch"]
        A, sa = _operand(gen, b * M, K, dtype, 1.0)
        B, sb = _operand(gen, b * (N if kc else K), K if kc else N, dtype, 1.0)
        s["A"], s["B"] = A.view(b, M, K), B.view(b, N if kc else K, K if kc else N)
        s["out"] = torch.empty((b, M, N), dtype=torch.float16 if dtype == "fp16" else torch.bfloat16, device="cuda")
        s["cfg"] = g.gemm_select_batched(M, N, K, b, _GEMM[dtype], layout)
        s["cfg"].alpha = sa * sb / math.sqrt(K)
    else:
        rows, alpha = _rows(case), 1.0
        s["tensors"] = []
        for m in rows:
            if m == 0:
                s["tensors"].append((None, None, None))
                continue
            A, B, alpha = _product(gen, case, m)
            s["tensors"].append((A, B, _out(m, N, dtype)))
        problems = g.make_problems([(m, N, K) for m in rows], 1 if kc else 0, s["tensors"])
        s["cfg"] = g.gemm_select_grouped(problems, _GEMM[dtype], layout)
        # (one alpha for the launch: the scale of the last group's operands stands for a model-wide one)
        s["cfg"].alpha = alpha
        s["table"], _ = g.gemm_grouped_plan(s["cfg"], problems)
        s["dev_table"] = g.table_to_device(s["table"])
    if kind in ("run", "batched"):
        need = g.gemm_workspace_bytes(s["cfg"])
        if need:
            s["ws"] = torch.empty((need + 3) // 4, dtype=torch.float32, device="cuda")
    return s


def run(state):
    if state["kind"] == "matmul":
        return api.matmul(state["A"], state["B"], out=state["out"], alpha=state["alpha"], beta=state["beta"],
                          b_k_contiguous=state["kc"])
    if state["kind"] == "grouped":
        g.gemm_run_grouped(state["cfg"], state["table"], state["dev_table"])
        return [c for _, _, c in state["tensors"] if c is not None]
    if state["ws"] is not None:
        g.gemm_set_workspace(state["ws"])
    g.gemm_run(state["cfg"], state["A"], state["B"], state["out"])
    return state["out"]


def _f64(x):
    return (x.float() if x.dtype == torch.float8_e4m3fn else x).double()


def exact(case, seed):
    s = prepare(case, seed)
    kc = case["kc"]

    def product(A, B, alpha):
        b = _f64(B)
        return alpha * (_f64(A) @ (b.t().contiguous() if kc else b.contiguous()))

    if case["kind"] == "grouped":
        alpha = float(np.float32(s["cfg"].alpha))
        return [product(A, B, alpha) for A, B, _ in s["tensors"] if A is not None]
    if case["kind"] == "batched":
        alpha = float(np.float32(s["cfg"].alpha))
        return torch.stack([product(s["A"][i], s["B"][i], alpha) for i in range(case["batch"])])
    c = product(s["A"], s["B"], float(np.float32(s["alpha"])))
    return c + case["beta"] * _f64(s["out"]) if case["beta"] else c
