"""`matmul`: the call a user of the paper's library makes -- hand over two tensors, get the product,
with the kernel chosen analytically for the shape (Section V-C: selection costs microseconds and
is cached per shape, no tuning run).  A thin convenience layer over `binding`: it looks up or
makes the cfg, keeps one workspace tensor per device and calls gemm_run; every step of the
computation runs in libgemm355.so.

    C = matmul(A, B)                       # A (M, K), B (K, N): bf16, fp16 or float8_e4m3fn
    C = matmul(X, W, b_k_contiguous=True)  # W stored (N, K), as an nn.Linear weight
"""
import ctypes

import torch

from . import binding as g

_DTYPES = {torch.bfloat16: g.GEMM_BF16, torch.float16: g.GEMM_FP16}
if hasattr(torch, "float8_e4m3fn"):
    _DTYPES[torch.float8_e4m3fn] = g.GEMM_FP8_E4M3

_cfg_cache = {}       # (M, N, K, dtype, b_layout) -> cfg; the selector is deterministic, so this is exact
_workspace = {}       # device index -> tensor
_plans = {}           # (M, N, K, dtype, b_layout, lda, ldb, ldc) -> _Plan
_MAX_PLANS = 4096     # a program with more shapes than this starts over


def select(M, N, K, dtype, b_layout=g.GEMM_B_ROW_MAJOR):
    """The analytic pick for a shape, memoised."""
    key = (M, N, K, dtype, b_layout)
    cfg = _cfg_cache.get(key)
    if cfg is None:
        cfg = _cfg_cache[key] = g.gemm_select_ex(M, N, K, dtype, b_layout)
    return cfg


class _Plan:
    """What one launch needs beside its pointers: the pick with the tensors' leading dimensions, alpha = 1 and beta = 0
    (never changed after it is made, so threads share it), and its workspace size."""
    __slots__ = ("base", "cfg", "ref", "need")

    def __init__(self, base, lda, ldb, ldc):
        self.base, self.cfg = base, base.copy()
        self.cfg.lda, self.cfg.ldb, self.cfg.ldc = lda, ldb, ldc
        self.cfg.alpha, self.cfg.beta = 1.0, 0.0
        self.ref = ctypes.byref(self.cfg)
        self.need = g.gemm_workspace_bytes(self.cfg)


def _plan(base, key):
    plan = _plans.get(key)
    if plan is None or plan.base is not base:      # (another base: the memo of picks was emptied since)
        if len(_plans) >= _MAX_PLANS:
            _plans.clear()
        plan = _plans[key] = _Plan(base, *key[5:])
    return plan


def _ensure_workspace(need, device):
    idx = device.index if device.index is not None else torch.cuda.current_device()
    cur = _workspace.get(idx)
    if cur is None or cur.numel() * 4 < need:
        # A larger buffer replaces the old one.  Launches enqueued earlier -- on whatever stream the caller
        # gave them -- may still be using the old one, and the allocator only knows about torch's current
        # stream: wait for the device before the old buffer can be handed out again.  (Rare: the buffer
        # only ever grows.)
        if cur is not None:
            torch.cuda.synchronize(device)
        cur = _workspace[idx] = torch.empty((need + 3) // 4, dtype=torch.float32, device=device)
    g.gemm_set_workspace(cur)


def matmul(A, B, out=None, alpha=1.0, beta=0.0, b_k_contiguous=False, stream=None):
    """out = alpha * A @ B + beta * out.  A: (M, K) row-major; B: (K, N) row-major, or (N, K)
    row-major with b_k_contiguous=True.  bf16 / fp8 inputs give a bf16 result, fp16 gives fp16."""
    a_dtype, device = A.dtype, A.device
    dtype = _DTYPES.get(a_dtype)
    if dtype is None or B.dtype != a_dtype:
        raise TypeError("matmul takes two tensors of one dtype out of %s" % sorted(str(d) for d in _DTYPES))
    if A.dim() != 2 or B.dim() != 2 or not A.is_cuda or not B.is_cuda or device != B.device:
        raise ValueError("matmul takes two 2-D tensors on one GPU")
    (lda, a_step), (ldb, b_step) = A.stride(), B.stride()
    if a_step != 1 or b_step != 1:
        raise ValueError("rows of A and B must be contiguous (leading dimensions are free)")
    M, K = A.shape
    N, K_b = B.shape if b_k_contiguous else B.shape[::-1]
    if K_b != K:
        raise ValueError("inner dimensions differ")
    out_dtype = torch.float16 if dtype == g.GEMM_FP16 else torch.bfloat16
    if out is None:
        if beta != 0.0:
            raise ValueError("beta != 0 needs out")
        # rows of C start on 16-byte boundaries: a ragged N gets a padded row stride (the result is a view)
        ldc = -(-N // 8) * 8
        out = torch.empty((M, ldc), dtype=out_dtype, device=device)
        if ldc != N:
            out = out[:, :N]
    else:
        if out.shape != (M, N) or out.dtype != out_dtype or out.stride(1) != 1 or out.device != device:
            raise ValueError("out must be a (%d, %d) %s tensor with contiguous rows" % (M, N, out_dtype))
        ldc = out.stride(0)
    layout = g.GEMM_B_K_CONTIGUOUS if b_k_contiguous else g.GEMM_B_ROW_MAJOR
    plan = _plan(select(M, N, K, dtype, layout), (M, N, K, dtype, layout, lda, ldb, ldc))
    cfg_ref = plan.ref
    if alpha != 1.0 or beta != 0.0:
        cfg = plan.cfg.copy()
        cfg.alpha, cfg.beta = alpha, beta
        cfg_ref = ctypes.byref(cfg)
    if torch.cuda.current_device() == device.index:
        _launch(plan.need, cfg_ref, A, B, out, device, stream)
    else:
        with torch.cuda.device(device):
            _launch(plan.need, cfg_ref, A, B, out, device, stream)
    return out


def _launch(need, cfg_ref, A, B, out, device, stream):
    """gemm_run with the tensors' device current: no error paths, no Python objects made per argument."""
    if need:
        _ensure_workspace(need, device)
    stream = g.current_stream_handle(device.index) if stream is None else g._stream_handle(stream)
    g._check(g._lib.gemm_run(cfg_ref, A.data_ptr(), B.data_ptr(), out.data_ptr(), stream), "gemm_run")
