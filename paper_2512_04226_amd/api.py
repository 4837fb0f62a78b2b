"""`matmul`: the call a user of the paper's library makes -- hand over two tensors, get the product,
with the kernel chosen analytically for the shape (Section V-C: selection costs microseconds and
is cached per shape, no tuning run).  A thin convenience layer over `binding`: it looks up or
makes the cfg, keeps one workspace tensor per stream and launches; every step of the computation
runs in libgemm355.so.  A call whose plan is known and needs no workspace goes the short way of a
compiled extension; all others, mistakes included, the general way below, and every call where the
extension is not built for this torch and Python (a warning says so; a call then takes some 3 us
more of host time).  Calls on several streams and from several threads need no order among
themselves.  (Graphs captured on one stream share its workspace: replays of two of them are to
be ordered.)

    C = matmul(A, B)                       # A (M, K), B (K, N): bf16, fp16 or float8_e4m3fn
    C = matmul(X, W, b_k_contiguous=True)  # W stored (N, K), as an nn.Linear weight
"""
import collections
import ctypes
import threading
import warnings

import torch

from . import binding as g     # (first: it says how to build what is missing)

try:
    from . import _fastcall
    if _fastcall.torch_version != torch.__version__:
        raise ImportError("built for torch %s, this is %s" % (_fastcall.torch_version, torch.__version__))
except (ImportError, AttributeError) as e:
    _fastcall = None
    warnings.warn("no compiled short way of matmul, run `python -m paper_2512_04226_amd.build`: %s" % e, RuntimeWarning)

_DTYPES = {torch.bfloat16: g.GEMM_BF16, torch.float16: g.GEMM_FP16}
if hasattr(torch, "float8_e4m3fn"):
    _DTYPES[torch.float8_e4m3fn] = g.GEMM_FP8_E4M3

_REAL = (float, int)
_cfg_cache = {}       # (M, N, K, dtype, b_layout) -> cfg; the selector is deterministic, so this is exact
_workspaces = collections.OrderedDict()     # (device index, stream handle, thread) -> _Workspace, least recently used first
_MAX_WORKSPACES = 32  # torch hands out 32 pooled streams per device; beyond that the oldest that no graph holds goes
_pinned = []          # outgrown buffers whose addresses captured graphs may hold
_workspace_lock = threading.RLock()    # (re-entered only by a finaliser that multiplies)
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

    def ref_for(self, alpha, beta):
        # (the fast way only for real numbers: whatever else equals 1 is for the field's own conversion to take or refuse)
        if type(alpha) in _REAL and type(beta) in _REAL and alpha == 1.0 and beta == 0.0:
            return self.ref
        cfg = self.cfg.copy()
        cfg.alpha, cfg.beta = alpha, beta
        return ctypes.byref(cfg)


def _plan(base, key):
    plan = _plans.get(key)
    if plan is None or plan.base is not base:      # (another base: the memo of picks was emptied since)
        if len(_plans) >= _MAX_PLANS:
            _plans.clear()
        plan = _plans[key] = _Plan(base, *key[5:])
    return plan


class _Workspace:
    """A buffer of one stream.  `pinned`: a graph may have been captured with its address."""
    __slots__ = ("tensor", "address", "nbytes", "pinned")

    def __init__(self, tensor):
        self.tensor, self.address, self.nbytes, self.pinned = tensor, tensor.data_ptr(), tensor.numel() * 4, False


def _allocate(nbytes, device, stream):
    """Device memory that the allocator knows as the stream's: once it is given up, only later work of the same stream gets
    it, so that nothing has to be waited for."""
    if stream == g.current_stream_handle(device.index):
        return torch.empty((nbytes + 15) // 16 * 4, dtype=torch.float32, device=device)
    with torch.cuda.stream(torch.cuda.ExternalStream(stream, device) if stream else torch.cuda.default_stream(device)):
        return torch.empty((nbytes + 15) // 16 * 4, dtype=torch.float32, device=device)


def _workspace_for(need, device, stream):
    """The stream's workspace of at least `need` bytes (with _workspace_lock held).  A buffer that a capture has seen is never
    given up, as replays write to it; it is replaced by one of at least twice its size, so that a stream holds at most twice
    what its largest call needs."""
    # handle 2 is the per-thread default stream: another stream in every thread
    key = (device.index, stream, threading.get_ident() if stream == 2 else 0)
    ws = _workspaces.get(key)
    if ws is None or ws.nbytes < need:
        if ws is not None and ws.pinned:
            _pinned.append(ws.tensor)
            need = max(need, 2 * ws.nbytes)
        ws = _workspaces[key] = _Workspace(_allocate(need, device, stream))
        if len(_workspaces) > _MAX_WORKSPACES:
            for old in [k for k, w in _workspaces.items() if not w.pinned and k != key][:1]:
                del _workspaces[old]
    else:
        _workspaces.move_to_end(key)
    if not ws.pinned and g.gemm_stream_capturing(stream):
        ws.pinned = True
    return ws


def matmul(A, B, out=None, alpha=1.0, beta=0.0, b_k_contiguous=False, stream=None):
    """out = alpha * A @ B + beta * out.  A: (M, K) row-major; B: (K, N) row-major, or (N, K)
    row-major with b_k_contiguous=True.  bf16 / fp8 inputs give a bf16 result, fp16 gives fp16."""
    if stream is None:
        result = _short_way(A, B, out, alpha, beta, b_k_contiguous, stream)
        if result is not None:
            return result
    return _matmul_general(A, B, out, alpha, beta, b_k_contiguous, stream)


def _fast_plan(*key):
    """For the short way: the pick, its key in the memo, the plan's cfg, that cfg's address and its workspace size.  (The cfg
    itself, as another thread may empty the plans before its address is used.)"""
    base = select(*key[:5])
    plan = _plan(base, key)
    return base, key[:5], plan.cfg, ctypes.addressof(plan.cfg), plan.need


if _fastcall is not None:
    _short_way = _fastcall.matmul
    _fastcall.init(ctypes.cast(g._lib.gemm_run, ctypes.c_void_p).value, ctypes.sizeof(g.gemm_cfg), _fast_plan, g._check, globals())
else:
    def _short_way(*call):
        return None


def _matmul_general(A, B, out, alpha, beta, b_k_contiguous, stream):
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
    if type(alpha) is float and alpha == 1.0 and type(beta) is float and beta == 0.0:
        cfg_ref = plan.ref
    else:
        cfg_ref = plan.ref_for(alpha, beta)
    if torch.cuda.current_device() == device.index:
        _launch(plan.need, cfg_ref, A, B, out, device, stream)
    else:
        with torch.cuda.device(device):
            _launch(plan.need, cfg_ref, A, B, out, device, stream)
    return out


def _launch(need, cfg_ref, A, B, out, device, stream):
    """One launch with the tensors' device current: no Python objects made per argument."""
    stream = g.current_stream_handle(device.index) if stream is None else g._stream_handle(stream)
    if not need:
        g._check(g._lib.gemm_run(cfg_ref, A.data_ptr(), B.data_ptr(), out.data_ptr(), stream), "gemm_run")
        return
    # a call is two kernels: no other thread may put its own on the stream between them
    with _workspace_lock:
        ws = _workspace_for(need, device, stream)
        g._check(g._lib.gemm_run_ws(cfg_ref, A.data_ptr(), B.data_ptr(), out.data_ptr(), stream, ws.address, ws.nbytes), "gemm_run_ws")
