"""The compiled short way of `api.matmul` against the general one.  (In a file of its own: torch deals its streams
round-robin onto four hardware queues, so a stream created before the tests of launches beside another stream
can put those two on one queue.)"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_the_short_way_of_matmul_gives_what_the_general_way_gives():
    """Every form the short way accepts, against the general way bit for bit; every form it has to leave alone."""
    from paper_2512_04226_amd import api, binding as g
    gen = torch.Generator(device="cuda").manual_seed(8)

    def operand(r, c, dtype, pad=0):
        per16 = 16 if dtype == torch.float8_e4m3fn else 8
        return torch.randn((r, -(-c // per16) * per16 + pad), device="cuda", generator=gen).to(dtype)[:, :c]

    for dtype in (torch.bfloat16, torch.float16, torch.float8_e4m3fn):
        for M, N, K, pad in ((96, 256, 128, 0), (1, 64, 64, 16), (33, 77, 101, 0), (50, 136, 64, 32)):
            for kc in (False, True):
                A, B = operand(M, K, dtype, pad), operand(*((N, K) if kc else (K, N)), dtype, pad)
                out_dtype = torch.float16 if dtype == torch.float16 else torch.bfloat16
                for alpha, beta, own in ((1.0, 0.0, False), (0.5, 0.0, False), (0.25, 0.0, True), (1.0, 0.5, True)):
                    cin = torch.randn((M, -(-N // 8) * 8 + pad), device="cuda", generator=gen).to(out_dtype)
                    outs = [cin.clone()[:, :N] if own else None for _ in range(2)]
                    short = api._fastcall.matmul(A, B, outs[0], alpha, beta, kc, None)
                    assert (short is not None) == (api.select(M, N, K, api._DTYPES[dtype], int(kc)).split_k == 1)
                    if short is None:
                        continue
                    want = api._matmul_general(A, B, outs[1], alpha, beta, kc, None)
                    assert short.dtype == want.dtype and short.shape == want.shape and short.stride() == want.stride()
                    assert torch.equal(short.view(torch.int16), want.view(torch.int16))
                    assert (short is outs[0]) == own and (short._is_view() == want._is_view())
    A, B = operand(64, 64, torch.bfloat16), operand(64, 64, torch.bfloat16)
    alike = (A, B, None, 1.0, 0.0, False, None)
    assert api._fastcall.matmul(*alike) is not None

    class Sub(torch.Tensor):
        pass

    for i, other in ((0, A.as_subclass(Sub)), (0, A.float()), (0, A.cpu()), (0, A[0]), (0, A.t()), (0, operand(64, 72, torch.bfloat16)),
                     (2, torch.empty(64, 65, dtype=torch.bfloat16, device="cuda")), (2, torch.empty(64, 64, device="cuda")), (3, 1), (3, np.float64(1)),
                     (3, 1j), (4, 0.5), (4, 0), (5, 1), (6, torch.cuda.current_stream())):
        assert api._fastcall.matmul(*(alike[:i] + (other,) + alike[i + 1:])) is None, (i, type(other))
    with torch.device("cuda"):         # a function mode
        assert api._fastcall.matmul(*alike) is None
    torch.func.vmap(lambda x: (torch.testing.assert_close(api._fastcall.matmul(x, B, None, 1.0, 0.0, False, None), None), x)[1])(A.expand(2, 64, 64).clone())
    # a memo that was emptied: the next call asks for the pick again
    base = api.select(64, 64, 64, g.GEMM_BF16)
    api._cfg_cache.clear()
    assert api._fastcall.matmul(*alike) is not None and api.select(64, 64, 64, g.GEMM_BF16) is not base
    # launches go to the current stream of the tensors' device
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        C = api.matmul(A, B)
    C.zero_()
    graph.replay()
    assert torch.equal(C, api.matmul(A, B))


def test_a_trace_sees_the_short_ways_allocation():
    """A trace records where the result comes from, as it does on the general way; allocated behind its back, the first call's
    result would stand in the traced program as a constant."""
    from paper_2512_04226_amd import api
    A, B = (torch.randn(64, 64, device="cuda").bfloat16() for _ in range(2))
    graphs = []
    for way in (lambda a, b: api._fastcall.matmul(a, b, None, 1.0, 0.0, False, None), lambda a, b: api._matmul_general(a, b, None, 1.0, 0.0, False, None)):
        traced = torch.jit.trace(lambda a, b: way(a, b) + 1, (A, B), check_trace=False)
        graphs.append([n.kind() for n in traced.graph.nodes() if n.kind() in ("aten::empty", "aten::add")])
    assert graphs[0] == graphs[1] == ["aten::empty", "aten::add"]
    assert torch.equal(api._fastcall.matmul(A, B, None, 1.0, 0.0, False, None), api._matmul_general(A, B, None, 1.0, 0.0, False, None))


def _operands(M, N, K):
    return tuple(torch.randn(s, device="cuda").bfloat16() for s in ((M, K), (K, N)))


@pytest.mark.parametrize("error", [KeyboardInterrupt, TimeoutError])
def test_what_a_signal_raises_while_a_plan_is_made_is_not_lost(error, monkeypatch):
    """The plan of a new shape is made by Python code, where a signal's handler may raise: whatever the kind, once."""
    from paper_2512_04226_amd import api
    A, B = _operands(40 if error is KeyboardInterrupt else 41, 72, 48)      # (a shape that has no plan yet)
    once, select = [error("a handler's")], api.select
    monkeypatch.setattr(api, "select", lambda *key: select(*key) if not once else (_ for _ in ()).throw(once.pop()))
    with pytest.raises(error):
        api.matmul(A, B)
    assert api._fastcall.matmul(A, B, None, 1.0, 0.0, False, None) is not None


def test_a_plan_made_twice_at_once_keeps_no_reference_of_the_first(monkeypatch):
    """A call that comes in while the same shape's plan is being made (another thread's, or one from a finaliser)."""
    import weakref
    from paper_2512_04226_amd import api
    A, B = _operands(56, 88, 64)
    first, select = [True], api.select

    def interrupted(*key):
        if first:
            first.clear()
            assert api._fastcall.matmul(A, B, None, 1.0, 0.0, False, None) is not None
        return select(*key)
    monkeypatch.setattr(api, "select", interrupted)
    api.matmul(A, B)
    pick = weakref.ref(select(56, 88, 64, 0))
    assert pick() is not None
    api._cfg_cache.clear()
    api._plans.clear()
    api.matmul(A, B)                   # (meets the emptied memo and drops what it held of the old pick)
    assert pick() is None


def test_other_threads_run_while_a_result_is_allocated():
    """The result's memory comes from cached blocks that have to be given back first, which waits for the device: half a
    second of work, during which a Python thread has to go on counting."""
    import threading
    import time
    from paper_2512_04226_amd import api
    M, N = 76800, 4096                 # 600 MB
    A, B = _operands(M, N, 16)
    assert api.select(M, N, 16, 0).split_k == 1
    api.matmul(A[:128], B)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    torch.cuda._sleep(1000000)
    e1.record()
    e1.synchronize()
    cycles = int(500.0 / e0.elapsed_time(e1) * 1000000)
    blocks = [torch.empty(512 << 20, dtype=torch.uint8, device="cuda") for _ in range(2)]
    del blocks
    total = torch.cuda.get_device_properties(0).total_memory
    gaps, stop = [], threading.Event()

    def count():
        last = time.perf_counter()
        while not stop.is_set():
            time.sleep(0.001)
            now = time.perf_counter()
            gaps.append(now - last)
            last = now
    thread = threading.Thread(target=count)
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        torch.cuda._sleep(cycles)
        thread.start()
        t0 = time.perf_counter()
        out = api.matmul(A, B)
        took = time.perf_counter() - t0
    finally:
        stop.set()
        thread.join()
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    assert out.shape == (M, N)
    print("the call took %.3f s, the thread waited %.3f s at most" % (took, max(gaps)))
    if took < 0.05:
        pytest.skip("the allocator did not wait for the device")
    assert max(gaps) < 0.5 * took, (max(gaps), took)
