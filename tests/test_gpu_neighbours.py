"""A launch's speed beside other work and under another descriptor: the tiles of a launch go to whatever CUs are free, and a
replaced hardware table (a study of the selector) does not shrink the launch.  Ratios of times with wide margins."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _fp8(g, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(5)
    ops = [torch.randn(s, device="cuda", generator=gen).to(torch.float8_e4m3fn) for s in ((M, K), (K, N))]
    cfg = g.gemm_select(M, N, K, g.GEMM_FP8_E4M3)
    assert cfg.split_k == 1 and not cfg.stream_k
    return cfg, ops[0], ops[1], torch.empty((M, N), dtype=torch.bfloat16, device="cuda")


def _us(fn, launches=3):
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(launches):
        fn()
    e1.record()
    return lambda: e0.elapsed_time(e1) * 1e3 / launches


def _bf16(g, M, N, K, block_m, block_n, kind):
    cfg = next(c for c in (g.gemm_cfg_at_ex(i, M, N, K, g.GEMM_BF16, 1) for i in range(0, g.gemm_cfg_count(g.GEMM_BF16), 7))
               if c is not None and (c.block_m, c.block_n, c.block_k) == (block_m, block_n, 64))
    assert g.gemm_launched_kernel(cfg)[0] == kind
    gen = torch.Generator(device="cuda").manual_seed(6)
    A, B = (torch.randn(s, device="cuda", generator=gen).bfloat16() for s in ((M, K), (N, K)))
    return cfg, A, B, torch.empty((M, N), dtype=torch.bfloat16, device="cuda")


# fp8: 1024 tiles on 256 CUs, eight of them held: five rounds instead of four (1.25) at most where the dispatcher deals the
# tiles one by one; a fixed share of the tiles per workgroup makes it 2.
# Chained: four tiles per workgroup and four such shares per CU, five with eight CUs held (measured 1.19 to 1.28); two shares of eight
# tiles measured 1.38 and 1.43.  64x64 tiles with 1.25 and 2 per slot: all dealt out at the start, five on a CU.
@pytest.mark.parametrize("what,bound", [("fp8", 1.45), ("chained 256x256", 1.36), ("chained 64x64, 1.25 rounds", 1.4), ("chained 64x64, 2 rounds", 1.4)])
def test_a_kernel_that_holds_a_few_cus_costs_a_launch_little(what, bound):
    from paper_2512_04226_amd import binding as g
    work = (_fp8(g, 8192, 8192, 2048) if what == "fp8" else _bf16(g, 32768, 8192, 512, 256, 256, "chained") if "256" in what
            else _bf16(g, 3200 if "1.25" in what else 5120, 2048, 192, 64, 64, "chained"))
    launches = 20 if "64x64" in what else 3
    M, N, K = 256, 2048, 65536                    # eight 256x256 tiles of a thousand K slabs each: some milliseconds
    hold = next(c for c in (g.gemm_cfg_at(i, M, N, K, g.GEMM_BF16) for i in range(g.gemm_cfg_count(g.GEMM_BF16)))
                if c is not None and (c.block_m, c.block_n, c.block_k, c.split_k, c.stream_k) == (256, 256, 64, 1, 0))
    A, B = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((M, K), (K, N)))
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    alone, beside = [], []
    for _ in range(12):
        g.gemm_run(*work)

    def held_by(other):
        """One sample beside a holder on `other`, or None where the holder ended first."""
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(2):
                g.gemm_run(hold, A, B, C)
            held = torch.cuda.Event(enable_timing=True)
            held.record()
        g.gemm_run(*work)                         # (the holder has started when this one is done)
        end = torch.cuda.Event(enable_timing=True)
        sample = _us(lambda: g.gemm_run(*work), launches)
        end.record()
        torch.cuda.synchronize()
        return sample if end.elapsed_time(held) > 0 else None

    # (torch deals its streams onto a few hardware queues; one that shares the current stream's queue runs after it, not beside)
    other = next(s for s in (torch.cuda.Stream() for _ in range(8)) if held_by(s) is not None)
    for _ in range(7):
        torch.cuda.synchronize()
        alone.append(_us(lambda: g.gemm_run(*work), launches))
        sample = held_by(other)
        if sample is not None:
            beside.append(sample)
    assert len(beside) >= 3
    alone, beside = (sorted(f() for f in x)[len(x) // 2] for x in (alone, beside))
    print("%s: alone %.1f us, beside %.1f us" % (what, alone, beside))
    assert beside <= bound * alone, (alone, beside)


def test_a_replaced_descriptor_does_not_shrink_the_launch():
    from paper_2512_04226_amd import binding as g
    work = _fp8(g, 4096, 8192, 2048)
    small = g.gemm_hw_get()
    small.n_cu = 32
    times = {}
    for _ in range(5):
        for name in ("own", "small"):
            if name == "small":
                g.gemm_hw_set(small)
            try:
                g.gemm_run(*work)
                times.setdefault(name, []).append(_us(lambda: g.gemm_run(*work)))
                torch.cuda.synchronize()
            finally:
                g.gemm_hw_reset()
    own, shrunk = (sorted(f() for f in times[n])[2] for n in ("own", "small"))
    print("own table %.1f us, table of 32 CUs %.1f us" % (own, shrunk))
    assert shrunk <= 1.5 * own, (own, shrunk)
