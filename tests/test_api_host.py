"""Argument checks of api.matmul that need no GPU, the sweep tool's summary of its own records, and the
calibration tool's reading of the variant table."""
import ctypes
import json
import subprocess
import threading
import time

import pytest
import torch


def test_matmul_rejects_what_it_cannot_run_before_touching_the_gpu():
    from paper_2512_04226_amd import api, binding as g
    a = torch.zeros((8, 16), dtype=torch.bfloat16)
    b = torch.zeros((16, 8), dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        api.matmul(a, b)                                   # CPU tensors
    with pytest.raises(TypeError):
        api.matmul(a.float(), b.float())                   # unsupported dtype
    with pytest.raises(TypeError):
        api.matmul(a, b.to(torch.float16))                 # mixed dtypes
    # the memoised pick is the selector's pick, for both layouts
    for layout in (g.GEMM_B_ROW_MAJOR, g.GEMM_B_K_CONTIGUOUS):
        c = api.select(300, 520, 72, g.GEMM_BF16, layout)
        ref = g.gemm_select_ex(300, 520, 72, g.GEMM_BF16, layout)
        assert bytes(c) == bytes(ref) and api.select(300, 520, 72, g.GEMM_BF16, layout) is c


def test_alpha_and_beta_are_taken_and_refused_by_the_cfg_field():
    """A number that equals the default without being a real one is still refused; one that converts is still taken."""
    from fractions import Fraction

    from paper_2512_04226_amd import api, binding as g
    plan = api._Plan(api.select(64, 64, 64, g.GEMM_BF16), 64, 64, 64)
    assert plan.ref_for(1.0, 0.0) is plan.ref and plan.ref_for(1, 0) is plan.ref
    for alpha, beta in ((1 + 0j, 0.0), (1.0, 0j), ("1", 0.0), (None, 0.0)):
        with pytest.raises(TypeError):
            plan.ref_for(alpha, beta)
    for alpha, beta in ((0.5, 0.0), (1.0, 2.0), (Fraction(1, 2), 0), (torch.tensor(0.5), torch.tensor(2.0)), (float("nan"), 0.0)):
        cfg = plan.ref_for(alpha, beta)._obj
        assert cfg is not plan.cfg and (cfg.alpha == float(alpha) or alpha != alpha) and cfg.beta == float(beta)
    assert (plan.cfg.alpha, plan.cfg.beta) == (1.0, 0.0)


def test_sweep_summary_of_records(tmp_path, capsys):
    from paper_2512_04226_amd import sweep
    rec = {"M": 64, "N": 128, "K": 256, "dtype": 0, "b_layout": 0, "n_cfgs": 3,
           "best": {"idx": 1, "cfg": "64x64x64 w2x4 mfma16 s3 split1 g8", "us": 4.0, "pred_us": 4.2},
           "pick": "64x64x64 w2x4 mfma16 s3 streamk256 g8", "pick_us": 5.0, "pick_pred_us": 4.1, "efficiency": 0.8,
           "best_tflops": 1.0, "pick_tflops": 0.8, "bottleneck": "launch", "top5": []}
    grp = {"set": "two groups", "groups": 2, "rows": [3, 4], "dtype": 0, "b_layout": 0,
           "best": {"idx": 0, "cfg": "64x64x64 w2x4 mfma16 s3 split1 g8 groups2", "us": 2.0, "pred_us": 2.0},
           "pick": "64x64x64 w2x4 mfma16 s3 split1 g8 groups2", "pick_us": 2.0, "pick_pred_us": 2.0, "efficiency": 1.0,
           "pick_tflops": 3.0, "best_tflops": 3.0, "separate_launches_us": 5.0, "top5": []}
    p1, p2 = tmp_path / "a_0.jsonl", tmp_path / "grouped.jsonl"
    p1.write_text(json.dumps(rec) + "\n")
    p2.write_text(json.dumps(grp) + "\n")
    sweep.summarize([str(p1), str(p2)])
    out = capsys.readouterr().out
    assert "a_0.jsonl" in out and "median 0.800" in out and "Stream-K picked 1, sweep-best 0" in out
    assert "grouped.jsonl (grouped)" in out and "two groups" in out and "separate launches" in out


def test_variant_table_loop_form_columns_cover_every_compiled_variant():
    """calibrate.py reprints the variant table and must carry the two K-loop-form columns over: its
    parser has to find one row per compiled variant, in table order, with a known form."""
    from paper_2512_04226_amd import binding as g, calibrate

    forms = calibrate.table_loop_forms()
    for sect, dtype in (("BF16", g.GEMM_BF16), ("FP8", g.GEMM_FP8_E4M3)):
        rows = [k for k in forms if k[0] == sect]
        assert len(rows) == g.gemm_variant_count(dtype)
        seen = set()
        for idx in range(g.gemm_cfg_count(dtype)):
            c = g.gemm_cfg_at(idx, 8192, 8192, 8192, dtype)
            if c is not None:
                seen.add((sect, c.block_m, c.block_n, c.block_k, c.waves_m, c.waves_n, c.mfma, c.stages))
        assert seen == set(rows)
    assert all(lf in range(7) and lf_kc in range(7) for lf, lf_kc in forms.values())


class _Recorder:
    """Stands in for the library: remembers (stream, workspace range, thread, times) of every launch with a workspace."""

    def __init__(self, seconds=0.0):
        self.calls, self.seconds = [], seconds

    def gemm_run_ws(self, cfg, a, b, c, stream, ws, nbytes):
        t0 = time.monotonic()
        time.sleep(self.seconds)
        self.calls.append((stream, ws, nbytes, threading.get_ident(), t0, time.monotonic()))
        return 0


class _Buffer:
    def data_ptr(self):
        return 4096


@pytest.fixture
def launcher(monkeypatch):
    """launch(need, stream handle) -> (address, bytes) of the workspace it got; no GPU involved."""
    from paper_2512_04226_amd import api, binding as g
    rec, state = _Recorder(), {"capturing": False, "current": 0}

    class Stream:
        def __init__(self, handle):
            self.handle = handle

        def __enter__(self):
            self.before, state["current"] = state["current"], self.handle

        def __exit__(self, *exc):
            state["current"] = self.before

    allocated_on = {}
    empty = torch.empty

    def on_cpu(*args, device, **kw):
        t = empty(*args, **kw)
        allocated_on[t.data_ptr()] = state["current"]
        return t

    monkeypatch.setattr(api, "_workspaces", type(api._workspaces)())
    monkeypatch.setattr(api, "_pinned", [])
    monkeypatch.setattr(torch, "empty", on_cpu)
    monkeypatch.setattr(g, "_lib", rec)
    monkeypatch.setattr(g, "current_stream_handle", lambda index: state["current"])
    monkeypatch.setattr(torch.cuda, "stream", lambda s: s)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device: Stream(handle))
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device: Stream(0))
    monkeypatch.setattr(g, "gemm_stream_capturing", lambda handle: state["capturing"])

    def launch(need, stream=None):
        x = _Buffer()
        api._launch(need, None, x, x, x, torch.device("cuda", 0), stream)
        handle, ws, nbytes = rec.calls[-1][:3]
        assert nbytes >= need and ws % 16 == 0 and allocated_on[ws] == handle
        return ws, nbytes

    launch.rec, launch.state, launch.api = rec, state, api
    return launch


def test_every_stream_has_a_workspace_of_its_own(launcher):
    """Two K-split calls in flight on two streams must not share their partial sums' buffer, whether the stream is torch's
    current one or an argument; calls of one stream reuse its buffer; an outgrown one is replaced on its own stream."""
    a, b, c = launcher(1000), launcher(1000, 77), launcher(1000, 78)
    assert len({a[0], b[0], c[0]}) == 3
    assert launcher(900) == a and launcher(1000, 77) == b
    launcher.state["current"] = 77
    assert launcher(10) == b and launcher(10, 0) == a
    assert launcher(5000, 78)[1] >= 5000 and launcher(1000, 78)[1] >= 5000 and launcher(1000) == b
    for handle in range(100, 200):                                     # bounded
        launcher(16, handle)
    assert len(launcher.api._workspaces) <= launcher.api._MAX_WORKSPACES


def test_a_workspace_that_a_capture_has_seen_is_kept(launcher):
    """Replays write to the address that was captured, whatever later calls need."""
    launcher.state["capturing"] = True
    a = launcher(1000, 77)
    launcher.state["capturing"] = False
    b = launcher(1200, 77)
    assert b[0] != a[0] and b[1] >= 2000 and [t.data_ptr() for t in launcher.api._pinned] == [a[0]]
    launcher.state["capturing"] = True
    c = launcher(1200, 78)
    launcher.state["capturing"] = False
    for handle in range(100, 200):
        launcher(16, handle)
    assert launcher(1200, 78) == c


def test_threads_do_not_interleave_their_launches(launcher):
    """A call with a workspace is two kernels on one stream: another thread's must not come between them."""
    launcher.rec.seconds = 0.005
    threads = [threading.Thread(target=lambda: [launcher.api._launch(64, None, _Buffer(), _Buffer(), _Buffer(), torch.device("cuda", 0), h)
                                                for h in (0, 77, 2)]) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    calls = sorted(launcher.rec.calls, key=lambda c: c[4])
    assert len(calls) == 12 and all(x[5] <= y[4] for x, y in zip(calls, calls[1:]))
    # handle 2 is the per-thread default stream: one buffer per thread
    assert len({c[1] for c in calls if c[0] == 2}) == len({c[3] for c in calls})
    assert len({c[1] for c in calls if c[0] == 77}) == 1


def test_a_second_build_of_the_library_gets_whole_pointers(tmp_path, monkeypatch):
    """The calibration tool runs other builds of the library through handles of its own.  A stand-in built here hands back
    the arguments its gemm_run received: addresses above 32 bits have to arrive whole."""
    from paper_2512_04226_amd import binding as g, calibrate

    src, lib = tmp_path / "echo.c", tmp_path / "echo.so"
    src.write_text("#include <stdint.h>\nuintptr_t seen[4];\n"
                   "int gemm_run(const void *cfg, void *a, void *b, void *c, void *s)\n"
                   "{ seen[0] = (uintptr_t)a; seen[1] = (uintptr_t)b; seen[2] = (uintptr_t)c; seen[3] = (uintptr_t)s; return cfg == 0; }\n")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)

    class Tensor:
        def __init__(self, address):
            self.data_ptr = lambda: address

    addresses = (0x7F1234567890, 0x7F12F4567890, 0x8000000000)
    monkeypatch.setattr(g, "_stream_handle", lambda stream: 0x55AA12345678)
    handle = g.open_library(str(lib))
    calibrate.run_in(handle, g.gemm_cfg(), *(Tensor(a) for a in addresses))
    assert tuple((ctypes.c_size_t * 4).in_dll(handle, "seen")) == addresses + (0x55AA12345678,)
    # and the tool opens its libraries in no other way
    assert "CDLL" not in open(calibrate.__file__).read()


@pytest.fixture
def timed(monkeypatch):
    """The cfgs that the calibration and the sweep hand to their timing functions; nothing is launched."""
    from paper_2512_04226_amd import binding as g, calibrate, sweep
    cfgs = []

    class Event:
        def __init__(self, **kw):
            pass

        record = synchronize = lambda self: None
        elapsed_time = lambda self, other: 1.0

    def note(cfg, *args, **kw):
        cfgs.append(cfg.copy())
        return 1.0 + len(cfgs) % 7

    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(g, "open_library", lambda path: path)
    monkeypatch.setattr(calibrate, "run_in", lambda lib, cfg, *args: note(cfg))
    for tool in (calibrate, sweep):
        monkeypatch.setattr(tool, "make_operands", lambda *a, **kw: tuple(torch.zeros(2, 2) for _ in range(3)))
    monkeypatch.setattr(calibrate, "_time_plain", note)
    monkeypatch.setattr(calibrate.Workspace, "ensure", lambda self, cfg: None)
    monkeypatch.setattr(sweep, "time_cfg", note)
    return cfgs


def _runs_its_own(g, cfg):
    return (cfg.stream_k or g.gemm_launched_tile(cfg) == (cfg.block_m, cfg.block_n, cfg.split_k)) and not g.gemm_launched_kernel(cfg)[0].startswith("sliced")


def test_calibration_times_the_kernels_that_the_cfgs_name(timed, capsys):
    """At 4096^3 and 8192^3 gemm_run runs the pipelined 256x256 tile in place of a third of the variants; a slab cost divided by
    another tile's count says nothing about either."""
    from paper_2512_04226_amd import binding as g, calibrate
    rows = sum((calibrate.measure_slab_clk(dt, n, bl, passes=1) for dt in (g.GEMM_BF16, g.GEMM_FP8_E4M3) for n in (4096, 8192) for bl in (0, 1)), [])
    assert len(rows) == len(timed) and len({id(r[0]) for r in rows}) == len(rows) > 200
    calibrate.compare_loop_forms(["a", "b"], passes=1)
    calibrate.decompose(list("abcd"))
    calibrate.compare_builds(["n=a"])
    assert all(_runs_its_own(g, c) for c in timed)
    # (and by themselves some would not)
    plain = [c.copy() for c in timed]
    for c in plain:
        c.own_tile = 0
    assert not all(_runs_its_own(g, c) for c in plain)


@pytest.mark.parametrize("shape,replaced", [((1152, 2240, 11696), True), ((40, 64, 8192), True), ((2304, 5120, 512), False)])
def test_sweep_times_entries_as_named_and_the_pick_as_launched(timed, shape, replaced):
    from paper_2512_04226_amd import binding as g, sweep
    rec, rows = sweep.sweep_shape(*shape, g.GEMM_BF16, None, b_layout=1)
    assert len(rows) == rec["n_cfgs"] > 50 and all(_runs_its_own(g, c) for c in timed[:len(rows)])
    pick = g.gemm_select_ex(*shape, g.GEMM_BF16, 1)
    assert rec["pick"] == pick.describe() and rec["pick_launched"] == list(g.gemm_launched_tile(pick))
    assert replaced == (not _runs_its_own(g, pick))
    as_launched = [c for c in timed[len(rows):] if not c.own_tile]
    assert len(as_launched) == (3 if replaced else 0) and all(c.describe() == pick.describe() for c in as_launched)


def test_uniform128_shapes_follow_the_papers_recipe():
    """Section V-A: dimensions are multiples of 128 up to 8192; the sample is seeded."""
    from paper_2512_04226_amd import workloads as wl

    s = wl.uniform128_shapes()
    assert len(s) == 192 and s == wl.uniform128_shapes()
    assert all(d % 128 == 0 and 128 <= d <= 8192 for shape in s for d in shape)
    assert len({d for shape in s for d in shape}) > 48          # spread over the 64 possible values


def test_the_short_ways_plan_keeps_the_cfg_whose_address_it_gives(monkeypatch):
    """Another thread that empties the plans while one is handed over must not free it: the cfg is part of the result."""
    from paper_2512_04226_amd import api, binding as g
    monkeypatch.setattr(api, "_plans", {})
    given = api._fast_plan(96, 64, 128, g.GEMM_BF16, 0, 128, 64, 64)
    api._plans.clear()
    kept = [x for x in given if isinstance(x, g.gemm_cfg) and ctypes.addressof(x) in given]
    assert len(kept) == 1 and kept[0].ldc == 64 and kept[0].M == 96
