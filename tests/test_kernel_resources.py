"""Register budget of the compiled kernels (no GPU needed: hipcc cross-compiles and reports resource usage).
The 256x256 tiles sit at the 256-register limit of an eight-wave workgroup, the four-wave ones at 512 with their
accumulators; a change of the K loop's source that costs a few registers shows as scratch (spills inside the loop) long
before any test of results notices."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_04226_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _usage(src, *defines):
    """Rows of a file of the library (or of a path of its own)."""
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", "-o", os.devnull, *defines, os.path.join(CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    rows, cur = [], None
    for line in r.stderr.split("\n"):
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = {"name": m.group(1)}
            rows.append(cur)
        for key, pat in (("vgprs", r"VGPRs: (\d+)"), ("scratch", r"ScratchSize \[bytes/lane\]: (\d+)"),
                         ("waves_per_simd", r"Occupancy \[waves/SIMD\]: (\d+)")):
            m = re.search(pat, line)
            if m and cur is not None:
                cur[key] = int(m.group(1))
    return rows


def _tile(es, bm, bn, bk, wm, wn, mi, ns, bl, ft, rg=0, st=0):
    """Regular expression for the whole-chunk (rg = 1: ragged) instantiation of a tile, whatever K-loop form it has.
    st = 0: the kernel of Stream-K and grouped launches, 3: of launches of one problem (direct)."""
    return "TileI" + "".join("Li%dE" % x for x in (es, bm, bn, bk, wm, wn, mi, ns, bl, ft)) + r"Li\d+ELi%dELi%dEEEEE" % (rg, st)


@pytest.fixture(scope="module")
def usage():
    """Resource rows of the kernels in three files: the 16-bit tiles with the 16x16 instruction, the larger fp8 tiles."""
    if shutil.which(HIPCC) is None and not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    with ThreadPoolExecutor(max_workers=3) as ex:
        return sum(ex.map(_usage, ["kernels_bf16_4.hip", "kernels_fp16_4.hip", "kernels_fp8_0.hip"]), [])


def _find(rows, tag):
    hit = [r for r in rows if re.search(tag, r["name"])]
    assert len(hit) == 1, (tag, [r["name"] for r in hit])
    return hit[0]


def test_ragged_tiles_keep_the_third_workgroup_of_a_cu(usage):
    """Six waves per SIMD: three eight-wave workgroups, which the 48 KB rings of these two tiles leave room for."""
    for bm, bn in ((128, 64), (64, 128)):
        for bl in (0, 1):
            r = _find(usage, _tile(2, bm, bn, 64, 2, 4, 16, 2, bl, 0, rg=1))
            assert r["waves_per_simd"] >= 6 and r["scratch"] <= 16, r


def test_ragged_256_tiles_on_eight_waves_do_not_spill_where_a_form_avoids_it(usage):
    for tile in ((2, 256, 256, 64, 2, 4, 16, 2, 0, 0), (1, 256, 256, 128, 2, 4, 32, 2, 1, 0), (2, 256, 256, 64, 4, 2, 16, 2, 0, 0)):
        r = _find(usage, _tile(*tile, rg=1))
        assert r["scratch"] == 0, r


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="needs hipcc")
def test_headline_kernels_keep_no_spills_and_no_kernel_spills_much(usage):
    rows = usage
    assert len(rows) >= 40
    # The bf16 256x256x64 tile on a 4x2 wave grid (row-major B) and on a 2x4 grid (K-contiguous B), fp8 256x256x128 on
    # four waves: the plain instantiations, which run at 8192^3's extents below twenty K slabs (of Stream-K and grouped
    # launches; the direct ones further down)
    for tag in (_tile(2, 256, 256, 64, 4, 2, 16, 2, 0, 0), _tile(2, 256, 256, 64, 2, 4, 16, 2, 1, 0),
                _tile(1, 256, 256, 128, 2, 2, 32, 2, 0, 0), _tile(1, 256, 256, 128, 2, 2, 32, 2, 1, 0)):
        r = _find(rows, tag)
        assert r["scratch"] == 0, r
    # nothing else in these files spills more than a few registers' worth
    worst = max(rows, key=lambda r: r.get("scratch", 0))
    assert worst.get("scratch", 0) <= 64, worst


def test_pipelined_kernels_have_no_scratch_and_the_spills_of_the_others_are_known(usage):
    """The four-wave kernels of the 256x256 tiles (K-loop form 7; what grouped launches of 8192^3's extents run, its own
    direct ones further down) hide nothing: no scratch, plain and ragged, both storages of B.  The kernels that do spill are listed, so that another one, or more of it, is noticed."""
    pipelined = [r for r in usage if re.search(r"TileI.*Li7ELi[01]ELi0EEEEE", r["name"])]
    assert len(pipelined) == 12             # {bf16, fp16, fp8} x storage of B x {plain, ragged}
    for r in pipelined:
        assert r["scratch"] == 0, r
    known = {_tile(1, 256, 256, 128, 2, 4, 32, 2, 0, 0, rg=1): 36, _tile(2, 256, 256, 64, 2, 4, 16, 2, 1, 0, rg=1): 20,
             _tile(2, 256, 256, 64, 2, 4, 16, 2, 1, 1, rg=1): 24, _tile(2, 256, 256, 64, 4, 2, 16, 2, 1, 1): 12}
    for ft in (0, 1):
        known[_tile(2, 256, 256, 64, 4, 2, 16, 2, 1, ft, rg=1)] = 12
        known[_tile(2, 64, 128, 64, 2, 4, 16, 2, 0, ft, rg=1)] = 12
        known[_tile(2, 128, 64, 64, 2, 4, 16, 2, 0, ft, rg=1)] = 8
    for r in usage:
        allowed = [b for tag, b in known.items() if re.search(tag, r["name"])]
        assert r.get("scratch", 0) <= (allowed[0] if allowed else 0), r


def test_direct_kernels_keep_no_spills_and_the_third_workgroup(usage):
    """What launches of one problem run: no scratch in any of them (8192^3 runs the pipelined ones, the extents below twenty
    K slabs the plain ones of the other tests), and three eight-wave workgroups on a CU for the two-stage 128x64 and 64x128
    tiles, ragged and with row-major B whole."""
    direct = [r for r in usage if re.search(r"11gemm_kernelI.*Li[34]EEEEE", r["name"])]
    assert 2 * len(direct) == len([r for r in usage if "11gemm_kernelI" in r["name"]]) >= 80      # each kernel twice
    for r in direct:
        assert r["scratch"] == 0, r
    assert len([r for r in direct if re.search(r"Li7ELi[01]ELi3EEEEE", r["name"])]) == 12         # the pipelined ones
    for ft in (0, 1):
        for bm, bn in ((128, 64), (64, 128)):
            for bl in (0, 1):
                r = _find(usage, _tile(2, bm, bn, 64, 2, 4, 16, 2, bl, ft, rg=1, st=3))
                assert r["waves_per_simd"] >= 6, r
            r = _find(usage, _tile(2, bm, bn, 64, 2, 4, 16, 2, 0, ft, st=3))
            assert r["waves_per_simd"] >= 6, r


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="needs hipcc")
def test_chained_kernels_fill_the_cu_as_their_walk_assumes():
    """The walk of a chained launch counts on as many resident workgroups as the LDS has room for; one has scratch."""
    with ThreadPoolExecutor(max_workers=3) as ex:
        rows = sum(ex.map(_usage, ["chained_bf16.hip", "chained_fp16.hip", "chained_fp8.hip"]), [])
    rows = [r for r in rows if "chained_kernel" in r["name"]]
    assert len(rows) == 77
    for r in rows:
        es, bm, bn, bk, wm, wn, mi, ns = map(int, re.search("TileI" + r"Li(\d+)E" * 8, r["name"]).groups())
        on_a_cu = 160 * 1024 // (ns * (bm + bn) * bk * es)
        assert r["waves_per_simd"] >= on_a_cu * wm * wn // 4, r
        spills = (es, bm, bn) == (1, 256, 256)
        assert r["scratch"] <= (20 if spills else 0), r


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("define", ["-DG355_FORCE_LOOP_FORM=3", "-DG355_DIAG_SKIP_FILL"])
def test_comparison_builds_hold_nothing_that_replaces_a_variant(define):
    """Builds that compare K-loop forms or leave a part of the loop out time the table's variants: were the pipelined tiles and the
    sliced kernel in them, in the forced form, launches would run those instead."""
    for src in ("pipelined_bf16.hip", "sliced_bf16.hip"):
        assert _usage(src, define) == []


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_kernels_that_replace_a_cfgs_keep_no_scratch(tmp_path):
    """Grouped launches of the pipelined 256x256 tiles, whose four loops need registers that a Stream-K part would not leave;
    the streaming tiles of up to 256 rows; the sliced kernel.  (192x256, the largest of the others: with its own tests.)"""
    kinds = {"grouped": ["Tile<%d, 256, 256, %d, 2, 2, %d, 2, %d, 0, 7, %d, 6>" % (es, 128 // es, 16 if es == 2 else 32, bl, rg)
                         for es in (1, 2) for bl in (0, 1) for rg in (0, 1)],
             "streaming": ["Tile<%d, %d, 128, %d, 2, 2, %d, 2, %d, 0, 7, 0, 4>" % (es, bm, 128 // es, 16 if es == 2 else 32, bl)
                           for es in (1, 2) for bl in (0, 1) for bm in (192, 256)],
             "sliced": ["Sliced<Tile<%d, 16, 16, %d, 1, 1, 16, 3, %d, 0, 0, %d, 3>, 4>" % (es, 256 // es, bl, rg)
                        for es in (1, 2) for bl in (0, 1) for rg in (0, 1)]}
    files = []
    for kind, tiles in kinds.items():
        for half in (0, 1):
            files.append(tmp_path / ("%s%d.hip" % (kind, half)))
            files[-1].write_text('#include "gemm_kernel.hpp"\nnamespace g355 {\n' + "".join(
                "template __global__ void gemm_kernel<%s>(const KernelArgs);\n" % t for t in tiles[half::2]) + "}\n")
    with ThreadPoolExecutor(max_workers=6) as ex:
        for f, rows in zip(files, ex.map(lambda f: _usage(str(f), "-I", CSRC), files)):
            assert len(rows) == 4, f
            for r in rows:
                assert r["scratch"] == 0, r
