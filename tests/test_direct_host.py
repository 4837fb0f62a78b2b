"""Tile coordinates of a direct launch (divisors inverted on the host) against the divisions they stand for, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include <random>
#include "fast_div.hpp"
using namespace g355;
int main()
{
    std::mt19937 rng(1);
    long n = 0, bad = 0;
    auto one = [&](uint32_t d, int64_t x) {
        if (x >= 0 && x <= 2147483647LL)
            ++n, bad += fast_div((int)x, fast_div_of(d)) != (int)(x / d);
    };
    auto divisor = [&](uint32_t d) {                // quotient edges, where a rounded reciprocal errs first
        for (int i = 0; i < 100; ++i)
            for (int e = -1; e <= 1; ++e)
                one(d, (int64_t)(rng() % (2147483647u / d + 1)) * d + e);
        one(d, 2147483647), one(d, 2147483647 / d * (int64_t)d - 1), one(d, 0), one(d, d), one(d, d - 1);
    };
    for (uint32_t d = 1; d < 3000; ++d)
        divisor(d);
    for (int b = 1; b < 31; ++b)
        divisor((1u << b) - 1), divisor(1u << b), divisor((1u << b) + 1), divisor(1 + rng() % (1u << b));
    divisor(2147483647u);
    for (int it = 0; it < 3000; ++it) {
        const int tm = 1 + rng() % 40, tn = 1 + rng() % 40, split = 1 + rng() % 4, group = 1 + rng() % (tm + 8), xcds = 1 + rng() % 10;
        const bool remap = rng() % 4;
        const DirectPlan p = direct_plan(tm, tn, split, group, xcds);
        const int grid = tm * tn * split;
        for (int pid = 0; pid < grid; ++pid, ++n) {
            int m, t, k, wm, wt;
            direct_coords(p, tm, tn, split, group, xcds, remap, pid, m, t, k);
            const int per = grid / xcds, rem = grid % xcds, x = pid % xcds, q = pid / xcds;
            const int l = remap ? x * per + (x < rem ? x : rem) + q : pid;      // one contiguous range per XCD
            logical_tile(tm, tn, group, l % (tm * tn), wm, wt);
            bad += m != wm || t != wt || k != l / (tm * tn);
        }
    }
    std::printf("%ld checks, %ld bad\n", n, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_direct_coordinates_equal_the_divisions_they_replace(tmp_path):
    src, exe = tmp_path / "direct.cpp", str(tmp_path / "direct")
    src.write_text(SOURCE)
    csrc = os.path.join(ROOT, "paper_2512_04226_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, "-I", os.path.join(ROOT, "include"), "-o", exe, str(src)], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
