// Division by a number known at launch, for the indexes of a kernel's first instructions (a division by a variable costs the
// device about twenty dependent instructions, this one three).  Granlund and Montgomery, "Division by invariant integers
// using multiplication" (1994), the round-up multiplier with the extra bit folded into an addition:
// floor(n / d) = (mulhi(n, m) + n) >> s with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1, for 0 <= n < 2^31.
#pragma once
#include <stdint.h>

#include "stream_k.hpp"

namespace g355 {
struct FastDiv {
    uint32_t mul, shift;
};

inline FastDiv fast_div_of(uint32_t d)      // d >= 1
{
    uint32_t s = 0;
    while (((uint64_t)1 << s) < d)
        ++s;
    return {(uint32_t)(((((uint64_t)1 << s) - d) << 32) / d + 1), s};
}

G355_HD inline int fast_div(int n, FastDiv f) { return (int)(((uint32_t)(((uint64_t)(uint32_t)n * f.mul) >> 32) + (uint32_t)n) >> f.shift); }

// Tile coordinates in a launch that is neither Stream-K nor grouped: logical_id and logical_tile with their divisors inverted
// on the host.
struct DirectPlan {
    FastDiv xcds, tiles, band, rows, last_rows;      // divisors: XCDs, tiles per slice, tiles of a band, its rows, the last band's
    int per_xcd, rem_xcd;                            // workgroups per XCD and how many XCDs have one more
};

inline DirectPlan direct_plan(int tiles_m, int tiles_n, int slices, int group_m, int n_xcd)   // slices: of K, or problems of a chain
{
    DirectPlan p;
    const int grid = tiles_m * tiles_n * slices;
    p.xcds = fast_div_of((uint32_t)(n_xcd > 0 ? n_xcd : 1));
    p.tiles = fast_div_of((uint32_t)(tiles_m * tiles_n));
    p.band = fast_div_of((uint32_t)(group_m * tiles_n));
    p.rows = fast_div_of((uint32_t)group_m);
    p.last_rows = fast_div_of((uint32_t)(tiles_m % group_m ? tiles_m % group_m : group_m));
    n_xcd = n_xcd > 0 ? n_xcd : 1;
    p.per_xcd = grid / n_xcd;
    p.rem_xcd = grid % n_xcd;
    return p;
}

// logical_tile
G355_HD inline void direct_tile(const DirectPlan &p, int tiles_m, int tiles_n, int group_m, int t, int &tm, int &tn)
{
    const int band = fast_div(t, p.band), first_m = band * group_m;
    const bool last = tiles_m - first_m < group_m;
    const int rows = last ? tiles_m - first_m : group_m, r = t - band * (group_m * tiles_n);
    tn = fast_div(r, {last ? p.last_rows.mul : p.rows.mul, last ? p.last_rows.shift : p.rows.shift});
    tm = first_m + r - tn * rows;
}

G355_HD inline void direct_coords(const DirectPlan &p, int tiles_m, int tiles_n, int split_k, int group_m, int n_xcd, bool remap, int pid,
                                  int &tm, int &tn, int &ks)
{
    int l = pid;
    if (remap) {
        const int q = fast_div(pid, p.xcds), x = pid - q * n_xcd;
        l = x * p.per_xcd + (x < p.rem_xcd ? x : p.rem_xcd) + q;
    }
    ks = split_k > 1 ? fast_div(l, p.tiles) : 0;
    direct_tile(p, tiles_m, tiles_n, group_m, l - ks * (tiles_m * tiles_n), tm, tn);
}
}  // namespace g355
