// Which kernel, tile and K slices a launch of one problem or strided batch really runs (host only).
//
// The selector ranks the variants of its table; their tiles halve and double, and so do its K splits, so that a pick can leave
// a third of the CUs without work, or compute a fifth of its rows for padding.  The pipelined kernels (K-loop form 7, four
// waves, one workgroup per CU) exist for tiles between those, and a launch may have any number of K slices that the cfg's
// workspace holds.  retile() prices all of them and the cfg's own tile by one rule and takes another where that promises at
// least the margins below; a launch whose cfg names the better tile runs it as before.
//
// What a launch costs (us; a slab is 128 bytes of K): per round of 256 workgroups `fixed` + slabs * the slab's time, which is
// `alone` while the chip has power to spare and grows with the share of busy CUs up to `full` (N(0,1) data: a chip with all
// matrix cores busy runs at 1.8 GHz instead of 2.4).  Fitted to 1500 launches of 168 drawn problems (16-bit and fp8 slabs take the
// same time within the fit's error, 14 % rms); the tile it takes is 2 % behind the best of the family in the mean.
#pragma once
#include <algorithm>
#include <cstdint>

namespace g355 {
struct PipelinedTile {
    int block_m, block_n;
    double fixed, alone, full;
};
constexpr PipelinedTile kPipelinedTiles[] = {
    {256, 256, 7.5, 1.20, 1.60}, {192, 256, 4.6, 1.00, 1.38}, {128, 256, 3.0, 0.76, 1.06}, {64, 256, 2.3, 0.55, 0.74},
    {256, 128, 3.1, 0.77, 1.12}, {192, 128, 3.6, 0.60, 0.84}, {128, 128, 2.8, 0.46, 0.63}, {64, 128, 2.0, 0.29, 0.43}};

struct Retiled {
    int block_m, block_n, split;      // block_m == 0: the cfg's own
};

struct RetileProblem {
    int64_t M, N, batch, slabs;       // slabs: of 128 bytes, in K
    int block_m, block_n, split;      // the cfg's
    bool two_resident;                // two workgroups of the cfg's kernel share a CU
    bool reads_c;                     // beta != 0: the old C is read, in the store stage or with the slices' sums
};

constexpr int64_t kRetileCus = 256;

inline double pipelined_us(const PipelinedTile &t, const RetileProblem &p, int64_t split, int64_t workgroups, int64_t per_slice,
                           int64_t cus = kRetileCus)
{
    const int64_t rounds = workgroups / cus, rest = workgroups % cus;
    double us = rounds * (t.fixed + per_slice * t.full);
    if (rest)
        us += t.fixed + per_slice * std::max(t.alone, t.full * rest / cus);
    // the slices' sums are added by a second kernel: 20 bytes per ps
    return split > 1 ? us + 3.2 + p.batch * p.M * p.N * (4. * split + 2.) * 5e-8 : us;
}

// Margins, and where the rule does not look, by the measured time over that of the cfg's own kernel, alone and beside another
// stream's kernel that holds eight CUs.  Of 1517 drawn launches that the price alone retiled 193 took more than 1.03 of it (up to 1.51; 0.91
// in the mean): what the price leaves out.  Of 1127 others that the lines below leave, 30 (up to 1.13; 0.87 in the mean, beside 0.87).
//  - fewer than kMinSlabs slabs per workgroup: a pipelined workgroup's prologue and store stage stand alone (0.96 - 1.2 below);
//  - fewer than kMinGrid workgroups: not what the selector picks these tiles for;
//  - 256x256 below twenty slabs runs an eight-wave kernel that is up to 8 % faster than the pipelined one it is priced as, and
//    launches priced between 0.85 and 0.95 went either way (0.85 - 1.09);
//  - two-stage 128x128 and 64x256 tiles, two to a CU, hide each other's store stage: priced at 0.93 one went to 1.04, up to 0.83 all
//    gained.  A round that nearly fills the chip with the former is priced as two (440 to 512 workgroups: 0.98 in the mean, three of 19 above 1.08);
//  - smaller tiles than 128x128 have three and more workgroups on a CU: 0.9 - 1.2;
//  - more bytes towards a CU's LDS than the cfg's kernel has: a launch that waits for its loads takes as much longer (fewer workgroups over
//    the same weights, three 64-row tiles in place of two of 128: by the ratio of the two up to 1.0 0.76 - 0.95 in the mean, from 1.1
//    0.98 - 1.08, one in two above 1.03; up to 64 rows, whose tiles load the same of B, 0.99 - 1.02 to 1.15);
//  - an old C that the store stage reads: two workgroups of a CU hide that too (up to 17 slabs 1.13 and 1.10 in the mean, to 23 slabs 0.98,
//    from 24 0.93, with the last above 1.1 at 27);
//  - batches: the problems' operands come from memory, and only tiles of 192x256 and 256x256 ask for them less often (0.88 in the mean;
//    the smaller ones 0.97, one in five above 1.03);
//  - 64x256 in place of another tile for more than 64 rows: 1.09 in the mean;
//  - what needs all CUs: the price on 248 of them must hold too (single rounds of 249 to 256 workgroups 1.11 beside).
// A price of 0.55 and less outweighs the last five, one of 0.65 (0.70 from K slices) that of a batch.
inline Retiled retile(const RetileProblem &p)
{
    constexpr int64_t kMinSlabs = 9, kMinGrid = 64, kMinRetiled = 100, kMinSlabsReadingC = 32, kHeldCus = 8;
    const Retiled own = {0, 0, 0};
    auto tiles = [&](int bm, int bn) {      // (M, N and K are at most 2^30)
        return (int64_t)(((uint32_t)p.M + bm - 1) / (uint32_t)bm) * (((uint32_t)p.N + bn - 1) / (uint32_t)bn) * p.batch;
    };
    if (p.block_m * p.block_n < 128 * 128 || p.slabs < kMinSlabs || tiles(p.block_m, p.block_n) * p.split < kMinGrid)
        return own;
    // rows and columns of a slab that a CU loads over all rounds
    auto loads = [&](int bm, int bn, int64_t workgroups, int64_t per_slice) {
        return (workgroups + kRetileCus - 1) / kRetileCus * per_slice * (std::min<int64_t>(bm, p.M) + std::min<int64_t>(bn, p.N));
    };
    const int64_t own_slabs = (p.slabs + p.split - 1) / p.split, own_grid = tiles(p.block_m, p.block_n) * p.split;
    if (p.two_resident && p.block_m == 128 && own_grid > 400 && own_grid <= 2 * kRetileCus)
        return own;
    double own_us = 0, own_held = 0;
    for (const PipelinedTile &t : kPipelinedTiles)
        if (t.block_m == p.block_m && t.block_n == p.block_n) {
            own_us = pipelined_us(t, p, p.split, own_grid, own_slabs);
            own_held = pipelined_us(t, p, p.split, own_grid, own_slabs, kRetileCus - kHeldCus);
        }
    const int64_t own_loads = loads(p.block_m, p.block_n, own_grid, own_slabs);
    double limit = own_us * ((p.block_m * p.block_n == 256 * 256 && own_slabs < 20) ? 0.85 : p.two_resident ? 0.90 : 0.95);
    // the K splits that leave no slice empty, with the slabs of a slice (the table's cfgs have up to 32)
    constexpr int kMaxSplits = 32;
    int splits[kMaxSplits], n_splits = 0;
    uint32_t per[kMaxSplits];
    const uint32_t slabs = (uint32_t)p.slabs;
    for (uint32_t split = 1; split <= (uint32_t)p.split && n_splits < kMaxSplits;) {
        const uint32_t per_slice = (slabs + split - 1) / split;
        if (per_slice < kMinSlabs)
            break;
        if ((slabs + per_slice - 1) / per_slice == split) {
            splits[n_splits] = (int)split;
            per[n_splits++] = per_slice;
        }
        ++split;
    }
    const double sum_us = p.batch * p.M * p.N * 5e-8;
    Retiled best = own;
    for (const PipelinedTile &t : kPipelinedTiles) {
        const int64_t n = tiles(t.block_m, t.block_n);
        // (whatever the split, the matrix cores' time on all CUs)
        if (t.full * n * p.slabs > 1.001 * kRetileCus * limit)
            continue;
        const bool narrow = t.block_m * t.block_n < 192 * 256;
        const bool rows64 = t.block_m == 64 && t.block_n == 256 && (p.block_m != 64 || p.block_n != 256) && p.M > 64;
        for (int i = 0; i < n_splits; ++i) {
            const int split = splits[i];
            const int64_t per_slice = per[i];
            if (n * split < kMinRetiled)
                continue;
            if (split > 1 && t.fixed + kMinSlabs * t.alone + 3.2 + sum_us * (4. * split + 2.) > 1.001 * limit)
                break;      // (the more slices, the longer their sums take)
            const double us = pipelined_us(t, p, split, n * split, per_slice);
            if (us > limit || (p.batch > 1 && narrow && us > (p.split > 1 ? 0.70 : 0.65) * own_us))
                continue;
            if (us > 0.55 * own_us &&
                (rows64 || (p.reads_c && split == 1 && own_slabs < kMinSlabsReadingC) ||
                 20 * loads(t.block_m, t.block_n, n * split, per_slice) > (p.M > 64 ? 21 : 23) * own_loads ||
                 pipelined_us(t, p, split, n * split, per_slice, kRetileCus - kHeldCus) > 0.97 * own_held))
                continue;
            limit = us;
            best = {t.block_m, t.block_n, split};
        }
    }
    return best.block_m == p.block_m && best.block_n == p.block_n && best.split == p.split ? own : best;
}

// The same for a launch of one tile row over weights beyond the memory-side cache: above 128 rows the pipelined streaming kernel,
// of 192 rows where they suffice, 128 columns to a tile, whose loads are spread over the matrix instructions.  What bounds it is
// the CU's vector-memory path, on which A's hits in the L2 wait behind B's misses (256x28672x8192 bf16: A alone 33 us, B alone 74,
// both 119 without a matrix instruction); a bit less of A is fetched for nothing, and nothing else waits.  Its time over the
// eight-wave kernel's, bf16 on six and fp8 on two shapes of weights, K splits halved where the cfg's tile has 256 columns:
//   160 rows  row-major .90-.94 (fp8 1.00-1.01), K-contiguous .86-.99 (fp8 .95)   256 rows  .86-.91 (.88-.89), .86-.97 (.95-.96)
// At 128 rows and below it is level with the 128x128 tile (.95-1.02) and behind the 128x256 one (1.0-1.25).  Row-major weights whose
// 128-column tiles take a second round where the cfg's 256-column ones do not: 1.01-1.07 (57344x4096, 448 workgroups for 224; K-contiguous
// .93-.99).
inline Retiled retile_streaming(const RetileProblem &p, bool kc)
{
    const int split = p.block_n == 256 && p.split > 1 ? p.split / 2 : p.split;
    const int64_t per_slice = (p.slabs + split - 1) / split;
    if (p.batch != 1 || p.M <= 128 || p.M > 256 || p.block_n < 128 || per_slice < 9 || (p.slabs + per_slice - 1) / per_slice != split)
        return {0, 0, 0};
    if (!kc && p.block_n == 256 && (p.N + 127) / 128 * split > kRetileCus)
        return {0, 0, 0};
    return {p.M <= 192 ? 192 : 256, 128, split};
}

// Whether a launch of few 16x16 tiles runs the sliced kernel (sliced.inc) in place of the cfg's.  At most one of its workgroups
// per CU; the cfg's own kernel must be one that is picked for such shapes (small tiles, or K slices of several workgroups).
// Time of the sliced kernel over what ran before, 15 shapes of 12 to 256 tiles (M = 1 to 1000), picks:
//                      K =  768      1024      1536      2048      3072      4096      8192       16384       28672
//   16-bit, K-contiguous  .94-1.00  .84- .90  .78-1.01  .73-1.02  .63- .99  .58-1.00  .49- .96   .55-1.17   .82-1.61
//   16-bit, row-major     .91-1.13  .85-1.10  .81-1.10  .74-1.02  .66-1.04  .40-1.12  .69-1.59  1.37-2.3   1.9-3.1
//   fp8, K-contiguous    1.15-1.29 1.07-1.13 1.02-1.15  .92- .99  .84-1.13  .75-1.10  .40- .85   .48-1.01   .70-1.26
//   fp8, row-major       1.09-1.29 1.05-1.30  .99-1.30  .92-1.33  .85-1.33  .79-1.31  .40-1.55   .88-2.0   1.2-2.9
// and of 2590 drawn launches that a rule of K and tiles alone sliced, by what that left out (1552 others that these lines leave: 0.77 in the
// mean, eight above 1.03, up to 1.16):
//  - K-contiguous B against K slices, which spread a long K over more CUs.  One tile row .70-.88 up to K = 12288 (16-bit) and above; more
//    than 16 tiles in 2-4 rows .66-.94 up to K = 10000, 1.03 and more in five of 13 beyond; in 5-8 rows .72-.82 up to 8192, 1.09 and 1.14
//    beyond; in more .86 up to 6000, .99 to 1.15 beyond; fp8 in 5 and more rows .77 up to 11000, .91 to 1.20 beyond; batches .82 and 1.00;
//  - of row-major B a 16-column tile reads 32 (fp8: 16) bytes of each k row: from the L2 that is level, from memory it is not, so
//    only few columns (128 tiles: .81-.98 at K = 1536, .66-.93 at 3072), and not against K slices that spread the reading (8 of them
//    1.12, 16 and 32 .40-.97; one tile row of more than 64 tiles whose rows are an odd number of half KB apart .92-1.07, else .79-.96);
//  - row-major B that many tile rows read again, or the problems of a batch bring along: nine and more rows of more than 64 tiles
//    .95 in the mean and one in five above 1.03, batches of 48 tiles and more the same; else .80, three of 430 above 1.03;
//  - row-major fp8: against 16x64 tiles of four waves and K slices up to 1.38, and so beyond 128 columns (one tile row: 256) and for batches of two dozen
//    tiles; else .79.
// A launch of most CUs over weights that come from memory is bound by those (1.00-1.13 in one piece).
// One tile row of 120 to 176 tiles in one piece, row-major, K = 1536 to 2816: 1.00-1.07 where the rows of B (b_pitch bytes apart) are
// not whole KB, .90-.97 where they are (32-byte and wider pieces then meet in the same channels and the cfg's kernel is the slower for
// it: 16x2304 7.0 us, 16x2560 9.7, sliced 7.3 and 9.0); up to 113 tiles .84-.96 at any pitch, several tile rows .84-1.01.
inline bool runs_sliced(int64_t M, int64_t N, int64_t K, int64_t batch, int64_t b_pitch, bool fp8, bool kc, int block_m, int block_n, int split)
{
    const int64_t rows = (M + 15) / 16, tiles = rows * ((N + 15) / 16) * batch;
    if (tiles > 256 || (split == 1 ? block_m * block_n > 16 * 64 : split < 4 || block_m * block_n > 64 * 128))
        return false;
    if (kc) {
        if (K < (fp8 ? 2048 : 896))
            return false;
        if (split == 1)
            return tiles <= 160 || N * K * batch * (fp8 ? 1 : 2) <= (8 << 20);
        if (batch > 1)
            return K <= (fp8 ? 10240 : 6144);
        if (tiles <= 16 || rows == 1)
            return K <= (fp8 ? 16384 : 12288);
        return K <= (rows <= 4 ? (fp8 ? 16384 : 10000) : fp8 ? 11264 : rows <= 8 ? 8192 : 6144);
    }
    if (fp8)
        return split == 1 && block_n == 16 && N <= (rows == 1 && batch == 1 ? 256 : 128) && tiles <= (batch > 1 ? 23 : 64) && K >= 4096 && K <= 8192;
    if (K < (tiles <= 128 ? 1536 : 2048) || K > 4096 || tiles > 192)
        return false;
    if (split > 1)
        return split >= 16 && !(rows == 1 && tiles > 64 && b_pitch % 1024 == 512);
    if (batch > 1)
        return tiles < 48;
    return !(rows > 8 && tiles > 64) && !(rows == 1 && tiles > 112 && b_pitch % 1024);
}

// Band height of the rasterisation: the 32 workgroups that an XCD holds cover a region about as high as it is wide.
inline int64_t retiled_group_m(int block_m, int block_n)
{
    int64_t g = 1;
    while (4 * g * g * block_m <= 64 * block_n)
        g *= 2;
    return g;
}
}  // namespace g355
