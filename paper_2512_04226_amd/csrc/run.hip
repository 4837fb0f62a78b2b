// gemm_run and the split-K workspace: the only entry points that touch the GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <mutex>

#include "../../include/gemm.h"
#include "gemm_kernel.hpp"
#include "launch.hpp"
#include "model.hpp"
#include "retile.hpp"

using namespace g355;

namespace g355 {
// Sum the split-K slabs in slice order (deterministic), scale, round to bf16.
// Scale four sums, add beta * C when beta != 0 (C is read before it is overwritten), round to
// the 16-bit output format (f16 != 0: IEEE fp16, else bf16) and store.
__device__ inline void scale_round_store(f32x4 s, float alpha, float beta, void *dst, int f16, int count = 4)
{
    // count < 4: the ragged right edge of C -- only the first `count` outputs exist; C is read (beta != 0)
    // as a whole quad all the same, which stays inside the row's leading dimension
    if (f16) {
        f16x4 o;
        const f16x4 c = (beta != 0.f) ? *(const f16x4 *)dst : f16x4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r)
            o[r] = (beta != 0.f) ? (_Float16)__builtin_fmaf(beta, (float)c[r], s[r] * alpha) : (_Float16)(s[r] * alpha);
        if (count >= 4) {
            *(f16x4 *)dst = o;
        } else {
#pragma unroll
            for (int r = 0; r < 3; ++r)
                if (r < count)
                    ((_Float16 *)dst)[r] = o[r];
        }
    } else {
        bf16x4 o;
        const bf16x4 c = (beta != 0.f) ? *(const bf16x4 *)dst : bf16x4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r)
            o[r] = (beta != 0.f) ? (__bf16)__builtin_fmaf(beta, (float)c[r], s[r] * alpha) : (__bf16)(s[r] * alpha);
        if (count >= 4) {
            *(bf16x4 *)dst = o;
        } else {
#pragma unroll
            for (int r = 0; r < 3; ++r)
                if (r < count)
                    ((__bf16 *)dst)[r] = o[r];
        }
    }
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ ws, uint16_t *C, int M, int N, int ldc,
                                                            int split_k, float alpha, float beta, int f16,
                                                            long long stride_c)
{
    // slab rows are N rounded up to 8 floats apart (the kernels store whole 32-byte pieces also at a ragged edge)
    const size_t nw = (size_t)(N + 7) / 8 * 8;
    ws += (size_t)blockIdx.y * split_k * M * nw;     // problem of the batch
    C += (size_t)blockIdx.y * stride_c;
    const size_t qpr = (size_t)(N + 3) / 4;          // quads per row, the last one possibly partial
    const size_t quads = (size_t)M * qpr;
    const size_t slab = (size_t)M * nw;
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < quads; q += (size_t)gridDim.x * blockDim.x) {
        const size_t m = q / qpr, n = (q % qpr) * 4;
        const float *p = ws + m * nw + n;
        f32x4 s = *(const f32x4 *)p;
        for (int k = 1; k < split_k; ++k) {
            f32x4 t = *(const f32x4 *)(p + k * slab);
            s += t;
        }
        const int count = (int)((size_t)N - n < 4 ? (size_t)N - n : 4);
        scale_round_store(s, alpha, beta, C + m * ldc + n, f16, count);
    }
}


// Stream-K second pass: for every stream-K tile that more than one worker contributed to,
// sum the workers' fp32 partial tiles, scale, round to bf16.  A block of 256 threads is R
// thread rows of 256 / R groups of 4 consecutive outputs; the rows share the contributor
// list (row r adds contributors r, r + R, ... in worker order) and are combined through LDS
// as a fixed binary tree.  The host picks R from the number of contributors per tile, so
// the result depends only on the plan: deterministic.
template <int R>
__global__ __launch_bounds__(256) void streamk_sum_kernel(const float *__restrict__ ws, uint16_t *C, int M, int N, int ldc,
                                                          float alpha, float beta, int f16, int tiles_m, int tiles_n,
                                                          int group_m, SkPlan sk, int BM, int BN, int blocks_per_tile)
{
    constexpr int Q = 256 / R;
    __shared__ f32x4 part[R][Q];
    const int j = blockIdx.x / blocks_per_tile;
    const int quad = threadIdx.x % Q, r = threadIdx.x / Q;
    const int q = (blockIdx.x % blocks_per_tile) * Q + quad;
    int g_first, g_last;
    sk_contributors(sk, j, &g_first, &g_last);
    if (g_first == g_last)
        return;   // one worker computed the whole tile and stored it (uniform over the block)
    int tm, tn;
    logical_tile(tiles_m, tiles_n, group_m, sk.dp_tiles + j, tm, tn);
    const int row = q / (BN / 4), col = (q % (BN / 4)) * 4;
    const int m = tm * BM + row, n = tn * BN + col;
    const bool live = q < BM * BN / 4 && m < M && n < N;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (live) {
        const size_t tile_elems = (size_t)BM * BN;
        const float *base = ws + (size_t)row * BN + col;
        // the first contributor's partial is its second segment unless its range starts with
        // this tile; every later contributor's range starts inside this tile (first segment)
        const int slot_first = sk_slot_of(sk, g_first, j);
#pragma unroll 4
        for (int g = g_first + r; g <= g_last; g += R) {
            const int slot = (g == g_first) ? slot_first : 0;
            s += *(const f32x4 *)(base + (size_t)(2 * g + slot) * tile_elems);
        }
    }
    if constexpr (R > 1) {
        part[r][quad] = s;
        __syncthreads();
#pragma unroll
        for (int half = R / 2; half >= 1; half /= 2) {
            if (r < half)
                part[r][quad] += part[r + half][quad];
            __syncthreads();
        }
        s = part[0][quad];
    }
    if (r == 0 && live)
        scale_round_store(s, alpha, beta, C + (size_t)m * ldc + n, f16, N - n < 4 ? N - n : 4);
}

}  // namespace g355

// Workspace of gemm_run_noalloc: device memory that belongs to the code object, one copy per GPU, from
// module load to process end.  In host code this name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[GEMM_NOALLOC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 16;
struct Workspace {
    void *ptr;
    size_t bytes;
};
// Registered by gemm_set_workspace, read by gemm_run: plain process-wide state, one entry per device.
// Callers that register and run from several threads order those calls themselves.
Workspace g_ws[kMaxDevices];

// Device address of `scratch` on each GPU (every GPU holds its own copy at its own address),
// looked up on the first gemm_run_noalloc call with that device current.
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];

int scratch_of_current_device(void **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return GEMM_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GEMM_OK;
}

// which: a gemm_kernel_kind
const VariantFns &launcher_of(int dtype, int id, int bl, int which)
{
    if (which == GEMM_KERNEL_CHAINED || which == GEMM_KERNEL_CHAINED_RAGGED) {
        const Variant &v = variant_at(dtype, id);
        const auto of = dtype == GEMM_FP16 ? chained_fp16 : dtype == GEMM_BF16 ? chained_bf16 : chained_fp8;
        return of(v.block_m, v.block_n, bl, which == GEMM_KERNEL_CHAINED_RAGGED);
    }
#define G355_COUNT(...) +1
    constexpr int n_b0 = 0 G355_VARIANTS_BF16_0(G355_COUNT);
    constexpr int n_b1 = 0 G355_VARIANTS_BF16_1(G355_COUNT);
    constexpr int n_b2 = 0 G355_VARIANTS_BF16_2(G355_COUNT);
    constexpr int n_b3 = 0 G355_VARIANTS_BF16_3(G355_COUNT);
    constexpr int n_b4 = 0 G355_VARIANTS_BF16_4(G355_COUNT);
    constexpr int n_f0 = 0 G355_VARIANTS_FP8_0(G355_COUNT);
#undef G355_COUNT
    if (dtype == GEMM_FP16) {
        if (id < n_b0)
            return kLaunchFp16_0(id, bl, which);
        if (id < n_b0 + n_b1)
            return kLaunchFp16_1(id - n_b0, bl, which);
        if (id < n_b0 + n_b1 + n_b2)
            return kLaunchFp16_2(id - n_b0 - n_b1, bl, which);
        if (id < n_b0 + n_b1 + n_b2 + n_b3)
            return kLaunchFp16_3(id - n_b0 - n_b1 - n_b2, bl, which);
        if (id < n_b0 + n_b1 + n_b2 + n_b3 + n_b4)
            return kLaunchFp16_4(id - n_b0 - n_b1 - n_b2 - n_b3, bl, which);
        return kLaunchFp16_5(id - n_b0 - n_b1 - n_b2 - n_b3 - n_b4, bl, which);
    }
    if (dtype == GEMM_BF16) {
        if (id < n_b0)
            return kLaunchBf16_0(id, bl, which);
        if (id < n_b0 + n_b1)
            return kLaunchBf16_1(id - n_b0, bl, which);
        if (id < n_b0 + n_b1 + n_b2)
            return kLaunchBf16_2(id - n_b0 - n_b1, bl, which);
        if (id < n_b0 + n_b1 + n_b2 + n_b3)
            return kLaunchBf16_3(id - n_b0 - n_b1 - n_b2, bl, which);
        if (id < n_b0 + n_b1 + n_b2 + n_b3 + n_b4)
            return kLaunchBf16_4(id - n_b0 - n_b1 - n_b2 - n_b3, bl, which);
        return kLaunchBf16_5(id - n_b0 - n_b1 - n_b2 - n_b3 - n_b4, bl, which);
    }
    if (id < n_f0)
        return kLaunchFp8_0(id, bl, which);
    return kLaunchFp8_1(id - n_f0, bl, which);
}

// The instantiation of a variant that a launch runs.  The pipelined one (four waves, K-loop form 7) has the faster loop
// and, with half the waves, the slower prologue and store stage (about 1 us in 16-bit types): it pays from about twenty
// K slabs per workgroup.  Time of the pipelined kernel over the plain (or ragged) one, 4096 x 4096 (4093 ragged), at
// 10 / 17 / 20 / 24 / 32 / 48 slabs:
//   bf16 4x2 grid, row-major B      1.07 1.01 0.99 0.97 0.96 0.92     ragged 1.10 1.04 1.01 1.00 0.98 0.95
//        4x2 grid, K-contiguous     1.05 1.01 0.98 0.95 0.95 0.92     ragged 1.06 1.01 1.00 0.98 0.97 0.95
//        2x4 grid, K-contiguous     1.08 1.04 1.03 1.00 1.00 0.96     ragged 1.05 1.03 1.01 1.01 0.99 0.97
//   fp16 4x2 grid, row-major B      1.06 1.01 0.99 0.97 0.97 0.90     ragged 1.10 1.05 1.02 1.00 0.98 0.96
//        2x4 grid, K-contiguous     1.07 1.05 1.02 1.00 1.00 0.95     ragged 1.04 1.02 1.00 0.99 1.00 0.97
//   fp8  2x4 grid, row-major B      1.06 1.00 0.99 0.97 0.96 0.93     ragged 1.07 1.02 1.00 0.99 0.96 0.91
//        2x4 grid, K-contiguous     1.02 0.97 0.95 0.94 0.94 0.91     ragged 1.01 0.98 0.97 0.95 0.95 0.94
// and of a group of sixteen products (100 to 2000 rows, N = 2048) at 12 / 16 / 20 / 24 / 32 slabs, equal in all groups or
// half and one and a half times that in turn (the mean decides): bf16 4x2 row-major 1.07 1.01 0.98 0.97 0.97, mixed
// 1.07 1.00 0.98 0.95 0.93; 2x4 K-contiguous 1.07 1.04 1.01 0.99 0.99, mixed 1.04 0.99 0.98 0.99 0.97.
// (One line for all: at twenty the slowest to gain, the 2x4 grid on K-contiguous B, still loses 2-3 %, the others have
// gained up to 5.  The four-wave fp8 tile runs form 7 at every K: level with form 5 up to K = 2048.)
constexpr int64_t kPipelinedSlabs = 20;
int kernel_of(int dtype, int id, int bl, bool ragged, bool streaming, int64_t slabs)
{
    if (streaming)
        return GEMM_KERNEL_STREAMING;
    const int pipelined = ragged ? GEMM_KERNEL_PIPELINED_RAGGED : GEMM_KERNEL_PIPELINED;
    if (slabs >= kPipelinedSlabs && launcher_of(dtype, id, bl, pipelined).launch)
        return pipelined;
    return ragged ? GEMM_KERNEL_RAGGED : GEMM_KERNEL_PLAIN;
}

inline int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The pipelined kernel of a tile of retile.hpp (nullptr: a comparison build has none).
const VariantFns *pipelined_of(int dtype, int block_m, int block_n, int b_layout, int ragged, int streaming)
{
    const VariantFns *f = nullptr;
    if (block_m == 256 && block_n == 256) {
        for (int id = 0; id < variant_count(dtype); ++id) {
            const Variant &v = variant_at(dtype, id);
            if (v.block_m == 256 && v.block_n == 256 && (!f || !f->launch))
                f = &launcher_of(dtype, id, b_layout, ragged ? GEMM_KERNEL_PIPELINED_RAGGED : GEMM_KERNEL_PIPELINED);
        }
    } else {
        f = &(dtype == GEMM_FP16 ? pipelined_fp16 : dtype == GEMM_BF16 ? pipelined_bf16 : pipelined_fp8)(block_m, block_n, b_layout, ragged,
                                                                                                          streaming ? PIPELINED_STREAMING : PIPELINED_DIRECT);
    }
    return f && f->launch ? f : nullptr;
}

// Tiles per workgroup of a chained launch, 0: the launch is not chained.  `c_bits`: C's address and the distances in bytes of
// its rows and problems, or-ed.  A tile of few slabs (128 bytes of K) is bound by the latency of its first loads and by its
// store stage, and a chained workgroup has the next tile's loads in flight under both; with more slabs the loop counts, which
// is the plain one of the K-loop forms.  Time of the chained kernel over the one that runs otherwise, by rounds (tiles over the
// workgroups the device holds) and slabs, alone and beside another stream's kernel that holds eight CUs; rows of C on
// 128-byte boundaries, mean of both layouts of B, of one problem with 32 tile columns, one with 4 and a batch of 256 tiles each:
//   16-bit             1/4 slab    1          2           4          8          16
//     256x256    4   1.05 1.21   .94 1.09   .90 1.04   .98 1.09   .99 1.13
//                8    .91 1.13   .84 1.05   .86 1.05   .89 1.09   .93 1.12
//               16    .90 1.02   .83  .95   .84  .92   .91  .97   .93 1.02
//     256x128    4    .92 1.11   .93 1.11   .98 1.18   .98 1.17  1.03 1.23              (128x256 alike)
//                8    .82  .97   .80  .96   .87 1.00   .91 1.09   .95 1.17  1.00 1.23
//               16    .76  .83   .77  .85   .82  .90   .91  .99   .94 1.05  1.01 1.11
//     128x128    4   1.03 1.08  1.03 1.09  1.04 1.09   .97 1.07   .95 1.02
//                8    .84  .92   .85  .89   .87  .94   .94 1.00   .98 1.05  1.01 1.07
//               16    .86  .88   .87  .85   .84  .86   .95  .94   .97  .97   .99 1.00
//     128x64     4    .96 1.00   .96 1.00   .97  .99   .98 1.01  1.02 1.05  1.05 1.11   (64x128 alike)
//                8    .86  .85   .87  .86   .90  .94   .91  .97   .98  .99  1.05 1.03
//     64x64   1.25    .95  .99   .95  .99   .95  .96   .93  .92   .95  .96  1.00 1.01
//                2    .86  .89   .85  .88   .85  .86   .86  .88  1.00  .95  1.09 1.03
//                8    .66  .69   .71  .71   .79  .79   .80  .82   .90  .88   .97  .97
//   fp8
//     256x256    8    .95 1.09   .94 1.07   .94 1.08   .99 1.15  1.02 1.20   (K-contiguous B; the row-major one spills)
//     256x128    8    .84  .97   .82  .94   .88 1.00   .92 1.08   .96 1.14  1.03 1.25
//     128x128    8    .90  .96   .93  .95   .93  .99   .98 1.02  1.02 1.08  1.01 1.07   (one problem, 12 rounds: 1.02 at one slab)
//     128x64     4    .89  .89   .90  .89   .90  .88   .96  .96  1.00 1.00
//     64x64      4    .91  .95   .91  .94   .92  .93   .94  .95   .99 1.01
// Among these, from four slabs on the large tiles gain less and lose more beside other work on one problem of 32 columns and
// more (256x128 at 8 rounds of 8 slabs 1.07 and 1.28 against .92 and 1.11 with 4 columns): the other launch has their
// panels in the L2.  A batch of problems of some hundred tiles and less gains most: the other launch deals every problem's tiles
// to all XCDs, the chained walk gives an XCD whole problems (problems of 4 to 64 tiles, from two or three rounds on: .50 to .95;
// 52 x 808x1720x576 fp16 on 128x128 tiles, nine slabs, 152 -> 138 us).
// Rows of C that start inside a 128-byte line: two tiles share a line, and the further apart in time they write it the more
// often the memory behind the L2 gets it in two parts.  16 rounds at 4 and at 2 tiles per workgroup: 16-bit 128x128 one slab
// 1.03 to 1.19 and .98 to 1.10, two to eight slabs .87 to .95 at both; fp8 128x128 1.00 to 1.29 and 1.00 to 1.19; 128x64 .86 to 1.08 and
// .82 to 1.02 and 64x64 .67 to 1.05 and .74 to 1.03, of which rows on 64-byte boundaries are level; the wider tiles gain as with
// whole lines, and so do the smaller ones while C fits well into the memory-side cache, where the parts meet (128x128 one slab,
// up to 150 MB .79 to .97, from 200 MB 1.10 to 1.41), and batches (.78 to .98).
// (The ragged kernels lie within 0.03 of these.)
int64_t chain_of(const Variant &v, int dtype, int64_t tiles_m, int64_t tiles_n, int64_t batch, int64_t k_bytes, int64_t c_bytes, int resident,
                 uint64_t c_bits)
{
    constexpr int64_t kXcds = 8, kMemorySideCache = 256 << 20;      // the chip's, whatever descriptor the selector works with
    const int64_t slots = kXcds * resident, slabs = cdiv64(k_bytes, 128), tiles = tiles_m * tiles_n * batch;
    const int size = v.block_m * v.block_n;
    const bool fp8 = dtype == GEMM_FP8_E4M3, thin = k_bytes < 64, lines = c_bits % 128 == 0;
    // (the tiles with slabs of 64 bytes compute no half slab beyond K, a chained one does: 5320x10560x160, 2.5 slabs, 1.07)
    const bool half = v.block_k * elem_bytes(dtype) < 128 && (k_bytes - 1) % 128 < 64;
    const bool cached = c_bytes <= kMemorySideCache / 8 * 5;
    const bool batched = batch > 1, small = batched && tiles_m * tiles_n <= 128, compact = batched || std::min(tiles_m, tiles_n) <= 8;
    int64_t most = 0;                 // slabs up to which it pays
    const auto from = [&](double rounds, int64_t limit) {
        if ((double)tiles >= rounds * (double)slots)
            most = std::max(most, limit);
    };
    if (size == 256 * 256) {
        if (small)
            from(3, fp8 ? 4 : 8);
        else if (!fp8 && !thin && (batched || !half))
            from(3, 4), from(compact ? 6 : 12, 8);
    } else if (size == 256 * 128) {
        if (fp8)
            from(8, small ? 16 : batched ? 8 : compact ? 4 : 2);
        else if (small)
            from(3, 8), from(8, 16);
        else
            from(6, compact ? 8 : 2), from(8, 4);
    } else if (size == 128 * 128) {
        if (fp8)
            from(8, batched ? 16 : 0);
        else if (batched)
            from(small ? (thin ? 6 : slabs < 2 ? 4 : 3) : 6, 8), from(8, 16);
        else if (lines)
            from(8, 4);
        else
            from(5, cached ? 4 : 0), from(6, slabs >= 2 ? 8 : 0);
    } else if (size == 128 * 64) {
        if (small)
            from(2, fp8 ? 16 : 32);
        else if (batched)
            from(lines ? 3 : 2, 2), from(fp8 ? 4 : 3, 8), from(6, 16);
        else
            from(lines ? 3 : 2, 2), from(fp8 ? 4 : 6, 4), from(6, fp8 && !compact ? 8 : 0);
    } else {
        from(fp8 ? 4 : 1.25, small ? (fp8 ? 8 : 16) : fp8 && batched ? 8 : 4);
        from(3, fp8 ? 0 : batched ? 16 : 8);
    }
    if (slabs > most)
        return 0;
    // From four rounds on half of the tiles or more are left to the dispatcher, which balances what other work holds CUs; at three a
    // third, and at two or less every tile is dealt out at the start, which only the smallest tiles bear (the 64x64 lines above,
    // beside; a CU holds five of them).  Beyond four tiles per workgroup little is gained alone, and a large tile, of which a CU
    // holds one at a time, loses beside other work (16 rounds at 2 / 4 / 8 tiles, alone and beside a kernel that holds eight CUs:
    // 256x256 one slab .88 .83 .82 and 1.00 .95 1.06, 256x128 four slabs .98 .91 .88 and 1.03 .99 1.09).
    return slabs < 2 && c_bits % (size < 128 * 128 ? 64 : 128) && !cached && !batched && size <= 128 * 128
               ? 2
               : std::max<int64_t>(2, std::min<int64_t>(4, cdiv64(tiles, slots) / 2));
}
}  // namespace

extern "C" int gemm_set_workspace(void *dev_ptr, size_t bytes)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices)
        return GEMM_ERR_HIP;
    if (dev_ptr && ((uintptr_t)dev_ptr & 15))
        return GEMM_ERR_ALIGN;
    g_ws[dev].ptr = dev_ptr;
    g_ws[dev].bytes = dev_ptr ? bytes : 0;
    return GEMM_OK;
}

// What a launch of a cfg that names one problem, or one strided batch, comes to.
struct Launch {
    const VariantFns *fns;
    SkPlan sk;                       // workers == 0 unless stream-K
    int block_m, block_n, split;     // the cfg's, or a pipelined tile's in its place (retile.hpp)
    int64_t group_m;
    int64_t kps, tiles_m, tiles_n;   // K elements per workgroup, tiles
    int chain;                       // tiles per workgroup of the chained kernels
    int kind;                        // gemm_kernel_kind
};

// Checks a cfg (aligned: whether its operands start on 16-byte boundaries) and plans its launch.  c_address: where C starts
// (0: on a boundary of any kind).
static int plan_launch(const gemm_cfg *cfg, bool aligned, uintptr_t c_address, Launch *out)
{
    if (cfg->abi_version != GEMM_ABI_VERSION)
        return GEMM_ERR_ABI;
    int rc = check_problem(cfg->M, cfg->N, cfg->K, cfg->dtype);
    if (rc)
        return rc;
    const int dtype = cfg->dtype;
    const int es = elem_bytes(dtype);
    if (cfg->kernel_id < 0 || cfg->kernel_id >= variant_count(dtype))
        return GEMM_ERR_CFG_ILLEGAL;
    const Variant &v = variant_at(dtype, cfg->kernel_id);
    const gemm_hw &hw = hw_current();
    // the descriptive fields must agree with the variant the id names
    if (cfg->block_m != v.block_m || cfg->block_n != v.block_n || cfg->block_k != v.block_k ||
        cfg->waves_m != v.waves_m || cfg->waves_n != v.waves_n || cfg->mfma != v.mfma || cfg->stages != v.stages)
        return GEMM_ERR_CFG_ILLEGAL;
    if (cfg->split_k < 1 || cfg->group_m < 1 || !variant_legal(hw, v, dtype, cfg->M, cfg->N, cfg->K, cfg->split_k, 0))
        return GEMM_ERR_CFG_ILLEGAL;
    if (cfg->b_layout > 1 || cfg->stream_k > 1)
        return GEMM_ERR_CFG_ILLEGAL;
    if (cfg->groups != 0)
        return GEMM_ERR_CFG_ILLEGAL;   // a grouped cfg runs through gemm_run_grouped
    if (cfg->batch < 1 || cfg->batch > 65535)
        return GEMM_ERR_SHAPE;
    if (cfg->batch > 1 && cfg->stream_k)
        return GEMM_ERR_CFG_ILLEGAL;
    // stream-K: the plan is rebuilt from the cfg's own worker count and must exist
    SkPlan &sk = out->sk;
    std::memset(&sk, 0, sizeof(sk));
    if (cfg->stream_k && !cfg_stream_k_plan(cfg, &sk))
        return GEMM_ERR_CFG_ILLEGAL;
    if (cfg->lda < cfg->K || cfg->ldb < (cfg->b_layout ? cfg->K : cfg->N) || cfg->ldc < cfg->N)
        return GEMM_ERR_SHAPE;
    const int per16 = 16 / es;
    if (!aligned || cfg->lda % per16 || cfg->ldb % per16 || cfg->ldc % 8)
        return GEMM_ERR_ALIGN;
    if (cfg->batch > 1) {
        // problems must not overlap and must keep the 16-byte alignment of the first one
        const int64_t a_min = (cfg->M - 1) * cfg->lda + cfg->K;
        const int64_t b_min = cfg->b_layout ? (cfg->N - 1) * cfg->ldb + cfg->K : (cfg->K - 1) * cfg->ldb + cfg->N;
        const int64_t c_min = (cfg->M - 1) * cfg->ldc + cfg->N;
        if (cfg->stride_a < a_min || cfg->stride_b < b_min || cfg->stride_c < c_min)
            return GEMM_ERR_SHAPE;
        if (cfg->stride_a % per16 || cfg->stride_b % per16 || cfg->stride_c % 8)
            return GEMM_ERR_ALIGN;
        if (cfg->stride_a >= ((int64_t)1 << 40) || cfg->stride_b >= ((int64_t)1 << 40) || cfg->stride_c >= ((int64_t)1 << 40))
            return GEMM_ERR_SHAPE;
    }
    const int64_t kps = k_per_split(v, cfg->K, cfg->split_k);
    const int64_t tiles_m = cdiv64(cfg->M, v.block_m), tiles_n = cdiv64(cfg->N, v.block_n);
    // the kernel addresses a tile's operands with 32-bit byte offsets below 2 GiB
    const int64_t lim = (int64_t)1 << 31;
    const int64_t b_window = cfg->b_layout ? (int64_t)v.block_n * cfg->ldb * es
                                           : (kps + (int64_t)v.stages * v.block_k) * cfg->ldb * es;
    if ((int64_t)v.block_m * cfg->lda * es >= lim || b_window >= lim ||
        tiles_m * tiles_n * cfg->split_k + cfg->sk_workers >= lim || cfg->M * cfg->N >= ((int64_t)1 << 40))
        return GEMM_ERR_SHAPE;

    // an N or K that is not a whole number of 16-byte chunks runs the instantiation that trims its last slab
    const int ragged = (cfg->N % per16 || cfg->K % per16) ? 1 : 0;
    // A grid of one tile row over weights larger than the memory-side cache runs the weight-streaming instantiation
    // (B's loads non-temporal, K walked in a rotated order where the weights' pitch asks for it).  Weights that fit
    // that cache are left to it: a caller that multiplies by the same weights again soon finds them there (fp8
    // M = 64, N = 28672, K = 8192, 235 MB, in a loop: 40 us cached, 48 us streamed).
    const int streaming = (!ragged && tiles_m == 1 && (double)cfg->N * (double)cfg->K * es > hw.mall_bytes) ? 1 : 0;
    // K slabs a workgroup walks: its slice of K, or a Stream-K worker's share where no tile is whole
    const int64_t slabs = (sk.workers > 0 && sk.dp_tiles == 0) ? sk.iters / sk.workers : kps / v.block_k;
    out->kind = kernel_of(dtype, cfg->kernel_id, cfg->b_layout, ragged, streaming, slabs);
    out->chain = 0;
    // (beta = 0 only: the chained store stage does not read C; a tile's rows of C are addressed with 32-bit offsets)
    const int chained = ragged ? GEMM_KERNEL_CHAINED_RAGGED : GEMM_KERNEL_CHAINED;
    if (!streaming && cfg->split_k == 1 && !cfg->stream_k && cfg->beta == 0.f && (int64_t)v.block_m * cfg->ldc * 2 < lim &&
        tiles_m * tiles_n * cfg->batch < lim) {
        const VariantFns &fns = launcher_of(dtype, cfg->kernel_id, cfg->b_layout, chained);
        const uint64_t c_bits = c_address | (uint64_t)cfg->ldc * 2 | (cfg->batch > 1 ? (uint64_t)cfg->stride_c * 2 : 0);
        if (fns.launch)
            out->chain = (int)chain_of(v, dtype, tiles_m, tiles_n, cfg->batch, cfg->K * es, 2 * cfg->M * cfg->N * cfg->batch,
                                      fns.resident, c_bits);
        if (out->chain)
            out->kind = chained;
    }
    out->kps = kps;
    out->tiles_m = tiles_m;
    out->tiles_n = tiles_n;
    out->block_m = v.block_m;
    out->block_n = v.block_n;
    out->split = cfg->split_k;
    out->group_m = cfg->group_m;
    out->fns = &launcher_of(dtype, cfg->kernel_id, cfg->b_layout, out->kind);
    if (cfg->stream_k || out->chain || cfg->own_tile)
        return GEMM_OK;
    const int bk = 128 / es;
    if (!streaming && runs_sliced(cfg->M, cfg->N, cfg->K, cfg->batch, cfg->ldb * es, es == 1, cfg->b_layout == GEMM_B_K_CONTIGUOUS, v.block_m, v.block_n, cfg->split_k)) {
        // (32-bit offsets as above; a wave's window holds its quarter of K, its ring asks for three slabs more)
        if (16 * cfg->lda * es >= lim || (cfg->b_layout ? (int64_t)16 : cdiv64(cfg->K, 4) + 8 * bk) * cfg->ldb * es >= lim)
            return GEMM_OK;
        const VariantFns &sliced = (dtype == GEMM_FP16 ? sliced_fp16 : dtype == GEMM_BF16 ? sliced_bf16 : sliced_fp8)(cfg->b_layout, ragged);
        if (!sliced.launch)
            return GEMM_OK;
        out->fns = &sliced;
        out->kind = ragged ? GEMM_KERNEL_SLICED_RAGGED : GEMM_KERNEL_SLICED;
        out->kps = cdiv64(cfg->K, 2 * bk) * (2 * bk);
        out->tiles_m = cdiv64(cfg->M, 16);
        out->tiles_n = cdiv64(cfg->N, 16);
        out->block_m = out->block_n = 16;
        out->split = 1;
        out->group_m = retiled_group_m(16, 16);
        return GEMM_OK;
    }
    const RetileProblem problem = {cfg->M, cfg->N, cfg->batch, cdiv64(cfg->K, bk), v.block_m, v.block_n, cfg->split_k,
                                   v.block_m * v.block_n == 128 * 128 && v.stages == 2, cfg->beta != 0.f};
    const Retiled r = streaming ? retile_streaming(problem, cfg->b_layout == GEMM_B_K_CONTIGUOUS) : retile(problem);
    if (!r.block_m)
        return GEMM_OK;
    const VariantFns *const fns = pipelined_of(dtype, r.block_m, r.block_n, cfg->b_layout, ragged, streaming);
    const int64_t r_kps = cdiv64(cdiv64(cfg->K, bk), r.split) * bk;
    // (its ring asks for at most six slabs more than the slice has; 32-bit offsets as above)
    if (!fns || (int64_t)r.block_m * cfg->lda * es >= lim ||
        (cfg->b_layout ? (int64_t)r.block_n : r_kps + 6 * bk) * cfg->ldb * es >= lim)
        return GEMM_OK;
    out->fns = fns;
    out->kind = streaming ? GEMM_KERNEL_STREAMING : ragged ? GEMM_KERNEL_PIPELINED_RAGGED : GEMM_KERNEL_PIPELINED;
    out->kps = r_kps;
    out->tiles_m = cdiv64(cfg->M, r.block_m);
    out->tiles_n = cdiv64(cfg->N, r.block_n);
    out->block_m = r.block_m;
    out->block_n = r.block_n;
    out->split = r.split;
    out->group_m = retiled_group_m(r.block_m, r.block_n);
    return GEMM_OK;
}

// The body of gemm_run, gemm_run_ws and gemm_run_noalloc.  own_ws: nullptr = the workspace registered for the
// current device, else the buffer of own_ws_bytes bytes to use instead.
static int run_impl(const gemm_cfg *cfg, const void *A, const void *B, void *C, void *hip_stream, void *own_ws,
                    size_t own_ws_bytes)
{
    if (!cfg || !A || !B || !C)
        return GEMM_ERR_NULL;
    Launch p;
    const int rc = plan_launch(cfg, !(((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15), (uintptr_t)C, &p);
    if (rc)
        return rc;
    const SkPlan &sk = p.sk;
    const Variant &v = variant_at(cfg->dtype, cfg->kernel_id);

    float *ws = nullptr;
    if ((cfg->split_k > 1 || cfg->stream_k) && own_ws) {
        if (own_ws_bytes < gemm_workspace_bytes(cfg))
            return GEMM_ERR_WORKSPACE;
        ws = (float *)own_ws;
    } else if (cfg->split_k > 1 || cfg->stream_k) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
            (void)hipGetLastError();
            return GEMM_ERR_HIP;
        }
        if (!g_ws[dev].ptr || g_ws[dev].bytes < gemm_workspace_bytes(cfg))
            return GEMM_ERR_WORKSPACE;
        ws = (float *)g_ws[dev].ptr;
    }

    KernelArgs a;
    a.A = A;
    a.B = B;
    a.C = C;
    a.ws = ws;
    a.M = (int)cfg->M;
    a.N = (int)cfg->N;
    a.K = (int)cfg->K;
    a.lda = (int)cfg->lda;
    a.ldb = (int)cfg->ldb;
    a.ldc = (int)cfg->ldc;
    a.alpha = cfg->alpha;
    a.beta = cfg->beta;
    a.tiles_m = (int)p.tiles_m;
    a.tiles_n = (int)p.tiles_n;
    a.split_k = p.split;
    a.k_per_split = (int)p.kps;
    a.group_m = (int)std::min<int64_t>(p.group_m, p.tiles_m);   // a band taller than the grid is the whole grid
    a.xcd_remap = cfg->xcd_remap ? 1 : 0;
    a.n_xcd = hw_current().n_xcd;
    a.batch = cfg->batch;
    a.stride_a = cfg->batch > 1 ? cfg->stride_a : 0;
    a.stride_b = cfg->batch > 1 ? cfg->stride_b : 0;
    a.stride_c = cfg->batch > 1 ? cfg->stride_c : 0;
    a.general = sk.workers > 0;
    if (a.general) {
        a.sk = sk;
        a.groups = nullptr;
        a.n_groups = 0;
    }
    a.chain = p.chain;
    if (p.chain) {
        // The workgroups of an XCD walk its tiles abreast.  Where two of their steps cover a band of the rasterisation, a band
        // twice as high halves how often new rows of A come from beyond the L2, which takes longest beside the stores
        // (65536x2048x128: 128x128 tiles 84 -> 78 us, 256x256 76 -> 73; wider grids lose up to a fifth, and so do batches,
        // whose B changes too: 32 x 2048x2048x128 96 -> 110).
        const int resident = p.fns->resident;
        if (a.batch == 1 && p.tiles_n * a.group_m <= 2 * resident)
            a.group_m = (int)std::min<int64_t>(2 * a.group_m, p.tiles_m);
    }
    if (!a.general)
        a.direct = direct_plan(a.tiles_m, a.tiles_n, p.chain ? a.batch : a.split_k, a.group_m, a.n_xcd);

    hipStream_t stream = (hipStream_t)hip_stream;
    const int f16 = (cfg->dtype == GEMM_FP16) ? 1 : 0;
    if (p.fns->launch(a, stream) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    if (cfg->stream_k) {
        // thread rows per output group: enough to keep one output's chain of contributors short
        const int contributors = sk.workers / sk.sk_tiles + 2;
        const int rows = contributors > 32 ? 8 : contributors > 8 ? 4 : 1;
        const int quads = 256 / rows;
        const int bpt = (v.block_m * v.block_n / 4 + quads - 1) / quads;
        const dim3 grid((unsigned)(sk.sk_tiles * bpt)), block(256);
        (void)hipGetLastError();
#define G355_SUM(R)                                                                                                   \
    hipLaunchKernelGGL(streamk_sum_kernel<R>, grid, block, 0, stream, ws, (uint16_t *)C, a.M, a.N, a.ldc, a.alpha,     \
                       a.beta, f16, a.tiles_m, a.tiles_n, a.group_m, sk, v.block_m, v.block_n, bpt)
        if (rows == 8)
            G355_SUM(8);
        else if (rows == 4)
            G355_SUM(4);
        else
            G355_SUM(1);
#undef G355_SUM
        if (hipGetLastError() != hipSuccess)
            return GEMM_ERR_HIP;
    } else if (p.split > 1) {
        const size_t quads = (size_t)cfg->M * (size_t)((cfg->N + 3) / 4);
        size_t blocks = (quads + 255) / 256;
        if (blocks > 256 * 8)
            blocks = 256 * 8;
        (void)hipGetLastError();
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)blocks, (unsigned)a.batch), dim3(256), 0, stream, ws, (uint16_t *)C, a.M,
                           a.N, a.ldc, a.split_k, a.alpha, a.beta, f16, a.stride_c);
        if (hipGetLastError() != hipSuccess)
            return GEMM_ERR_HIP;
    }
    return GEMM_OK;
}

extern "C" int gemm_run(const gemm_cfg *cfg, const void *A, const void *B, void *C, void *hip_stream)
{
    return run_impl(cfg, A, B, C, hip_stream, nullptr, 0);
}

extern "C" int gemm_run_ws(const gemm_cfg *cfg, const void *A, const void *B, void *C, void *hip_stream, void *workspace,
                           size_t workspace_bytes)
{
    if (!cfg)
        return GEMM_ERR_NULL;
    if ((uintptr_t)workspace & 15)
        return GEMM_ERR_ALIGN;
    // (so that a missing buffer never falls back to the registered one)
    if (!workspace && (cfg->split_k > 1 || cfg->stream_k))
        return GEMM_ERR_WORKSPACE;
    return run_impl(cfg, A, B, C, hip_stream, workspace, workspace_bytes);
}

extern "C" int gemm_stream_capturing(void *hip_stream, int *capturing)
{
    if (!capturing)
        return GEMM_ERR_NULL;
    *capturing = 0;
    if (!hip_stream)
        return GEMM_OK;   // the default stream cannot record, and asking would disturb a recording of another
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing((hipStream_t)hip_stream, &status) == hipSuccess;
    if (!known)
        (void)hipGetLastError();
    *capturing = !known || status != hipStreamCaptureStatusNone;
    return GEMM_OK;
}

extern "C" int gemm_run_noalloc(const gemm_cfg *cfg, const void *A, const void *B, void *C, void *hip_stream)
{
    if (!cfg)
        return GEMM_ERR_NULL;
    // sizes beyond the built-in buffer are refused before anything else is looked at
    if (gemm_workspace_bytes(cfg) > (size_t)GEMM_NOALLOC_WORKSPACE_BYTES)
        return GEMM_ERR_WORKSPACE;
    void *ws = nullptr;
    const int rc = scratch_of_current_device(&ws);
    if (rc)
        return rc;
    return run_impl(cfg, A, B, C, hip_stream, ws, (size_t)GEMM_NOALLOC_WORKSPACE_BYTES);
}

extern "C" int gemm_variant_occupancy(int dtype, int variant, int b_layout, int *blocks_per_cu)
{
    if (!blocks_per_cu)
        return GEMM_ERR_NULL;
    if (dtype != GEMM_BF16 && dtype != GEMM_FP8_E4M3 && dtype != GEMM_FP16)
        return GEMM_ERR_DTYPE;
    if (variant < 0 || variant >= variant_count(dtype))
        return GEMM_ERR_INDEX;
    if (b_layout != GEMM_B_ROW_MAJOR && b_layout != GEMM_B_K_CONTIGUOUS)
        return GEMM_ERR_CFG_ILLEGAL;
    (void)hipGetLastError();
    if (launcher_of(dtype, variant, b_layout, 0).occupancy(blocks_per_cu) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    return GEMM_OK;
}

static_assert(sizeof(gemm_group_rec) == sizeof(GroupRec) && offsetof(gemm_group_rec, M) == offsetof(GroupRec, M) &&
                  offsetof(gemm_group_rec, tile_start) == offsetof(GroupRec, tile_start) &&
                  offsetof(gemm_group_rec, group_m) == offsetof(GroupRec, group_m),
              "the public record is the kernel's record");

// The workgroups of a grouped launch (0: every group is empty) and its kernel.
static int plan_grouped(const gemm_cfg *cfg, int n_groups, const gemm_group_rec *host_table, int64_t *total, int *kind, const VariantFns **fns,
                        GroupedTail *tail)
{
    const int X = grouped_xcds(cfg);
    int64_t slots = 0;
    int64_t tiles = 0, tile_slabs = 0;
    int ragged = 0;   // one group with a ragged N or K sends the whole launch through the trimming instantiation
    const int per16 = 16 / elem_bytes(cfg->dtype);
    for (int i = 0; i < n_groups; ++i) {
        const int rc = check_group_rec(cfg, &host_table[i], slots);
        if (rc)
            return rc;
        slots += group_slots((int64_t)host_table[i].tiles_m * host_table[i].tiles_n, X);
        if (slots * X >= ((int64_t)1 << 31))
            return GEMM_ERR_SHAPE;
        if (host_table[i].M > 0 && (host_table[i].N % per16 || host_table[i].K % per16))
            ragged = 1;
        const int64_t t = (int64_t)host_table[i].tiles_m * host_table[i].tiles_n;
        tiles += t;
        tile_slabs += t * cdiv64(host_table[i].K, cfg->block_k);
    }
    *total = slots * X;
    // one kernel for all groups: the mean slab count over the tiles decides
    *kind = kernel_of(cfg->dtype, cfg->kernel_id, cfg->b_layout, ragged, false, tiles ? tile_slabs / tiles : 0);
    *fns = &launcher_of(cfg->dtype, cfg->kernel_id, cfg->b_layout, *kind);
    // (the pipelined tiles are all 256x256 with one slab depth per type)
    *tail = {slots, 1};
    if ((*kind == GEMM_KERNEL_PIPELINED || *kind == GEMM_KERNEL_PIPELINED_RAGGED) && (*fns)->loop_form == 7) {
        *fns = &(cfg->dtype == GEMM_FP16 ? pipelined_fp16 : cfg->dtype == GEMM_BF16 ? pipelined_bf16 : pipelined_fp8)(
            cfg->block_m, cfg->block_n, cfg->b_layout, ragged, PIPELINED_GROUPED);
        *tail = grouped_tail(slots, X);
        *total = (slots + (slots - tail->slot) * (tail->parts - 1)) * X;
    }
    return GEMM_OK;
}

extern "C" int gemm_run_grouped(const gemm_cfg *cfg, int n_groups, const gemm_group_rec *host_table, const void *dev_table,
                                void *hip_stream)
{
    if (!cfg || !host_table || !dev_table)
        return GEMM_ERR_NULL;
    int rc = check_grouped_cfg(cfg, n_groups);
    if (rc)
        return rc;
    if ((uintptr_t)dev_table & 15)
        return GEMM_ERR_ALIGN;
    int64_t total = 0;   // the grid: X workgroups per slot
    int kind = GEMM_KERNEL_PLAIN;
    const VariantFns *fns = nullptr;
    GroupedTail tail;
    rc = plan_grouped(cfg, n_groups, host_table, &total, &kind, &fns, &tail);
    if (rc)
        return rc;
    if (total == 0)
        return GEMM_OK;   // every group is empty
    const gemm_hw &hw = hw_current();
    KernelArgs a;
    std::memset(&a, 0, sizeof(a));
    a.alpha = cfg->alpha;
    a.beta = cfg->beta;
    a.tiles_m = (int)total;
    a.tiles_n = 1;
    a.split_k = 1;
    a.group_m = 1;
    a.xcd_remap = cfg->xcd_remap ? 1 : 0;
    a.n_xcd = hw.n_xcd;
    a.batch = 1;
    a.general = 1;
    a.groups = (const GroupRec *)dev_table;
    a.n_groups = n_groups;
    a.tail_slot = (int)tail.slot;
    a.tail_parts = tail.parts;
    if (fns->launch(a, (hipStream_t)hip_stream) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    return GEMM_OK;
}

extern "C" int gemm_grouped_launched(const gemm_cfg *cfg, int n_groups, const gemm_group_rec *table, int64_t workgroup, int32_t out5[5],
                                     int64_t *workgroups_out)
{
    if (!cfg || !table || !out5)
        return GEMM_ERR_NULL;
    int rc = check_grouped_cfg(cfg, n_groups), kind;
    int64_t total = 0;
    const VariantFns *fns;
    GroupedTail tail;
    if (!rc)
        rc = plan_grouped(cfg, n_groups, table, &total, &kind, &fns, &tail);
    if (rc)
        return rc;
    if (workgroups_out)
        *workgroups_out = total;
    if (workgroup < 0 || workgroup >= total)
        return GEMM_ERR_INDEX;
    const int X = grouped_xcds(cfg), x = (int)(workgroup % X);
    const GroupedPart part = grouped_part((int)(workgroup / X), (int)tail.slot, tail.parts, cfg->block_m);
    int32_t at[3];
    rc = gemm_grouped_locate(cfg, n_groups, table, (int64_t)part.slot * X + x, at);
    if (rc)
        return rc;
    const int64_t rows = at[0] < 0 ? 0 : (int64_t)table[at[0]].M - (int64_t)at[1] * cfg->block_m - part.first_row;
    for (int i = 0; i < 3; ++i)
        out5[i] = rows > 0 ? at[i] : -1;
    out5[3] = rows > 0 ? part.first_row : 0;
    out5[4] = rows > 0 ? (int32_t)std::min<int64_t>(rows, part.rows) : 0;
    return GEMM_OK;
}

extern "C" int gemm_launched_kernel(const gemm_cfg *cfg, int n_groups, const gemm_group_rec *host_table, int32_t out4[4])
{
    if (!cfg || !out4 || (n_groups != 0 && !host_table))
        return GEMM_ERR_NULL;
    int rc, kind = GEMM_KERNEL_PLAIN;
    const VariantFns *fns = nullptr;
    if (n_groups != 0) {
        int64_t total = 0;
        GroupedTail tail;
        rc = check_grouped_cfg(cfg, n_groups);
        if (!rc)
            rc = plan_grouped(cfg, n_groups, host_table, &total, &kind, &fns, &tail);
    } else {
        Launch p;
        rc = plan_launch(cfg, true, 0, &p);
        if (!rc) {
            kind = p.kind;
            fns = p.fns;
        }
    }
    if (rc)
        return rc;
    out4[0] = kind;
    out4[1] = fns->waves_m;
    out4[2] = fns->waves_n;
    out4[3] = fns->loop_form;
    return GEMM_OK;
}

extern "C" int gemm_launched_tile(const gemm_cfg *cfg, int32_t out3[3])
{
    if (!cfg || !out3)
        return GEMM_ERR_NULL;
    Launch p;
    const int rc = plan_launch(cfg, true, 0, &p);
    if (rc)
        return rc;
    out3[0] = p.block_m;
    out3[1] = p.block_n;
    out3[2] = p.split;
    return GEMM_OK;
}
