// The chained kernel: a workgroup computes several output tiles one after the other and treats their K slabs as one
// stream through the LDS ring, so that the first slabs of a tile are under way while the tile before it is finished
// and stored.  For launches of many tiles with few slabs each, where a tile's time is the latency of its first loads
// and of its store stage (see chain_of in run.hip for when a launch takes it).
// What bounds it: reads that come from beyond the L2 wait behind the writes of C there, and a wave's loads complete after
// the stores it issued before them.  65536x2048x256 bf16 with 256x256 tiles: 100 us (114 in a launch of one workgroup per
// tile), 90 with every read an L2 hit, 64 without the stores, 42 without either and without the matrix instructions; at
// K = 16 all that is left is the stores, 57 us = 4.7 TB/s (a plain fill of the same bytes 40).  Measured on the way, 128x128
// tiles at K = 128: a contiguous run of tiles per workgroup instead of the abreast walk 95 us (84); rings of five stages with
// one workgroup per CU 94; sixteen waves 106; eight waves instead of four level.  (With up to eight tiles per workgroup; at
// four, as launched now, 1.00 to 1.02 times these.)
#pragma once
#include "gemm_kernel.hpp"

namespace g355 {

// The tiles of a workgroup.  Every XCD owns a contiguous range of the launch's tiles (problem by problem, each in its
// rasterisation order), as in a launch of one workgroup per tile; the workgroups that are resident on it at a time
// walk a part of that range abreast, `step` tiles further each time, so that at any moment they work on neighbouring
// tiles and share panels through the L2.  (A contiguous run of tiles per workgroup re-reads A from beyond the L2.)
struct TileWalk {
    int item, step, end;        // next tile, tiles until the workgroup's next one, end of its part
    int bz, tm, tn;
    // Workgroups per XCD of a launch: whole blocks of `resident` workgroups with a.chain tiles each, then one block that
    // shares the rest evenly.
    __host__ __device__ static inline int grid_per_xcd(const KernelArgs &a, int resident)
    {
        const int X = a.xcd_remap ? a.n_xcd : 1, own = (a.tiles_m * a.tiles_n * a.batch + X - 1) / X;
        const int whole = own / (resident * a.chain), rest = own - whole * resident * a.chain;
        return whole * resident + (rest < resident ? rest : resident);
    }
    // false: nothing to do
    __device__ inline bool start(const KernelArgs &a, int resident)
    {
        int q = (int)blockIdx.x, base = 0, own = a.tiles_m * a.tiles_n * a.batch;
        if (a.xcd_remap) {      // the grid is a multiple of n_xcd
            q = fast_div(q, a.direct.xcds);
            const int x = (int)blockIdx.x - q * a.n_xcd, rem = a.direct.rem_xcd;
            base = x * a.direct.per_xcd + (x < rem ? x : rem);
            own = a.direct.per_xcd + (x < rem ? 1 : 0);
        }
        const int block = q / resident, first = block * resident * a.chain;   // the block's tiles start here
        const int size = (own - first < resident * a.chain) ? own - first : resident * a.chain;
        step = size < resident ? size : resident;
        item = base + first + (q - block * resident);
        end = base + first + size;
        if (item >= end)
            return false;
        locate(a);
        return true;
    }
    __device__ inline int count() const { return (end - item + step - 1) / step; }
    __device__ inline void locate(const KernelArgs &a)
    {
        bz = fast_div(item, a.direct.tiles);
        direct_tile(a.direct, a.tiles_m, a.tiles_n, a.group_m, item - bz * (a.tiles_m * a.tiles_n), tm, tn);
    }
    __device__ inline void next(const KernelArgs &a)
    {
        item += step;
        locate(a);
    }
};

template <class T>
__global__ __launch_bounds__(T::NT, T::CHAIN_WAVES) void chained_kernel(const KernelArgs args)
{
    constexpr int ES = T::ES, BM = T::BM, BN = T::BN, BK = T::BK, MI = T::MI, EPC = 16 / ES;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[T::LDS_BYTES];
    G355_LDS uint8_t *const lds = (G355_LDS uint8_t *)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WN, wn = wave % T::WN;

    TileWalk ahead;
    if (!ahead.start(args, T::CHAIN_RESIDENT))
        return;     // (the whole workgroup: nothing was started)
    const int count = ahead.count();
    const int KT = (args.K + BK - 1) / BK;      // slabs per tile

    // ---- the stream of slab requests ----
    // Lane offsets inside a tile's operands are the same for all tiles: a tile moves the buffer windows.  Rows beyond the
    // matrix lie outside the window.  So do columns of row-major B beyond N in its last row; in the rows before, they
    // are whatever follows there, and end up only in columns of C that are not stored.
    // (a wave's load instructions of one operand are a whole number of swizzle periods of rows apart)
    constexpr int A_STEP = T::NW * 64 / T::CA, B_STEP = T::NW * 64 / T::CB;
    static_assert(A_STEP % (T::A_ROWS_PER_WIN * (T::A_KEY_MASK + 1)) == 0 && (T::BL == 1 || B_STEP % 16 == 0) &&
                  (T::BL == 0 || B_STEP % (T::A_ROWS_PER_WIN * (T::A_KEY_MASK + 1)) == 0), "one swizzle key per lane and operand");
    const int a_row_l = (wave * 64 + lane) / T::CA, a_kcol = ((lane % T::CA) ^ T::a_key(a_row_l)) * EPC;
    const int b_row_l = (wave * 64 + lane) / T::CB, b_kcol = (T::BL == 0) ? 0 : ((lane % T::CB) ^ T::a_key(b_row_l)) * EPC;
    const unsigned a_voff = (unsigned)(a_row_l * args.lda + a_kcol) * ES;
    const unsigned b_voff = (unsigned)(b_row_l * args.ldb + b_kcol) * ES + (T::BL == 0 ? ((wave * 64 + lane) % T::CB * 16) ^ T::b_key(b_row_l) : 0);
    __amdgpu_buffer_rsrc_t rsA, rsB;
    int ahead_left = count, ahead_kt = 0;
    auto windows = [&]() __attribute__((always_inline)) {
        const int m0 = ahead.tm * BM, n0 = ahead.tn * BN;
        const int m_valid = (args.M - m0 < BM) ? args.M - m0 : BM, n_valid = (args.N - n0 < BN) ? args.N - n0 : BN;
        const uint8_t *const A = (const uint8_t *)args.A + (ahead.bz * args.stride_a + (size_t)m0 * args.lda) * ES;
        const uint8_t *const B = (const uint8_t *)args.B + (ahead.bz * args.stride_b + (T::BL == 0 ? (size_t)n0 : (size_t)n0 * args.ldb)) * ES;
        const bool any = ahead_left > 0;        // past the last tile nothing is read
        // (windows end with whole chunks: a ragged row's last one is fetched whole, inside its leading-dimension span)
        const int k_w = (args.K + EPC - 1) / EPC * EPC, n_w = (args.N - n0 + EPC - 1) / EPC * EPC;
        rsA = make_rsrc(A, any ? (unsigned)((m_valid - 1) * args.lda + k_w) * ES : 0u);
        rsB = make_rsrc(B, any ? (unsigned)(T::BL == 0 ? (args.K - 1) * args.ldb + n_w : (n_valid - 1) * args.ldb + k_w) * ES : 0u);
    };
    // the load instructions of the next slab of the stream
    auto request = [&](G355_LDS uint8_t *stage) __attribute__((always_inline)) {
        const int kk = ahead_kt * BK;
        const unsigned a0 = (a_kcol + kk < args.K) ? a_voff + (unsigned)(kk * ES) : OOB_OFFSET;
        const unsigned b0 = (T::BL == 0) ? b_voff + (unsigned)kk * (unsigned)(args.ldb * ES)
                                         : (b_kcol + kk < args.K) ? b_voff + (unsigned)(kk * ES) : OOB_OFFSET;
#pragma unroll
        for (int i = 0; i < T::A_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (G355_LDS void *)(stage + (i * T::NW + wave) * 1024), 16,
                                                     a0 + (unsigned)(i * A_STEP) * (unsigned)(args.lda * ES), 0, 0, G355_LOAD_DEFAULT);
#pragma unroll
        for (int i = 0; i < T::B_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (G355_LDS void *)(stage + T::A_BYTES + (i * T::NW + wave) * 1024), 16,
                                                     b0 + (unsigned)(i * B_STEP) * (unsigned)(args.ldb * ES), 0, 0, G355_LOAD_DEFAULT);
        if (++ahead_kt == KT) {
            ahead_kt = 0;
            --ahead_left;
            ahead.next(args);
            windows();
        }
    };

    // ---- fragments (the layouts of gemm_kernel) ----
    typedef typename std::conditional<MI == 32, f32x16, f32x4>::type acc_t;
    typedef typename std::conditional<ES == 2, bf16x8, i32x8>::type frag_t;
    acc_t acc[T::TN][T::TM];
    frag_t af[2][T::TM], bfr[2][T::TN];
    const int a_row = wm * T::WTM + lane % MI, b_row = wn * T::WTN + lane % MI, kg = lane / MI;
    const int g16 = lane >> 4, i16 = lane & 15;
    constexpr int LPR = (ES == 2) ? 4 : 2, TRK = 16 / LPR;
    const int b_krow_l = (MI == 32 ? g16 >> 1 : g16) * T::KL + i16 / LPR;
    const int b_ncol = wn * T::WTN + (MI == 32 ? (g16 & 1) * 16 : 0) + (i16 % LPR) * (8 / ES);
    auto kc_frag = [&](frag_t &dst, const G355_LDS uint8_t *p, int row, int k0) __attribute__((always_inline)) {
        const int chunk = (k0 + kg * T::KL) / EPC;
        if constexpr (ES == 2) {
            dst = *(const G355_LDS frag_t *)(p + T::a_off(row, chunk));
        } else {
            const i32x4 lo = *(const G355_LDS i32x4 *)(p + T::a_off(row, chunk));
            const i32x4 hi = *(const G355_LDS i32x4 *)(p + T::a_off(row, chunk + 1));
            dst = __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    };
    auto load_frags = [&](const G355_LDS uint8_t *stage, int kstep, int buf) __attribute__((always_inline)) {
        const G355_LDS uint8_t *const sB = stage + T::A_BYTES;
        const int k0 = kstep * T::KI;
#pragma unroll
        for (int i = 0; i < T::TM; ++i)
            kc_frag(af[buf][i], stage, a_row + i * MI, k0);
#pragma unroll
        for (int j = 0; j < T::TN; ++j) {
            if constexpr (T::BL == 1) {
                kc_frag(bfr[buf][j], sB, b_row + j * MI, k0);
            } else if constexpr (ES == 2) {
                const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((G355_LDS short4_t *)(sB + T::b_off(k0 + b_krow_l, (b_ncol + j * MI) * 2)));
                const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((G355_LDS short4_t *)(sB + T::b_off(k0 + b_krow_l + TRK, (b_ncol + j * MI) * 2)));
                bfr[buf][j] = __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            } else {
                int2_t q[4];
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    q[h] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((G355_LDS int2_t *)(sB + T::b_off(k0 + b_krow_l + h * TRK, b_ncol + j * MI)));
                const i32x4 lo = __builtin_shufflevector(q[0], q[1], 0, 1, 2, 3), hi = __builtin_shufflevector(q[2], q[3], 0, 1, 2, 3);
                bfr[buf][j] = __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
    };
    auto mma_kstep = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < T::TN; ++j)
#pragma unroll
            for (int i = 0; i < T::TM; ++i) {
                if constexpr (ES == 2 && T::FT == 1 && MI == 16)
                    acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, bfr[buf][j]), __builtin_bit_cast(f16x8, af[buf][i]), acc[j][i], 0, 0, 0);
                else if constexpr (ES == 2 && MI == 16)
                    acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[buf][j], af[buf][i], acc[j][i], 0, 0, 0);
                else
                    acc[j][i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bfr[buf][j], af[buf][i], acc[j][i], 0, 0, 0, 0, 0, 0);
            }
    };
    static_assert(MI == 16 ? ES == 2 && T::TN % 2 == 0 : ES == 1, "16x16x32 for the 16-bit types, 32x32x64 for fp8");

    // ---- store stage: lanes exchange halves of their results so that each holds 8 consecutive columns of one row, and
    //      store them: 64 (32x32: 32) bytes of a row per instruction, no LDS and no barrier.  Every wave issues the same
    //      number of stores whatever the tile's valid part: what lies outside C goes to an offset beyond its window. ----
    typedef typename std::conditional<T::FT == 1, _Float16, __bf16>::type out_t;
    typedef typename std::conditional<T::FT == 1, f16x4, bf16x4>::type out4_t;
    constexpr int STORES = T::TM * T::TN * T::ACC / 8;       // per wave and tile
    constexpr int FULL = T::A_LOADS + T::B_LOADS;
    static_assert(T::A_UNITS % T::NW == 0 && T::B_UNITS % T::NW == 0, "every wave issues every load");
    TileWalk done;
    const float alpha = args.alpha;
    auto store_tile = [&]() __attribute__((always_inline)) {
        const int m0 = done.tm * BM, n0 = done.tn * BN;
        const int m_valid = (args.M - m0 < BM) ? args.M - m0 : BM;
        const __amdgpu_buffer_rsrc_t rsC =
            make_rsrc((const uint8_t *)args.C + (done.bz * args.stride_c + (size_t)m0 * args.ldc + n0) * 2,
                      (unsigned)((m_valid - 1) * args.ldc + (args.N - n0)) * 2);
        const int q = lane / 16;
        const int m_l = wm * T::WTM + (lane % MI);
        const int n_l = wn * T::WTN + (MI == 16 ? (q & 1) * 16 + (q >> 1) * 8 : (lane >> 5) * 8);
        const unsigned off0 = (unsigned)(m_l * args.ldc + n_l) * 2;
        auto pack = [&](const acc_t &v, int g) __attribute__((always_inline)) {
            out4_t o;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                o[r] = (out_t)(v[g * 4 + r] * alpha);
            return __builtin_bit_cast(int2_t, o);
        };
        auto put = [&](auto pieces, int2_t x, int2_t y, int i, int col) __attribute__((always_inline)) {
            i32x4 v;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int xr = x[r], yr = y[r];
                auto s = [&] {
                    if constexpr (MI == 16)
                        return __builtin_amdgcn_permlane16_swap(xr, yr, false, false);
                    else
                        return __builtin_amdgcn_permlane32_swap(xr, yr, false, false);
                }();
                v[r] = (int)s[0];
                v[2 + r] = (int)s[1];
            }
            // (rows below the matrix lie beyond the window by themselves; the scalar offset stays 0, it would take part in
            // the window's check with a wrap-around)
            const unsigned at = off0 + (unsigned)(i * MI * args.ldc + col) * 2;
            const int left_n = args.N - n0 - (n_l + col);       // valid columns from this lane's first
            if constexpr (!decltype(pieces)::value) {
                __builtin_amdgcn_raw_buffer_store_b128(v, rsC, left_n >= 8 ? at : OOB_OFFSET, 0, 0);
            } else {
                // the group that holds column N - 1: element by element, nothing beyond it is written
#pragma unroll
                for (int r = 0; r < 7; ++r)
                    __builtin_amdgcn_raw_buffer_store_b16((short)(v[r / 2] >> (r % 2 * 16)), rsC, (left_n < 8 && r < left_n) ? at + r * 2 : OOB_OFFSET, 0, 0);
            }
        };
        auto all = [&](auto pieces) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < T::TM; ++i) {
                if constexpr (MI == 16) {
#pragma unroll
                    for (int j = 0; j < T::TN; j += 2)
                        put(pieces, pack(acc[j][i], 0), pack(acc[j + 1][i], 0), i, j * 16);
                } else {
#pragma unroll
                    for (int j = 0; j < T::TN; ++j)
#pragma unroll
                        for (int p = 0; p < 2; ++p)
                            put(pieces, pack(acc[j][i], 2 * p), pack(acc[j][i], 2 * p + 1), i, j * 32 + p * 16);
                }
            }
        };
        all(std::false_type{});
        if constexpr (T::RG) {
            if (args.N % 8 != 0 && args.N - n0 < BN) {
                // (packed again from the sums: kept from above they would be a quarter of the registers)
#pragma unroll
                for (int j = 0; j < T::TN; ++j)
#pragma unroll
                    for (int i = 0; i < T::TM; ++i)
                        asm volatile("" : "+v"(acc[j][i])::"memory");
                all(std::true_type{});
            }
        }
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < T::TN; ++j)
#pragma unroll
            for (int i = 0; i < T::TM; ++i)
#pragma unroll
                for (int r = 0; r < T::ACC; ++r)
                    acc[j][i][r] = 0.f;
    };

    // Ragged instantiation: the chunk of every row of a K-contiguous operand that straddles the end of K is cleared beyond it
    // in the last slab of a tile, which has landed and whose fragments are not yet read (gemm_kernel's trim_last_slab).
    auto trim = [&](G355_LDS uint8_t *pa) __attribute__((always_inline)) {
        const int valid = args.K % EPC;
        if (!T::RG || valid == 0)
            return;
        G355_LDS uint8_t *const pb = pa + T::A_BYTES;
        const int chunk = args.K % BK / EPC;
        for (int r = tid; r < BM + (T::BL == 1 ? BN : 0); r += T::NT) {
            G355_LDS i32x4 *const c = (G355_LDS i32x4 *)(r < BM ? pa + T::a_off(r, chunk) : pb + T::a_off(r - BM, chunk));
            i32x4 v = *c;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int keep = valid - d * (4 / ES);
                v[d] = (int)((unsigned)v[d] & (keep >= 4 / ES ? 0xffffffffu : keep <= 0 ? 0u : ((1u << (keep * 8 * ES)) - 1u)));
            }
            *c = v;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };

    // ---- the stream ----
    static_assert(T::KSTEPS % 2 == 0, "fragment double buffering needs an even number of k-steps");
    constexpr int ALLOW = (T::NS - 2) * FULL;
    static_assert(ALLOW + STORES <= 63 && (T::NS - 1) * FULL <= 63, "vmcnt is a 6-bit counter");
    // k-steps 0 .. KSTEPS-2 of the slab in `cur`, then its barrier, which certifies the next slab: all of a wave's newer
    // requests may still be in flight, and the stores of the `fresh` tiles that it stored after asking for that slab --
    // memory operations of a wave complete in order
    constexpr int MAXF = (63 - ALLOW) / STORES < T::NS - 1 ? (63 - ALLOW) / STORES : T::NS - 1;
    auto until_barrier = [&](const G355_LDS uint8_t *cur, int fresh) __attribute__((always_inline)) {
#pragma unroll
        for (int kstep = 0; kstep < T::KSTEPS - 1; ++kstep) {
            load_frags(cur, kstep + 1, (kstep + 1) & 1);
            mma_kstep(kstep & 1);
        }
        if (MAXF >= 3 && fresh >= 3)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(ALLOW + (MAXF >= 3 ? 3 : 0) * STORES) : "memory");
        else if (MAXF >= 2 && fresh >= 2)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(ALLOW + (MAXF >= 2 ? 2 : 0) * STORES) : "memory");
        else if (fresh >= 1)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(ALLOW + STORES) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(ALLOW) : "memory");
    };
    done = ahead;
    windows();
#pragma unroll
    for (int s = 0; s < T::NS; ++s)
        request(lds + s * T::STAGE);
    clear();
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((T::NS - 1) * FULL) : "memory");
    if (KT == 1)
        trim(lds);
    load_frags(lds, 0, 0);
    until_barrier(lds, 0);
    int kt = 0, stage = 0, left = count * KT;      // kt: slab of its tile in `stage`
    int stored = 0;                                // tiles stored so far, up to NS
    // from the barrier of one slab to the barrier of the next (gemm_kernel's after_barrier)
    auto span = [&](G355_LDS uint8_t *__restrict__ freed, G355_LDS uint8_t *__restrict__ next) __attribute__((always_inline)) {
        const bool last = ++kt == KT;
        if ((last ? 1 : kt + 1) == KT)
            trim(next);
        request(freed);
        if (!last)
            load_frags(next, 0, 0);
        mma_kstep((T::KSTEPS - 1) & 1);
        if (last) {
            asm volatile("" ::: "memory");      // the stores follow the requests: until_barrier counts on it
            store_tile();
            asm volatile("" ::: "memory");
            done.next(args);
            clear();
            kt = 0;
            stored += stored < T::NS;
            load_frags(next, 0, 0);             // (not before: the registers of these fragments are the store's)
        }
        int fresh;
        if (--left > 0) {
            // tiles that ended in the last NS-1 spans
            fresh = kt < T::NS - 1 ? 1 + (KT == 1 ? T::NS - 2 - kt : KT == 2 ? (T::NS - 2 - kt) / 2 : KT == 3 ? (T::NS - 2 - kt) / 3 : 0) : 0;
            until_barrier(next, fresh < stored ? fresh : stored);
        }
    };
    while (left > 0) {
        const int next = (stage + 1 == T::NS) ? 0 : stage + 1;
        span(lds + stage * T::STAGE, lds + next * T::STAGE);
        stage = next;
    }
    // requests past the last tile write zeros to LDS: none may be in flight when the workgroup ends (its stores may)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STORES) : "memory");
}

}  // namespace g355
