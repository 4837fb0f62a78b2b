#pragma once
#include <hip/hip_runtime.h>

#include "../../include/gemm.h"
#include "gemm_kernel.hpp"

// Builds that force a K-loop form or leave a part of the loop out, for comparisons, hold the variants of the table only: neither
// pipelined instantiations nor sliced ones, so that every launch runs its cfg's own tile.
#if defined(G355_FORCE_LOOP_FORM) || defined(G355_DIAG_SKIP_FILL) || defined(G355_DIAG_SKIP_FRAG) || \
    defined(G355_DIAG_SKIP_MFMA) || defined(G355_DIAG_PANEL) || defined(G355_DIAG_FILL_MODE)
#define G355_COMPARISON_BUILD
#endif

namespace g355 {
typedef hipError_t (*LaunchFn)(const KernelArgs &, hipStream_t);
// One launch by the runtime's own entry: the <<<>>> form pushes its configuration, calls a stub that pops it, and leaves its
// error for another call to fetch.  (An error that an earlier, unrelated runtime call left behind is not ours.)
template <class A>
inline hipError_t launch_kernel(void (*kernel)(A), dim3 grid, dim3 block, A args, hipStream_t stream)
{
    (void)hipGetLastError();
    void *list[] = {&args};
    return hipLaunchKernel((const void *)kernel, grid, block, list, 0, stream);
}
typedef hipError_t (*OccupancyFn)(int *blocks_per_cu);
struct VariantFns {
    LaunchFn launch;
    OccupancyFn occupancy;   // the runtime's resident-workgroups-per-CU figure for the instantiation (chained ones: none)
    int waves_m, waves_n, loop_form;
    int resident;            // chained kernels: workgroups that an XCD holds at a time
};
// (variant index inside the translation unit's list, storage of B: 0 row-major K x N, 1 K-contiguous N x K,
//  instantiation: a gemm_kernel_kind; of the pipelined ones launch is null for a tile that has none)
const VariantFns &kLaunchBf16_0(int, int, int),
    &kLaunchBf16_1(int, int, int),
    &kLaunchBf16_2(int, int, int),
    &kLaunchBf16_3(int, int, int),
    &kLaunchFp8_0(int, int, int),
    &kLaunchFp8_1(int, int, int),
    &kLaunchFp16_0(int, int, int),
    &kLaunchFp16_1(int, int, int),
    &kLaunchFp16_2(int, int, int),
    &kLaunchFp16_3(int, int, int),
    &kLaunchBf16_4(int, int, int),
    &kLaunchFp16_4(int, int, int),
    &kLaunchBf16_5(int, int, int),
    &kLaunchFp16_5(int, int, int);   // fp16 shares the bf16 variant lists

// The chained kernel of a tile size (ragged: the instantiation that trims), whatever slab depth and wave grid the variant has;
// launch is null for sizes that have none.
const VariantFns &chained_bf16(int block_m, int block_n, int b_layout, int ragged), &chained_fp16(int, int, int, int), &chained_fp8(int, int, int, int);
// The pipelined kernels of a tile size: direct ones of the sizes other than 256x256, streaming ones for one tile row over large
// weights, and of 256x256 one for grouped launches; launch is null for sizes that have none, and in a comparison build for all.
enum PipelinedForm { PIPELINED_DIRECT, PIPELINED_STREAMING, PIPELINED_GROUPED };
const VariantFns &pipelined_bf16(int block_m, int block_n, int b_layout, int ragged, int form), &pipelined_fp16(int, int, int, int, int),
    &pipelined_fp8(int, int, int, int, int);
// The sliced kernel: 16x16 tiles, four K slices in a workgroup (launch: as above).
const VariantFns &sliced_bf16(int b_layout, int ragged), &sliced_fp16(int, int), &sliced_fp8(int, int);
}  // namespace g355
