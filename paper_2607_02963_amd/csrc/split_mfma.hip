// Launches of the matrix-core split kernels (kernel_mfma.h).  This
// translation unit is compiled on its own, with the IEEE mode bit clear and
// without NaN semantics (see the build script): the compiler then drops the
// quieting v_max(x, x) it otherwise puts before every operand of the
// softmax's maxima, which matters in the vector-ALU-bound block loop.  The
// vector-ALU kernels, whose code the same flags make slower, stay in
// pdec_api.hip.
#include <hip/hip_runtime.h>

#include "kernel_mfma.h"
#include "kernel_mfma32.h"
#include "kernel_branch.h"

namespace pdec {

namespace {

template <int D, bool PLAN>
void launch_shape(const StepArgs& a, int shape, int grid, hipStream_t s)
{
    if constexpr (D == 128) {
        // 32-row tiles (decode step at D = 128): 256 rows as eight row waves,
        // 128 rows as four row waves x two key groups
        if (shape == 4) {
            hipLaunchKernelGGL((split_m32_kernel<8, 1, PLAN>), dim3(grid), dim3(512), 0, s, a);
            return;
        }
        if (shape == 5) {
            hipLaunchKernelGGL((split_m32_kernel<4, 2, PLAN>), dim3(grid), dim3(512), 0, s, a);
            return;
        }
    }
    switch (shape) {
    case 1: hipLaunchKernelGGL((split_mfma_kernel<D, 1, 4, 2, PLAN>), dim3(grid), dim3(512), 0, s, a); break;
    case 2:
        // 128 rows: eight one-tile row waves x two key groups at D = 128
        // (3-4% faster than four two-tile row waves on the decode loop and
        // the ragged batch); four two-tile row waves otherwise (D = 64, and
        // the self-only plan mask, whose sixteen-wave form the compiler gives
        // private memory)
        if constexpr (D == 128 && !PLAN)
            hipLaunchKernelGGL((split_mfma_kernel<D, 1, 8, 2, PLAN>), dim3(grid), dim3(1024), 0, s, a);
        else
            hipLaunchKernelGGL((split_mfma_kernel<D, 2, 4, 2, PLAN>), dim3(grid), dim3(512), 0, s, a);
        break;
    default:
        // 256 rows: sixteen one-tile row waves at D = 128 (four waves per SIMD
        // hide more latency than eight two-tile waves); eight two-tile waves
        // at D = 64, whose sixteen-wave form the compiler gives private-memory
        // arrays
        if constexpr (D == 128)
            hipLaunchKernelGGL((split_mfma_kernel<D, 1, 16, 1, PLAN>), dim3(grid), dim3(1024), 0, s, a);
        else
            hipLaunchKernelGGL((split_mfma_kernel<D, 2, 8, 1, PLAN>), dim3(grid), dim3(512), 0, s, a);
        break;
    }
}

}  // namespace

// The self-only plan mask has kernels of its own, so that the full design's
// inner loop carries none of its tests.
void launch_split_mfma(const StepArgs& a, int shape, int grid, hipStream_t stream)
{
    const bool plan = a.plan_T > 0;
    if (a.D == 128) {
        if (plan) launch_shape<128, true>(a, shape, grid, stream);
        else launch_shape<128, false>(a, shape, grid, stream);
    } else {
        if (plan) launch_shape<64, true>(a, shape, grid, stream);
        else launch_shape<64, false>(a, shape, grid, stream);
    }
}

namespace {

template <int D, bool CROSS>
void launch_branch_rows(const StepArgs& a, int own_bound, bool rows_first, hipStream_t s)
{
    const dim3 grid((unsigned)(8 * ((a.n_items + 7) / 8))), block(256);
    if (a.rows_per_item == 256) hipLaunchKernelGGL((branch_kernel<D, 2, 4, CROSS>), grid, block, 0, s, a, own_bound, (int)rows_first);
    else hipLaunchKernelGGL((branch_kernel<D, 1, 4, CROSS>), grid, block, 0, s, a, own_bound, (int)rows_first);
}

}  // namespace

// Whole branches: 64 rows per wave (two tiles) in groups of 256 rows, 32 in
// groups of 128.  The causal-attention variant has kernels of its own.
void launch_branch(const StepArgs& a, int own_bound, bool rows_first, hipStream_t s)
{
    if (a.D == 128) {
        if (a.cross) launch_branch_rows<128, true>(a, own_bound, rows_first, s);
        else launch_branch_rows<128, false>(a, own_bound, rows_first, s);
    } else {
        if (a.cross) launch_branch_rows<64, true>(a, own_bound, rows_first, s);
        else launch_branch_rows<64, false>(a, own_bound, rows_first, s);
    }
}

}  // namespace pdec
