/* Ragged kernel of size class 2, sizes 1..16 (see kernels_ragged.h): 114 VGPRs,
 * 4 waves per SIMD. An earlier form of it (the ds_bpermute solver, a resident
 * grid, 4 waves per SIMD) spilled 144 bytes per lane, 80 once the lane table
 * became word-sized, and returned wrong, run-to-run different solutions for some
 * size-16 systems (7 to 42 of 200 sampled per run), while the per-size kernels
 * of the same solver without scratch were exact. The cause is unknown. A test on
 * the host checks that this kernel, like all others, uses no scratch memory. */
#include "kernels_ragged.h"

namespace lupp {

__global__ void __launch_bounds__(kRaggedThreads)
    __attribute__((amdgpu_waves_per_eu(ragged_class_waves(2), ragged_class_waves(2)))) k_ragged_c2(RaggedArgs a)
{
    ragged_class<2>(a);
}

hipError_t ragged_c2_launch(const RaggedArgs &a, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_ragged_c2, dim3(grid), dim3(kRaggedThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace lupp
