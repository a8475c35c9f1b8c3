/* Ragged kernel of size class 2, sizes 1..16 (see kernels_ragged.h): 113 VGPRs,
 * 4 waves per SIMD. A build of an earlier form of this kernel that spilled returned wrong,
 * run-to-run different solutions for some size-16 systems: it is kept free of
 * scratch memory. */
#include "kernels_ragged.h"

namespace lupp {

__global__ void __launch_bounds__(kRaggedThreads)
    __attribute__((amdgpu_waves_per_eu(ragged_class_waves(2), ragged_class_waves(2)))) k_ragged_c2(RaggedArgs a)
{
    ragged_class_item<2>(a);
}

hipError_t ragged_c2_launch(const RaggedArgs &a, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_ragged_c2, dim3(grid), dim3(kRaggedThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace lupp
