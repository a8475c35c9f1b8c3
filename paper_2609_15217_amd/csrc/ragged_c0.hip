/* Ragged kernel of size class 0, sizes 22..32 (see kernels_ragged.h): 166
 * VGPRs, 3 waves per SIMD. */
#include "kernels_ragged.h"

namespace lupp {

__global__ void __launch_bounds__(kRaggedThreads)
    __attribute__((amdgpu_waves_per_eu(ragged_class_waves(0), ragged_class_waves(0)))) k_ragged_c0(RaggedArgs a)
{
    ragged_class<0>(a);
}

hipError_t ragged_c0_launch(const RaggedArgs &a, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_ragged_c0, dim3(grid), dim3(kRaggedThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace lupp
