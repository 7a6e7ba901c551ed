// bf16 expert FFN for passes with groups of any size (see ffn_bf16.h).
#include "ffn_bf16.h"

namespace moe {

hipError_t launch_ffn_bf16(const FfnArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_ffn_bf16<true>, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace moe
