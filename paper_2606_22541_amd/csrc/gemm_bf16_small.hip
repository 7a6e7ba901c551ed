// bf16 expert FFN for passes all of whose groups are known to be small (see
// ffn_bf16.h): the kernel without the large tiles' code.
#include "ffn_bf16.h"

namespace moe {

hipError_t launch_ffn_bf16_small(const FfnArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_ffn_bf16<false>, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace moe
