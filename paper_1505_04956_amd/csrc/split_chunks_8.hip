// Assignment kernel for rows of up to 128 columns.
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_assign_8(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s)
{
    hipError_t e = hipFuncSetAttribute((const void *)split_assign_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_assign_kernel<8>, dim3(blocks), dim3(threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace asgd
