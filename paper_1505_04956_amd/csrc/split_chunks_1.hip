// Step and Eq. 8 kernels for rows of 1 to 16 columns.
#include "split_quant_screen.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_local_1(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_local<1>(r, blocks, threads, lds, s);
}
hipError_t launch_split_assign_1(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_phase<11>(l, blocks, threads, lds, s);
}
hipError_t launch_split_quant_1(const SplitQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return split_launch_quant<1>(a, blocks, lds, s);
}
hipError_t launch_screen_quant_1(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return launch_screen_quant<1, true>(a, blocks, lds, s);          // (always kept)
}

}  // namespace asgd
