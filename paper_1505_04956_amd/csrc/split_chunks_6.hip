// Step and Eq. 8 kernels for rows of 81 to 96 columns.
#include "split_quant_screen.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_local_6(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_local<6>(r, blocks, threads, lds, s);
}
hipError_t launch_split_assign_6(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_phase<16>(l, blocks, threads, lds, s);
}
hipError_t launch_screen_quant_6(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return a.keep ? launch_screen_quant<6, true>(a, blocks, lds, s) : launch_screen_quant<6, false>(a, blocks, lds, s);
}

}  // namespace asgd
