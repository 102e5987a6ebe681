// Step and Eq. 8 kernels for rows of 65 to 80 columns.
#include "split_quant_screen.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_local_5(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_local<5>(r, blocks, threads, lds, s);
}
hipError_t launch_split_assign_5(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_phase<15>(l, blocks, threads, lds, s);
}
hipError_t launch_screen_quant_5(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return a.keep ? launch_screen_quant<5, true>(a, blocks, lds, s) : launch_screen_quant<5, false>(a, blocks, lds, s);
}

}  // namespace asgd
