// Step and Eq. 8 kernels for rows of 17 to 32 columns.
#include "split_quant_screen.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_local_2(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_local<2>(r, blocks, threads, lds, s);
}
hipError_t launch_split_assign_2(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_phase<12>(l, blocks, threads, lds, s);
}
hipError_t launch_screen_quant_2(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return launch_screen_quant<2, true>(a, blocks, lds, s);          // (always kept)
}

}  // namespace asgd
