// Step and Eq. 8 kernels for rows of more than 128 columns.
#include "split_quant.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_local_0(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return split_launch_local<0>(r, blocks, threads, lds, s);
}
hipError_t launch_split_assign_0(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    return l.run.a.wide ? split_launch_phase<9>(l, blocks, threads, lds, s) : split_launch_phase<10>(l, blocks, threads, lds, s);
}
hipError_t launch_split_quant_0(const SplitQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    return split_launch_quant<0>(a, blocks, lds, s);
}

}  // namespace asgd
