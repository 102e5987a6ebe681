// Where the launches of a call end, in one place: asgd_run_steps() and a host-only check (tests/host/check_launch_cuts.cpp)
// use these.  Steps are counted from 0; a call runs the steps [t, t_end).  Plain C++, no HIP types.
#pragma once

namespace asgd {

// Rounds one launch with in-kernel waits covers at most (a longer call becomes several such launches): the waits of a workgroup
// draw on one budget of polls per launch, which the short waits of a healthy run must not use up however long the call is.
constexpr long long ONE_LAUNCH_MAX_ROUNDS = 1024;

// The streaming kernel looks out for elements beyond its limits in the first epoch after loading (6 % of the time of an epoch;
// looking at all samples while loading took as long as an epoch).  A call that begins with that epoch and goes on for fifteen
// more and longer is cut after it.  S: steps of an epoch, E: steps of a round, 0 where a launch may end at any step.  Never past t_end.
inline long long first_epoch_cut(long long t_end, long long S, long long E)
{
    const long long cut = E > 0 ? (S + E - 1) / E * E : S;
    return t_end - cut > 15 * S ? cut : t_end;
}

// End of a launch with in-kernel waits that begins at step a: a multiple of E or t_end.
inline long long one_launch_end(long long a, long long t_end, long long cut, long long E)
{
    long long b = (a / E + ONE_LAUNCH_MAX_ROUNDS) * E;
    if (b > cut) b = cut;
    return b < t_end ? b : t_end;
}

}  // namespace asgd
