// Where the launches of a call end, in one place: asgd_run_steps() and a host-only check (tests/host/check_launch_cuts.cpp)
// use these.  Steps are counted from 0; a call runs the steps [t, t_end).  Plain C++, no HIP types.
#pragma once

namespace asgd {

// Rounds one launch with in-kernel waits covers at most (a longer call becomes several such launches): the waits of a workgroup
// draw on one budget of polls per launch, which the short waits of a healthy run must not use up however long the call is.
constexpr long long ONE_LAUNCH_MAX_ROUNDS = 1024;

// Mini-batches of the shards that the streaming kernel has looked at since the samples were loaded: those of the steps [from, to).
// Step t works on mini-batch t mod S.
struct SeenSteps {
    long long from = 0, to = 0;
    bool all(long long S) const { return to - from >= S; }
    void begin(long long t, long long S)          // a run goes on at step t
    {
        if (!all(S) && (t < from || t > to)) from = to = t;
    }
    void ran(long long t)                         // ... and has got to step t
    {
        if (t > to) to = t;
    }
};

// The streaming kernel looks out for elements beyond its limits in the first S steps after loading, an epoch, or after a jump of the step
// counter (6 % of the time of an epoch, more where it meets some; looking at all samples while loading took as long as an epoch).  A call
// that begins with them and has more than an epoch and 2^29 elements to go after them is cut there: the wait and the second launch cost
// some 20 us, 6 % of that time at 5.6 TB/s.  first: where they began; E: steps of a round, 0 where a launch may end at any step;
// elements: of a step of all workers.  Never past t_end.
inline long long first_epoch_cut(long long t_end, long long first, long long S, long long E, double elements)
{
    const long long cut = E > 0 ? (first + S + E - 1) / E * E : first + S;
    return t_end - cut > S && (double)(t_end - cut) * elements > 536870912.0 ? cut : t_end;
}

// End of a launch with in-kernel waits that begins at step a: a multiple of E or t_end.
inline long long one_launch_end(long long a, long long t_end, long long cut, long long E)
{
    long long b = (a / E + ONE_LAUNCH_MAX_ROUNDS) * E;
    if (b > cut) b = cut;
    return b < t_end ? b : t_end;
}

}  // namespace asgd
