// Host-only check of where the launches of a call end (csrc/launch_cuts.h), built with the plain C++ compiler: whatever the
// epoch, the round and the length of the call, the launches are the steps of the call, each once and no more.
#include <cstdio>
#include <initializer_list>

#include "launch_cuts.h"

using namespace asgd;

#define REQUIRE(c) do { if (!(c)) { printf("FAIL %s: S %lld E %lld t %lld steps %lld\n", #c, S, E, t, steps); return 1; } } while (0)

int main()
{
    long long calls = 0, cuts = 0;
    for (long long S : {1LL, 2LL, 3LL, 7LL, 97LL, 50000LL})
        for (long long E : {0LL, 1LL, 2LL, 8LL, 100LL, 2000LL, 1000000LL, 2000000000LL})
            for (long long steps : {1LL, S, 15 * S, 16 * S, 16 * S + 1, 17 * S, 17 * S + 3, 40 * S + 1, 16 * S + E, 17 * S + E + 2})
                for (long long t : {0LL, 1LL, S - 1, E, 5 * S}) {
                    const long long t_end = t + steps, cut = first_epoch_cut(t_end, t, S, E, 1e7);
                    REQUIRE(cut <= t_end);
                    REQUIRE(cut == t_end || (cut >= t + S && cut < t_end && (E == 0 || cut % E == 0)));
                    REQUIRE(steps <= 2 * S + E || steps <= S + E + 54 || cut < t_end);
                    cuts += cut < t_end;
                    ++calls;
                    if (E == 0) continue;
                    int launches = 0;
                    for (long long a = t; a < t_end;) {
                        const long long b = one_launch_end(a, t_end, a < cut ? cut : t_end, E);
                        REQUIRE(b > a && b <= t_end && (b == t_end || b % E == 0));
                        REQUIRE(b / E - a / E <= ONE_LAUNCH_MAX_ROUNDS);
                        a = b;
                        ++launches;
                    }
                    REQUIRE(launches <= 2 + steps / E / ONE_LAUNCH_MAX_ROUNDS + 1);
                }
    // the cut would lie behind the end of the call
    const double all = 1.024e7;                            // 1024 workers, 1000 samples of ten columns: 97 steps are 4 GB
    if (first_epoch_cut(1649, 0, 97, 2000, all) != 1649 || one_launch_end(0, 1649, first_epoch_cut(1649, 0, 97, 2000, all), 2000) != 1649) return 1;
    if (first_epoch_cut(51, 0, 3, 100, all) != 51 || first_epoch_cut(3 * 97, 0, 97, 8, all) != 104 || first_epoch_cut(3 * 97, 0, 97, 0, all) != 97) return 1;
    if (first_epoch_cut(2 * 97, 0, 97, 0, all) != 2 * 97 || first_epoch_cut(16 * 3, 0, 3, 0, all) != 16 * 3 || first_epoch_cut(20 * 3, 0, 3, 0, all) != 3) return 1;
    // runs in pieces, a step back, a jump: only an unbroken stretch of S steps is all mini-batches
    SeenSteps seen;
    for (long long t : {0LL, 40LL, 10LL}) {
        seen.begin(t, 97);
        seen.ran(t + 40);
        if (seen.all(97)) return 1;
    }
    seen.begin(1000, 97);
    seen.ran(1050);
    if (seen.all(97) || seen.from != 1000) return 1;
    seen.begin(1050, 97);
    seen.ran(1097);
    if (!seen.all(97)) return 1;
    seen.begin(5, 97);
    seen.ran(6);
    if (!seen.all(97)) return 1;
    printf("ok %lld calls, %lld cut\n", calls, cuts);
    return 0;
}
