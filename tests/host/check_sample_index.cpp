// Host-only check of the elements that column maxima over a part of the samples look at (csrc/sample_index.h): every one lies
// inside the samples and in the thread's column; small data are looked at whole.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "sample_index.h"

using namespace asgd;

int main(int argc, char **argv)
{
    const int d = argc > 1 ? atoi(argv[1]) : 10;
    const long long lo = argc > 2 ? atoll(argv[2]) : 1, hi = argc > 3 ? atoll(argv[3]) : 100;
    long long looked = 0;
    for (long long rows = lo; rows <= hi; ++rows) {
        const long long total = rows * d, pieces = sample_pieces(total, d), every = sample_every(pieces);
        std::vector<char> seen(every == 1 ? total : 0);
        for (long long q = 0; q < pieces; q += every)
            for (int u = 0; u < SAMPLE_SWEEPS; ++u)
                for (int t = 0; t < sample_threads(d); ++t) {
                    const long long e = sample_element(q, u, t, total, d);
                    if (e < 0 || e >= total || e % d != t % d) {
                        printf("FAIL rows %lld piece %lld sweep %d thread %d: element %lld\n", rows, q, u, t, e);
                        return 1;
                    }
                    if (every == 1) seen[e] = 1;
                    ++looked;
                }
        for (char s : seen)
            if (!s) {
                printf("FAIL rows %lld: not looked at whole\n", rows);
                return 1;
            }
    }
    printf("ok %lld\n", looked);
    return 0;
}
