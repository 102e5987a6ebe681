// Which elements of the samples the streaming kernel's column maxima are formed of when the samples are loaded, in one place:
// the kernel (kernels_generic.hip) and a host-only check (tests/host/check_sample_index.cpp) use these.  Plain C++, no HIP types.
#pragma once

#include "exchange_index.h"      // ASGD_HD

namespace asgd {

// The samples are total = rows * d floats (d <= 16).  Pieces of 16 sweeps of a workgroup of T threads, T a multiple of d, so that a
// thread stays in one column.  All pieces up to 8191 (128 MB), then 4096 and more evenly spread ones, 1 in 128 at the least;
// whoever uses the maxima looks out for elements beyond them.  (All samples of N = 1e8, d = 10: 675 us, as long as an epoch over them.)
constexpr int SAMPLE_SWEEPS = 16;
ASGD_HD inline int sample_threads(int d) { return 256 - 256 % d; }
ASGD_HD inline long long sample_pieces(long long total, int d)
{
    const long long piece = (long long)SAMPLE_SWEEPS * sample_threads(d);
    return (total + piece - 1) / piece;
}
ASGD_HD inline long long sample_every(long long pieces)
{
    const long long n = pieces / 4096;
    return n < 1 ? 1 : n > 128 ? 128 : n;
}
// Element that thread t looks at in a sweep of a piece: past the end of the samples the first one of the thread's column.
ASGD_HD inline long long sample_element(long long piece, int sweep, int t, long long total, int d)
{
    const long long e = (piece * SAMPLE_SWEEPS + sweep) * sample_threads(d) + t;
    return e < total ? e : t % d;
}

}  // namespace asgd
