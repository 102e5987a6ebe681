// Host-only check of the limit of a term whose column maximum was formed of a part of the samples (csrc/fixed_point_sums.h).
#include <cstdio>
#include <cstdlib>

#include "fixed_point_sums.h"

using namespace asgd;

#define REQUIRE(c) do { if (!(c)) { printf("FAIL %s: b %d xmax %g most %g limit %d\n", #c, b, x, most, limit); return 1; } } while (0)

int main(int argc, char **argv)
{
    const int b = argc > 1 ? atoi(argv[1]) : 1000;
    for (double x = 1e-20; x < 1e20; x *= 1.0371) {
        const float scale = fx_column_scale(b, (float)x);
        const double most = (double)(float)x * scale;
        const int limit = fx_term_limit(b, (float)most);
        REQUIRE(scale > 0.0f && limit % 2 == 0);
        REQUIRE((double)b * limit <= 2147483647.0);                       // a sum of b terms keeps to 32 bits
        REQUIRE(limit < 4194304 && 2.0 * limit < 8388608.0);             // magic constant; offset and term among the denormal numbers
        // a quarter above the largest element wherever the two bounds above leave room; never below it by more than the rounding to even
        const double room = 2147483647.0 / b < 4194303.0 ? 2147483647.0 / b : 4194303.0;
        REQUIRE(limit + 2.0 >= (1.25 * most < room ? 1.25 * most : room));
        REQUIRE(limit + 2.0 >= most);
    }
    printf("ok %d\n", b);
    return 0;
}
