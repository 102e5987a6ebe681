// Host-only check of the LDS layout of the step kernels with fp16-split operands (csrc/split_plan.h): whatever the state and the
// mini-batch, a workgroup's LDS fits a compute unit, the regions do not overlap, and the two mini-batches of a kept worker have room
// for what their fetch writes.
#include <cstdio>
#include <cstdlib>

#include "split_plan.h"

using namespace asgd;

#define REQUIRE(c) do { if (!(c)) { printf("FAIL %s: k %d d %d b %d W %d local %d\n", #c, k, d, b, W, local); return 1; } } while (0)

int main(int argc, char **argv)
{
    const int d = argc > 1 ? atoi(argv[1]) : 7, W = argc > 2 ? atoi(argv[2]) : 192;
    long long plans = 0, kept = 0, full = 0;
    for (int k = 2; k <= 7680; k += k < 1200 ? 1 : 61)
        for (int b = 1; b <= 20000; b += b < 3000 ? 3 : 59)
            for (int local = 0; local < 2; ++local) {
                const SplitPlan q = split_plan(k, d, b, W, local != 0);
                REQUIRE(q.lds <= SPLIT_LDS_ALL && q.lds_sums <= SPLIT_LDS_ALL);
                REQUIRE(q.off_cells % 16 == 0 && q.off_cnt % 16 == 0 && q.off_hs % 16 == 0 && q.off_ms % 16 == 0 && q.off_args % 16 == 0 && q.off_batch % 16 == 0);
                REQUIRE(q.off_cells >= (q.resident ? q.frag_bytes : 0) && q.off_hs >= q.off_cnt + (q.fused ? 4u * k : 0));
                REQUIRE(!q.fused || q.off_cnt >= q.off_cells + 8u * k * ((d + 1) / 2 * 2));
                REQUIRE(q.off_ms >= q.off_hs + 4u * q.kpad && q.off_args >= q.off_ms + 4u * q.dpad);
                if (q.kept) {
                    REQUIRE(local && q.fused && q.resident && q.shares == 1 && q.waves == 8);
                    REQUIRE(q.off_batch >= q.off_args + 8 * 64 * 4 && q.off_batch + 2 * q.batch_bytes + SPLIT_LDS_SHARED <= q.lds);
                    REQUIRE(q.batch_bytes % 1024 == 0 && q.batch_bytes >= 4u * b * d);       // sweeps of 1 KB (16 bytes a lane) or 256 bytes
                    ++kept;
                    full += q.lds > SPLIT_LDS_ALL - 1024;
                }
                if (q.screen) {
                    const unsigned pair = q.nch * 2 * SPLIT_PIECE, operands = SPLIT_LISTED / 32 * pair, best = 8 * SPLIT_LISTED / 64 * 5 * 64 * 4;
                    REQUIRE(q.stage_pairs >= 1 && q.stages * q.stage_pairs >= q.npair && (q.stages - 1) * q.stage_pairs < q.npair);
                    REQUIRE(q.off_cells >= (q.stages > 1 ? 2 : 1) * q.stage_pairs * pair && q.off_cells >= operands && q.off_cells >= best && q.off_cells >= SPLIT_HARD * 8 * 16);
                    REQUIRE(q.off_list >= q.off_args + 2 * SPLIT_LISTED / 32 * 64 * 4 && q.off_list + 4 * SPLIT_LIST + SPLIT_LDS_SHARED <= q.lds);
                    REQUIRE(SPLIT_LIST >= 2 * 8 * 128);            // a sweep of eight waves adds at most as many as there is room
                    REQUIRE(q.off_cells >= 2u * q.nch * 4 * SPLIT_PIECE && !q.fused && !q.resident);            // the stages of the item without screening
                }
                if (q.wide) {
                    REQUIRE(q.longrow && q.waves == 8 && q.off_cells >= 64u * 4 * q.dpad && q.off_args + 8 * 64 * 4 * 7 + SPLIT_LDS_SHARED <= q.lds);
                    REQUIRE(SPLIT_HARD * 8 * 16 <= 8 * 64 * 4 * 5 && (!local || q.shares == 1));
                    // no other cut leaves a compute unit fewer groups of 64 samples one after the other, starts counted as half a group
                    auto cost = [&](long long shares, long long len) { return (W * shares + SPLIT_CUS - 1) / SPLIT_CUS * (2 * len + 1); };
                    for (int len = 1; !local && k % 32 == 0 && len <= 64; ++len) {
                        const int shares = ((b + 63) / 64 + len - 1) / len;
                        REQUIRE(shares > 64 || cost(q.shares, q.share_len / 64) <= cost(shares, len));
                    }
                }
                ++plans;
            }
    printf("ok %lld plans, %lld kept, %lld of them within 1 KB of the limit\n", plans, kept, full);
    return 0;
}
