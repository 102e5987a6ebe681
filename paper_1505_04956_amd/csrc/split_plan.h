// Step kernels with fp16-split operands: what lies where in the LDS of a workgroup, how a mini-batch is cut into shares, and when a
// worker is kept in the LDS from step to step.  The launcher and a host-only check (tests/host/check_split_plan.cpp) use it.  Plain
// C++, no HIP types.
#pragma once

#include <stddef.h>

namespace asgd {

constexpr int SPLIT_PIECE = 1024;                 // bytes of 32 rows x 16 columns of one part
constexpr unsigned SPLIT_LDS_SHARED = 512;        // what all phases share, before everything else
constexpr unsigned SPLIT_LDS_ALL = 160 * 1024;    // LDS of a compute unit
constexpr unsigned SPLIT_LDS = 150 * 1024;        // what operands and cells may take of it
constexpr int SPLIT_CUS = 256;
constexpr int SPLIT_HARD = 32;                    // samples that may wait for a scan of all the rows by a whole workgroup
constexpr int SPLIT_LISTED = 128;                 // of them at a time
constexpr int SPLIT_LIST = 2048;                  // undecided samples of a screened mini-batch that are noted before they are scored again
constexpr int SPLIT_UNSCREENED = 15;              // items without screening after one that was given up
constexpr int SPLIT_KEPT_CHUNKS = 4;              // longest rows of a kept worker: beyond, its kernel needs more registers than there are

struct SplitPlan {
    int nch, dpad, nblk, kpad, npair;
    size_t frag_bytes;
    bool longrow, fused, resident, kept;
    bool wide;                     // rows of more than 128 columns, the operands of 64 samples fit the LDS
    bool screen;                   // samples are screened (split_screen.h)
    int stage_pairs, stages;       // row pairs of a stage of high parts; stages of the state (one: it stays)
    unsigned off_list;
    int waves, shares, share_len, grid;
    unsigned off_cells, off_cnt, off_hs, off_ms, off_args, off_batch, batch_bytes, lds;
    int dc, ncol, sum_shares, sum_len;      // sums in a launch of their own: columns per workgroup, shares
    unsigned lds_sums;
    int g, upd_blocks;             // update: lanes per row, workgroups per worker
};

inline int split_padded_row(int d) { return d > 128 ? (d + 127) / 128 * 128 : (d + 15) / 16 * 16; }
inline unsigned split_round16(size_t v) { return (unsigned)((v + 15) / 16 * 16); }

// Of `screened` samples of a workgroup `open` are undecided: is the rest better off without screening?  An undecided sample costs its screening, a
// second read and conversion and all three products, with few other samples to share the state's operands.  Microseconds per step with three
// products for all, with all of them screened, and given up (samples next to one of two equal rows, share): k = 1024, d = 128, b = 4096: 10 %
// 13510, 11070, -, 20 % 20720, 20310, 20720, 30 % 21870, 28730, 21890, all 30150, 83880, 30130; k = 600, d = 60, b = 1500: 20 % 211, 210, -, 30 % 219, 230, 238, all 273,
// 381, 294; k = 2000, d = 20, b = 800: 30 % 262, 229, -, 50 % 273, 267, 282, all 297, 350, 310.  One column a thousand times as wide as the others:
// k = 1024, d = 64, b = 1500 6457, 18126, 6477.
inline constexpr bool split_screen_gives_up(int open, int screened, int nch) { return (long long)open * (nch <= 3 ? 2 : nch == 4 ? 4 : 6) > screened; }

// Rows of more than 128 columns, phases, one workgroup per compute unit: the cut of a mini-batch of `groups` groups of 64 samples that takes the fewest
// groups one after the other, half a group counted for a workgroup's start.  `even`: in one round that fills the device,
// or of two groups at most.
// (256 / W shares, rounded down, one beyond 256 workers: microseconds per step with those and with these, k = 160, d = 200, b = 2000: W = 100 258, 239, 129
// 432, 308, 190 482, 413, 257 838, 582, 380 939, 779, 600 1507, 1331; k = 256, d = 384, b = 512: W = 150 287, 271, 300 560, 497; the same cut at W = 64, 120, 256,
// 512.)
struct SplitCut { int shares; bool even; };
inline SplitCut split_wide_cut(int W, int groups)
{
    SplitCut best = {1, true};
    long long least = -1;
    for (int s = 1; s <= groups && s <= 64; ++s) {
        const int len = (groups + s - 1) / s, cut = (groups + len - 1) / len;
        const long long rounds = ((long long)W * cut + SPLIT_CUS - 1) / SPLIT_CUS, cost = rounds * (2 * len + 1);
        if (least >= 0 && cost >= least) continue;
        least = cost;
        best.shares = cut;
        best.even = rounds == 1 && (len <= 2 || 4LL * W * cut >= 3 * SPLIT_CUS);
    }
    return best;
}

inline SplitPlan split_plan(int k, int d, int b, int W, bool local)
{
    SplitPlan q = {};
    q.longrow = d > 128;
    q.dpad = split_padded_row(d);
    q.nch = q.dpad / 16;
    q.nblk = (k + 31) / 32;
    q.npair = (q.nblk + 1) / 2;
    q.kpad = q.npair * 64;
    q.frag_bytes = (size_t)q.npair * q.nch * 4 * SPLIT_PIECE;
    const size_t cells = (size_t)k * ((d + 1) & ~1) * 8 + (size_t)k * 4;
    const size_t fixed = (size_t)q.kpad * 4 + (size_t)q.dpad * 4 + 8 * 64 * 4 + 64;
    const size_t stage2 = q.longrow ? 0 : (size_t)2 * q.nch * 4 * SPLIT_PIECE;
    const size_t group = (size_t)64 * q.dpad * 4, wide_others = (size_t)q.kpad * 4 + (size_t)q.dpad * 4 + 8 * 64 * 4 * 7 + 64;
    // One workgroup per compute unit, 64 samples at a time, its waves share the state's blocks of 32 rows: with few blocks only as long as there are few
    // groups of 64 for a workgroup, because elsewhere every wave has one of its own.  Microseconds per step before and with it: k = 256, d = 384,
    // b = 512: W = 64 171, 110, W = 256 497, 374; k = 300, d = 500, b = 1000, W = 16 196, 78; k = 160, d = 200, b = 4000, W = 256 1394, 1067; k = 128 974,
    // 949; d = 150: k = 100, b = 2000, W = 256 523, 515; k = 20, b = 1000, W = 64 (four groups) 73, 71, b = 2000 90, 118; k = 50, b = 2000, W = 256 368, 473.
    // Four groups that do not fill the device, one or two blocks: k = 20, d = 150, b = 250, W = 150 50, 58, W = 300 98, 111; fewer groups: k = 20, d = 150, b = 130,
    // W = 150 47, 46, W = 300 81, 76; b = 64, W = 600 106, 74; b = 500, W = 4 50, 32.
    const int groups = (b + 63) / 64, one_round = W < SPLIT_CUS && !local ? SPLIT_CUS / W : 1;
    const SplitCut cut = q.longrow && !local ? split_wide_cut(W, groups) : SplitCut{1, true};
    const bool wide_few = (groups + one_round - 1) / one_round <= 4 && (q.nblk == 3 || cut.even || groups <= 3);
    q.wide = q.longrow && group + wide_others <= SPLIT_LDS && (q.nblk >= 4 || wide_few);
    if (q.longrow) {
        q.resident = q.fused = false;
    } else if (q.frag_bytes + cells + fixed <= SPLIT_LDS) {
        q.resident = q.fused = true;
    } else if (stage2 + cells + fixed <= SPLIT_LDS) {
        q.resident = false;
        q.fused = true;
    } else {
        q.fused = false;
        q.resident = q.frag_bytes + fixed <= SPLIT_LDS;
    }
    // Screening (split_screen.h) saves two of three products and pays one pass over the state, and barriers, for the few samples it leaves open: where
    // the state has to be streamed in any case and a step is one workgroup's.  Microseconds of a step, all three products and
    // screened: k = 1024, d = 128: b = 100 323, 348, 500 383, 373, 2000 705, 543, 4096 1130, 780; k = 512, d = 128: b = 1000 293, 288, 4096 685, 544; k = 1024, d = 64: b = 1500
    // 318, 254.  (Not where the state stays in the LDS: k = 200, d = 100, b = 2000 119, 142; not in phases, whose launches are
    // as long as the slowest of the workgroups with something left open: k = 300, d = 128, W = 8, b = 500 36, 57.)
    q.screen = local && !q.longrow && !q.fused && !q.resident && q.nch >= 2 && b >= 384;
    unsigned o = split_round16(q.resident ? q.frag_bytes : stage2);
    if (q.screen) {
        const size_t pair = (size_t)q.nch * 2 * SPLIT_PIECE, others = fixed + SPLIT_LIST * 4;
        const size_t listed = (size_t)SPLIT_LISTED / 32 * (q.nch > 3 ? q.nch : 3) * 2 * SPLIT_PIECE;      // (operands, then the best scores of eight waves)
        q.resident = false;
        q.stage_pairs = q.npair;
        if (q.npair * pair + others > SPLIT_LDS) q.stage_pairs = (int)((SPLIT_LDS - others) / (2 * pair));
        q.stages = (q.npair + q.stage_pairs - 1) / q.stage_pairs;
        o = (unsigned)((q.stages > 1 ? 2 : 1) * q.stage_pairs * pair);
        if (o < listed) o = (unsigned)listed;
    }
    if (q.wide) o = (unsigned)group;
    q.off_cells = o;
    if (q.fused) o += split_round16((size_t)k * ((d + 1) & ~1) * 8);
    q.off_cnt = o;
    if (q.fused) o += split_round16((size_t)k * 4);
    q.off_hs = o;  o += split_round16((size_t)q.kpad * 4);
    q.off_ms = o;  o += split_round16((size_t)q.dpad * 4);
    q.off_args = o; o += 8 * 64 * 4 * (q.wide ? 7 : q.longrow ? 5 : 1);
    q.off_list = o; o += q.screen ? SPLIT_LIST * 4 : 0;
    // (two mini-batches of a kept worker: the next one arrives while the current one is worked on; a fetch writes whole KBs)
    q.batch_bytes = (unsigned)(((size_t)(b < 16384 ? b : 16384) * d * 4 + 1023) / 1024 * 1024);
    q.kept = local && q.fused && q.resident && q.nch <= SPLIT_KEPT_CHUNKS && W <= SPLIT_CUS && b <= 16384 && (size_t)o + 2 * (size_t)q.batch_bytes + SPLIT_LDS_SHARED <= SPLIT_LDS_ALL;
    // (at whole KBs where there is room: k = 64, d = 32, W = 256, b = 500, E = 1, 31 steps 1303 -> 1300 us)
    const unsigned whole = (o + 1023) / 1024 * 1024;
    if (q.kept && (size_t)whole + 2 * (size_t)q.batch_bytes + SPLIT_LDS_SHARED <= SPLIT_LDS_ALL) o = whole;
    q.off_batch = o;
    if (q.kept) o += 2 * q.batch_bytes;
    q.lds = o;
    // Phases: waves of a workgroup and shares of a mini-batch - enough workgroups for the compute units first, then as many
    // waves per workgroup as share the staged operands, and as many workgroups as are resident at once (three waves per
    // SIMD up to 32 columns, two above).
    q.waves = 8;
    q.shares = 1;
    if (q.longrow) {
        // (the waves of a workgroup share the rows of its groups of samples, see split_assign_wide_item and split_assign_long_item)
        int rsplit = q.wide ? 8 : 1;
        while (2 * rsplit <= q.npair && 2 * rsplit <= 8) rsplit *= 2;
        const int max_shares = (groups + 8 / rsplit - 1) / (8 / rsplit);
        if (!local) q.shares = q.wide ? cut.shares : (2 * SPLIT_CUS + W - 1) / W;
        if (q.shares > max_shares) q.shares = max_shares;
        if (q.shares > 64) q.shares = 64;
    } else if (!local) {
        int nw = q.lds <= 50 * 1024 ? 4 : 8;
        // (with one workgroup per compute unit a second round must not begin)
        const int fill = q.lds > 78 * 1024 ? SPLIT_CUS * 3 / 8 : SPLIT_CUS;
        while (nw > 1 && (long long)W * ((groups + nw - 1) / nw) < fill) nw /= 2;
        q.waves = nw;
        const int max_shares = (groups + nw - 1) / nw;
        const int want = SPLIT_CUS * (q.nch <= 2 && q.lds <= 50 * 1024 ? 12 : 8) / nw;
        q.shares = (want + W - 1) / W;
        if (q.shares > max_shares) q.shares = max_shares;
        if (q.shares > 64) q.shares = 64;
    }
    q.share_len = (groups + q.shares - 1) / q.shares * 64;
    q.shares = (b + q.share_len - 1) / q.share_len;
    if (!q.fused) {
        auto bytes = [&](int dc) { return (size_t)k * ((dc + 1) * 8 + 4); };
        int dc = 64;
        while (dc > 8 && bytes(dc) > 72 * 1024) dc /= 2;
        if (dc < 16 && bytes(16) <= SPLIT_LDS) dc = 16;         // (rows in pieces of 64 bytes, even with one workgroup per compute unit)
        while (dc > 1 && bytes(dc) > SPLIT_LDS) dc /= 2;
        q.dc = dc;
        q.ncol = (d + dc - 1) / dc;
        q.lds_sums = split_round16(bytes(dc));
        // (every share writes and the update reads the sums of a whole state: no more than fill the device)
        int ss = local ? 1 : 2 * SPLIT_CUS / (W * q.ncol);
        if (ss > groups / 8) ss = groups / 8;
        if (ss < 1) ss = 1;
        q.sum_len = (groups + ss - 1) / ss * 64;
        q.sum_shares = (b + q.sum_len - 1) / q.sum_len;
    } else {
        q.sum_shares = q.shares;
        q.sum_len = q.share_len;
    }
    int g = 1;
    while (g < q.dpad / 8 && g < 64) g *= 2;
    q.g = g;
    // workgroups of the update per worker (256 threads): enough for four on every compute unit, as long as each has rows to do
    q.upd_blocks = local ? 1 : (4 * SPLIT_CUS + W - 1) / W;
    const int row_groups = (k + 256 / g - 1) / (256 / g);
    if (q.upd_blocks > row_groups) q.upd_blocks = row_groups;
    q.grid = W < SPLIT_CUS ? W : SPLIT_CUS;
    if (local && !q.fused && q.lds < q.lds_sums) q.lds = q.lds_sums;
    q.lds_sums += SPLIT_LDS_SHARED;
    q.lds += SPLIT_LDS_SHARED;
    return q;
}

}  // namespace asgd
