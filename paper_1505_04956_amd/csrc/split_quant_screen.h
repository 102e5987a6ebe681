// Eq. 8 for rows of 8 to 128 columns: the state is split once per call (splitq_operands_kernel) and streamed through the LDS, samples
// are screened with the high parts alone (split_screen.h), and the few that are not decided by that are noted and scored with all
// three products, 64 at a time, as in split_quant.h.  All add the direct distance to their nearest row in fp64, those alone excepted of which no score says
// anything (split_quant.h: "decided in direct form"): they add the smallest of their fp32 distances to all the rows.
//
// Two workgroups of four waves per compute unit, whose barriers are their own.  A wave takes up to four tiles of 32 samples, 4 NC
// registers each, so that a state operand read from the LDS is used as often.  k = 1024, d = 128, 5e6 samples: 4.8 ms with three
// products and the state split by every workgroup for every 512 samples, 1.6 now, of which the matrix instructions and insertions take
// 0.85, loading and converting the samples 0.6 (4.3 TB/s) and the distances 0.4; waves that start apart, priorities and a
// deeper queue of stages changed nothing.  k = 37, d = 75, 4e6 samples: 507 us, 283 now (4.2 TB/s).  Where every sample has two nearest rows, the
// second case takes as long as with three products for all (2e6 samples: 389 us, 367 now), the first a tenth (500000: 12270, 1090).
//
// The samples share one power-of-two scale, from 64 of them, which leaves room for elements a hundred times as large as those;
// larger ones go to the list, where every sample has its own.  So the offsets of the rows are the same for all samples and are
// read from the LDS as the first accumulator.
#pragma once

#include "split_quant.h"
#include "split_screen.h"

namespace asgd {

constexpr int SCREENQ_THREADS = 256;
constexpr int SCREENQ_WAVES = SCREENQ_THREADS / 64;
constexpr int SCREENQ_ROWS = 64;                 // samples the common scale is taken from
constexpr int SCREENQ_SAMPLE = 8;                // their largest element below 2^8
constexpr float SCREENQ_LIMIT = 6.0e4f;          // norm of a scaled sample whose elements are fp16 numbers
constexpr int SCREENQ_LIST = 256;                // undecided samples a wave may note: two sweeps' worth
constexpr int SCREENQ_QUEUE = 1024;              // bytes a wave has for their candidates: the nearest of 64 samples, two times 64 pairs of a sample and a row

// Where more than one in this many samples is left open, the others are not screened.  Microseconds with all of them screened, and given up (samples next to
// one of two equal rows, share): k = 37, d = 75, 2e6 samples: 20 % 255, 322, 40 % 388, 350, all 650, 347; k = 300, d = 48, 1e6: 20 % 148, 180, 40 %
// 201, 209, all 301, 216; k = 100, d = 100, 1e6: 20 % 197, 265, 40 % 290, 296, all 498, 299.
constexpr int SCREENQ_OPEN_SHARE = 2;

struct ScreenQuant {
    SplitQuant q;
    // operands of the state, see splitq_operands_kernel: m by slot, offsets, high parts, low parts ([row pair][chunk][block] pieces
    // of 1 KB), sizes of the rows of a pair
    float *head, *m, *hs, *sizes;
    unsigned char *hi, *lo;
    int pairs_per_stage, keep;
    unsigned off_ms, off_list, off_stage;
};
struct ScreenqHead { float sw, ratio, direct; int sw_exp; };       // at `head`

struct ScreenqSize { SplitqSize rows; float rest; };

// Tiles of a wave.  KEEP: its samples stay in the registers as they came, for the distances.
constexpr int screenq_tiles(int chunks, bool keep) { return !keep || chunks <= 2 ? 4 : chunks <= 6 ? 2 : 1; }

// The sample of the wave that entry `code` of its list stands for: 128 times the sweep, and the place among the wave's samples of it.  `full`
// sweeps are of `per` samples per wave, one more may follow with half as many.
typedef __attribute__((address_space(3))) unsigned char *ScreenqQueue;           // (LDS instructions, which keep their order)
struct ScreenqWave { int full, waves, wave, per; };
__device__ __forceinline__ long long screenq_sample(int code, const ScreenqWave &w)
{
    const int sweep = code >> 7, at = code & 127;
    return (long long)sweep * w.waves * w.per + (long long)w.wave * (sweep < w.full ? w.per : w.per / 2) + at;
}

// The smaller one of the direct distances of the lanes' samples `own` to their rows `arg` (below zero: none) and `second` (below zero: to `arg` only), as below.
template <int NC>
__device__ __forceinline__ double screenq_distances(const float *x, const float *w, long long own, int arg, int second, int d)
{
    constexpr int LANES = NC == 1 ? 4 : 8, U = (NC + 1) / 2, SAMPLES = 64 / LANES;
    const int lane = split_lane(), own_lane = lane & (LANES - 1), own_sample = lane / LANES;
    const int count = 64 - __clzll((long long)__ballot(arg >= 0));
    struct Pass { float4u x[U], a[U], b[U]; int c; };
    const bool pairs = __ballot(second >= 0) != 0;
    auto fetch = [&](Pass &p, int at0) {
        const int at = min(at0 + own_sample, 63), c2 = __shfl(second, at, 64);
        p.c = __shfl(arg, at, 64);
        const float *row = x + (size_t)max(__shfl(own, at, 64), 0LL) * d;
        const unsigned ao = (unsigned)(max(p.c, 0) * d), bo = (unsigned)(max(c2 >= 0 ? c2 : p.c, 0) * d);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned j = (unsigned)min(32 * u + 4 * own_lane, d - 4);
            p.x[u] = *reinterpret_cast<const float4u *>(row + j);
            p.a[u] = *reinterpret_cast<const float4u *>(w + (ao + j));
            if (pairs) p.b[u] = *reinterpret_cast<const float4u *>(w + (bo + j));
        }
    };
    auto distance = [&](const float4u (&xv)[U], const float4u (&wv)[U]) {
        double far = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = 32 * u + 4 * own_lane;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double t = (double)xv[u][e] - (double)(u + 1 < U || (j < d && min(j, d - 4) + e >= j) ? wv[u][e] : xv[u][e]);
                far = fma(t, t, far);
            }
        }
#pragma unroll
        for (int off = LANES / 2; off > 0; off >>= 1) far += __shfl_xor(far, off, 64);
        return far;
    };
    double sum = 0.0;
    auto add = [&](const Pass &p) {
        double far = distance(p.x, p.a);
        if (pairs) far = fmin(far, distance(p.x, p.b));
        // (infinite where an fp32 number is, as in the other kernels)
        if (p.c >= 0 && own_lane == 0) sum += far <= 3.402823466e38 ? far : INFINITY;
    };
    if (count == 0) return 0.0;
    Pass a, b;
    fetch(a, 0);
    for (int at = 0; at < count; at += 2 * SAMPLES) {             // (two passes in flight; past the last one the last sample again)
        fetch(b, at + SAMPLES);
        add(a);
        __builtin_amdgcn_sched_barrier(0);
        fetch(a, at + 2 * SAMPLES);
        add(b);
        __builtin_amdgcn_sched_barrier(0);
    }
    return 0.5 * sum;
}

// What up to 64 samples (`own`: the lane's, below zero if it has none) add to Eq. 8: scores with all three products, the state's operands straight from the L2.
typedef const __attribute__((address_space(4))) ScreenQuant *ScreenQuantPtr;
template <int NC>
__device__ __forceinline__ double screenq_group(ScreenQuantPtr a, ScreenqQueue queue, long long own, SplitqSize size, int sw_exp)
{
    const int lane = split_lane(), half = lane >> 5, l32 = lane & 31, d = a->q.d, nblk = a->q.nblk;
    const float *m = a->m;
    half8 bh[2][NC], bl[2][NC];
    float n2[2] = {0.0f, 0.0f}, ratio[2];
    bool direct[2];
    SplitTop top[2];
    const float big = split_opaque_infinity();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float *row = a->q.x + (size_t)max(__shfl(own, 32 * q + l32, 64), 0LL) * d;
        float v[NC][8], most = 0.0f;
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) split_load8<false>(v[ch], row, ch + 1 < NC ? ch * 16 + 8 * half : min(ch * 16 + 8 * half, d - 8), d);
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
            const int slot = ch * 16 + 8 * half;
            const float4 m0 = *reinterpret_cast<const float4 *>(m + slot), m1 = *reinterpret_cast<const float4 *>(m + slot + 4);
            const float mm[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[ch][e] = ch + 1 < NC || split_slot_used(slot + e, d) ? v[ch][e] - mm[e] : 0.0f;
                most = fmaxf(most, fabsf(v[ch][e]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        most = fmaxf(most, __shfl_xor(most, 32, 64));
        const int e = splitq_exponent(most, SPLITQ_SAMPLE), r = most > 0.0f ? min(e - sw_exp, SPLITQ_RATIO_MAX) : 0;
        direct[q] = r < SPLITQ_RATIO_MIN;
        const float scale = ldexpf(1.0f, max(-126, min(126, r + sw_exp)));
        ratio[q] = ldexpf(1.0f, max(r, SPLITQ_RATIO_MIN));
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
#pragma unroll
            for (int e2 = 0; e2 < 8; ++e2) {
                const float y = v[ch][e2] * scale;
                bh[q][ch][e2] = (_Float16)y;
                bl[q][ch][e2] = (_Float16)(y - (float)bh[q][ch][e2]);
                n2[q] = fmaf(y, y, n2[q]);
            }
            asm volatile("" : "+v"(bh[q][ch]), "+v"(bl[q][ch]));             // (packed here, as in screen_convert())
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" : "+v"(n2[q]));
        top[q].v1 = top[q].v2 = top[q].v3 = -INFINITY;
        top[q].i1 = top[q].i2 = 0;
    }
    auto scores = [&](sfloatx16 (&acc)[2], int blk) {
        const float *hp = a->hs + blk * 32 + 4 * half;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const float4 h = *reinterpret_cast<const float4 *>(hp + 8 * r4);
            acc[0][4 * r4 + 0] = h.x * ratio[0]; acc[0][4 * r4 + 1] = h.y * ratio[0]; acc[0][4 * r4 + 2] = h.z * ratio[0]; acc[0][4 * r4 + 3] = h.w * ratio[0];
            acc[1][4 * r4 + 0] = h.x * ratio[1]; acc[1][4 * r4 + 1] = h.y * ratio[1]; acc[1][4 * r4 + 2] = h.z * ratio[1]; acc[1][4 * r4 + 3] = h.w * ratio[1];
        }
        const size_t at = (((size_t)(blk >> 1) * NC) * 2 + (blk & 1)) * SPLIT_PIECE + lane * 16;
#pragma unroll
        for (int ch = 0; ch < NC; ++ch) {
            const half8 ah = *reinterpret_cast<const half8 *>(a->hi + at + (size_t)ch * 2 * SPLIT_PIECE);
            const half8 al = *reinterpret_cast<const half8 *>(a->lo + at + (size_t)ch * 2 * SPLIT_PIECE);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[0][ch], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[1][ch], acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[0][ch], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[1][ch], acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[0][ch], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[1][ch], acc[1], 0, 0, 0);
        }
    };
    for (int blk = 0; blk < nblk; ++blk) {
        sfloatx16 acc[2];
        scores(acc, blk);
        split_insert(top[0], acc[0], blk, big);
        split_insert(top[1], acc[1], blk, big);
    }
    SplitTop t;
    split_combine(top, t, half);
    swap2(n2[0], n2[1]);
    int arg = min(max(t.i1, 0), a->q.k - 1), second = min(max(t.i2, 0), a->q.k - 1);
    const SplitqOpen open = splitq_open(t, arg, second, own >= 0, n2[0] + n2[1], half ? ratio[1] : ratio[0], half ? direct[1] : direct[0], size, a->q.dpad);
    const bool near = open.more && open.limit < INFINITY;
    if (__ballot(near)) {
        // More than two candidates: the scores once more, and the direct distances to the rows within the bound of the best.  (To all k rows: k = 1024,
        // d = 128, 500000 samples, one column a thousand times as wide as the others 12000 us, now 1520; eight copies of every row 12280, 1250.)  They are
        // collected, 64 at a time, so that eight lanes can share one; every lane its own took 2600 and 1960.
        auto *nearest = (__attribute__((address_space(3))) u64 *)queue;             // by sample: distance, row
        auto *pairs = (__attribute__((address_space(3))) int *)(queue + 512);
        nearest[lane] = ~0ULL;
        int queued = 0;
        auto drain = [&](int n) {
            queued -= n;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            constexpr int U = (NC + 1) / 2;
            const int l8 = lane & 7;
            for (int from = 0; from < n; from += 8) {
                const int at = from + (lane >> 3), pair = pairs[queued + min(at, n - 1)], sample = pair >> 13, c = pair & 8191;
                const float *row = a->q.x + (size_t)max(__shfl(own, sample, 64), 0LL) * d, *wrow = a->q.w + (unsigned)(c * d);
                float far = 0.0f;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = 32 * u + 4 * l8;
                    const float4u xv = *reinterpret_cast<const float4u *>(row + min(j, d - 4)), wv = *reinterpret_cast<const float4u *>(wrow + min(j, d - 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float diff = u + 1 < U || (j < d && min(j, d - 4) + e >= j) ? xv[e] - wv[e] : 0.0f;
                        far = fmaf(diff, diff, far);
                    }
                }
#pragma unroll
                for (int off = 4; off > 0; off >>= 1) far += __shfl_xor(far, off, 64);
                if (l8 == 0 && at < n) __hip_atomic_fetch_min(&nearest[sample], (u64)__float_as_uint(far) << 32 | (u64)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        for (int blk = 0; blk < nblk; ++blk) {
            sfloatx16 acc[2];
            scores(acc, blk);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float limit = __shfl(open.limit, 32 * q + l32, 64);
                unsigned hit = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) hit |= acc[q][r] >= limit ? 1u << r : 0u;
                for (unsigned long long some; (some = __ballot(hit != 0)) != 0; hit &= hit - 1) {
                    const int r = __builtin_ctz(hit | 0x10000u), c = blk * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (hit) pairs[queued + __popcll(some & ((1ULL << lane) - 1))] = (32 * q + l32) << 13 | min(c, a->q.k - 1);
                    queued += __popcll(some);
                    if (queued >= 64) drain(64);
                }
            }
        }
        if (queued) drain(queued);
        if (near) arg = min((int)(nearest[lane] & 8191), a->q.k - 1);
    }
    const bool scan = open.more && !near;
    const float scanned = splitq_scan((SplitQuantPtr)a, __ballot(scan), own, lane);
    double sum = screenq_distances<NC>(a->q.x, a->q.w, own, own >= 0 && !scan ? arg : -1, open.two ? second : -1, d);
    if (scan) sum += 0.5 * (double)scanned;
    return sum;
}

// The samples of codes[0 .. n), or (no codes) n samples of the wave from the start of sweep `from` on.  A function that is really called, with registers of its
// own; the loop is in it because a call saves and restores half of them.
template <int NC>
__device__ __noinline__ double screenq_listed(u64 args, ScreenqQueue queue, const int *codes, int from, int n_any, ScreenqWave w_any, SplitqSize size, int sw_exp_any)
{
    const ScreenQuantPtr a = (ScreenQuantPtr)split_uniform64(args);
    const int sw_exp = __builtin_amdgcn_readfirstlane(sw_exp_any), n = __builtin_amdgcn_readfirstlane(n_any), lane = split_lane();
    const ScreenqWave w = {__builtin_amdgcn_readfirstlane(w_any.full), __builtin_amdgcn_readfirstlane(w_any.waves), __builtin_amdgcn_readfirstlane(w_any.wave),
                           __builtin_amdgcn_readfirstlane(w_any.per)};
    double sum = 0.0;
    for (int r0 = 0; r0 < n; r0 += 64) {
        const int r = min(r0 + lane, n - 1);
        const long long own = screenq_sample(codes ? codes[r] : (from + r / w.per) * 128 + r % w.per, w);
        sum += screenq_group<NC>(a, queue, r0 + lane < n && own < a->q.N ? own : -1, size, sw_exp);
    }
    return sum;
}

// The direct distances of the wave's samples gw .. gw + 63 to their nearest rows (lane l: `arg` of sample gw + l, below zero: not
// decided).  Eight lanes per sample, sixteen bytes each, so that a load takes whole lines of eight rows.
template <int NC>
__device__ __forceinline__ double screenq_distances(const float *x, const float *w, long long gw, long long N, int d, int arg)
{
    const int lane = split_lane(), l8 = lane & 7, s8 = lane >> 3;
    constexpr int U = (NC + 1) / 2;                       // 32 columns each
    const float *xb = x + (size_t)gw * d;
    const int last = (int)min(63LL, N - 1 - gw);
    auto fetch = [&](float4u (&xv)[U], float4u (&wv)[U], int &c, int p) {
        const int at = 8 * p + s8;
        c = __shfl(arg, at, 64);
        const unsigned xo = (unsigned)(min(at, last) * d), wo = (unsigned)(max(c, 0) * d);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned j = (unsigned)min(32 * u + 4 * l8, d - 4);
            xv[u] = *reinterpret_cast<const float4u *>(xb + (xo + j));
            wv[u] = *reinterpret_cast<const float4u *>(w + (wo + j));
        }
    };
    double sum = 0.0;
    auto add = [&](const float4u (&xv)[U], const float4u (&wv)[U], int c) {
        double far = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = 32 * u + 4 * l8;                // (the last sixteen bytes of a row hold columns of those before them)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double t = (double)xv[u][e] - (double)(u + 1 < U || (j < d && min(j, d - 4) + e >= j) ? wv[u][e] : xv[u][e]);
                far = fma(t, t, far);                     // (as fast as in fp32, whose squares of numbers with few digits are biased by 5e-11 of the sum)
            }
        }
        far = c >= 0 ? far : 0.0;                         // (no branch: behind one, the loads of all passes came first, 120 spills)
        asm volatile("" : "+v"(far));
        sum += far;
    };
    float4u xa[U], wa[U], xn[U], wn[U];
    int ca, cn;
    fetch(xa, wa, ca, 0);
#pragma unroll
    for (int p = 0; p < 8; p += 2) {
        fetch(xn, wn, cn, p + 1);
        add(xa, wa, ca);
        __builtin_amdgcn_sched_barrier(0);            // (two passes in flight, not as many as there are loads)
        if (p + 2 < 8) fetch(xa, wa, ca, p + 2);
        add(xn, wn, cn);
        __builtin_amdgcn_sched_barrier(0);
    }
    return 0.5 * sum;
}

template <int NC, bool KEEP>
__global__ __launch_bounds__(SCREENQ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void screen_quant_kernel(ScreenQuant a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double red[SCREENQ_WAVES];
    __shared__ int open_all;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int d = a.q.d, nblk = a.q.nblk, npair = (nblk + 1) / 2;
    const long long N = a.q.N, waves = (long long)gridDim.x * SCREENQ_WAVES, wv = (long long)blockIdx.x * SCREENQ_WAVES + wave;
    const u64 args = (u64)__builtin_amdgcn_kernarg_segment_ptr();
    float *hs = reinterpret_cast<float *>(smem), *ms = reinterpret_cast<float *>(smem + a.off_ms);
    int *list = reinterpret_cast<int *>(smem + a.off_list) + wave * SCREENQ_LIST;
    unsigned char *stage = smem + a.off_stage;
    const ScreenqQueue queue = (ScreenqQueue)(smem + a.off_list + SCREENQ_WAVES * SCREENQ_LIST * 4 + wave * SCREENQ_QUEUE);
    const int nstage = (npair + a.pairs_per_stage - 1) / a.pairs_per_stage;
    const unsigned stage_bytes = (unsigned)a.pairs_per_stage * NC * 2 * SPLIT_PIECE;

    // Sweeps of four tiles per wave; what is left is one more of them, or of two
    constexpr int TILES = screenq_tiles(NC, KEEP), PER = 32 * TILES;
    const long long whole = waves * PER, rest = N % whole, few = TILES > 1 ? waves * (PER / 2) : 0, full = N / whole + (rest > few);
    const bool half_sweep = rest > 0 && rest <= few;
    if ((long long)blockIdx.x * SCREENQ_WAVES * (full > 0 ? PER : PER / 2) >= N) {
        if (tid == 0) a.q.partials[blockIdx.x] = 0.0;
        return;
    }
    const ScreenqHead head = *reinterpret_cast<const ScreenqHead *>(a.head);
    const float scale = head.sw * head.ratio;
    for (int c = tid; c < a.q.kpad; c += SCREENQ_THREADS) hs[c] = a.hs[c] * head.ratio;
    for (int j = tid; j < a.q.dpad; j += SCREENQ_THREADS) ms[j] = -a.m[j] * scale;
    ScreenqSize size = {{INFINITY, 0.0f, INFINITY}, 0.0f};
    for (int r = 0; r < npair; ++r) {
        const float4 s = reinterpret_cast<const float4 *>(a.sizes)[r];
        size.rows.vmin = fminf(size.rows.vmin, s.x);
        size.rows.vmax = fmaxf(size.rows.vmax, s.y);
        size.rows.vfar = fminf(size.rows.vfar, s.z);
        size.rest = fmaxf(size.rest, s.w);
    }
    size.rows.vmax = sqrtf(size.rows.vmax) * 1.0001f;
    size.rows.vmin = sqrtf(size.rows.vmin) * 1.0001f;
    size.rows.vfar = sqrtf(size.rows.vfar) * 0.9999f;
    size.rest = sqrtf(size.rest) * 1.0001f;

    // Norm of a sample, in scaled units, whose squared distance to the smallest row an fp32 number holds (others are infinite, which the list sees to)
    const float yn_limit = fminf(SCREENQ_LIMIT, 1.8e19f * scale - size.rows.vmin * head.ratio);

    double sum = 0.0;
    int listed = 0, turn = 0, open_own = 0;
    bool staged = false;
    if (tid == 0) open_all = 0;
    const ScreenqWave here = {(int)full, (int)waves, (int)wv, PER};
    auto flush = [&](int from, int n) {
        sum += screenq_listed<NC>(args, queue, list + from, 0, n, here, size.rows, head.sw_exp);
    };
    // (a third and a fourth stage on their way changed nothing)
    auto stage_fetch = [&](int st, int buf) {
        const int pairs = min(a.pairs_per_stage, npair - st * a.pairs_per_stage);
        split_stage(a.hi + (size_t)st * stage_bytes, stage + buf * stage_bytes, pairs * NC * 2);
    };
    // one sweep over this wave's 32 * T samples from gw on
    auto sweep = [&](auto tiles, long long gw, int code0, bool last) {
        constexpr int T = decltype(tiles)::value;
        constexpr int HC = (NC + 1) / 2, SETS = KEEP ? 2 * T : 3;
        half8 b[T][NC];
        float n2[T], r2[T], v[SETS][HC][8];
        ScreenTop top[T];
        {
            const long long base = min(gw, N - 1);
            const float *xb = a.q.x + (size_t)base * d;
            const int most = (int)min((long long)(32 * T - 1), N - 1 - base);
            // units of half a tile, two on their way while one is converted (KEEP: all of them)
            auto load = [&](float (&to)[HC][8], int u) {
                const float *row = xb + (unsigned)(min(32 * (u >> 1) + l32, most) * d);
#pragma unroll
                for (int q = 0; q < HC; ++q) {
                    const int ch = (u & 1) * HC + q;
                    if (ch < NC) split_load8<false>(to[q], row, ch + 1 < NC ? ch * 16 + 8 * half : min(ch * 16 + 8 * half, d - 8), d);
                }
            };
#pragma unroll
            for (int u = 0; u < (KEEP ? 2 * T : 2); ++u) load(v[u], u);
#pragma unroll
            for (int u = 0; u < 2 * T; ++u) {
                const int t = u >> 1;
                if (!KEEP && u + 2 < 2 * T) load(v[(u + 2) % SETS], u + 2);
                if ((u & 1) == 0) n2[t] = r2[t] = 0.0f;
                const int hf = split_lane() >> 5;             // (ms is read again for every tile, not kept in 64 registers)
#pragma unroll
                for (int q = 0; q < HC; ++q) {
                    const int ch = (u & 1) * HC + q;
                    if (ch + 1 < NC) screen_convert<false>(v[u % SETS][q], scale, ms, ch * 16 + 8 * hf, d, b[t][ch], n2[t], r2[t]);
                    else if (ch + 1 == NC) screen_convert<true>(v[u % SETS][q], scale, ms, ch * 16 + 8 * hf, d, b[t][ch], n2[t], r2[t]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                asm volatile("" : "+v"(n2[t]), "+v"(r2[t]));
                if (u & 1) {
                    top[t].v1 = top[t].v2 = -INFINITY;
                    top[t].i1 = 0;
                }
            }
        }
        for (int st = 0; st < nstage; ++st) {
            if (nstage > 1 || !staged) split_stage_wait();                 // this stage is there, and nobody reads the other one any more
            staged = true;
            if (nstage > 1 && !(last && st + 1 == nstage)) stage_fetch(st + 1 < nstage ? st + 1 : 0, (turn + 1) & 1);
            const unsigned char *from = stage + (turn & 1) * stage_bytes;
            turn += nstage > 1;
            const int blk0 = st * a.pairs_per_stage * 2, blks = min(a.pairs_per_stage * 2, nblk - blk0);
            for (int q = 0; q < blks; ++q) {
                const half8 *A = reinterpret_cast<const half8 *>(from + ((q >> 1) * NC * 2 + (q & 1)) * SPLIT_PIECE) + lane;
                sfloatx16 h, acc[T];
                split_init_acc(h, hs, blk0 + q, half);
                half8 ah = A[0];
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) {
                    half8 nh = ah;
                    if (ch + 1 < NC) nh = A[(ch + 1) * 128];
#pragma unroll
                    for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, b[t][ch], ch == 0 ? h : acc[t], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    ah = nh;
                }
#pragma unroll
                for (int t = 0; t < T; ++t) screen_insert(top[t], acc[t], blk0 + q);
            }
        }
        if (gw < N) {
#pragma unroll
            for (int p = 0; p < (T + 1) / 2; ++p) {
                ScreenTop t, none = {-INFINITY, -INFINITY, 0};
                float n2b = 0.0f, r2b = 0.0f;
                screen_combine(top[2 * p], 2 * p + 1 < T ? top[(2 * p + 1) % T] : none, t, half);
                swap2(n2[2 * p], 2 * p + 1 < T ? n2[(2 * p + 1) % T] : n2b);
                swap2(r2[2 * p], 2 * p + 1 < T ? r2[(2 * p + 1) % T] : r2b);
                n2b = 2 * p + 1 < T ? n2[(2 * p + 1) % T] : n2b;
                r2b = 2 * p + 1 < T ? r2[(2 * p + 1) % T] : r2b;
                const float yn = sqrtf(n2[2 * p] + n2b) * 1.0001f, rl = sqrtf(r2[2 * p] + r2b) * 1.0001f, yr = yn / head.ratio;
                // (why rows of that size are enough: split_quant.h; one that is larger has a rest of 2^-11 of it at most)
                const float vn = fminf(size.rows.vmax, 4.0f * yr + 2.0f * size.rows.vmin), vl = fminf(size.rest, 4.8877e-4f * vn + 1.0e-6f);
                const float thr = screen_bound(yn, rl, vn, vl, 0.5f * vn * vn * head.ratio, a.q.dpad);
                const bool all = head.direct != 0.0f || !(yn < yn_limit) || !(size.rows.vmin < INFINITY) ||
                                 (size.rows.vfar < INFINITY && !(2.02f * yr + size.rows.vmin < size.rows.vfar));
                const bool valid = gw + 64 * p + lane < N && (T > 1 || half == 0), open = valid && (all || !(t.v1 - t.v2 > thr));
                const unsigned long long o = __ballot(open);
                if (open) list[listed + __popcll(o & ((1ULL << lane) - 1))] = code0 + 64 * p + lane;
                listed += __popcll(o);
                open_own += __popcll(o);
                const int arg = valid && !open ? min(max(t.i1, 0), a.q.k - 1) : -1;
                if constexpr (KEEP) {
                    // the samples are in the registers still, a lane's columns against those of its sample's nearest row
#pragma unroll
                    for (int q = 0; q < 2 && 2 * p + q < T; ++q) {
                        const int c = __shfl(arg, 32 * q + l32, 64);
                        const float *row = a.q.w + (unsigned)(max(c, 0) * d);
                        float wv[NC][8];
                        double far = 0.0;
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) split_load8<false>(wv[ch], row, ch + 1 < NC ? ch * 16 + 8 * half : min(ch * 16 + 8 * half, d - 8), d);
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float x = v[(2 * (2 * p + q) + ch / HC) % SETS][ch % HC][e];
                                const double diff = (double)x - (double)(ch + 1 < NC || split_slot_used(ch * 16 + 8 * half + e, d) ? wv[ch][e] : x);
                                far = fma(diff, diff, far);
                            }
                        }
                        sum += c >= 0 ? 0.5 * far : 0.0;
                    }
                } else if (gw + 64 * p < N) {
                    sum += screenq_distances<NC>(a.q.x, a.q.w, gw + 64 * p, N, d, arg);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        while (listed >= 64) {
            listed -= 64;
            flush(listed, 64);
        }
        __builtin_amdgcn_wave_barrier();
    };
    stage_fetch(0, 0);
    __syncthreads();                                  // (hs and ms are complete)
    // Data of which screening decides little: the rest is scored with all three products right away.  Where the state is staged the waves have to agree.
    // (Nobody adds to open_all again before all have read it: there are the barriers of the next sweep's stages.)
    auto gives_up = [&](long long sweeps) {
        if (nstage == 1) return open_own * SCREENQ_OPEN_SHARE > sweeps * PER;
        if (lane == 0) atomicAdd(&open_all, open_own);
        open_own = 0;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(open_all) * SCREENQ_OPEN_SHARE > sweeps * PER * SCREENQ_WAVES;
    };
    long long s = 0;
    bool screens = true;
    for (; s < full; ++s) {
        sweep(std::integral_constant<int, TILES>{}, (s * waves + wv) * PER, (int)(s * 128), !half_sweep && s + 1 == full);
        if ((s + 1 < full || half_sweep) && gives_up(s + 1)) { screens = false; ++s; break; }
    }
    if (screens) {
        if constexpr (TILES > 1)
            if (half_sweep) sweep(std::integral_constant<int, TILES / 2>{}, full * whole + wv * (PER / 2), (int)(full * 128), true);
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // (a stage may be on its way)
        sum += screenq_listed<NC>(args, queue, nullptr, (int)s, (int)(full - s) * PER + (half_sweep ? PER / 2 : 0), here, size.rows, head.sw_exp);
    }
    if (listed > 0) flush(0, listed);
    sum = split_wave_sum(sum);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0;
        for (int v = 0; v < SCREENQ_WAVES; ++v) tot += red[v];
        a.q.partials[blockIdx.x] = tot;
    }
}

template <int NC, bool KEEP>
hipError_t launch_screen_quant(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    const hipError_t e = hipFuncSetAttribute((const void *)screen_quant_kernel<NC, KEEP>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((screen_quant_kernel<NC, KEEP>), dim3(blocks), dim3(SCREENQ_THREADS), lds, s, a);
    return hipGetLastError();
}

}  // namespace asgd
