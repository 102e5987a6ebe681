// Eq. 8 on the fp16 matrix instructions, rows of less than 8 and of more than 128 columns, few samples and centroids of up to 16 columns (the others:
// split_quant_screen.h, which shares the decisions and what follows about odd rows).  Scores with fp16-split operands (split_core.h) only screen: the
// error of a score is bounded, and a sample whose runner-up lies within the bound is decided by distances in direct form -
// two candidates by theirs, more by those to all the centroids.  So every sample adds the smallest of its direct fp32
// distances, whatever the scores are worth, and the sum over the samples is fp64.
//
// One workgroup of eight waves per compute unit walks groups of 512 samples; a wave takes 64 of them and keeps their
// operands in registers.  Nothing is known about the samples beforehand, so every sample gets a power-of-two scale of its
// own from its largest |x_j - m_j|.  The state is split by every workgroup: once per launch when it fits the LDS, else
// block by block for every group of samples, the next block's rows on their way meanwhile (that costs 2 * 8 * 5 vector
// instructions per wave and pair of row blocks, next to 96 matrix instructions of 32 cycles).
//
// What one odd row can do.  m is the middle of nine rows of the state, and the scale of the state's operands comes from the
// middle of the sizes of the same rows: up to three dead or outlying prototypes among them move neither.  Rows 2^10 times as
// large as that and more are not scored at all.  With |y| the norm of the sample relative to m and |v|min that of the
// smallest row, a row cannot be nearest if |v_c| > 2 |y| + |v|min (its distance is |v_c| - |y| or more, that of the smallest
// row |y| + |v|min or less); a sample for which this does not rule out all the rows left out is decided in direct form.  For the
// same reason the bound of a score need not hold for the largest row, only for rows up to 4 |y| + 2 |v|min: a larger one
// scores below -|v_c|^2/8, the smallest row above -|v_c||v|min/4, and the difference is far above both errors.
#pragma once

#include "split_core.h"

namespace asgd {

struct SplitQuant {
    const float *x, *w;
    long long N;
    double *partials;
    int k, d, kpad, nblk, dpad, resident;
    int nan_is_inf;                        // a sample without a finite distance counts as infinitely far, else with its distance to row 0
    unsigned off_hs, off_m;
};

constexpr int SPLITQ_THREADS = 512;

// index of half-piece (hi; lo is 64 further) of eight slots of row c in fragments of `nch` chunks
__device__ __forceinline__ int split_frag_at(int c, int slot, int nch)
{
    return (((c >> 6) * nch + (slot >> 4)) * 4 + ((c >> 5) & 1) * 2) * 64 + (c & 31) + 32 * ((slot >> 3) & 1);
}

// eight slots of a state row relative to m, unscaled; zero where not in use
__device__ __forceinline__ void splitq_row(float (&v)[8], const float *w, const float *m, int c, int k, int slot, int d)
{
    const bool real = c < k && slot < d;
    split_load8<true>(v, w + (size_t)(real ? c : 0) * d, real ? slot : 0, d);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = real && split_slot_used(slot + e, d) ? v[e] - m[slot + e] : 0.0f;
}
__device__ __forceinline__ void splitq_put(half8 *at, const float (&v)[8], float s, bool scored)
{
    half8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float y = scored ? v[e] * s : 0.0f;
        hi[e] = (_Float16)y;
        lo[e] = (_Float16)(y - (float)hi[e]);
    }
    at[0] = hi;
    at[64] = lo;
}

// The median of the medians of three triples: any three of the nine numbers may be outliers.  (Four instructions; a kernel this
// short is mostly the fetch of its own code: an exact median of fifteen by counting ranks cost 14 us.)
__device__ __forceinline__ float splitq_middle(const float (&v)[9])
{
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_fmed3f(v[0], v[1], v[2]), __builtin_amdgcn_fmed3f(v[3], v[4], v[5]),
                                   __builtin_amdgcn_fmed3f(v[6], v[7], v[8]));
}

// of nine rows spread over the state, the column of slot j
__device__ __forceinline__ float splitq_middle_of(const float *w, int k, int d, int j)
{
    if (!split_slot_used(j, d)) return 0.0f;
    const float *col = w + split_column(j, d);
    float v[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) v[q] = col[(size_t)(q * k / 9) * d];
#pragma unroll
    for (int q = 0; q < 9; ++q)
        if (!(fabsf(v[q]) < INFINITY)) v[q] = 0.0f;
    return splitq_middle(v);
}

// exponent of the power of two that takes `most` to [2^(to - 1), 2^to) (some exponent when it is zero or not finite)
__device__ __forceinline__ int splitq_exponent(float most, int to)
{
    int q = 0;
    if (most > 0.0f && most < INFINITY) (void)frexpf(most, &q);
    return max(-124, min(100, to - q));
}
constexpr int SPLITQ_TYPICAL = 5, SPLITQ_LIMIT = 15;      // operands of a typical row below 2^5, of a scored one below 2^15
constexpr int SPLITQ_SAMPLE = 13;                         // of a sample below 2^13
// scale of a sample over that of the state: between 2^-40 (the padding rows' offset has to stay below all the scores) and
// 2^16 (the offset of a large row has to stay finite)
constexpr int SPLITQ_RATIO_MIN = -40, SPLITQ_RATIO_MAX = 16;

// distance of the lane pair's sample to centroid c, direct form; a lane adds the slots of its half-wave
// TAIL: the columns need not fill the last four chunks
template <bool TAIL>
__device__ __forceinline__ float splitq_distance(const float *row, const float *wrow, int d, int half)
{
    float d2 = 0.0f;
    // (Four chunks at a time, then those that are left one by one: every load takes sixteen bytes of 64 rows, and of those at d = 75
    // three in eight were past the end: 4e6 samples, k = 37: 632 us, 548 without them.)
    auto add = [&](const float (&xv)[8], const float (&wv)[8], int slot) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float t = split_slot_used(slot + e, d) ? xv[e] - wv[e] : 0.0f;
            d2 = fmaf(t, t, d2);
        }
    };
    int s0 = 0;
    for (; s0 + (TAIL ? 48 : 0) < d; s0 += 64) {
        float xv[4][8], wv[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int slot = min(s0 + 16 * u + 8 * half, (d - 1) & ~7);
            split_load8<true>(xv[u], row, slot, d);
            split_load8<true>(wv[u], wrow, slot, d);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) add(xv[u], wv[u], s0 + 16 * u + 8 * half);
    }
    for (; TAIL && s0 < d; s0 += 16) {
        const int slot = min(s0 + 8 * half, (d - 1) & ~7);
        float xv[8], wv[8];
        split_load8<true>(xv, row, slot, d);
        split_load8<true>(wv, wrow, slot, d);
        add(xv, wv, s0 + 8 * half);
    }
    return d2;
}

// smallest direct distance of the lane's own sample `xl` to any of the k rows (infinite if none is finite)
__device__ inline float splitq_scan_own(const float *xl, const float *w, int k, int d)
{
    float best = INFINITY;
    for (int c0 = 0; c0 < k; c0 += 8) {
        float s[8];
        const float *wr[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            s[q] = 0.0f;
            wr[q] = w + (size_t)min(c0 + q, k - 1) * d;
        }
        int j = 0;
        for (; j + 4 <= d; j += 4) {
            const float4u x4 = *reinterpret_cast<const float4u *>(xl + j);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float4u w4 = *reinterpret_cast<const float4u *>(wr[q] + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = x4[e] - w4[e];
                    s[q] = fmaf(t, t, s[q]);
                }
            }
        }
        for (; j < d; ++j) {
            const float xj = xl[j];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float t = xj - wr[q][j];
                s[q] = fmaf(t, t, s[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (s[q] < best) best = s[q];
    }
    return best;
}
// the same of ONE sample by the whole wave: sixteen lanes per row, four columns each, sixteen rows in flight
__device__ inline float splitq_scan_wave(const float *xl, const float *w, int k, int d, int lane)
{
    const int l16 = lane & 15, quarter = lane >> 4;
    float best = INFINITY;
    for (int c0 = 0; c0 < k; c0 += 16) {
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const float *wr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) wr[q] = w + (size_t)min(c0 + 4 * q + quarter, k - 1) * d;
        for (int j = 4 * l16; j < d; j += 64) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (j + e >= d) continue;
                const float xj = xl[j + e];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float t = xj - wr[q][j + e];
                    s[q] = fmaf(t, t, s[q]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) s[q] += __shfl_xor(s[q], off, 64);
            if (s[q] < best) best = s[q];
        }
    }
    best = fminf(best, __shfl_xor(best, 16, 64));
    return fminf(best, __shfl_xor(best, 32, 64));
}

typedef const __attribute__((address_space(4))) SplitQuant *SplitQuantPtr;
struct SplitqSize { float vmin, vmax, vfar; };       // of the scored rows, scaled; smallest |v_c| of those that are not scored

// What the scores of a sample leave open: two candidates, or more.  Of those, the nearest row's score is `limit` or more (infinite where no score says
// anything about it).
struct SplitqOpen { bool two, more; float limit; };
__device__ __forceinline__ SplitqOpen splitq_open(const SplitTop &t, int arg, int second, bool valid, float n2, float ratio, bool direct, const SplitqSize &size, int dpad)
{
    const float yn = sqrtf(n2) * 1.0001f, yr = yn / ratio;              // |y|, and in the units of the state
    const float v = fminf(size.vmax, 4.0f * yr + 2.0f * size.vmin);
    const float thr = split_c1(dpad) * (yn * v + 0.5f * v * v * ratio) + split_c2(dpad) * (yn + v);
    // no scored row, scores out of their range (or not a number), a row that was not scored may be nearest
    const bool all = direct || !(yn < 1.0e18f) || !(size.vmin < INFINITY) ||
                     (size.vfar < INFINITY && !(2.02f * yr + size.vmin < size.vfar));
    SplitqOpen o;
    const bool close2 = valid && (all || !(t.v1 - t.v2 > thr));
    o.more = close2 && (all || !(t.v1 - t.v3 > thr) || __float_as_int(t.v1) == __float_as_int(t.v2) || second == arg);
    o.two = close2 && !o.more;
    // (the bound holds the tags' part of a score; those of the score zero, where y and v are zero and it too, are below 2^-144)
    o.limit = o.more && !all && fabsf(t.v1 - thr) < INFINITY ? t.v1 - thr - 1.0e-37f : INFINITY;
    return o;
}
// Smallest direct distance to any of the rows for the samples of the lanes in `some` (n: the lane's sample, -1 without one).
__device__ __forceinline__ float splitq_scan(SplitQuantPtr a, unsigned long long some, long long n, int lane)
{
    float scanned = INFINITY;
    if (!some) return scanned;
    const float *xl = a->x + (size_t)max(n, 0LL) * a->d;
    if (__popcll(some) <= 8) {
        for (unsigned long long left = some; left; left &= left - 1) {
            const int L = __builtin_ctzll(left);           // (a valid sample)
            const float best = splitq_scan_wave(a->x + (size_t)__shfl(n, L, 64) * a->d, a->w, a->k, a->d, lane);
            if (lane == L) scanned = best;
        }
    } else if (some >> lane & 1) {
        scanned = splitq_scan_own(xl, a->w, a->k, a->d);
    }
    if ((some >> lane & 1) && !(scanned < INFINITY) && !a->nan_is_inf) {
        scanned = 0.0f;
        for (int j = 0; j < a->d; ++j) scanned = fmaf(xl[j] - a->w[j], xl[j] - a->w[j], scanned);
    }
    return scanned;
}

// What the samples of a wave add to Eq. 8 once their scores are known (lane l: sample gw + l).  For rows whose operands stay in
// registers this is a function that is really called, with registers of its own: inlined it was 2 to 10 % faster where few samples are
// undecided and up to twice as slow where many are (microseconds called and inlined, 2e6 samples: k = 100, d = 5 144, 133, k = 1000 526, 563, one
// column a thousand times as wide as the others 2376, 3414; k = 300, d = 3, every row twice 355, 523).  For long rows the registers saved around the
// call were the dearer (k = 256, d = 384, 250000: called 0.98 ms, inlined 0.55).  A call passes its arguments in vector
// registers; what is uniform is read back into scalar ones.
template <bool TAIL>
__device__ __forceinline__ double splitq_finish_here(u64 args, long long gw_any, SplitTop t, float n2, float ratio, bool direct, SplitqSize size)
{
    const SplitQuantPtr a = (SplitQuantPtr)split_uniform64(args);
    const long long gw = (long long)split_uniform64((u64)gw_any), N = a->N;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31, k = a->k, d = a->d;
    const float *x = a->x, *w = a->w;
    const int arg = min(max(t.i1, 0), k - 1), second = min(max(t.i2, 0), k - 1);
    const SplitqOpen open = splitq_open(t, arg, second, gw + lane < N, n2, ratio, direct, size, a->dpad);
    const unsigned long long pairs = __ballot(open.two), many = __ballot(open.more);
    const float scanned = splitq_scan(a, many, gw + lane < N ? gw + lane : -1, lane);
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int at = 32 * q + l32;
        const long long n = gw + at;
        const float *row = x + (size_t)(n < N ? n : N - 1) * d;
        float d2 = splitq_distance<TAIL>(row, w + (size_t)__shfl(arg, at, 64) * d, d, half);
        d2 += __shfl_xor(d2, 32, 64);
        if (pairs) {
            const int c2 = __shfl(open.two ? second : arg, at, 64);
            float o2 = splitq_distance<TAIL>(row, w + (size_t)c2 * d, d, half);
            o2 += __shfl_xor(o2, 32, 64);
            d2 = o2 < d2 ? o2 : d2;
        }
        const float s2 = __shfl(scanned, at, 64);
        if (many >> at & 1) d2 = s2;
        if (half == 0 && n < N) sum += 0.5 * (double)d2;
    }
    return sum;
}

__device__ __noinline__ inline double splitq_finish(u64 args, long long gw, SplitTop t, float n2, float ratio, bool direct, SplitqSize size)
{
    return splitq_finish_here<true>(args, gw, t, n2, ratio, direct, size);
}

template <int NC>
__global__ __launch_bounds__(SPLITQ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_quant_kernel(SplitQuant a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double red[8];
    __shared__ float redf[3][8];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int k = a.k, d = a.d, npair = (a.nblk + 1) / 2;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs), *m = reinterpret_cast<float *>(smem + a.off_m);
    half8 *frag = reinterpret_cast<half8 *>(smem);

    if ((long long)blockIdx.x * SPLITQ_THREADS >= a.N) {
        if (tid == 0) a.partials[blockIdx.x] = 0.0;
        return;
    }
    // m by slot: middle of nine rows spread over the state (any value would do; one near the data keeps the operands small)
    for (int j = tid; j < a.dpad; j += SPLITQ_THREADS) m[j] = splitq_middle_of(a.w, k, d, j);
    __syncthreads();
    // Two passes over the state, g lanes per row.  First the largest |v_cj| of every row (infinite if one is not finite), from
    // which the scale follows; then h_c = -|v_c|^2/2 in scaled units and the smallest and largest |v_c|.
    int g = 1;
    while (g < a.dpad / 8 && g < 64) g *= 2;
    int sw_exp = 0;
    float sw = 1.0f, vmin = INFINITY, vmax = 0.0f, vfar = INFINITY;     // vfar: smallest |v_c| of the rows that are not scored
    for (int pass = 0; pass < 2; ++pass) {
        const int lane_g = tid & (g - 1), ngrp = SPLITQ_THREADS / g;
        for (int c0 = tid / g; c0 < a.kpad; c0 += 4 * ngrp) {
            float sq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            unsigned vb[4] = {0, 0, 0, 0};
            for (int slot = 8 * lane_g; slot < a.dpad; slot += 8 * g) {
                float v[4][8];
#pragma unroll
                for (int q = 0; q < 4; ++q) splitq_row(v[q], a.w, m, c0 + q * ngrp, k, slot, d);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float vs = v[q][e] * sw;
                        sq[q] = fmaf(vs, vs, sq[q]);
                        vb[q] = max(vb[q], __float_as_uint(v[q][e]) & 0x7fffffffu);
                    }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                for (int off = g / 2; off > 0; off >>= 1) {
                    sq[q] += __shfl_xor(sq[q], off, 64);
                    vb[q] = max(vb[q], (unsigned)__shfl_xor((int)vb[q], off, 64));
                }
                const int c = c0 + q * ngrp;
                if (lane_g != 0 || c >= a.kpad) continue;
                const float most = __uint_as_float(min(vb[q], 0x7f800000u));
                if (pass == 0) {
                    hs[c] = most;
                    if (most < INFINITY) vmax = fmaxf(vmax, most);
                } else if (c >= k) {
                    hs[c] = SPLIT_PAD_SCORE;
                } else if (most * sw < (float)(1 << SPLITQ_LIMIT)) {
                    hs[c] = -0.5f * sq[q];
                    vmin = fminf(vmin, sq[q]);
                    vmax = fmaxf(vmax, sq[q]);
                } else {
                    hs[c] = SPLIT_PAD_SCORE;
                    // (no distance to a row that is not finite is below infinity)
                    if (most < INFINITY) vfar = fminf(vfar, sq[q] < 1.0e37f ? sq[q] : 1.0e37f);
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            vmax = fmaxf(vmax, __shfl_xor(vmax, off, 64));
            vmin = fminf(vmin, __shfl_xor(vmin, off, 64));
            vfar = fminf(vfar, __shfl_xor(vfar, off, 64));
        }
        __syncthreads();                                   // (the first pass' values have been read; hs is complete)
        if (lane == 0) { redf[0][wave] = vmax; redf[1][wave] = vmin; redf[2][wave] = vfar; }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            vmax = fmaxf(vmax, redf[0][q]);
            vmin = fminf(vmin, redf[1][q]);
            vfar = fminf(vfar, redf[2][q]);
        }
        if (pass == 0) {
            // a typical row of the same nine; at m itself: the largest of all
            float v[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) v[q] = hs[q * k / 9];
            float typical = splitq_middle(v);
            if (!(typical > 0.0f && typical < INFINITY)) typical = vmax;
            sw_exp = splitq_exponent(typical, SPLITQ_TYPICAL);
            sw = ldexpf(1.0f, sw_exp);
            vmax = 0.0f;
            __syncthreads();                               // (hs is written again)
        }
    }
    vmax = sqrtf(vmax) * 1.0001f;
    vmin = sqrtf(vmin) * 1.0001f;
    vfar = sqrtf(vfar) * 0.9999f;
    const SplitqSize size = {vmin, vmax, vfar};
    const SplitQuantPtr args = (SplitQuantPtr)__builtin_amdgcn_kernarg_segment_ptr();

    // operands of row pair rp, columns of `cg` groups of 8 chunks (NC == 0) or all of them, into `dst`
    constexpr int SC = NC == 0 ? 8 : NC;                   // chunks of a stage
    constexpr int NU = (64 * SC * 2 + SPLITQ_THREADS - 1) / SPLITQ_THREADS;
    auto stage_load = [&](float (&v)[NU][8], int rp, int cg) {
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int un = min(tid + q * SPLITQ_THREADS, 64 * SC * 2 - 1), c = un / (SC * 2), slot = (un - c * (SC * 2)) * 8;
            splitq_row(v[q], a.w, m, rp * 64 + c, k, cg * 128 + slot, d);
        }
    };
    auto stage_put = [&](const float (&v)[NU][8], half8 *dst, int rp) {
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int un = tid + q * SPLITQ_THREADS, c = un / (SC * 2), slot = (un - c * (SC * 2)) * 8;
            if (un < 64 * SC * 2) splitq_put(dst + split_frag_at(c, slot, SC), v[q], sw, hs[rp * 64 + c] != SPLIT_PAD_SCORE);
        }
    };
    constexpr int STAGE = SC * 256;                        // half8 per stage
    if (NC != 0 && a.resident) {
        for (int rp = 0; rp < npair; ++rp) {
            float v[NU][8];
            stage_load(v, rp, 0);
            stage_put(v, frag + (size_t)rp * STAGE, rp);
        }
    }
    __syncthreads();

    double sum = 0.0;
    for (long long g0 = (long long)blockIdx.x * SPLITQ_THREADS; g0 < a.N; g0 += (long long)gridDim.x * SPLITQ_THREADS) {
        const long long gw = g0 + wave * 64;
        const float *row[2];
        float ratio[2], scale[2], n2[2] = {0.0f, 0.0f};    // n2: |y|^2 in scaled units, this half-wave's slots
        bool direct[2];                                    // scores out of their range
        SplitTop top[2];
        const float big = split_opaque_infinity();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const long long n = gw + 32 * q + l32;
            row[q] = a.x + (size_t)(n < a.N ? n : a.N - 1) * d;
            top[q].v1 = top[q].v2 = top[q].v3 = -INFINITY;
            top[q].i1 = top[q].i2 = 0;
        }
        auto own_scale = [&](int q, float most) {
            most = fmaxf(most, __shfl_xor(most, 32, 64));
            const int e = splitq_exponent(most, SPLITQ_SAMPLE), r = most > 0.0f ? min(e - sw_exp, SPLITQ_RATIO_MAX) : 0;
            direct[q] = r < SPLITQ_RATIO_MIN;
            scale[q] = ldexpf(1.0f, max(-126, min(126, r + sw_exp)));
            ratio[q] = ldexpf(1.0f, max(r, SPLITQ_RATIO_MIN));
        };
        auto init = [&](sfloatx16 &acc, int q, int blk) {
            const float4 *hp = reinterpret_cast<const float4 *>(hs + blk * 32 + 4 * half);
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float4 h = hp[2 * r4];
                acc[4 * r4 + 0] = h.x * ratio[q]; acc[4 * r4 + 1] = h.y * ratio[q];
                acc[4 * r4 + 2] = h.z * ratio[q]; acc[4 * r4 + 3] = h.w * ratio[q];
            }
        };
        auto multiply = [&](const half8 *A, const half8 &bh0, const half8 &bl0, const half8 &bh1, const half8 &bl1, sfloatx16 (&acc)[2]) {
            const half8 ah = A[0], al = A[64];
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl1, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh1, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh1, acc[1], 0, 0, 0);
        };
        auto convert = [&](const float (&v)[8], float s, half8 &hi, half8 &lo, float &sq) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float y = v[e] * s;
                hi[e] = (_Float16)y;
                lo[e] = (_Float16)(y - (float)hi[e]);
                sq = fmaf(y, y, sq);
            }
        };
        // eight slots of a sample relative to m; zero where not in use
        auto load = [&](float (&v)[8], const float *r, int slot) { split_load8<true>(v, r, min(slot, (d - 1) & ~7), d); };
        auto centre = [&](float (&v)[8], int slot) {
            const float4 m0 = *reinterpret_cast<const float4 *>(m + slot), m1 = *reinterpret_cast<const float4 *>(m + slot + 4);
            const float mm[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = split_slot_used(slot + e, d) ? v[e] - mm[e] : 0.0f;
        };

        if constexpr (NC != 0) {
            half8 bh[2][SC], bl[2][SC];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float v[SC][8], most = 0.0f;
#pragma unroll
                for (int ch = 0; ch < SC; ++ch) {
                    if (ch + 1 < SC) split_load8<false>(v[ch], row[q], ch * 16 + 8 * half, d);
                    else load(v[ch], row[q], ch * 16 + 8 * half);
                }
#pragma unroll
                for (int ch = 0; ch < SC; ++ch) {
                    if (ch + 1 < SC) {
                        const float4 m0 = *reinterpret_cast<const float4 *>(m + ch * 16 + 8 * half), m1 = *reinterpret_cast<const float4 *>(m + ch * 16 + 8 * half + 4);
                        v[ch][0] -= m0.x; v[ch][1] -= m0.y; v[ch][2] -= m0.z; v[ch][3] -= m0.w;
                        v[ch][4] -= m1.x; v[ch][5] -= m1.y; v[ch][6] -= m1.z; v[ch][7] -= m1.w;
                    } else {
                        centre(v[ch], ch * 16 + 8 * half);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) most = fmaxf(most, fabsf(v[ch][e]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                own_scale(q, most);
#pragma unroll
                for (int ch = 0; ch < SC; ++ch) {
                    convert(v[ch], scale[q], bh[q][ch], bl[q][ch], n2[q]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // (formed here: left to the compiler the squares were formed after the products, the 128 elements spilled till then)
                asm volatile("" : "+v"(n2[q]));
            }
            float st[NU][8];
            if (!a.resident) {
                __syncthreads();                           // nobody still reads the first stage
                stage_load(st, 0, 0);
                stage_put(st, frag, 0);
                __syncthreads();
            }
            for (int rp = 0; rp < npair; ++rp) {
                const half8 *base = frag + (size_t)(a.resident ? rp : (rp & 1)) * STAGE + lane;
                if (!a.resident && rp + 1 < npair) stage_load(st, rp + 1, 0);
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    if (2 * rp + blk >= a.nblk) break;
                    sfloatx16 acc[2];
                    init(acc[0], 0, 2 * rp + blk);
                    init(acc[1], 1, 2 * rp + blk);
#pragma unroll
                    for (int ch = 0; ch < SC; ++ch) {
                        multiply(base + ch * 256 + blk * 128, bh[0][ch], bl[0][ch], bh[1][ch], bl[1][ch], acc);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    split_insert(top[0], acc[0], 2 * rp + blk, big);
                    split_insert(top[1], acc[1], 2 * rp + blk, big);
                }
                if (!a.resident && rp + 1 < npair) {
                    stage_put(st, frag + (size_t)((rp + 1) & 1) * STAGE, rp + 1);
                    __syncthreads();
                }
            }
        } else {
            // long rows: a pass for the scales, then the columns again for every pair of row blocks
            const int ncg = a.dpad / 128;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float most = 0.0f;
                for (int slot = 8 * half; slot < a.dpad; slot += 64) {
                    float v[4][8];
#pragma unroll
                    for (int u = 0; u < 4; ++u) load(v[u], row[q], slot + 16 * u);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        centre(v[u], slot + 16 * u);
#pragma unroll
                        for (int e = 0; e < 8; ++e) most = fmaxf(most, fabsf(v[u][e]));
                    }
                }
                own_scale(q, most);
            }
            float st[NU][8];
            __syncthreads();
            stage_load(st, 0, 0);
            stage_put(st, frag, 0);
            __syncthreads();
            sfloatx16 acc[2][2];
            int rp = 0, cg = 0;
            for (int it = 0; it < npair * ncg; ++it) {
                const int ncgx = cg + 1 < ncg ? cg + 1 : 0, nrp = cg + 1 < ncg ? rp : rp + 1;
                const bool more = it + 1 < npair * ncg;
                if (more) stage_load(st, nrp, ncgx);
                if (cg == 0) {
                    // (kpad is a multiple of 64: the second block of the last pair may be padding altogether)
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                        for (int q = 0; q < 2; ++q) init(acc[blk][q], q, 2 * rp + blk);
                }
                const half8 *base = frag + (size_t)(it & 1) * STAGE + lane;
                for (int c4 = 0; c4 < 8; c4 += 2) {
                    float v[2][2][8];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int q = 0; q < 2; ++q) load(v[u][q], row[q], cg * 128 + (c4 + u) * 16 + 8 * half);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        half8 bh[2], bl[2];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const int slot = cg * 128 + (c4 + u) * 16 + 8 * half;
                            centre(v[u][q], slot);
                            float sq = 0.0f;
                            convert(v[u][q], scale[q], bh[q], bl[q], sq);
                            n2[q] += rp == 0 ? sq : 0.0f;
                            asm volatile("" : "+v"(n2[q]));
                        }
                        multiply(base + (c4 + u) * 256, bh[0], bl[0], bh[1], bl[1], acc[0]);
                        multiply(base + (c4 + u) * 256 + 128, bh[0], bl[0], bh[1], bl[1], acc[1]);
                    }
                }
                if (cg + 1 == ncg) {
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk) {
                        if (2 * rp + blk < a.nblk) {
                            split_insert(top[0], acc[blk][0], 2 * rp + blk, big);
                            split_insert(top[1], acc[blk][1], 2 * rp + blk, big);
                        }
                    }
                }
                if (more) {
                    stage_put(st, frag + (size_t)((it + 1) & 1) * STAGE, nrp);
                    __syncthreads();
                }
                cg = ncgx;
                rp = nrp;
            }
        }
        SplitTop t;
        split_combine(top, t, half);
        swap2(n2[0], n2[1]);
        if constexpr (NC == 0) sum += splitq_finish_here<false>((u64)args, gw, t, n2[0] + n2[1], half ? ratio[1] : ratio[0], half ? direct[1] : direct[0], size);
        else sum += splitq_finish((u64)args, gw, t, n2[0] + n2[1], half ? ratio[1] : ratio[0], half ? direct[1] : direct[0], size);
    }
    sum = split_wave_sum(sum);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        double tot = 0.0;
        for (int v = 0; v < 8; ++v) tot += red[v];
        a.partials[blockIdx.x] = tot;
    }
}

template <int NC>
hipError_t split_launch_quant(const SplitQuant &a, int blocks, unsigned lds, hipStream_t s)
{
    const hipError_t e = hipFuncSetAttribute((const void *)split_quant_kernel<NC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_quant_kernel<NC>, dim3(blocks), dim3(SPLITQ_THREADS), lds, s, a);
    return hipGetLastError();
}

}  // namespace asgd
