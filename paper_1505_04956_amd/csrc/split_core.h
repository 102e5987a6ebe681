// Scores of the matrix-core kernels that take any row length: x.w_c - |w_c|^2/2 with fp32 operands split into two fp16
// parts each (v_mfma_f32_32x32x16_f16, sixteen times the rate of the fp32 matrix instruction; three products per pair of
// operands, so a little over five times the fp32 rate), the running top three of a sample and the exact decision between
// close candidates.
//
// Both operands are taken relative to a fixed point m (near the middle of the data), y = x - m and v = w - m: the
// nearest centroid does not change, |y| and |v| - and with them the rounding error of a score - are as small as the
// spread of the data, however far it lies from the origin.  y and v are rounded to fp32 (relative 2^-24), scaled by a
// power of two so that nothing reaches the largest fp16 number, and split: hi = fp16(y), lo = fp16(y - hi); what is
// left is at most 2^-22 |y| (or half the smallest fp16 subnormal, 2^-25 in scaled units).
//
// Error of a score.  Per element: rounding of y and v 2 * 2^-24, rest of the two splits 2 * 2^-22, product lo * lo that is
// not formed 2^-22 - fourteen units of 2^-24 |y_j v_j|, and by Cauchy's inequality of |y||v|; subnormal rests 2^-25
// sqrt(d) (|y| + |v|) in scaled units.  Accumulation: a matrix instruction adds sixteen exact products to a running
// fp32 sum, 3 d/16 of them per score; each is allowed SPLIT_ULP_PER_MFMA = 6 units of 2^-23 of |y||v| + |h| (measured
// on the device: below 1.1 on random and cancelling operands of one size, 4.0 on operands built to lose the most, one
// large product and fifteen that are cut off below its last place).  h = -|v|^2/2 is a sum of d squares, lane-local chains
// and a butterfly: at most d/64 + 16 roundings.  The tag in the low mantissa bits: 2^-18 of the score.
#pragma once

#include <type_traits>

#include "asgd_internal.h"
#include "split_plan.h"

namespace asgd {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float sfloatx16 __attribute__((ext_vector_type(16)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));      // rows of any length: 4-byte aligned
typedef unsigned long long u64;

constexpr float SPLIT_PAD_SCORE = -1.0e30f;       // offset of the padding rows: never the nearest
constexpr float SPLIT_ULP_PER_MFMA = 6.0f;

// thr = c1 * (|y||v|max + |v|max^2/2) + c2 * (|y| + |v|max), all in scaled units, for row length `dpad`
__device__ __forceinline__ float split_c1(int dpad)
{
    const float u = 5.9604645e-8f;
    const float acc = SPLIT_ULP_PER_MFMA * 2.0f * 3.0f * (float)(dpad / 16);
    return 2.0f * u * (acc + 14.0f + (float)(dpad / 64) + 20.0f) + 7.62939453125e-6f;
}
__device__ __forceinline__ float split_c2(int dpad) { return 2.0f * 2.98023224e-8f * 1.001f * sqrtf((float)dpad); }

// The lane number as a value of its own: what is derived from it (addresses, masks) is formed where it is used instead of
// being kept in registers across the loop over the samples - 60 of them, spilled around every group.
__device__ __forceinline__ int split_lane()
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

struct SplitTop {
    float v1, v2, v3;      // three largest scores, the accumulator register in the low mantissa bits
    int i1, i2;            // block of 32 rows (later: row) the two largest came from
};

__device__ __forceinline__ float split_opaque_infinity()
{
    float big = INFINITY;
    asm volatile("" : "+s"(big));
    return big;
}

// Inserts the 16 scores a lane holds of a block of 32 rows: four instructions per score (tag, three v_med3_f32; the
// median with +infinity is the maximum without the NaN-quieting instruction the compiler puts before v_max_f32).
__device__ __forceinline__ void split_insert(SplitTop &t, const sfloatx16 &acc, int block, float big)
{
    const int o1 = __float_as_int(t.v1), o2 = __float_as_int(t.v2);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float s = __int_as_float((__float_as_int(acc[r]) & ~31) | r);
        t.v3 = __builtin_amdgcn_fmed3f(t.v2, t.v3, s);
        t.v2 = __builtin_amdgcn_fmed3f(t.v1, t.v2, s);
        t.v1 = __builtin_amdgcn_fmed3f(t.v1, s, big);
    }
    const int n1 = __float_as_int(t.v1), n2 = __float_as_int(t.v2);
    const int b2 = n2 == o2 ? t.i2 : (n2 == o1 ? t.i1 : block);
    t.i1 = n1 != o1 ? block : t.i1;
    t.i2 = b2;
}

__device__ __forceinline__ void split_merge(SplitTop &t, float s, int c)
{
    const bool g1 = s > t.v1, g2 = s > t.v2, g3 = s > t.v3;
    t.v3 = g2 ? t.v2 : (g3 ? s : t.v3);
    t.i2 = g1 ? t.i1 : (g2 ? c : t.i2);
    t.v2 = g1 ? t.v1 : (g2 ? s : t.v2);
    t.i1 = g1 ? c : t.i1;
    t.v1 = g1 ? s : t.v1;
}

// After swap2(a, b) the lower half-wave holds in `a` its own a and in `b` the upper half-wave's a; the upper one in `a`
// the lower half-wave's b and in `b` its own: both halves of the sample a lane owns.
__device__ __forceinline__ void swap2(unsigned &a, unsigned &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap2(float &a, float &b)
{
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    swap2(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
__device__ __forceinline__ void swap2(int &a, int &b)
{
    unsigned x = (unsigned)a, y = (unsigned)b;
    swap2(x, y);
    a = (int)x;
    b = (int)y;
}

// A lane holds results of two samples (columns l mod 32 of the two tiles of its wave), each for half of the rows.
// Afterwards `t` is the result over all rows for ONE sample, number `lane` of the wave's 64.
__device__ __forceinline__ void split_combine(SplitTop (&top)[2], SplitTop &t, int half)
{
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        // register r of a 32x32 result is row 8*(r/4) + 4*half + r%4
        const int r1 = __float_as_int(top[m].v1) & 15, r2 = __float_as_int(top[m].v2) & 15;
        top[m].i1 = top[m].i1 * 32 + 8 * (r1 >> 2) + 4 * half + (r1 & 3);
        top[m].i2 = top[m].i2 * 32 + 8 * (r2 >> 2) + 4 * half + (r2 & 3);
    }
    swap2(top[0].v1, top[1].v1);
    swap2(top[0].v2, top[1].v2);
    swap2(top[0].v3, top[1].v3);
    swap2(top[0].i1, top[1].i1);
    swap2(top[0].i2, top[1].i2);
    t = top[0];
    split_merge(t, top[1].v1, top[1].i1);
    split_merge(t, top[1].v2, top[1].i2);
    t.v3 = fmaxf(t.v3, top[1].v3);
}

__device__ __forceinline__ double split_wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Nearest of all k centroids in fp64, every lane its own sample `xl`; four centroids and four columns in flight (one of
// each was a chain of latencies: every sample of k = 1024, d = 128, b = 4096 decided here took 383 ms per step, now 34).
__device__ inline int split_scan_own(const float *xl, const float *w, int k, int d)
{
    double best = INFINITY;
    int arg = 0;
    for (int c0 = 0; c0 < k; c0 += 4) {
        double sd[4] = {0.0, 0.0, 0.0, 0.0};
        const float *wr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) wr[q] = w + (size_t)min(c0 + q, k - 1) * d;
        int j = 0;
        for (; j + 4 <= d; j += 4) {
            const float4u x4 = *reinterpret_cast<const float4u *>(xl + j);
            float4u w4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) w4[q] = *reinterpret_cast<const float4u *>(wr[q] + j);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double x = (double)x4[e];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double diff = x - (double)w4[q][e];
                    sd[q] += diff * diff;
                }
            }
        }
        for (; j < d; ++j) {
            const double x = (double)xl[j];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double diff = x - (double)wr[q][j];
                sd[q] += diff * diff;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (c0 + q < k && sd[q] < best) { best = sd[q]; arg = c0 + q; }
    }
    return arg;
}

// Nearest of the rows [c_lo, c_hi) in fp64 to ONE sample, by a wave: sixteen lanes per centroid, four columns each, so that sixteen centroids are in
// flight (a lane per centroid was a chain of d loads and took 0.2 ms for one sample, k = 256, d = 384).
__device__ __forceinline__ void split_scan_wave(const float *xl, const float *w, int c_lo, int c_hi, int d, double &best, int &barg)
{
    const int lane = split_lane(), l16 = lane & 15, quarter = lane >> 4;
    best = INFINITY;
    barg = 0;
    for (int c0 = c_lo; c0 < c_hi; c0 += 16) {
        double sd[4] = {0.0, 0.0, 0.0, 0.0};
        const float *wr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) wr[q] = w + (size_t)min(c0 + 4 * q + quarter, c_hi - 1) * d;
        for (int j = 4 * l16; j < d; j += 64) {
            float xv[4], wv[4][4];
            if (j + 4 <= d) {
                const float4u x4 = *reinterpret_cast<const float4u *>(xl + j);
                float4u w4[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) w4[q] = *reinterpret_cast<const float4u *>(wr[q] + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xv[e] = x4[e];
#pragma unroll
                    for (int q = 0; q < 4; ++q) wv[q][e] = w4[q][e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = j + e < d;
                    xv[e] = in ? xl[j + e] : 0.0f;
#pragma unroll
                    for (int q = 0; q < 4; ++q) wv[q][e] = in ? wr[q][j + e] : 0.0f;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double diff = (double)xv[e] - (double)wv[q][e];
                    sd[q] += diff * diff;
                }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) sd[q] += __shfl_xor(sd[q], off, 64);
            const int cq = c0 + 4 * q + quarter;
            if (cq < c_hi && sd[q] < best) { best = sd[q]; barg = cq; }
        }
    }
#pragma unroll
    for (int off = 32; off > 8; off >>= 1) {
        const double ob = __shfl_xor(best, off, 64);
        const int oa = __shfl_xor(barg, off, 64);
        if (ob < best || (ob == best && oa < barg)) { best = ob; barg = oa; }
    }
}

// The exact-arithmetic nearest centroid of the fp32 state for the samples of a wave: a lane owns the sample in row `own` of
// `xb` (valid or not, that of lane 0 always), `t` its best scores.  Closer than thr: decided in fp64, two candidates by the sign of
// sum_j (w_aj - w_bj)(w_aj + w_bj - 2 x_j), more by all k distances in direct form; the lowest index wins exact ties.
// thr may be infinite (then everything is decided in fp64); scores may be NaN.
// DEFER: where all k distances are asked for, the sample's row goes to the workgroup's list `hard` as long as there is room, and the
// result is -1 (split_scan_hard()); without it `own` is the lane.
template <bool DEFER>
__device__ __forceinline__ int split_settle(const SplitTop &t, float thr, bool valid, const float *xb, int own, const float *w, int k,
                                            int d, int &rechecks, int *hard = nullptr, int *hard_count = nullptr)
{
    const int lane = split_lane();
    int arg = min(max(t.i1, 0), k - 1);
    const int second = min(max(t.i2, 0), k - 1);
    const bool close2 = valid && !(t.v1 - t.v2 > thr);
    bool close3 = close2 && (!(t.v1 - t.v3 > thr) || __float_as_int(t.v1) == __float_as_int(t.v2) || second == arg);
    rechecks += close2 ? 1 : 0;
    unsigned long long pm = __ballot(close2 && !close3);
    if constexpr (DEFER) {
        const unsigned long long all = __ballot(close3);
        if (all) {
            int base = 0;
            if (lane == 0) base = atomicAdd(hard_count, __popcll(all));
            const int at = __builtin_amdgcn_readfirstlane(base) + __popcll(all & ((1ULL << lane) - 1));
            if (close3 && at < SPLIT_HARD) {
                hard[at] = own;
                arg = -1;
                close3 = false;
            }
        }
    }
    while (pm) {
        int L[4], ca[4], cb[4], at[4];
        double dd[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            L[q] = -1; ca[q] = 0; cb[q] = 0; dd[q] = 0.0;
            at[q] = DEFER ? __builtin_amdgcn_readfirstlane(own) : 0;
            if (pm) {
                L[q] = __builtin_ctzll(pm);
                pm &= pm - 1;
                ca[q] = __builtin_amdgcn_readlane(arg, L[q]);
                cb[q] = __builtin_amdgcn_readlane(second, L[q]);
                at[q] = DEFER ? __builtin_amdgcn_readlane(own, L[q]) : L[q];
            }
        }
        for (int j0 = 0; j0 < d; j0 += 128) {
            float wa[2][4], wb[2][4], xx[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = j0 + 64 * h + lane, jc = j < d ? j : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    wa[h][q] = w[(size_t)ca[q] * d + jc];
                    wb[h][q] = w[(size_t)cb[q] * d + jc];
                    xx[h][q] = xb[(size_t)at[q] * d + jc];
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double a = (double)wa[h][q], b = (double)wb[h][q];
                    if (j0 + 64 * h + lane < d) dd[q] += (a - b) * ((a + b) - 2.0 * (double)xx[h][q]);
                }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double s = split_wave_sum(dd[q]);
            const int res = s < 0.0 ? ca[q] : (s > 0.0 ? cb[q] : min(ca[q], cb[q]));
            if (lane == L[q]) arg = res;
        }
    }
    unsigned long long fm = __ballot(close3);
    if (__popcll(fm) <= 8) {
        // few: one sample at a time
        while (fm) {
            const int L = __builtin_ctzll(fm);
            fm &= fm - 1;
            const float *xl = xb + (size_t)(DEFER ? __builtin_amdgcn_readlane(own, L) : L) * d;
            double best;
            int barg;
            split_scan_wave(xl, w, 0, k, d, best, barg);
            // (no distance below infinity: centroid 0, like a scan that starts there)
            if (lane == L) arg = best < INFINITY ? barg : 0;
        }
    } else if (close3) {
        arg = split_scan_own(xb + (size_t)(DEFER ? own : lane) * d, w, k, d);
    }
    return arg;
}

// Column of a row that slot j of its operands holds (columns go to the slots in order, eight at a time).  The last group
// of a row whose length is not a multiple of eight takes the row's LAST eight columns, so that it can be loaded like the
// others; those that the group before it holds already count as zero, like the groups past the end.
__host__ __device__ inline int split_column(int slot, int d)
{
    const int g = slot & ~7;
    return d >= 8 && g + 8 > d ? d - 8 + (slot & 7) : slot;
}
__host__ __device__ inline bool split_slot_used(int slot, int d)
{
    const int c = split_column(slot, d);
    return c < d && c >= (slot & ~7);
}

// The columns of the eight slots from `slot` on.  TAIL: not all of them may be in use (the values of the others are
// columns of the same row, nothing past its end is read).
template <bool TAIL>
__device__ __forceinline__ void split_load8(float (&v)[8], const float *row, int slot, int d)
{
    if (!TAIL || d >= 8) {
        const float *p = row + (TAIL ? min(slot, d - 8) : slot);
        const float4u a = *reinterpret_cast<const float4u *>(p), b = *reinterpret_cast<const float4u *>(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = row[min(e, d - 1)];
    }
}
// hi and lo parts of y = fma(x, s, ms) (ms = -m * s by slot, exact products: s is a power of two); adds y^2 to n2
template <bool TAIL>
__device__ __forceinline__ void split_convert(const float (&v)[8], float s, const float *ms, int slot, int d, half8 &hi,
                                              half8 &lo, float &n2)
{
    const float4 m0 = *reinterpret_cast<const float4 *>(ms + slot), m1 = *reinterpret_cast<const float4 *>(ms + slot + 4);
    const float mm[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float y = fmaf(v[e], s, mm[e]);
        if (TAIL) y = split_slot_used(slot + e, d) ? y : 0.0f;
        const _Float16 h = (_Float16)y;
        hi[e] = h;
        lo[e] = (_Float16)(y - (float)h);
        n2 = fmaf(y, y, n2);
    }
}

// 1 KB pieces [0, n) from global memory to LDS, the waves of the workgroup in turn; no registers pass the data
__device__ __forceinline__ void split_stage(const unsigned char *src, unsigned char *dst, int n)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    for (int q = wave; q < n; q += nw)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (size_t)q * SPLIT_PIECE + lane * 16),
                                         (__attribute__((address_space(3))) void *)(dst + q * SPLIT_PIECE), 16, 0, 0);
}
__device__ __forceinline__ void split_stage_wait()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

__device__ __forceinline__ void split_init_acc(sfloatx16 &acc, const float *hs, int block, int half)
{
    const float4 *hp = reinterpret_cast<const float4 *>(hs + block * 32 + 4 * half);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 h = hp[2 * q];
        acc[4 * q + 0] = h.x; acc[4 * q + 1] = h.y; acc[4 * q + 2] = h.z; acc[4 * q + 3] = h.w;
    }
}

// (a call passes its arguments in vector registers; what is uniform is read back into scalar ones)
__device__ __forceinline__ u64 split_uniform64(u64 v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v), hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return (u64)hi << 32 | lo;
}

}  // namespace

}  // namespace asgd
