// Screening: scores from the high fp16 parts of both operands alone (split_core.h), one matrix instruction where the full
// scores take three.  The error of such a score is bounded with the norms of what the rounding to fp16 left over, measured for every
// sample and for the rows of the state (a third of what Cauchy's inequality with 2^-11 allows): a sample whose best score
// leads by more than the bound is decided, the others - a few in a hundred of ordinary data - are noted in a list and
// scored again with all three products.  So only the best score, where it came from, and the second best are
// kept: nine instructions for four scores (the full scores: sixteen).
//
// Error of a score.  With y = yh + yl and v = vh + vl, y.v - yh.vh = yl.v + yh.vl, at most |yl||v| + (|y| + |yl|)|vl|.  The rest
// is as in split_core.h, with d/16 matrix instructions per score.
#pragma once

#include "split_core.h"

namespace asgd {

namespace {

struct ScreenTop {
    float v1, v2;      // two largest scores, the accumulator register in the low mantissa bits
    int i1;            // block of 32 rows (later: row) the largest came from
};

__device__ __forceinline__ float screen_max3(float a, float b, float c)
{
    // (the compiler quiets NaNs of every operand first; these are results of integer instructions, no matrix results)
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Inserts the 16 scores a lane holds of a block of 32 rows.
__device__ __forceinline__ void screen_insert(ScreenTop &t, const sfloatx16 &acc, int block)
{
    const int o1 = __float_as_int(t.v1);
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = __int_as_float((__float_as_int(acc[r + e]) & ~15) | (r + e));
        // the second largest of the best so far and two more
        const float ma = __builtin_amdgcn_fmed3f(t.v1, s[0], s[1]);
        t.v1 = screen_max3(t.v1, s[0], s[1]);
        const float mb = __builtin_amdgcn_fmed3f(t.v1, s[2], s[3]);
        t.v1 = screen_max3(t.v1, s[2], s[3]);
        t.v2 = screen_max3(t.v2, ma, mb);
    }
    t.i1 = __float_as_int(t.v1) != o1 ? block : t.i1;
}

// As split_combine(): afterwards `t` is the result over all rows for the sample number `lane` of the 64 of two tiles.
__device__ __forceinline__ void screen_combine(ScreenTop &a, ScreenTop &b, ScreenTop &t, int half)
{
    const int ra = __float_as_int(a.v1) & 15, rb = __float_as_int(b.v1) & 15;
    a.i1 = a.i1 * 32 + 8 * (ra >> 2) + 4 * half + (ra & 3);
    b.i1 = b.i1 * 32 + 8 * (rb >> 2) + 4 * half + (rb & 3);
    swap2(a.v1, b.v1);
    swap2(a.v2, b.v2);
    swap2(a.i1, b.i1);
    t.v1 = fmaxf(a.v1, b.v1);
    t.v2 = fmaxf(fminf(a.v1, b.v1), fmaxf(a.v2, b.v2));
    t.i1 = b.v1 > a.v1 ? b.i1 : a.i1;
}

// Twice the error of a score, in units of score: yn >= |y|, rl >= |yl| in scaled units of the sample, v >= |v| and vl >= |vl| in
// those of the state, offset >= |h|.
__device__ __forceinline__ float screen_bound(float yn, float rl, float v, float vl, float offset, int dpad)
{
    const float u = 5.9604645e-8f;
    const float acc = SPLIT_ULP_PER_MFMA * 2.0f * (float)(dpad / 16);
    const float c1 = 2.0f * u * (acc + 14.0f + (float)(dpad / 64) + 20.0f) + 7.62939453125e-6f;
    return 2.0002f * (rl * v + (yn + rl) * vl) + c1 * (yn * v + offset);
}

// hi parts of y = fma(x, s, ms) as in split_convert(); adds y^2 to n2 and the square of what is left over to r2
template <bool TAIL>
__device__ __forceinline__ void screen_convert(const float (&v)[8], float s, const float *ms, int slot, int d, half8 &hi, float &n2, float &r2)
{
    const float4 m0 = *reinterpret_cast<const float4 *>(ms + slot), m1 = *reinterpret_cast<const float4 *>(ms + slot + 4);
    const float mm[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float y = fmaf(v[e], s, mm[e]);
        if (TAIL) y = split_slot_used(slot + e, d) ? y : 0.0f;
        const _Float16 h = (_Float16)y;
        hi[e] = h;
        const float rest = y - (float)h;
        n2 = fmaf(y, y, n2);
        r2 = fmaf(rest, rest, r2);
    }
    asm volatile("" : "+v"(hi));             // (packed here: left to the compiler they stayed apart, in twice the registers, until they were used)
}

}  // namespace

}  // namespace asgd
