// Eq. 8 on the fp16 matrix instructions, any row length: the nearest centroid of a sample from scores with fp16-split
// operands (split_core.h), the distance to it formed directly in fp32 and added in fp64.
//
// One workgroup of eight waves per compute unit walks groups of 512 samples; a wave takes 64 of them and keeps their
// operands in registers.  Nothing is known about the samples beforehand, so every sample gets a power-of-two scale of its
// own from its largest |x_j - m_j| (m: middle of some rows of the state) and a score is h_c + (products) * 1/scale, one
// more instruction than an accumulator that starts at h_c.  The state is split by every workgroup: once per launch when it
// fits the LDS, else block by block for every group of samples, the next block's rows on their way meanwhile (that costs
// 2 * 8 * 5 vector instructions per wave and pair of row blocks, next to 96 matrix instructions of 32 cycles).
#pragma once

#include "split_core.h"

namespace asgd {

struct SplitQuant {
    const float *x, *w;
    long long N;
    double *partials;
    int k, d, kpad, nblk, dpad, resident;
    int nan_is_inf;                        // a distance that is not a number counts as infinite
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
__device__ __forceinline__ void splitq_put(half8 *at, const float (&v)[8], float s)
{
    half8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float y = v[e] * s;
        hi[e] = (_Float16)y;
        lo[e] = (_Float16)(y - (float)hi[e]);
    }
    at[0] = hi;
    at[64] = lo;
}

// power of two that takes `most` to [2^12, 2^13) (any number when it is zero or not finite)
__device__ __forceinline__ float splitq_scale(float most)
{
    int q = 0;
    if (most > 0.0f && most < 3.0e38f) (void)frexpf(most, &q);
    return ldexpf(1.0f, max(-100, min(100, 13 - q)));
}

// distance of the lane pair's sample to centroid c, direct form; a lane adds the slots of its half-wave
__device__ __forceinline__ float splitq_distance(const float *row, const float *wrow, int d, int half)
{
    float d2 = 0.0f;
    for (int s0 = 0; s0 < d; s0 += 64) {
        float xv[4][8], wv[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int slot = min(s0 + 16 * u + 8 * half, (d - 1) & ~7);
            split_load8<true>(xv[u], row, slot, d);
            split_load8<true>(wv[u], wrow, slot, d);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int slot = s0 + 16 * u + 8 * half;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float t = split_slot_used(slot + e, d) ? xv[u][e] - wv[u][e] : 0.0f;
                d2 = fmaf(t, t, d2);
            }
        }
    }
    return d2;
}

template <int NC>
__global__ __launch_bounds__(SPLITQ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_quant_kernel(SplitQuant a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ double red[8];
    __shared__ float redf[8];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int k = a.k, d = a.d, nch = a.dpad / 16, npair = (a.nblk + 1) / 2;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs), *m = reinterpret_cast<float *>(smem + a.off_m);
    half8 *frag = reinterpret_cast<half8 *>(smem);

    // m by slot: mean of the first rows of the state (any value would do; one near the data keeps the operands small)
    for (int j = tid; j < a.dpad; j += SPLITQ_THREADS) {
        float s = 0.0f;
        if (split_slot_used(j, d)) {
            const float *col = a.w + split_column(j, d);
            float v[16];
            const int n = min(k, 16);
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = col[(size_t)min(q, n - 1) * d];
#pragma unroll
            for (int q = 0; q < 16; ++q) s += q < n ? v[q] : 0.0f;
            s /= (float)n;
            if (!(fabsf(s) < 3.0e38f)) s = 0.0f;
        }
        m[j] = s;
    }
    __syncthreads();
    // h_c = -|v_c|^2/2 and the largest |v|: g lanes per row
    int g = 1;
    while (g < a.dpad / 8 && g < 64) g *= 2;
    float vabs = 0.0f;
    {
        const int lane_g = tid & (g - 1), ngrp = SPLITQ_THREADS / g;
        for (int c0 = tid / g; c0 < a.kpad; c0 += 4 * ngrp) {
            float sq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int slot = 8 * lane_g; slot < a.dpad; slot += 8 * g) {
                float v[4][8];
#pragma unroll
                for (int q = 0; q < 4; ++q) splitq_row(v[q], a.w, m, c0 + q * ngrp, k, slot, d);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        sq[q] = fmaf(v[q][e], v[q][e], sq[q]);
                        const float av = fabsf(v[q][e]);
                        if (av < 3.0e38f) vabs = fmaxf(vabs, av);
                    }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                for (int off = g / 2; off > 0; off >>= 1) sq[q] += __shfl_xor(sq[q], off, 64);
                const int c = c0 + q * ngrp;
                if (lane_g == 0 && c < a.kpad) hs[c] = c < k ? -0.5f * sq[q] : SPLIT_PAD_SCORE;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) vabs = fmaxf(vabs, __shfl_xor(vabs, off, 64));
    if (lane == 0) redf[wave] = vabs;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) vabs = fmaxf(vabs, redf[q]);
    const float sw = splitq_scale(vabs);

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
    auto stage_put = [&](const float (&v)[NU][8], half8 *dst) {
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            const int un = tid + q * SPLITQ_THREADS, c = un / (SC * 2), slot = (un - c * (SC * 2)) * 8;
            if (un < 64 * SC * 2) splitq_put(dst + split_frag_at(c, slot, SC), v[q], sw);
        }
    };
    constexpr int STAGE = SC * 256;                        // half8 per stage
    if (NC != 0 && a.resident) {
        for (int rp = 0; rp < npair; ++rp) {
            float v[NU][8];
            stage_load(v, rp, 0);
            stage_put(v, frag + (size_t)rp * STAGE);
        }
    }
    __syncthreads();

    double sum = 0.0;
    for (long long g0 = (long long)blockIdx.x * SPLITQ_THREADS; g0 < a.N; g0 += (long long)gridDim.x * SPLITQ_THREADS) {
        const long long gw = g0 + wave * 64;
        const float *row[2];
        float inv[2], best[2] = {-INFINITY, -INFINITY}, scale[2];
        int bblk[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const long long n = gw + 32 * q + l32;
            row[q] = a.x + (size_t)(n < a.N ? n : a.N - 1) * d;
        }
        auto own_scale = [&](float most) {
            most = fmaxf(most, __shfl_xor(most, 32, 64));
            return splitq_scale(most);
        };
        auto score = [&](const sfloatx16 &acc, int q, int blk) {
            const float4 *hp = reinterpret_cast<const float4 *>(hs + blk * 32 + 4 * half);
            float bm = -INFINITY;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float4 h = hp[2 * r4];
                const float hv[4] = {h.x, h.y, h.z, h.w};
                float t[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float sc = fmaf(acc[4 * r4 + r], inv[q], hv[r]);
                    t[r] = __int_as_float((__float_as_int(sc) & ~15) | (4 * r4 + r));
                }
                bm = fmaxf(fmaxf(fmaxf(bm, t[0]), t[1]), fmaxf(t[2], t[3]));
            }
            if (bm > best[q]) { best[q] = bm; bblk[q] = blk; }
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
        auto convert = [&](const float (&v)[8], float s, int slot, half8 &hi, half8 &lo) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float y = v[e] * s;
                hi[e] = (_Float16)y;
                lo[e] = (_Float16)(y - (float)hi[e]);
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
                scale[q] = own_scale(most);
                inv[q] = 1.0f / (scale[q] * sw);
#pragma unroll
                for (int ch = 0; ch < SC; ++ch) {
                    convert(v[ch], scale[q], ch * 16 + 8 * half, bh[q][ch], bl[q][ch]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            float st[NU][8];
            if (!a.resident) {
                __syncthreads();                           // nobody still reads the first stage
                stage_load(st, 0, 0);
                stage_put(st, frag);
                __syncthreads();
            }
            for (int rp = 0; rp < npair; ++rp) {
                const half8 *base = frag + (size_t)(a.resident ? rp : (rp & 1)) * STAGE + lane;
                if (!a.resident && rp + 1 < npair) stage_load(st, rp + 1, 0);
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    if (2 * rp + blk >= a.nblk) break;
                    sfloatx16 acc[2];
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.0f;
#pragma unroll
                    for (int ch = 0; ch < SC; ++ch) {
                        multiply(base + ch * 256 + blk * 128, bh[0][ch], bl[0][ch], bh[1][ch], bl[1][ch], acc);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    score(acc[0], 0, 2 * rp + blk);
                    score(acc[1], 1, 2 * rp + blk);
                }
                if (!a.resident && rp + 1 < npair) {
                    stage_put(st, frag + (size_t)((rp + 1) & 1) * STAGE);
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
                scale[q] = own_scale(most);
                inv[q] = 1.0f / (scale[q] * sw);
            }
            float st[NU][8];
            __syncthreads();
            stage_load(st, 0, 0);
            stage_put(st, frag);
            __syncthreads();
            sfloatx16 acc[2][2];
            int rp = 0, cg = 0;
            for (int it = 0; it < npair * ncg; ++it) {
                const int ncgx = cg + 1 < ncg ? cg + 1 : 0, nrp = cg + 1 < ncg ? rp : rp + 1;
                const bool more = it + 1 < npair * ncg;
                if (more) stage_load(st, nrp, ncgx);
                if (cg == 0) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[0][0][r] = acc[0][1][r] = acc[1][0][r] = acc[1][1][r] = 0.0f;
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
                            convert(v[u][q], scale[q], slot, bh[q], bl[q]);
                        }
                        multiply(base + (c4 + u) * 256, bh[0], bl[0], bh[1], bl[1], acc[0]);
                        multiply(base + (c4 + u) * 256 + 128, bh[0], bl[0], bh[1], bl[1], acc[1]);
                    }
                }
                if (cg + 1 == ncg) {
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk) {
                        if (2 * rp + blk < a.nblk) {
                            score(acc[blk][0], 0, 2 * rp + blk);
                            score(acc[blk][1], 1, 2 * rp + blk);
                        }
                    }
                }
                if (more) {
                    stage_put(st, frag + (size_t)((it + 1) & 1) * STAGE);
                    __syncthreads();
                }
                cg = ncgx;
                rp = nrp;
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = __float_as_int(best[q]) & 15;
            int c = bblk[q] * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            const float ob = __shfl_xor(best[q], 32, 64);       // the other half-wave saw the other rows
            const int oc = __shfl_xor(c, 32, 64);
            if (ob > best[q] || (ob == best[q] && oc < c)) c = oc;
            c = min(c, k - 1);
            float d2 = splitq_distance(row[q], a.w + (size_t)c * d, d, half);
            d2 += __shfl_xor(d2, 32, 64);
            if (a.nan_is_inf && d2 != d2) d2 = INFINITY;
            if (half == 0 && gw + 32 * q + l32 < a.N) sum += (double)(0.5f * d2);
        }
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
