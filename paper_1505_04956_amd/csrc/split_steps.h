// Step kernels for any row length: a step is an assignment launch over (worker, share of the mini-batch), for large
// states a launch that forms the gradient sums, and an update launch over the workers.  Shared declarations and the
// assignment kernels; see kernels_split.hip for the others.
#pragma once

#include "split_core.h"

namespace asgd {

// Operands of a worker's state rows, as the matrix instructions want them: rows in pairs of 32-row blocks, columns in
// chunks of 16; [row pair][chunk][block of the pair][hi, lo] pieces of 1 KB, piece = 64 lanes x 8 fp16, lane l holding row
// l % 32, columns 8 * (l / 32) .. + 7 of the chunk.
constexpr int SPLIT_PIECE = 1024;                    // bytes
constexpr int SPLIT_STAGE = 8 * 4 * SPLIT_PIECE;     // a row pair's eight chunks: what the long-row kernel stages at a time

struct SplitState {                // one per worker and step modulo 3
    float sw;                      // scale of the operands
    unsigned vabs, n2;             // bit patterns of the largest |v_cj| and |v_c|^2; above those of all numbers if not finite
    unsigned pad[29];              // a cache line each: atomics on one line wait for each other, and that took 15 us
};

struct SplitArgs {
    const float *x, *w;              // samples, states
    const unsigned char *frag;       // W x frag_bytes
    const float *hs;                 // W x kpad: -|v_c|^2/2 * sx * sw, SPLIT_PAD_SCORE for the padding rows
    const SplitState *state;         // W
    const float *ms;                 // dpad: -m_j * sx, zero past d
    const float *xmeta;              // sx
    const double *colscale;          // d scales of the fixed-point sums, then d inverse scales
    int *idx;                        // W x b assignments (null: not stored)
    float *part;                     // shares x W x k x d sums of a share's samples
    int *cntpart;                    // shares x W x k samples per centroid
    int32_t *dump;                   // W x b of this step, or null
    long long *counters;
    size_t frag_bytes;
    long long H, row0;
    int k, d, b, W, kpad, nblk, dpad;
    int shares, share_len;           // share_len: samples of a share, a multiple of 64
    int resident, fused, vec4;
    unsigned off_cells, off_cnt, off_hs, off_ms, off_args;
};

// A term x * scale is rounded to an integer by adding 1.5 * 2^52 in the fused multiply-add and its bit pattern is added
// to a 64-bit cell; the count times the bit pattern of 1.5 * 2^52 comes off when the cell is read, modulo 2^64.
constexpr double SPLIT_MAGIC = 6755399441055744.0;
__device__ __forceinline__ u64 split_term(float x, double scale)
{
    return (u64)__double_as_longlong(fma((double)x, scale, SPLIT_MAGIC));
}
__device__ __forceinline__ void split_add(u64 *cell, u64 v)
{
    (void)__hip_atomic_fetch_add(cell, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ float split_sum(u64 cell, int count, double inv)
{
    const u64 bias = (u64)__double_as_longlong(SPLIT_MAGIC);
    return (float)((double)(long long)(cell - (u64)count * bias) * inv);
}

// The samples of a wave (rows 0 .. nv-1 of xg, their centroids in args) into the cells.  A lane keeps its columns (four,
// or two where rows are not 16-byte aligned) and their scales; eight or sixteen rows in flight: the reads hit a cache, and
// with fewer in flight this pass was a chain of their latencies (75 columns, 256 workers: half of the launch).
__device__ inline void split_accumulate(const SplitArgs &a, const float *xg, int nv, const int *args, u64 *cells, int *cnt)
{
    const int lane = threadIdx.x & 63, d = a.d;
    if (lane < nv) atomicAdd(&cnt[args[lane]], 1);
    if (a.vec4) {
        const int q4 = d >> 2, R = 64 / q4, r = lane / q4, c = lane - r * q4;
        if (r < R) {
            constexpr int U = 8;
            double s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = a.colscale[4 * c + e];
            const float4 *src = reinterpret_cast<const float4 *>(xg) + c;
            for (int n0 = r; n0 < nv; n0 += U * R) {
                float4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = src[(unsigned)(min(n0 + u * R, nv - 1) * q4)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (n0 + u * R < nv) {
                        u64 *cell = cells + args[n0 + u * R] * d + 4 * c;
                        split_add(cell + 0, split_term(v[u].x, s[0]));
                        split_add(cell + 1, split_term(v[u].y, s[1]));
                        split_add(cell + 2, split_term(v[u].z, s[2]));
                        split_add(cell + 3, split_term(v[u].w, s[3]));
                    }
                }
            }
        }
    } else {
        // pairs of columns; the last lane of an odd row loads the pair before the end and uses its second half
        constexpr int U = 16;
        const int q2 = (d + 1) >> 1, R = 64 / q2, r = lane / q2, c = 2 * (lane - r * q2);
        if (r < R) {
            const bool odd = c + 1 == d;                       // one column left
            const int c0 = odd ? max(d - 2, 0) : c;
            const double s0 = a.colscale[c], s1 = a.colscale[odd ? c : c + 1];
            for (int n0 = r; n0 < nv; n0 += U * R) {
                float v0[U], v1[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const unsigned o = (unsigned)(min(n0 + u * R, nv - 1) * d + c0);
                    v0[u] = xg[o];
                    v1[u] = xg[o + (d > 1 ? 1 : 0)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (n0 + u * R < nv) {
                        u64 *cell = cells + args[n0 + u * R] * d + c;
                        split_add(cell, split_term(odd ? v1[u] : v0[u], s0));
                        if (!odd) split_add(cell + 1, split_term(v1[u], s1));
                    }
                }
            }
        }
    }
}

// Sums and counts of a workgroup's cells to the share's row of `part`.
__device__ inline void split_flush(const SplitArgs &a, int worker, int share, const u64 *cells, const int *cnt)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6, d = a.d;
    float *out = a.part + ((size_t)share * a.W + worker) * a.k * d;
    const int R = d < 64 ? 64 / d : 1, r = d < 64 ? lane / d : 0;
    if (r < R)
        for (int j = d < 64 ? lane - r * d : lane; j < d; j += 64) {
            const double inv = a.colscale[d + j];
            for (int c = wave * R + r; c < a.k; c += nw * R) out[c * d + j] = split_sum(cells[c * d + j], cnt[c], inv);
        }
    int *oc = a.cntpart + ((size_t)share * a.W + worker) * a.k;
    for (int c = threadIdx.x; c < a.k; c += blockDim.x) oc[c] = cnt[c];
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

// What a workgroup does once a group's best scores are known, the same in both assignment kernels.
__device__ __forceinline__ void split_finish_group(const SplitArgs &a, SplitTop (&top)[2], float (&n2)[2], int worker, int g,
                                                   int n_hi, const float *xb, int half, int *args, u64 *cells, int *cnt,
                                                   int &rechecks)
{
    const int lane = threadIdx.x & 63;
    SplitTop t;
    split_combine(top, t, half);
    swap2(n2[0], n2[1]);
    const float yn = sqrtf(n2[0] + n2[1]) * 1.0001f;
    const SplitState st = a.state[worker];
    const float sw = st.sw, vmax = sqrtf(__uint_as_float(st.n2)) * 1.0001f * sw, sx = a.xmeta[0];
    float thr = split_c1(a.dpad) * (yn * vmax + 0.5f * vmax * vmax * (sx / sw)) + split_c2(a.dpad) * (yn + vmax);
    // a state that is not finite, or has outgrown the scale of its fp16 operands: everything in fp64
    if (st.n2 >= 0x7f800000u || st.vabs >= 0x7f800000u || !(__uint_as_float(st.vabs) * sw < 32768.0f)) thr = INFINITY;
    const float *xg = xb + (size_t)g * a.d;
    const bool valid = g + lane < n_hi;
    const int arg = split_settle(t, thr, valid, xg, a.w + (size_t)worker * a.k * a.d, a.k, a.d, rechecks);
    if (valid) {
        if (a.idx) a.idx[(size_t)worker * a.b + g + lane] = arg;
        if (a.dump) a.dump[(size_t)worker * a.b + g + lane] = arg;
    }
    if (a.fused) {
        args[lane] = valid ? arg : 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        split_accumulate(a, xg, min(64, n_hi - g), args, cells, cnt);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

__device__ __forceinline__ void split_count_rechecks(const SplitArgs &a, int worker, int rechecks)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rechecks += __shfl_xor(rechecks, off, 64);
    if ((threadIdx.x & 63) == 0 && rechecks)
        atomicAdd((u64 *)&a.counters[(size_t)worker * CNT_STRIDE + CNT_RECHECK], (u64)rechecks);
}

// Assignment for rows of at most 16 * NC columns, NC <= 8.  A wave takes 64 samples at a time and keeps their operands in
// registers (NC * 16 registers); the state's operands come from LDS, resident when they fit, else one row pair at a time
// through two stages.  fused: the gradient sums are formed right away from a second, coalesced read of the wave's
// samples (in a cache still), in 64-bit fixed-point cells in LDS.
template <int NC>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NC <= 2 ? 3 : 2, NC <= 2 ? 3 : 2))) void split_assign_kernel(SplitArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int worker = blockIdx.x % a.W, share = blockIdx.x / a.W;
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, npair = (a.nblk + 1) / 2;
    u64 *cells = reinterpret_cast<u64 *>(smem + a.off_cells);
    int *cnt = reinterpret_cast<int *>(smem + a.off_cnt);
    float *hs = reinterpret_cast<float *>(smem + a.off_hs);
    float *ms = reinterpret_cast<float *>(smem + a.off_ms);
    int *args = reinterpret_cast<int *>(smem + a.off_args) + wave * 64;
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)a.row0) * a.d;
    const float sx = a.xmeta[0];

    if (a.resident) split_stage(frag, smem, npair * NC * 4);
    for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
    for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
    if (a.fused) {
        for (int e = tid; e < a.k * a.d; e += blockDim.x) cells[e] = 0;
        for (int c = tid; c < a.k; c += blockDim.x) cnt[c] = 0;
    }
    split_stage_wait();

    int rechecks = 0;
    const int span = nw * 64;
    for (int g0 = n_lo; g0 < n_hi; g0 += span) {
        const int g = g0 + wave * 64;
        const bool active = g < n_hi;
        if (a.resident && !active) break;
        half8 bh[2][NC], bl[2][NC];
        float n2[2] = {0.0f, 0.0f};
        if (active) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int n = g + 32 * m + l32;
                const float *row = xb + (size_t)(n < n_hi ? n : g) * a.d;
                float v[NC][8];
#pragma unroll
                for (int ch = 0; ch + 1 < NC; ++ch) split_load8<false>(v[ch], row, ch * 16 + 8 * half, a.d);
                split_load8<true>(v[NC - 1], row, (NC - 1) * 16 + 8 * half, a.d);
#pragma unroll
                for (int ch = 0; ch + 1 < NC; ++ch) {
                    split_convert<false>(v[ch], sx, ms, ch * 16 + 8 * half, a.d, bh[m][ch], bl[m][ch], n2[m]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                split_convert<true>(v[NC - 1], sx, ms, (NC - 1) * 16 + 8 * half, a.d, bh[m][NC - 1], bl[m][NC - 1], n2[m]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        SplitTop top[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            top[m].v1 = top[m].v2 = top[m].v3 = -INFINITY;
            top[m].i1 = top[m].i2 = 0;
        }
        const float big = split_opaque_infinity();
        if (!a.resident) {
            __syncthreads();                    // nobody still reads the first stage
            split_stage(frag, smem, NC * 4);
        }
        for (int rp = 0; rp < npair; ++rp) {
            const unsigned char *st = smem + (size_t)(a.resident ? rp : (rp & 1)) * NC * 4 * SPLIT_PIECE;
            if (!a.resident) {
                split_stage_wait();
                if (rp + 1 < npair)
                    split_stage(frag + (size_t)(rp + 1) * NC * 4 * SPLIT_PIECE, smem + ((rp + 1) & 1) * NC * 4 * SPLIT_PIECE, NC * 4);
                if (!active) continue;
            }
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                if (2 * rp + blk >= a.nblk) break;
                sfloatx16 acc[2];
                split_init_acc(acc[0], hs, 2 * rp + blk, half);
                acc[1] = acc[0];
                // the operands of the next chunk are read under the matrix work of this one; the scheduling barrier keeps
                // the compiler from hoisting the reads of all chunks (registers)
                const half8 *A = reinterpret_cast<const half8 *>(st + blk * 2 * SPLIT_PIECE) + lane;
                half8 ah = A[0], al = A[64];
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) {
                    half8 nh = ah, nl = al;
                    if (ch + 1 < NC) { nh = A[(ch + 1) * 256]; nl = A[(ch + 1) * 256 + 64]; }
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[0][ch], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[1][ch], acc[1], 0, 0, 0);
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[0][ch], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[1][ch], acc[1], 0, 0, 0);
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[0][ch], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[1][ch], acc[1], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    ah = nh; al = nl;
                }
                split_insert(top[0], acc[0], 2 * rp + blk, big);
                split_insert(top[1], acc[1], 2 * rp + blk, big);
            }
        }
        if (active) split_finish_group(a, top, n2, worker, g, n_hi, xb, half, args, cells, cnt, rechecks);
    }
    split_count_rechecks(a, worker, rechecks);
    if (a.fused) {
        __syncthreads();
        split_flush(a, worker, share, cells, cnt);
    }
}

}  // namespace asgd
