// Step kernel for any row length.  A step of a worker is an assignment of its mini-batch, for large states gradient sums in
// a pass of their own, at merge points Eq. 4, and an update; each is written as an item of work for one workgroup, and
// there are two forms of putting them together:
//   - local: all the steps of a call are ONE cooperative launch, a workgroup of eight waves per compute unit does all the
//     items of its workers, and workers wait for each other's messages only.  Chosen where the workers fill the device.
//   - phases: every phase of a step is a launch of its own over all workers, whose items are cut further (shares of the
//     mini-batch, columns, rows), so that a few workers fill the device too.
// (Tried between the two: one launch with barriers over the whole grid between the phases - 10 us a barrier, mostly the
// write-back and invalidation of the L2 by every workgroup; 35 us per step where phases take 22.)
#pragma once

#include "split_screen.h"

namespace asgd {

// Operands of a worker's state rows, as the matrix instructions want them: rows in pairs of 32-row blocks, columns in
// chunks of 16; [row pair][chunk][block of the pair][hi, lo] pieces of 1 KB, piece = 64 lanes x 8 fp16, lane l holding row
// l % 32, columns 8 * (l / 32) .. + 7 of the chunk.
constexpr int SPLIT_THREADS = 512;

struct SplitState {                // one per worker and step modulo 3
    float sw;                      // scale of the operands
    unsigned vabs, n2;             // bit patterns of the largest |v_cj| and of the largest |sw v_c|^2; above those of all numbers if not finite
    unsigned rest;                 // of the largest |sw v_c - its high parts|^2
    unsigned pad[28];              // a cache line each: atomics on one line wait for each other, and that took 15 us
};

struct SplitSize { float sw; unsigned vabs, n2; };

struct SplitStep {                         // what is the same for all workers in a step
    int slot, slot_next, slot_after;       // step modulo 3
    int merge, send, round;                // merge point, messages go out, round number
    int read_parity, send_parity, local;
    int batch;                             // which of a kept worker's two buffers holds the mini-batch
    const SplitState *state;               // W, of this step's slot
    int32_t *dump;                         // W x b of this step, or null
    long long row0, row0_next;             // first row of the mini-batch in a shard, and of the next one (-1: none)
    int shift[MAX_BUFFERS];                // deterministic schedule of the round
};

// The arguments stay in the kernel argument segment and are read again (scalar loads) by every item that needs them: kept
// in scalar registers across the phases they were 500 spills.
#define SPLIT_ARG const __attribute__((address_space(4)))

struct SplitArgs {
    const float *x, *w;              // samples, states
    const unsigned char *frag;       // W x frag_bytes
    const float *hs;                 // W x kpad: -|sw v_c|^2/2 * sx / sw, SPLIT_PAD_SCORE for the padding rows
    const float *ms;                 // dpad: -m_j * sx, zero past d
    const float *xmeta;              // sx
    const double *colscale;          // d scales of the fixed-point sums, then d inverse scales
    int *idx;                        // W x b assignments (null: not stored)
    float *part;                     // shares x W x k x d sums of a share's samples
    int *cntpart;                    // shares x W x k samples per centroid
    long long *counters;
    size_t frag_bytes;
    long long H;
    int k, d, b, W, kpad, nblk, dpad;
    int shares, share_len;           // share_len: samples of a share, a multiple of 64
    int sum_shares, sum_len, dc, ncol;       // sums in a phase of their own: shares, columns per item, groups of columns
    int resident, fused, vec4, wide;
    int stage_pairs, stages;         // screened samples
    int kept;                        // local form, one worker per workgroup: its operands, sums and counts stay in the LDS, and two mini-batches take turns there
    unsigned off_cells, off_cnt, off_hs, off_ms, off_args, off_batch, batch_bytes, off_list;
};

struct SplitShared {                       // start of the LDS: the step, and space of the gate and update phases
    SplitStep now;
    double red[8];
    int delta;
    unsigned most[3][8];
    int listed;                            // undecided samples in the list
    int hard;                              // samples that wait for a scan of all the rows, SPLIT_HARD of them at most in `hard_rows`
    int hard_rows[SPLIT_HARD];
    int unscreened;                        // items that this workgroup does not screen
    SplitSize size[3];                     // SplitState of a kept worker
};

// The LDS starts with what all phases share.
extern __shared__ __attribute__((aligned(16))) unsigned char split_lds[];
static_assert(sizeof(SplitShared) <= SPLIT_LDS_SHARED, "room at the start of the LDS");
__device__ __forceinline__ SplitShared &split_shared() { return *reinterpret_cast<SplitShared *>(split_lds); }

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

// Gradient sums of a wave's samples.  A lane keeps its columns (four, or two where rows are not 16-byte aligned) and their
// scales; a centroid's cells lie in the order (j mod 4, j / 4), or (j mod 2, j / 2), so that neighbouring lanes add to
// neighbouring cells (in the order of j the adds of a wave fell into a quarter, or half, of the banks).  The rows come
// from a cache; two sets of them take turns, one in flight while the other is added (with one set the pass was a chain of
// latencies: k = d = 100, W = 512: a quarter of the launch).
__device__ __forceinline__ int split_cell_stride(SPLIT_ARG SplitArgs &a) { return a.vec4 ? a.d : (a.d + 1) & ~1; }
__device__ __forceinline__ int split_cell(SPLIT_ARG SplitArgs &a, int j)
{
    return a.vec4 ? (j & 3) * (a.d >> 2) + (j >> 2) : (j & 1) * ((a.d + 1) >> 1) + (j >> 1);
}
// rows 0 .. nv-1 of xg, their centroids in args
__device__ __forceinline__ void split_accumulate(SPLIT_ARG SplitArgs &a, const float *xg, int nv, const int *args, u64 *cells, int *cnt)
{
    const int lane = split_lane(), d = a.d;
    if (lane < nv) atomicAdd(&cnt[args[lane]], 1);
    if (a.vec4) {
        const int q4 = d >> 2, R = 64 / q4, r = lane / q4, c = lane - r * q4;
        if (r < R) {
            constexpr int U = 4;
            double s[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = a.colscale[4 * c + e];
            const float4 *src = reinterpret_cast<const float4 *>(xg) + c;
            auto fetch = [&](float4 (&v)[U], int n0) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = src[(unsigned)(min(n0 + u * R, nv - 1) * q4)];
            };
            auto add = [&](const float4 (&v)[U], int n0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (n0 + u * R < nv) {
                        u64 *cell = cells + args[n0 + u * R] * d + c;
                        split_add(cell, split_term(v[u].x, s[0]));
                        split_add(cell + q4, split_term(v[u].y, s[1]));
                        split_add(cell + 2 * q4, split_term(v[u].z, s[2]));
                        split_add(cell + 3 * q4, split_term(v[u].w, s[3]));
                    }
                }
            };
            float4 va[U], vb[U];
            fetch(va, r);
            for (int n0 = r; n0 < nv; n0 += 2 * U * R) {
                fetch(vb, n0 + U * R);
                add(va, n0);
                fetch(va, n0 + 2 * U * R);
                add(vb, n0 + U * R);
            }
        }
    } else {
        // pairs of columns; the last lane of an odd row loads the pair before the end and uses its second half
        constexpr int U = 8;
        const int q2 = (d + 1) >> 1, R = 64 / q2, r = lane / q2, c = lane - r * q2;
        if (r < R) {
            const bool odd = 2 * c + 1 == d;                   // one column left
            const int c0 = odd ? max(d - 2, 0) : 2 * c, c1 = c0 + (d > 1 ? 1 : 0), stride = 2 * q2;
            const double s0 = a.colscale[2 * c], s1 = a.colscale[odd ? 2 * c : 2 * c + 1];
            auto fetch = [&](float (&v0)[U], float (&v1)[U], int n0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float *row = xg + (unsigned)(min(n0 + u * R, nv - 1) * d);
                    v0[u] = row[c0];
                    v1[u] = row[c1];
                }
            };
            auto add = [&](const float (&v0)[U], const float (&v1)[U], int n0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (n0 + u * R < nv) {
                        u64 *cell = cells + args[n0 + u * R] * stride + c;
                        split_add(cell, split_term(odd ? v1[u] : v0[u], s0));
                        if (!odd) split_add(cell + q2, split_term(v1[u], s1));
                    }
                }
            };
            float xa[U], ya[U], xb[U], yb[U];
            fetch(xa, ya, r);
            for (int n0 = r; n0 < nv; n0 += 2 * U * R) {
                fetch(xb, yb, n0 + U * R);
                add(xa, ya, n0);
                fetch(xa, ya, n0 + 2 * U * R);
                add(xb, yb, n0 + U * R);
            }
        }
    }
}

// Sums and counts of a workgroup's cells to the share's row of `part`.
__device__ inline void split_flush(SPLIT_ARG SplitArgs &a, int worker, int share, const u64 *cells, const int *cnt)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6, d = a.d;
    float *out = a.part + ((size_t)share * a.W + worker) * a.k * d;
    const int R = d < 64 ? 64 / d : 1, r = d < 64 ? lane / d : 0;
    if (r < R)
        for (int j = d < 64 ? lane - r * d : lane; j < d; j += 64) {
            const double inv = a.colscale[d + j];
            const int at = split_cell(a, j), stride = split_cell_stride(a);
            for (int c = wave * R + r; c < a.k; c += nw * R) out[c * d + j] = split_sum(cells[c * stride + at], cnt[c], inv);
        }
    int *oc = a.cntpart + ((size_t)share * a.W + worker) * a.k;
    for (int c = threadIdx.x; c < a.k; c += blockDim.x) oc[c] = cnt[c];
}

// A mini-batch of a kept worker on its way to the LDS.
__device__ __forceinline__ void split_batch_fetch(SPLIT_ARG SplitArgs &a, int worker, long long row0, unsigned char *dst)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6, total = a.b * a.d;
    const float *src = a.x + ((size_t)worker * a.H + (size_t)row0) * a.d;
    if (a.vec4) {
        for (int q = wave; q * 256 < total; q += nw)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + min(q * 256 + lane * 4, total - 4)),
                                             (__attribute__((address_space(3))) void *)(dst + q * 1024), 16, 0, 0);
    } else {
        for (int q = wave; q * 64 < total; q += nw)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + min(q * 64 + lane, total - 1)),
                                             (__attribute__((address_space(3))) void *)(dst + q * 256), 4, 0, 0);
    }
}

// Twice the error of a score of a sample with norm `yn`, infinite where everything is decided in fp64: a state that is not finite, has
// outgrown the scale of its fp16 operands or has shrunk so far below it that its squares lose their last places, scores
// that come near the offset of the padding rows.  rl: norm of the sample's low parts, where high parts alone were multiplied.
template <bool SCREEN>
__device__ __forceinline__ float split_threshold(SPLIT_ARG SplitArgs &a, const SplitSize &st, float rest, float yn, float rl)
{
    const float sw = st.sw, n2max = __uint_as_float(st.n2), vmax = sqrtf(n2max) * 1.0001f, ratio = a.xmeta[0] / sw;
    const float offset = 0.5f * vmax * vmax * ratio;
    float thr;
    if (SCREEN) thr = screen_bound(yn, rl, vmax, sqrtf(rest) * 1.0001f, offset, a.dpad);
    else thr = split_c1(a.dpad) * (yn * vmax + offset) + split_c2(a.dpad) * (yn + vmax);
    if (st.n2 >= 0x7f800000u || st.vabs >= 0x7f800000u || !(__uint_as_float(st.vabs) * sw < 32768.0f) || !(n2max > 1.0e-27f) ||
        !(yn * vmax + offset < -0.1f * SPLIT_PAD_SCORE))
        thr = INFINITY;
    return thr;
}

// What a wave does once the best scores of its 64 samples are known (lane l: sample l), the same in both assignment items.
template <bool KEPT>
__device__ __forceinline__ void split_finish_group(SPLIT_ARG SplitArgs &a, const SplitStep &now, const SplitTop &t, float n2, int worker, int g,
                                                   int n_hi, const float *xb, int *args, u64 *cells, int *cnt, int &rechecks)
{
    const int lane = split_lane();
    const float yn = sqrtf(n2) * 1.0001f;
    SplitSize st;
    if constexpr (KEPT) st = split_shared().size[now.slot];
    else st = SplitSize{now.state[worker].sw, now.state[worker].vabs, now.state[worker].n2};
    const float thr = split_threshold<false>(a, st, 0.0f, yn, 0.0f);
    const float *xg = xb + (size_t)g * a.d;
    const bool valid = g + lane < n_hi;
    const int arg = split_settle<false>(t, thr, valid, xg, lane, a.w + (size_t)worker * a.k * a.d, a.k, a.d, rechecks);
    if (valid) {
        if (a.idx) a.idx[(size_t)worker * a.b + g + lane] = arg;
        if (now.dump) now.dump[(size_t)worker * a.b + g + lane] = arg;
    }
    if (a.fused) {
        args[lane] = valid ? arg : 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (KEPT)
            split_accumulate(a, reinterpret_cast<const float *>(split_lds + SPLIT_LDS_SHARED + a.off_batch + now.batch * a.batch_bytes) + g * a.d,
                             min(64, n_hi - g), args, cells, cnt);
        else
            split_accumulate(a, xg, min(64, n_hi - g), args, cells, cnt);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

__device__ __forceinline__ void split_count_rechecks(SPLIT_ARG SplitArgs &a, int worker, int rechecks)
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
// `first`: samples of the share that are decided already.
template <int NC, bool KEPT>
__device__ void split_assign_item(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, unsigned char *smem, int first = 0)
{
    const int n_lo = share * a.share_len + first, n_hi = min(a.b, share * a.share_len + a.share_len);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, npair = (a.nblk + 1) / 2;
    u64 *cells = reinterpret_cast<u64 *>(smem + a.off_cells);
    int *cnt = reinterpret_cast<int *>(smem + a.off_cnt);
    float *hs = reinterpret_cast<float *>(smem + a.off_hs);
    float *ms = reinterpret_cast<float *>(smem + a.off_ms);
    int *args = reinterpret_cast<int *>(smem + a.off_args) + wave * 64;
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0) * a.d;
    const float sx = a.xmeta[0];
    const float *batch = reinterpret_cast<const float *>(smem + a.off_batch + now.batch * a.batch_bytes);

    // (this wave's rows of the new state, for the exact decisions, and its part of the mini-batch)
    if constexpr (KEPT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                            // (the item before this one is done with the LDS)
    if constexpr (KEPT) {
        if (now.row0_next >= 0) split_batch_fetch(a, worker, now.row0_next, smem + a.off_batch + (now.batch ^ 1) * a.batch_bytes);
    }
    if constexpr (!KEPT) {
        if (a.resident) split_stage(frag, smem, npair * NC * 4);
        for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
        for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
        if (a.fused) {
            for (int e = tid; e < a.k * split_cell_stride(a); e += blockDim.x) cells[e] = 0;
            for (int c = tid; c < a.k; c += blockDim.x) cnt[c] = 0;
        }
        split_stage_wait();
    }
    const bool resident = KEPT || a.resident;

    int rechecks = 0;
    const int span = nw * 64;
    for (int g0 = n_lo; g0 < n_hi; g0 += span) {
        const int g = g0 + wave * 64;
        const bool active = g < n_hi;
        if (resident && !active) break;
        half8 bh[2][NC], bl[2][NC];
        float n2[2] = {0.0f, 0.0f};
        // (Fetching a group's columns while the group before it is finished changed nothing where there are registers for
        // it, and spilled where rows are long; a wave's neighbour on the SIMD works meanwhile.)
        if (active) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                float v[NC][8];
                const int n = g + 32 * m + l32;
                if (KEPT) {
                    const float *row = batch + (n < n_hi ? n : n_lo) * a.d;
                    if (a.vec4 && a.d >= 8) {
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) {
                            const int slot = ch * 16 + 8 * half;
                            const float *q = row + (ch + 1 < NC ? slot : min(slot, a.d - 8));
                            const float4 p0 = *reinterpret_cast<const float4 *>(q), p1 = *reinterpret_cast<const float4 *>(q + 4);
                            v[ch][0] = p0.x; v[ch][1] = p0.y; v[ch][2] = p0.z; v[ch][3] = p0.w;
                            v[ch][4] = p1.x; v[ch][5] = p1.y; v[ch][6] = p1.z; v[ch][7] = p1.w;
                        }
                    } else {
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch)
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                v[ch][e] = row[min(split_column(ch * 16 + 8 * half < a.d ? ch * 16 + 8 * half + e : e, a.d), a.d - 1)];
                    }
                } else {
                    const float *row = xb + (size_t)(n < n_hi ? n : n_lo) * a.d;
#pragma unroll
                    for (int ch = 0; ch + 1 < NC; ++ch) split_load8<false>(v[ch], row, ch * 16 + 8 * half, a.d);
                    split_load8<true>(v[NC - 1], row, (NC - 1) * 16 + 8 * half, a.d);
                }
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
        if (!resident) {
            __syncthreads();                    // nobody still reads the first stage
            split_stage(frag, smem, NC * 4);
        }
        for (int rp = 0; rp < npair; ++rp) {
            const unsigned char *st = smem + (size_t)(resident ? rp : (rp & 1)) * NC * 4 * SPLIT_PIECE;
            if (!resident) {
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
        if (active) {
            SplitTop t;
            split_combine(top, t, half);
            swap2(n2[0], n2[1]);
            split_finish_group<KEPT>(a, now, t, n2[0] + n2[1], worker, g, n_hi, xb, args, cells, cnt, rechecks);
        }
    }
    split_count_rechecks(a, worker, rechecks);
    // (one launch: Eq. 4 and the update of this worker come next and take the sums from the cells)
    if (!KEPT && a.fused && !now.local) {
        __syncthreads();
        split_flush(a, worker, share, cells, cnt);
    }
}

// The samples in the workgroup's list of hard ones, by all its waves: a wave takes a part of the rows.  (One wave for all of them: 45 us
// for one sample of k = 1024, d = 128, which the others waited for.)  `results`: SPLIT_HARD x waves x 16 bytes of LDS; the
// caller's barriers are before and after.
struct SplitHard { double best; int arg, pad; };
__device__ inline void split_scan_hard(SPLIT_ARG SplitArgs &a, const float *xb, const float *w, int *idx, int32_t *dump, SplitHard *results)
{
    const int lane = split_lane(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int count = min(__builtin_amdgcn_readfirstlane(split_shared().hard), SPLIT_HARD);
    const int part = ((a.k + nw - 1) / nw + 15) & ~15, c_lo = min(wave * part, a.k), c_hi = min(c_lo + part, a.k);
    for (int q = 0; q < count; ++q) {
        double best = INFINITY;
        int arg = 0;
        if (c_lo < c_hi) split_scan_wave(xb + (size_t)split_shared().hard_rows[q] * a.d, w, c_lo, c_hi, a.d, best, arg);
        if (lane == 0) results[q * nw + wave] = SplitHard{best, arg, 0};
    }
    __syncthreads();
    if ((int)threadIdx.x < count) {
        const int row = split_shared().hard_rows[threadIdx.x];
        double best = INFINITY;
        int arg = 0;                          // (no distance below infinity: centroid 0, like a scan that starts there)
        for (int v = 0; v < nw; ++v) {
            const SplitHard r = results[threadIdx.x * nw + v];
            if (r.best < best) { best = r.best; arg = r.arg; }
        }
        idx[row] = arg;
        if (dump) dump[row] = arg;
    }
    if (threadIdx.x == 0) split_shared().hard = 0;
}

// ---- screened assignment: rows of 17 to 128 columns, a state that is streamed, sums in a pass of their own ----
// High parts alone, up to four tiles of 32 samples per wave, the state's high parts through LDS stages; samples that are not decided by that go
// to a list and are scored with all three products.  The decisions are those of the other items.  A workgroup that finds too many of its samples
// open (split_screen_gives_up()) goes on with the item without screening, and begins the next SPLIT_UNSCREENED mini-batches with it.
// k = 1024, d = 128, b = 4096, W = 256, microseconds per step: 1130 with three products for all, 780 now: loading and converting the samples and
// the stages 230, matrix instructions and insertions 130, the 3 % that are listed 95, sums 175, update 125.

// The listed samples: 128 at a time, their operands in the LDS (where the stages were), every wave its own blocks of the state's rows with both
// parts straight from the L2, a block ahead.
template <int NC>
__device__ __forceinline__ void split_listed(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, unsigned char *smem)
{
    const SplitState *state = now.state;
    int32_t *dump = now.dump;
    const int n_lo = share * a.share_len;
    const int lane = split_lane(), half = lane >> 5, l32 = lane & 31, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = blockDim.x >> 6, d = a.d, nblk = a.nblk;
    constexpr int HC = (NC + 1) / 2, TILES = SPLIT_LISTED / 32;
    const float *hs = reinterpret_cast<const float *>(smem + a.off_hs), *ms = reinterpret_cast<const float *>(smem + a.off_ms);
    float *norms = reinterpret_cast<float *>(smem + a.off_args);          // [tile][half of the chunks][64]
    float *tops = reinterpret_cast<float *>(smem);                        // [wave][pair of tiles][5][64], once the operands are used
    half8 *operands = reinterpret_cast<half8 *>(smem);                    // [tile][chunk][hi, lo] pieces
    const int *list = reinterpret_cast<const int *>(smem + a.off_list);
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0 + n_lo) * d;
    const float sx = a.xmeta[0];
    const SplitSize st = {state[worker].sw, state[worker].vabs, state[worker].n2};
    const int listed = __builtin_amdgcn_readfirstlane(split_shared().listed);
    int rechecks = 0;
    for (int p0 = 0; p0 < listed; p0 += SPLIT_LISTED) {
        const int here = min(SPLIT_LISTED, listed - p0);
        for (int un = wave; un < 2 * TILES; un += nw) {
            const int tile = un >> 1, hh = un & 1;
            const float *row = xb + (size_t)list[p0 + min(32 * tile + l32, here - 1)] * d;
            float v[HC][8], n2 = 0.0f;
#pragma unroll
            for (int q = 0; q < HC; ++q) {
                const int slot = (hh * HC + q) * 16 + 8 * half;
                split_load8<false>(v[q], row, min(slot, d - 8), d);
            }
#pragma unroll
            for (int q = 0; q < HC; ++q) {
                const int ch = hh * HC + q;
                if (ch >= NC) continue;
                half8 hi, lo;
                split_convert<true>(v[q], sx, ms, ch * 16 + 8 * half, d, hi, lo, n2);
                half8 *to = operands + (tile * NC + ch) * 128 + lane;
                to[0] = hi;
                to[64] = lo;
            }
            norms[un * 64 + lane] = n2;
        }
        SplitTop top[TILES];
        const float big = split_opaque_infinity();
#pragma unroll
        for (int m = 0; m < TILES; ++m) {
            top[m].v1 = top[m].v2 = top[m].v3 = -INFINITY;
            top[m].i1 = top[m].i2 = 0;
        }
        half8 A[2][2 * NC];
        auto fetch = [&](half8 (&to)[2 * NC], int blk) {
            const half8 *src = reinterpret_cast<const half8 *>(frag + ((size_t)(blk >> 1) * NC * 4 + (blk & 1) * 2) * SPLIT_PIECE) + lane;
#pragma unroll
            for (int ch = 0; ch < NC; ++ch) { to[2 * ch] = src[ch * 256]; to[2 * ch + 1] = src[ch * 256 + 64]; }
        };
        auto multiply = [&](const half8 (&from)[2 * NC], int blk) {
#pragma unroll
            for (int m = 0; m < TILES; ++m) {
                if (32 * m >= here) break;
                const half8 *B = reinterpret_cast<const half8 *>(smem) + m * NC * 128 + lane;
                sfloatx16 acc;
                split_init_acc(acc, hs, blk, half);
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) {
                    const half8 bh = B[ch * 128], bl = B[ch * 128 + 64];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(from[2 * ch], bl, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(from[2 * ch + 1], bh, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(from[2 * ch], bh, acc, 0, 0, 0);
                    if (ch % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
                split_insert(top[m], acc, blk, big);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (wave < nblk) fetch(A[0], wave);
        __syncthreads();                          // (the operands are there)
        for (int blk = wave; blk < nblk; blk += 2 * nw) {
            if (blk + nw < nblk) fetch(A[1], blk + nw);
            multiply(A[0], blk);
            if (blk + nw < nblk) {
                if (blk + 2 * nw < nblk) fetch(A[0], blk + 2 * nw);
                multiply(A[1], blk + nw);
            }
        }
        __syncthreads();                          // (and used)
#pragma unroll
        for (int p = 0; p < TILES / 2; ++p) {
            SplitTop t, pair[2] = {top[2 * p], top[2 * p + 1]};
            split_combine(pair, t, half);
            float *mine = tops + (wave * (TILES / 2) + p) * 5 * 64 + lane;
            mine[0] = t.v1; mine[64] = t.v2; mine[128] = t.v3;
            mine[192] = __int_as_float(t.i1); mine[256] = __int_as_float(t.i2);
        }
        __syncthreads();
        // every wave settles its share of the samples
        const int each = SPLIT_LISTED / nw;
        for (int s0 = 0; s0 < each; s0 += 64) {
            const int s = min(wave * each + s0 + lane, SPLIT_LISTED - 1);
            const bool valid = s0 + lane < each && wave * each + s0 + lane < here;
            SplitTop t = {-INFINITY, -INFINITY, -INFINITY, 0, 0};
            for (int q = 0; q < nw; ++q) {
                const float *o = tops + (q * (TILES / 2) + (s >> 6)) * 5 * 64 + (s & 63);
                split_merge(t, o[0], __float_as_int(o[192]));
                split_merge(t, o[64], __float_as_int(o[256]));
                t.v3 = fmaxf(t.v3, o[128]);
            }
            const float *nr = norms + (s >> 5) * 128 + (s & 31);
            const float thr = split_threshold<false>(a, st, 0.0f, sqrtf((nr[0] + nr[32]) + (nr[64] + nr[96])) * 1.0001f, 0.0f);
            const int own = list[p0 + min(s, here - 1)];
            const int arg = split_settle<true>(t, thr, valid, xb, own, a.w + (size_t)worker * a.k * d, a.k, d, rechecks, split_shared().hard_rows,
                                               &split_shared().hard);
            if (valid && arg >= 0) {
                a.idx[(size_t)worker * a.b + n_lo + own] = arg;
                if (dump) dump[(size_t)worker * a.b + n_lo + own] = arg;
            }
        }
        __syncthreads();                          // (tops are used, the list of hard ones is complete)
        if (split_shared().hard > 0)
            split_scan_hard(a, xb, a.w + (size_t)worker * a.k * d, a.idx + (size_t)worker * a.b + n_lo, dump ? dump + (size_t)worker * a.b + n_lo : nullptr,
                            reinterpret_cast<SplitHard *>(smem));
        __syncthreads();                          // (operands and norms are written again)
    }
    split_count_rechecks(a, worker, rechecks);
    if (threadIdx.x == 0) split_shared().listed = 0;
    __syncthreads();
}

// Returns the first sample of the share that is left to the item without screening, -1 if all are decided.
template <int NC>
__device__ int split_screen_item(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, unsigned char *smem)
{
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len), n = n_hi - n_lo;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, npair = (a.nblk + 1) / 2, nstage = a.stages;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs), *ms = reinterpret_cast<float *>(smem + a.off_ms);
    int *list = reinterpret_cast<int *>(smem + a.off_list);
    const unsigned stage_bytes = (unsigned)a.stage_pairs * NC * 2 * SPLIT_PIECE;
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0 + n_lo) * a.d;
    const float sx = a.xmeta[0];
    // the high parts of a stage: every other piece
    auto stage_fetch = [&](int st, int buf) {
        const unsigned char *src = frag + (size_t)st * 2 * stage_bytes + lane * 16;
        unsigned char *dst = smem + buf * stage_bytes;
        const int pieces = min(a.stage_pairs, npair - st * a.stage_pairs) * NC * 2;
        for (int q = wave; q < pieces; q += nw)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (size_t)q * 2 * SPLIT_PIECE),
                                             (__attribute__((address_space(3))) void *)(dst + q * SPLIT_PIECE), 16, 0, 0);
    };
    __syncthreads();                            // (the item before this one is done with the LDS)
    stage_fetch(0, 0);
    for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
    for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
    if (tid == 0) split_shared().listed = split_shared().hard = 0;
    __syncthreads();

    int turn = 0, done = 0;                     // done: samples before it are decided, none of them is in the list
    bool staged = false;
    // one sweep over this wave's 32 * T samples from g on (of the share)
    auto sweep = [&](auto tiles, int g, bool last) {
        constexpr int T = decltype(tiles)::value, HC = (NC + 1) / 2;
        half8 b[T][NC];
        float n2[T], r2[T];
        ScreenTop top[T];
        {
            float v[3][HC][8];
            // half tiles, two on their way while one is converted
            auto load = [&](float (&to)[HC][8], int u) {
                const float *row = xb + (unsigned)(min(g + 32 * (u >> 1) + l32, n - 1) * a.d);
#pragma unroll
                for (int q = 0; q < HC; ++q) {
                    const int ch = (u & 1) * HC + q;
                    if (ch < NC) split_load8<false>(to[q], row, ch + 1 < NC ? ch * 16 + 8 * half : min(ch * 16 + 8 * half, a.d - 8), a.d);
                }
            };
            load(v[0], 0);
            load(v[1], 1);
#pragma unroll
            for (int u = 0; u < 2 * T; ++u) {
                const int t = u >> 1;
                if (u + 2 < 2 * T) load(v[(u + 2) % 3], u + 2);
                if ((u & 1) == 0) n2[t] = r2[t] = 0.0f;
                const int hf = split_lane() >> 5;             // (ms is read again for every tile, not kept in 64 registers)
#pragma unroll
                for (int q = 0; q < HC; ++q) {
                    const int ch = (u & 1) * HC + q;
                    if (ch + 1 < NC) screen_convert<false>(v[u % 3][q], sx, ms, ch * 16 + 8 * hf, a.d, b[t][ch], n2[t], r2[t]);
                    else if (ch + 1 == NC) screen_convert<true>(v[u % 3][q], sx, ms, ch * 16 + 8 * hf, a.d, b[t][ch], n2[t], r2[t]);
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
            if (nstage > 1 || !staged) split_stage_wait();    // this stage is there, and nobody reads the other one any more
            staged = true;
            if (nstage > 1 && !(last && st + 1 == nstage)) stage_fetch(st + 1 < nstage ? st + 1 : 0, (turn + 1) & 1);
            const unsigned char *from = smem + (turn & 1) * stage_bytes;
            turn += nstage > 1;
            const int blk0 = st * a.stage_pairs * 2, blks = g < n ? min(a.stage_pairs * 2, a.nblk - blk0) : 0;
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
        if (g < n) {
            const SplitSize st = {now.state[worker].sw, now.state[worker].vabs, now.state[worker].n2};
            const float rest = __uint_as_float(now.state[worker].rest);
#pragma unroll
            for (int p = 0; p < T / 2; ++p) {
                ScreenTop t;
                screen_combine(top[2 * p], top[2 * p + 1], t, half);
                swap2(n2[2 * p], n2[2 * p + 1]);
                swap2(r2[2 * p], r2[2 * p + 1]);
                const float thr = split_threshold<true>(a, st, rest, sqrtf(n2[2 * p] + n2[2 * p + 1]) * 1.0001f, sqrtf(r2[2 * p] + r2[2 * p + 1]) * 1.0001f);
                const int at = g + 64 * p + lane;
                const bool valid = at < n, open = valid && !(t.v1 - t.v2 > thr);
                const unsigned long long o = __ballot(open);
                int base = 0;
                if (o != 0 && lane == 0) base = atomicAdd(&split_shared().listed, __popcll(o));
                base = __builtin_amdgcn_readfirstlane(base);
                if (open) list[base + __popcll(o & ((1ULL << lane) - 1))] = at;
                if (valid && !open) {
                    const int arg = min(max(t.i1, 0), a.k - 1);
                    a.idx[(size_t)worker * a.b + n_lo + at] = arg;
                    if (now.dump) now.dump[(size_t)worker * a.b + n_lo + at] = arg;
                }
            }
        }
    };
    for (int g0 = 0; g0 < n;) {
        const bool four = n - g0 > nw * 64;
        const int next = g0 + nw * (four ? 128 : 64);
        if (four) sweep(std::integral_constant<int, 4>{}, g0 + wave * 128, next >= n);
        else sweep(std::integral_constant<int, 2>{}, g0 + wave * 64, next >= n);
        g0 = next;
        __syncthreads();
        const int listed = __builtin_amdgcn_readfirstlane(split_shared().listed);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // (the stage that is on its way: the listed samples take its place)
        __syncthreads();                          // (everybody has read the number before anybody adds to it)
        if (split_screen_gives_up(listed, min(g0, n) - done, NC)) return done;
        if (listed > 0 && (g0 >= n || listed > SPLIT_LIST - nw * 128)) {
            split_listed<NC>(a, now, worker, share, smem);
            if (g0 < n) stage_fetch(0, turn & 1);
            staged = false;
            done = g0;
        }
    }
    return -1;
}

// ---- assignment for rows of more than 128 columns ----
// The operands of the samples do not fit the registers: for every pair of row blocks the samples' columns are read
// again (from a cache) and split again.  The waves of a workgroup share out the row pairs of a group of 64 samples (as far
// as there are any), so that few samples still make many waves, and read the state's operands straight from the L2 into
// registers, two chunks ahead: no stage, no barrier inside (staged in LDS with a wave per group of samples, k = 256,
// d = 384, 64 workers: 135 us per launch, most of it waiting at the barriers of the stage).
__device__ __forceinline__ int split_long_rows(int npair, int waves)       // waves that share a group's row pairs
{
    int r = 1;
    while (2 * r <= npair && 2 * r <= waves) r *= 2;
    return r;
}
__device__ inline void split_assign_long_item(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, unsigned char *smem)
{
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, npair = (a.nblk + 1) / 2, nch = a.dpad / 16;
    const int rsplit = split_long_rows(npair, nw), rw = wave % rsplit, gw = wave / rsplit, ng = nw / rsplit;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs);
    float *ms = reinterpret_cast<float *>(smem + a.off_ms);
    float *tops = reinterpret_cast<float *>(smem + a.off_args);          // [wave][5][64]
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0) * a.d;
    const float sx = a.xmeta[0];
    __syncthreads();
    for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
    for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
    __syncthreads();

    int rechecks = 0;
    for (int g0 = n_lo; g0 < n_hi; g0 += ng * 64) {
        const int g = g0 + gw * 64;
        const bool active = g < n_hi;
        const float *row[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int n = g + 32 * m + l32;
            row[m] = xb + (size_t)(n < n_hi ? n : n_lo) * a.d;
        }
        float n2[2] = {0.0f, 0.0f};
        SplitTop top[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            top[m].v1 = top[m].v2 = top[m].v3 = -INFINITY;
            top[m].i1 = top[m].i2 = 0;
        }
        const float big = split_opaque_infinity();
        for (int rp = rw; active && rp < npair; rp += rsplit) {
            sfloatx16 acc[2][2];                  // [block of the pair][tile of samples]
            split_init_acc(acc[0][0], hs, 2 * rp, half);
            acc[0][1] = acc[0][0];
            split_init_acc(acc[1][0], hs, 2 * rp + 1, half);
            acc[1][1] = acc[1][0];
            const half8 *A = reinterpret_cast<const half8 *>(frag + (size_t)rp * nch * 4 * SPLIT_PIECE) + lane;
            // two chunks per set: operands of the state, columns of the samples
            auto fetch = [&](half8 (&av)[2][4], float (&v)[2][2][8], int ch) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = min(ch + u, nch - 1);
#pragma unroll
                    for (int q = 0; q < 4; ++q) av[u][q] = A[c * 256 + q * 64];
#pragma unroll
                    for (int m = 0; m < 2; ++m) split_load8<true>(v[u][m], row[m], min(c * 16 + 8 * half, (a.d - 1) & ~7), a.d);
                }
            };
            auto multiply = [&](const half8 (&av)[2][4], const float (&v)[2][2][8], int ch) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    half8 bh[2], bl[2];
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        float q = 0.0f;
                        split_convert<true>(v[u][m], sx, ms, (ch + u) * 16 + 8 * half, a.d, bh[m], bl[m], q);
                        n2[m] += rp == rw ? q : 0.0f;
                    }
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][2 * blk], bl[m], acc[blk][m], 0, 0, 0);
                            acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][2 * blk + 1], bh[m], acc[blk][m], 0, 0, 0);
                            acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][2 * blk], bh[m], acc[blk][m], 0, 0, 0);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            half8 a0[2][4], a1[2][4];
            float v0[2][2][8], v1[2][2][8];
            fetch(a0, v0, 0);
            for (int ch = 0; ch < nch; ch += 4) {          // (nch is a multiple of eight)
                fetch(a1, v1, ch + 2);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a0, v0, ch);
                fetch(a0, v0, ch + 4);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a1, v1, ch + 2);
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                split_insert(top[m], acc[0][m], 2 * rp, big);
                split_insert(top[m], acc[1][m], 2 * rp + 1, big);
            }
        }
        SplitTop t;
        split_combine(top, t, half);
        float *mine = tops + wave * 5 * 64 + lane;
        if (rw != 0) {
            mine[0] = t.v1; mine[64] = t.v2; mine[128] = t.v3;
            mine[192] = __int_as_float(t.i1); mine[256] = __int_as_float(t.i2);
        }
        __syncthreads();
        if (rw == 0 && active) {
            for (int q = 1; q < rsplit; ++q) {
                const float *o = mine + q * 5 * 64;
                split_merge(t, o[0], __float_as_int(o[192]));
                split_merge(t, o[64], __float_as_int(o[256]));
                t.v3 = fmaxf(t.v3, o[128]);
            }
            swap2(n2[0], n2[1]);
            split_finish_group<false>(a, now, t, n2[0] + n2[1], worker, g, n_hi, xb, nullptr, nullptr, nullptr, rechecks);
        }
        __syncthreads();                          // (tops are written again)
    }
    split_count_rechecks(a, worker, rechecks);
}

// Rows whose operands fit the LDS for 64 samples (up to some 500 columns): they are split once, by all the waves, and every wave multiplies them
// with its own blocks of the state's rows, whose operands come straight from the L2, two chunks ahead.  No barrier inside.  The next 64
// samples are on their way meanwhile.
// (k = 256, d = 384, b = 512, W = 64: 110 us per launch where every wave split its samples for itself and one wave decided for 64; 45 now.)
__device__ inline void split_assign_wide_item(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, unsigned char *smem)
{
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, nch = a.dpad / 16, d = a.d;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs), *ms = reinterpret_cast<float *>(smem + a.off_ms);
    float *tops = reinterpret_cast<float *>(smem + a.off_args), *norms = tops + 8 * 5 * 64;          // [wave][5][64], [wave][tile][64]
    half8 *operands = reinterpret_cast<half8 *>(smem);                    // [tile][chunk][hi, lo] pieces
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0) * d;
    const float sx = a.xmeta[0];
    __syncthreads();
    for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
    for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
    if (tid == 0) split_shared().hard = 0;
    // the columns of a wave's chunks wave, wave + nw, .. of 32 samples of each tile, up to LOADS chunks ahead in registers
    constexpr int LOADS = 4;
    float v[LOADS][2][8];
    auto load = [&](int g, int q, float (&to)[2][8]) {
        const int ch = wave + q * nw;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int n = g + 32 * m + l32;
            split_load8<false>(to[m], xb + (size_t)(n < n_hi ? n : n_lo) * d, min(min(ch, nch - 1) * 16 + 8 * half, d - 8), d);
        }
    };
#pragma unroll
    for (int q = 0; q < LOADS; ++q) load(n_lo, q, v[q]);
    __syncthreads();

    int rechecks = 0;
    for (int g = n_lo; g < n_hi; g += 64) {
        float n2[2] = {0.0f, 0.0f};
        auto put = [&](int q, const float (&from)[2][8]) {
            const int ch = wave + q * nw;
            if (ch >= nch) return;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                half8 hi, lo;
                split_convert<true>(from[m], sx, ms, ch * 16 + 8 * half, d, hi, lo, n2[m]);
                half8 *to = operands + (m * nch + ch) * 128 + lane;
                to[0] = hi;
                to[64] = lo;
            }
        };
#pragma unroll
        for (int q = 0; q < LOADS; ++q) put(q, v[q]);
        for (int q = LOADS; wave + q * nw < nch; ++q) {
            float w8[2][8];
            load(g, q, w8);
            put(q, w8);
        }
        norms[(wave * 2 + 0) * 64 + lane] = n2[0];
        norms[(wave * 2 + 1) * 64 + lane] = n2[1];
        __syncthreads();                          // (the operands are there)
        if (g + 64 < n_hi) {
#pragma unroll
            for (int q = 0; q < LOADS; ++q) load(g + 64, q, v[q]);
        }
        SplitTop top[2];
        const float big = split_opaque_infinity();
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            top[m].v1 = top[m].v2 = top[m].v3 = -INFINITY;
            top[m].i1 = top[m].i2 = 0;
        }
        for (int blk = wave; blk < a.nblk; blk += nw) {
            const half8 *A = reinterpret_cast<const half8 *>(frag + ((size_t)(blk >> 1) * nch * 4 + (blk & 1) * 2) * SPLIT_PIECE) + lane;
            const half8 *B = operands + lane;
            sfloatx16 acc[2];
            split_init_acc(acc[0], hs, blk, half);
            acc[1] = acc[0];
            half8 a0[2][2], a1[2][2];             // two chunks per set: high and low parts
            auto fetch = [&](half8 (&av)[2][2], int ch) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = min(ch + u, nch - 1);
                    av[u][0] = A[c * 256];
                    av[u][1] = A[c * 256 + 64];
                }
            };
            auto multiply = [&](const half8 (&av)[2][2], int ch) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const half8 bh = B[(m * nch + ch + u) * 128], bl = B[(m * nch + ch + u) * 128 + 64];
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][0], bl, acc[m], 0, 0, 0);
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][1], bh, acc[m], 0, 0, 0);
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][0], bh, acc[m], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            half8 a2[2][2], a3[2][2];
            fetch(a0, 0);
            fetch(a1, 2);
            fetch(a2, 4);
            for (int ch = 0; ch < nch; ch += 8) {          // (nch is a multiple of eight)
                fetch(a3, ch + 6);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a0, ch);
                fetch(a0, ch + 8);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a1, ch + 2);
                fetch(a1, ch + 10);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a2, ch + 4);
                fetch(a2, ch + 12);
                __builtin_amdgcn_sched_barrier(0);
                multiply(a3, ch + 6);
            }
            split_insert(top[0], acc[0], blk, big);
            split_insert(top[1], acc[1], blk, big);
        }
        SplitTop t;
        split_combine(top, t, half);
        float *mine = tops + wave * 5 * 64 + lane;
        mine[0] = t.v1; mine[64] = t.v2; mine[128] = t.v3;
        mine[192] = __int_as_float(t.i1); mine[256] = __int_as_float(t.i2);
        __syncthreads();
        // every wave settles its share of the samples
        {
            const int each = 64 / nw, s = min(wave * each + lane, 63), n = min(g + s, n_hi - 1);
            const bool valid = lane < each && g + s < n_hi;
            float n2s = 0.0f;
            t = SplitTop{-INFINITY, -INFINITY, -INFINITY, 0, 0};
            for (int q = 0; q < nw; ++q) {
                const float *o = tops + q * 5 * 64 + s;
                split_merge(t, o[0], __float_as_int(o[192]));
                split_merge(t, o[64], __float_as_int(o[256]));
                t.v3 = fmaxf(t.v3, o[128]);
                const float *nr = norms + (q * 2 + (s >> 5)) * 64 + (s & 31);
                n2s += nr[0] + nr[32];
            }
            const SplitSize st = {now.state[worker].sw, now.state[worker].vabs, now.state[worker].n2};
            const float thr = split_threshold<false>(a, st, 0.0f, sqrtf(n2s) * 1.0001f, 0.0f);
            const int arg = split_settle<true>(t, thr, valid, xb, n, a.w + (size_t)worker * a.k * d, a.k, d, rechecks, split_shared().hard_rows,
                                               &split_shared().hard);
            if (valid && arg >= 0) {
                a.idx[(size_t)worker * a.b + n] = arg;
                if (now.dump) now.dump[(size_t)worker * a.b + n] = arg;
            }
        }
        __syncthreads();                          // (tops are used, the list of hard ones is complete)
        if (split_shared().hard > 0) {
            split_scan_hard(a, xb, a.w + (size_t)worker * a.k * d, a.idx + (size_t)worker * a.b, now.dump ? now.dump + (size_t)worker * a.b : nullptr,
                            reinterpret_cast<SplitHard *>(tops));
            __syncthreads();
        }
    }
    split_count_rechecks(a, worker, rechecks);
}

// ---- gradient sums of a (worker, share, group of dc columns) where the cells of a whole state do not fit LDS ----
// 64-bit fixed-point cells as in the fused form, a centroid's row padded by one so that rows start in different banks.
// Aligned rows: four columns per lane, four rows per lane in flight (one column per lane took 356 us for 256 workers of
// 4096 x 128 samples and 1024 centroids, most of it issuing loads).
__device__ inline void split_sums_item(SPLIT_ARG SplitArgs &a, const SplitStep &now, int worker, int share, int chunk, unsigned char *smem)
{
    const int dc = a.dc, stride = dc + 1, k = a.k, d = a.d, tid = threadIdx.x;
    u64 *cells = reinterpret_cast<u64 *>(smem);
    int *cnt = reinterpret_cast<int *>(smem + (size_t)k * stride * sizeof(u64));
    const int n_lo = share * a.sum_len, n_hi = min(a.b, n_lo + a.sum_len);
    __syncthreads();
    for (int e = tid; e < k * stride; e += blockDim.x) cells[e] = 0;
    for (int c = tid; c < k; c += blockDim.x) cnt[c] = 0;
    __syncthreads();
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)now.row0) * d;
    const int *idx = a.idx + (size_t)worker * a.b;
    if (a.vec4 && dc % 4 == 0) {
        constexpr int U = 4;
        const int L = dc / 4, col = tid % L, j = chunk * dc + 4 * col, R = blockDim.x / L, r = tid / L;
        const bool ok = j < d;                           // (d is a multiple of four)
        double s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = a.colscale[ok ? j + e : 0];
        const float *xc = xb + (ok ? j : 0);
        float4 va[U], vb[U];
        int ca[U], cb[U];
        auto fetch = [&](float4 (&v)[U], int (&c)[U], int n0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int n = min(n0 + u * R, n_hi - 1);
                c[u] = idx[n];
                v[u] = *reinterpret_cast<const float4 *>(xc + (size_t)n * d);
            }
        };
        auto add = [&](const float4 (&v)[U], const int (&c)[U], int n0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (n0 + u * R >= n_hi) continue;
                u64 *cell = cells + c[u] * stride + col;
                split_add(cell, split_term(v[u].x, s[0]));
                split_add(cell + L, split_term(v[u].y, s[1]));
                split_add(cell + 2 * L, split_term(v[u].z, s[2]));
                split_add(cell + 3 * L, split_term(v[u].w, s[3]));
                if (col == 0) atomicAdd(&cnt[c[u]], 1);
            }
        };
        if (n_lo + r < n_hi) {
            fetch(va, ca, n_lo + r);
            for (int n0 = n_lo + r; n0 < n_hi; n0 += 2 * U * R) {
                fetch(vb, cb, n0 + U * R);
                add(va, ca, n0);
                fetch(va, ca, n0 + 2 * U * R);
                add(vb, cb, n0 + U * R);
            }
        }
    } else {
        const int col = tid % dc, j = chunk * dc + col, R = blockDim.x / dc;
        const bool ok = j < d;
        const float *xc = xb + (ok ? j : 0);
        const double s = a.colscale[ok ? j : 0];
        for (int n0 = n_lo + tid / dc; n0 < n_hi; n0 += 8 * R) {
            float v[8];
            int c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int n = min(n0 + u * R, n_hi - 1);
                c[u] = idx[n];
                v[u] = xc[(size_t)n * d];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (n0 + u * R < n_hi) {
                    split_add(cells + c[u] * stride + col, split_term(v[u], s));
                    if (col == 0) atomicAdd(&cnt[c[u]], 1);
                }
        }
    }
    __syncthreads();
    float *out = a.part + ((size_t)share * a.W + worker) * k * d;
    {
        const int col = tid % dc, j = chunk * dc + col;
        const int at = a.vec4 && dc % 4 == 0 ? (col & 3) * (dc / 4) + (col >> 2) : col;
        if (j < d) {
            const double inv = a.colscale[d + j];
            for (int c = tid / dc; c < k; c += blockDim.x / dc) out[(size_t)c * d + j] = split_sum(cells[c * stride + at], cnt[c], inv);
        }
    }
    if (chunk == 0) {
        int *oc = a.cntpart + ((size_t)share * a.W + worker) * k;
        for (int c = tid; c < k; c += blockDim.x) oc[c] = cnt[c];
    }
}

// ---- merge, update, send and the operands of the next assignment ----
// A worker's rows are dealt to `blocks` workgroups.  What they need to know of the whole state goes through device
// memory between phases: the three sums of Eq. 4 (partial sums per workgroup, added in order), the largest |v| and
// row norm (integer maxima of bit patterns, which do not depend on the order), and the power of two the fp16 operands
// are scaled with, which follows the state one step behind.
struct SplitGate { double lhs, rhs, nrm; };
struct SplitMail { int has, round[MAX_BUFFERS]; };     // messages of a merge point: buffers that hold one, their rounds

struct SplitUpdate {
    unsigned char *frag;
    float *hs;
    SplitState *state;                     // 3 x W
    SplitGate *gate;                       // W x buffers x blocks
    SplitMail *mail;                       // W
    const float *m, *xmeta, *part;
    const int *cntpart;
    size_t frag_bytes;
    int kpad, dpad, shares, g, blocks;     // g: lanes per row, a power of two; blocks: workgroups per worker
};

// scale that takes the largest |v| to [2^9, 2^10): 2^6 below the largest fp16 number, should the state grow
__device__ __forceinline__ float split_state_scale(unsigned vabs)
{
    int q = 0;
    const float v = __uint_as_float(vabs);
    if (v > 0.0f && v < INFINITY) (void)frexpf(v, &q);
    return ldexpf(1.0f, max(-120, min(126, 10 - q)));
}

// the columns of the slots [j0, j0 + 8) of an array row (see split_column)
__device__ __forceinline__ void split_row8(float (&v)[8], const float *row, int j0, int d) { split_load8<true>(v, row, j0, d); }
__device__ __forceinline__ void split_put8(float *row, const float (&v)[8], int j0, int d)
{
    if (j0 + 8 <= d) {
        float4u a, b;
#pragma unroll
        for (int e = 0; e < 4; ++e) { a[e] = v[e]; b[e] = v[4 + e]; }
        *reinterpret_cast<float4u *>(row + j0) = a;
        *reinterpret_cast<float4u *>(row + j0 + 4) = b;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (split_slot_used(j0 + e, d)) row[split_column(j0 + e, d)] = v[e];
    }
}
// samples of centroid c, sums of eight columns of a row over the shares of the mini-batch, four shares in flight
__device__ __forceinline__ int split_count(SPLIT_ARG SplitUpdate &u, int W, int k, int i, int c)
{
    int n = 0;
    for (int s0 = 0; s0 < u.shares; s0 += 4) {
        int v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = u.cntpart[((size_t)min(s0 + q, u.shares - 1) * W + i) * k + c];
#pragma unroll
        for (int q = 0; q < 4; ++q) n += s0 + q < u.shares ? v[q] : 0;
    }
    return n;
}
// (The shares are rounded to fp32, added in fp64 and rounded once more: 2^-23 of the sum at worst, however many they are, and
// as their roundings are independent about 2^-24.  Added in fp32, 64 shares of a column far from the origin were several times
// that off.  Their 64-bit integers instead cost 11 % of a step, k = 64, d = 32, b = 500, W = 256, for twice the bytes.)
__device__ __forceinline__ void split_sums8(float (&sm)[8], SPLIT_ARG SplitUpdate &u, int W, int k, int i, int c, int j0, int d)
{
    split_row8(sm, u.part + ((size_t)i * k + c) * d, j0, d);
    if (u.shares == 1) return;
    double total[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) total[e] = (double)sm[e];
    for (int s0 = 1; s0 < u.shares; s0 += 4) {
        float v[4][8];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_row8(v[q], u.part + (((size_t)min(s0 + q, u.shares - 1) * W + i) * k + c) * d, j0, d);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) total[e] += s0 + q < u.shares ? (double)v[q][e] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) sm[e] = (float)total[e];
}

// The same of a kept worker, from the cells themselves.
__device__ __forceinline__ void split_kept_sums8(float (&sm)[8], SPLIT_ARG SplitArgs &a, const unsigned char *smem, int c, int cn, int j0, int d)
{
    const u64 *cells = reinterpret_cast<const u64 *>(smem + a.off_cells) + c * split_cell_stride(a);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int j = min(split_column(j0 + e, d), d - 1);
        sm[e] = split_sum(cells[split_cell(a, j)], cn, a.colscale[d + j]);
    }
}
__device__ __forceinline__ void split_kept_clear8(SPLIT_ARG SplitArgs &a, unsigned char *smem, int c, int j0, int d)
{
    u64 *cells = reinterpret_cast<u64 *>(smem + a.off_cells) + c * split_cell_stride(a);
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (split_slot_used(j0 + e, d)) cells[split_cell(a, split_column(j0 + e, d))] = 0;
}

// Messages between workgroups of one launch: written and read past the caches that are not shared, element by element, so that
// neither side needs a fence (which writes back or invalidates a whole L2: k = 64, d = 32, b = 500, a message every step, 105 us
// per step with fences).
// (sixteen bytes with the scope bit of an agent-scope access; a load waits in the same block.  A store of more than eight bytes
// reads its data late: two wait states before anything may write these registers, which the compiler, who does not look into the
// block, would not leave.)
__device__ __forceinline__ void split_message_put16(float *row, const float (&v)[8])
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 a = {v[0], v[1], v[2], v[3]}, b = {v[4], v[5], v[6], v[7]};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\tglobal_store_dwordx4 %0, %2, off offset:16 sc1\n\ts_nop 1" ::"v"(row), "v"(a), "v"(b) : "memory");
}
__device__ __forceinline__ void split_message_row16(float (&v)[8], const float *row)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    f4 a, b;
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %2, off offset:16 sc1\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(a), "=&v"(b) : "v"(row) : "memory");
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}
__device__ __forceinline__ void split_message_put8(float *row, const float (&v)[8], int j0, int d)
{
    if (j0 + 8 <= d) {
        split_message_put16(row + j0, v);
        return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (split_slot_used(j0 + e, d)) __hip_atomic_store(row + split_column(j0 + e, d), v[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void split_message_row8(float (&v)[8], const float *row, int j0, int d)
{
    if (d >= 8) {
        split_message_row16(v, row + min(j0, d - 8));
        return;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = __hip_atomic_load(row + min(split_column(j0 + e, d), d - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ double split_block_sum(double v, double *red)
{
    v = split_wave_sum(v);
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    double t = 0.0;
    for (int q = 0; q < nw; ++q) t += red[q];
    return t;
}

// The three sums of Eq. 4 over the used slots of a group of eight columns.
__device__ __forceinline__ void split_gate8(const float (&wv)[8], const float (&sm)[8], const float (&ev)[8], int cn, int j0,
                                            SPLIT_ARG StepParams &p, double &lhs, double &rhs, double &nrm)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const bool used = split_slot_used(j0 + e, p.d);
        const float gq = ((float)cn * wv[e] - sm[e]) / (float)p.b;          // descent gradient of Eq. 9, (c_k w_k - S_k) / b
        const double we = used ? (double)ev[e] : 0.0;
        const double q = used ? ((double)wv[e] - (double)p.eps * (double)gq) - we : 0.0, q2 = used ? (double)wv[e] - we : 0.0;
        lhs += q * q; rhs += q2 * q2; nrm += we * we;
    }
}

// Eq. 4 at a merge point: which buffers hold a message, and (whole states) the sums over a workgroup's rows, in fp64.
// CELLS: the sums are in the LDS still, where the assignment left them.
template <bool KEPT, bool CELLS>
__device__ inline void split_gate_item(SPLIT_ARG StepParams &p, SPLIT_ARG SplitUpdate &u, SPLIT_ARG SplitArgs &a, const SplitStep &now, int i, int blk, double *red)
{
    unsigned char *smem = split_lds + SPLIT_LDS_SHARED;
    __syncthreads();
    const int k = p.k, d = p.d;
    const int lane_g = threadIdx.x & (u.g - 1), ngrp = (int)blockDim.x / u.g, grp = threadIdx.x / u.g;
    const size_t kd = (size_t)k * d;
    const int det = p.mode == ASGD_MODE_DETERMINISTIC;
    SplitMail mail;
    mail.has = 0;
    for (int n = 0; n < MAX_BUFFERS; ++n) {
        mail.round[n] = -1;
        if (n >= p.nb) continue;
        const int st = __hip_atomic_load(p.stamp + exchange_buffer(now.read_parity, p.nb, n, p.W, i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (det ? (st == now.round - 1) : (st >= 0)) mail.has |= 1 << n;
        mail.round[n] = st;
    }
    if (blk == 0 && threadIdx.x == 0) u.mail[i] = mail;
    if (p.parts > 1) return;
    const float *w = p.w + (size_t)i * kd;
    for (int n = 0; n < p.nb; ++n) {
        double lhs = 0.0, rhs = 0.0, nrm = 0.0;
        if (mail.has >> n & 1) {
            const float *ext = p.slot + exchange_buffer(now.read_parity, p.nb, n, p.W, i) * kd;
            for (int c = blk * ngrp + grp; c < k; c += u.blocks * ngrp) {
                const int cn = CELLS ? reinterpret_cast<const int *>(smem + a.off_cnt)[c] : split_count(u, p.W, k, i, c);
                for (int j0 = lane_g * 8; j0 < d; j0 += u.g * 8) {
                    float wv[8], sm[8], ev[8];
                    split_row8(wv, w + (size_t)c * d, j0, d);
                    if constexpr (KEPT) split_message_row8(ev, ext + (size_t)c * d, j0, d);
                    else split_row8(ev, ext + (size_t)c * d, j0, d);
                    if constexpr (CELLS) split_kept_sums8(sm, a, smem, c, cn, j0, d);
                    else split_sums8(sm, u, p.W, k, i, c, j0, d);
                    split_gate8(wv, sm, ev, cn, j0, p, lhs, rhs, nrm);
                }
            }
        }
        lhs = split_block_sum(lhs, red); rhs = split_block_sum(rhs, red); nrm = split_block_sum(nrm, red);
        if (threadIdx.x == 0) u.gate[((size_t)i * p.nb + n) * u.blocks + blk] = SplitGate{lhs, rhs, nrm};
    }
}

__device__ __forceinline__ bool split_gate_at_once(SPLIT_ARG SplitArgs &a, SPLIT_ARG SplitUpdate &u)
{
    return a.k * u.g <= (int)blockDim.x && u.dpad <= 8 * u.g;
}

// MODE 0: size of the states; 1: their operands; 2: a step; 3: a step with the 1/count step size (no exchange there);
// 4: a step with partial messages.
// REST: also the norms of what the rows' high parts leave over, for screened samples.
// (A template: a phase this short is mostly the fetch of its own code.)
template <int MODE, bool KEPT, bool REST, bool CELLS>
__device__ inline void split_update_item(SPLIT_ARG StepParams &p, SPLIT_ARG SplitUpdate &u, SPLIT_ARG SplitArgs &a, const SplitStep &now, int i, int blk,
                                         SplitShared &sh)
{
    unsigned char *smem = split_lds + SPLIT_LDS_SHARED;
    int *kept_cnt = reinterpret_cast<int *>(smem + a.off_cnt);
    constexpr bool STEP = MODE >= 2, INV_COUNT = MODE == 3, ROWWISE = MODE == 4;
    const int tid = threadIdx.x, k = p.k, d = p.d;
    const int lane_g = tid & (u.g - 1), ngrp = (int)blockDim.x / u.g, grp = tid / u.g;
    const size_t kd = (size_t)k * d;
    float *w = p.w + (size_t)i * kd;
    unsigned char *frag = KEPT ? smem : u.frag + (size_t)i * u.frag_bytes;
    float *hs = KEPT ? reinterpret_cast<float *>(smem + a.off_hs) : u.hs + (size_t)i * u.kpad;
    SplitState *st_now = u.state + (size_t)now.slot * p.W + i, *st_next = u.state + (size_t)now.slot_next * p.W + i,
               *st_after = u.state + (size_t)now.slot_after * p.W + i;
    const float sx = u.xmeta[0];
    __syncthreads();                                 // (the item before this one is done with the LDS)
    const float sw = MODE == 0 ? 1.0f : split_state_scale(KEPT ? sh.size[now.slot].vabs : st_now->vabs);

    SplitMail mail;
    mail.has = 0;
    int delta_mask = 0;
    // A kept state of no more than a unit per thread: Eq. 4 here, its messages are read once and stay in registers.
    const bool at_once = KEPT && STEP && !INV_COUNT && split_gate_at_once(a, u);
    float evs[KEPT ? MAX_BUFFERS : 1][8];
    if (at_once && now.merge) {
        const bool det = p.mode == ASGD_MODE_DETERMINISTIC;
        const int j0 = lane_g * 8;
        double *gred = reinterpret_cast<double *>(smem + a.off_args);            // [wave][buffer][3]
        int st[MAX_BUFFERS];
        float wv[8], sm[8];
        const bool mine = grp < k && j0 < d;
        const int cn = mine ? kept_cnt[grp] : 0;
        if (mine) {
            split_row8(wv, w + (size_t)grp * d, j0, d);
            split_kept_sums8(sm, a, smem, grp, cn, j0, d);
        }
#pragma unroll
        for (int n = 0; n < MAX_BUFFERS; ++n) {
            if (n >= p.nb) continue;
            const size_t buf = exchange_buffer(now.read_parity, p.nb, n, p.W, i);
            st[n] = __hip_atomic_load(p.stamp + buf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            double lhs = 0.0, rhs = 0.0, nrm = 0.0;
            if (mine) {
                split_message_row8(evs[n], p.slot + buf * kd + (size_t)grp * d, j0, d);
                split_gate8(wv, sm, evs[n], cn, j0, p, lhs, rhs, nrm);
            }
            lhs = split_wave_sum(lhs); rhs = split_wave_sum(rhs); nrm = split_wave_sum(nrm);
            if ((tid & 63) == 0) {
                double *at = gred + ((tid >> 6) * MAX_BUFFERS + n) * 3;
                at[0] = lhs; at[1] = rhs; at[2] = nrm;
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // (the stamps have been read before thread 0 empties them)
        __syncthreads();
        int received = 0, near = 0;
#pragma unroll
        for (int n = 0; n < MAX_BUFFERS; ++n) {
            if (n >= p.nb || !(det ? st[n] == now.round - 1 : st[n] >= 0)) continue;
            double lhs = 0.0, rhs = 0.0, nrm = 0.0;
            for (int q = 0; q < (int)(blockDim.x >> 6); ++q) {
                const double *at = gred + (q * MAX_BUFFERS + n) * 3;
                lhs += at[0]; rhs += at[1]; nrm += at[2];
            }
            if (nrm > 0.0) {                               // lambda of Eq. 3: an all-zero buffer is empty
                received += 1;
                if (p.parzen ? (lhs < rhs) : 1) delta_mask |= 1 << n;
                if (rhs > 0.0 && fabs(lhs - rhs) / rhs < 1e-6) near += 1;
            }
        }
        if (tid == 0) {
            long long *cnp = p.counters + (size_t)i * CNT_STRIDE;
            if (received) {
                cnp[CNT_RECEIVED] += received;
                cnp[CNT_ACCEPTED] += __builtin_popcount(delta_mask);
                cnp[CNT_PARZEN_NEAR] += near;
            }
            for (int n = 0; n < p.nb; ++n)                 // (emptied when it was looked at, as below)
                __hip_atomic_store(p.stamp + exchange_buffer(now.read_parity, p.nb, n, p.W, i), -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else if (STEP && !INV_COUNT && now.merge) {
        // which buffers take part: Eq. 4 over the whole state, every buffer on its own (Eq. 6)
        mail = u.mail[i];
        if (tid == 0) {
            int received = 0, near = 0;
            for (int n = 0; n < p.nb && !ROWWISE; ++n) {
                if (!(mail.has >> n & 1)) continue;
                double lhs = 0.0, rhs = 0.0, nrm = 0.0;
                for (int q = 0; q < u.blocks; ++q) {
                    const SplitGate gt = u.gate[((size_t)i * p.nb + n) * u.blocks + q];
                    lhs += gt.lhs; rhs += gt.rhs; nrm += gt.nrm;
                }
                if (nrm > 0.0) {                       // lambda of Eq. 3: an all-zero buffer is empty
                    received += 1;
                    if (p.parzen ? (lhs < rhs) : 1) delta_mask |= 1 << n;
                    if (rhs > 0.0 && fabs(lhs - rhs) / rhs < 1e-6) near += 1;
                }
            }
            sh.delta = delta_mask;
            if (blk == 0) {
                long long *cnp = p.counters + (size_t)i * CNT_STRIDE;
                if (received) {
                    cnp[CNT_RECEIVED] += received;
                    cnp[CNT_ACCEPTED] += __builtin_popcount(delta_mask);
                    cnp[CNT_PARZEN_NEAR] += near;
                }
                // A buffer is emptied when it is looked at, in either mode: mode and interval may change between two runs.
                // (Deterministic mode: the sender's next stamp goes into this buffer two rounds on.)
                for (int n = 0; n < p.nb; ++n)
                    __hip_atomic_store(p.stamp + exchange_buffer(now.read_parity, p.nb, n, p.W, i), -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        delta_mask = sh.delta;
    }
    if (blk == 0 && tid == 0) {
        if constexpr (KEPT) {
            if (MODE != 0) sh.size[now.slot_next].sw = sw;
        } else {
            if (MODE != 0) st_next->sw = sw;
            st_after->vabs = st_after->n2 = st_after->rest = 0;           // (nobody looks at it in this launch)
        }
    }
    auto peer_of = [&](int n) -> int {                   // recipient of copy n of this worker's message, -1: lost on the way
        if (p.drop_thr && message_dropped(p.seed, now.round, i, p.drop_thr, n)) return -1;
        if (p.mode != ASGD_MODE_DETERMINISTIC) return peer_free(p.seed, now.round, i, p.W, n);
        const int q = i + now.shift[n];
        return q < p.W ? q : q - p.W;
    };

    // ---- Eq. 6 (one buffer: Eq. 7), Alg. 5, update and send; operands of the new state ----
    const int units = u.dpad / 8, nch = u.dpad / 16;
    unsigned vabs = 0, n2max = 0, restmax = 0;
    const float inv_all = 1.0f / (float)(__builtin_popcount(delta_mask) + 1);
    int nz = 0, accd = 0, near_row = 0;
    const int rows = MODE == 1 ? u.kpad : k;             // padding rows are written once
    // One launch, a unit per lane and row: what does not depend on the row is fetched once, a state row while the one before it is worked
    // on; row after row was a chain of latencies.
    const bool one = !KEPT && (CELLS || REST) && units <= u.g;
    const int c_step = u.blocks * ngrp, j_one = lane_g * 8;
    float mid_one[8], w_next[8];
    int at_one[CELLS ? 8 : 1];
    double inv_one[CELLS ? 8 : 1];
    if (one && j_one < d) {
        split_row8(mid_one, u.m, j_one, d);
        split_row8(w_next, w + (size_t)min(blk * ngrp + grp, k - 1) * d, j_one, d);
        if constexpr (CELLS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int j = min(split_column(j_one + e, d), d - 1);
                at_one[e] = split_cell(a, j);
                inv_one[e] = a.colscale[d + j];
            }
        }
    }
    for (int c = blk * ngrp + grp; c < rows; c += u.blocks * ngrp) {
        const bool real = MODE != 1 || c < k;
        const int cn = STEP ? (CELLS ? kept_cnt[c] : split_count(u, p.W, k, i, c)) : 0;
        int rowmask = delta_mask;
        float inv = inv_all;
        if (ROWWISE) {
            // partial messages: lambda, Eq. 4 and Eq. 6 row by row
            rowmask = 0;
            for (int n = 0; n < p.nb; ++n) {
                if (!(mail.has >> n & 1) || !row_travels(c, mail.round[n], i, n, p.parts)) continue;
                const float *ext = p.slot + exchange_buffer(now.read_parity, p.nb, n, p.W, i) * kd;
                double lhs = 0.0, rhs = 0.0, nrm = 0.0;
                for (int j0 = lane_g * 8; j0 < d; j0 += u.g * 8) {
                    float wv[8], sm[8], ev[8];
                    split_row8(wv, w + (size_t)c * d, j0, d);
                    split_row8(ev, ext + (size_t)c * d, j0, d);
                    split_sums8(sm, u, p.W, k, i, c, j0, d);
                    split_gate8(wv, sm, ev, cn, j0, p, lhs, rhs, nrm);
                }
                for (int off = u.g / 2; off > 0; off >>= 1) {
                    lhs += __shfl_xor(lhs, off, 64); rhs += __shfl_xor(rhs, off, 64); nrm += __shfl_xor(nrm, off, 64);
                }
                if (!(nrm > 0.0)) continue;
                nz |= 1 << n;
                if (rhs > 0.0 && fabs(lhs - rhs) / rhs < 1e-6) near_row = 1;
                if (p.parzen ? (lhs < rhs) : 1) rowmask |= 1 << n;
            }
            accd |= rowmask;
            inv = 1.0f / (float)(__builtin_popcount(rowmask) + 1);
        }
        long long seen = 0;
        if (INV_COUNT) {
            seen = p.ncum[(size_t)i * k + c] + cn;
            if (lane_g == 0) p.ncum[(size_t)i * k + c] = seen;
        }
        float sq = 0.0f, rest = 0.0f;
        for (int un = lane_g; un < units; un += u.g) {
            const int j0 = un * 8;
            const int lo_e = j0 + 8 <= d ? 0 : (d >= 8 ? 8 - (d - j0) : 0), hi_e = d >= 8 || j0 + 8 <= d ? 8 : d - j0;   // slots in use
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.0f;
            if (real && j0 < d) {
                float wn[8], mid[8];
                if (one) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) { wn[e] = w_next[e]; mid[e] = mid_one[e]; }
                    split_row8(w_next, w + (size_t)min(c + c_step, k - 1) * d, j0, d);      // (another row: the stores below do not touch it)
                } else {
                    split_row8(wn, w + (size_t)c * d, j0, d);
                    split_row8(mid, u.m, j0, d);
                }
                if (STEP) {
                    float sm[8];
                    if constexpr (CELLS) {
                        if (one) {
                            const u64 *cells = reinterpret_cast<const u64 *>(smem + a.off_cells) + c * split_cell_stride(a);
#pragma unroll
                            for (int e = 0; e < 8; ++e) sm[e] = split_sum(cells[at_one[e]], cn, inv_one[e]);
                        } else {
                            split_kept_sums8(sm, a, smem, c, cn, j0, d);
                        }
                        if constexpr (KEPT) split_kept_clear8(a, smem, c, j0, d);
                    } else {
                        split_sums8(sm, u, p.W, k, i, c, j0, d);
                    }
                    if (INV_COUNT) {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (cn > 0) wn[e] = wn[e] + (sm[e] - (float)cn * wn[e]) / (float)seen;
                    } else {
                        float sum[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) sum[e] = wn[e];
                        for (int n = 0; n < p.nb; ++n)
                            if (rowmask >> n & 1) {
                                float ev[8];
                                const float *ext = p.slot + exchange_buffer(now.read_parity, p.nb, n, p.W, i) * kd + (size_t)c * d;
                                if constexpr (KEPT) {
                                    if (at_once) {
#pragma unroll
                                        for (int e = 0; e < 8; ++e) ev[e] = n == 0 ? evs[0][e] : n == 1 ? evs[1][e] : n == 2 ? evs[2][e] : evs[3][e];
                                    } else {
                                        split_message_row8(ev, ext, j0, d);
                                    }
                                } else {
                                    split_row8(ev, ext, j0, d);
                                }
#pragma unroll
                                for (int e = 0; e < 8; ++e) sum[e] += ev[e];
                            }
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            float g = ((float)cn * wn[e] - sm[e]) / (float)p.b;
                            if (rowmask) g += wn[e] - inv * sum[e];
                            wn[e] = wn[e] - p.eps * g;
                        }
                    }
                    split_put8(w + (size_t)c * d, wn, j0, d);
                    if (!INV_COUNT && now.send)
                        for (int n = 0; n < p.nb; ++n) {
                            const int peer = peer_of(n);
                            float *to = p.slot + exchange_buffer(now.send_parity, p.nb, n, p.W, peer >= 0 ? peer : 0) * kd + (size_t)c * d;
                            if (peer >= 0 && (!ROWWISE || c % p.parts == message_part(now.round, peer, n, p.parts))) {
                                if constexpr (KEPT) split_message_put8(to, wn, j0, d);
                                else split_put8(to, wn, j0, d);
                            }
                        }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = e >= lo_e && e < hi_e ? wn[e] - mid[e] : 0.0f;
                    vabs = max(vabs, __float_as_uint(v[e]) & 0x7fffffffu);
                    v[e] *= sw;                            // (squares of scaled numbers neither overflow nor vanish)
                    sq = fmaf(v[e], v[e], sq);
                }
            }
            if (MODE != 0) {
                half8 hi, lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    hi[e] = (_Float16)v[e];
                    const float left = v[e] - (float)hi[e];
                    lo[e] = (_Float16)left;
                    if (REST) rest = fmaf(left, left, rest);
                }
                half8 *dst = reinterpret_cast<half8 *>(frag + ((((size_t)(c >> 6) * nch + (j0 >> 4)) * 2 + ((c >> 5) & 1)) * 2) * SPLIT_PIECE) +
                             (c & 31) + 32 * ((j0 >> 3) & 1);
                dst[0] = hi;
                dst[64] = lo;
            }
        }
        for (int off = u.g / 2; off > 0; off >>= 1) {
            sq += __shfl_xor(sq, off, 64);
            if (REST && MODE != 0) rest += __shfl_xor(rest, off, 64);
        }
        n2max = max(n2max, __float_as_uint(sq) & 0x7fffffffu);
        if (REST && MODE != 0) restmax = max(restmax, __float_as_uint(rest) & 0x7fffffffu);
        if (MODE != 0 && lane_g == 0) hs[c] = real ? -0.5f * sq * (sx / sw) : SPLIT_PAD_SCORE;
        if (KEPT && STEP && lane_g == 0) kept_cnt[c] = 0;        // (the lanes of a row are lanes of one wave: all have read it)
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        vabs = max(vabs, (unsigned)__shfl_xor((int)vabs, off, 64));
        n2max = max(n2max, (unsigned)__shfl_xor((int)n2max, off, 64));
        if (REST && MODE != 0) restmax = max(restmax, (unsigned)__shfl_xor((int)restmax, off, 64));
        if (ROWWISE) { nz |= __shfl_xor(nz, off, 64); accd |= __shfl_xor(accd, off, 64); near_row |= __shfl_xor(near_row, off, 64); }
    }
    if ((tid & 63) == 0) {
        sh.most[0][tid >> 6] = vabs;
        sh.most[1][tid >> 6] = n2max;
        if (REST) sh.most[2][tid >> 6] = restmax;
        if (ROWWISE && mail.has) {
            // buffers with a non-empty row, with an accepted row, a near-tie: whoever sets a flag first counts it
            const int flags = nz << 8 | accd << 16 | near_row << 24, fresh = flags & ~atomicOr(&u.mail[i].has, flags);
            u64 *cnp = (u64 *)(p.counters + (size_t)i * CNT_STRIDE);
            if (fresh >> 8 & 15) atomicAdd(cnp + CNT_RECEIVED, (u64)__builtin_popcount(fresh >> 8 & 15));
            if (fresh >> 16 & 15) atomicAdd(cnp + CNT_ACCEPTED, (u64)__builtin_popcount(fresh >> 16 & 15));
            if (fresh >> 24) atomicAdd(cnp + CNT_PARZEN_NEAR, (u64)1);
        }
    }
    __syncthreads();
    if (tid < (REST && MODE != 0 ? 3 : 2)) {
        // mode 0 prepares the slot that mode 1 reads, mode 1 the one the first step reads
        unsigned *at;
        if constexpr (KEPT) {
            SplitSize *dst = sh.size + (MODE == 0 ? now.slot : now.slot_next);
            at = tid == 0 ? &dst->vabs : &dst->n2;
        } else {
            SplitState *dst = MODE == 0 ? st_now : st_next;
            at = tid == 0 ? &dst->vabs : tid == 1 ? &dst->n2 : &dst->rest;
        }
        unsigned v = 0;
        for (int q = 0; q < (int)(blockDim.x >> 6); ++q) v = max(v, sh.most[tid][q]);
        if (KEPT || u.blocks == 1) *at = v;
        else atomicMax(at, v);
    }
    if (STEP && !INV_COUNT && now.send) {
        if (now.local) {                        // the message first, then its stamp (in the phases form the launch ends in between)
            if constexpr (KEPT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            else __threadfence();
            __syncthreads();
        }
        if (blk != 0 || tid != 0) return;
        for (int n = 0; n < p.nb; ++n) {
            const int peer = peer_of(n);
            if (peer >= 0)
                __hip_atomic_store(p.stamp + exchange_buffer(now.send_parity, p.nb, n, p.W, peer), now.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        p.counters[(size_t)i * CNT_STRIDE + CNT_SENT] += 1;
    }
}


// ---- the launches ----
struct SplitRun {
    StepParams p;
    SplitArgs a;
    SplitUpdate u;
    long long t0, t1, round0;              // local form: steps of the launch, round of the first
    int te0;                               // first step's place in its round
    int sync;                              // workers wait for each other's messages (deterministic exchange)
    int *arrived;                          // workgroups that have started (zero before the launch), SPLIT_NOBODY or'ed in to call it off
    int expected;                          // workgroups that have to have started before any begins
    int wait_polls;                        // polls a workgroup may spend on one wait
};
constexpr int SPLIT_NOBODY = 1 << 30;
constexpr int SPLIT_ARRIVAL_POLLS = 1 << 20;       // polls until the launch is called off (half a second and more)
struct SplitLaunch {                       // arguments of a phase
    SplitRun run;
    SplitStep now;
};

// The items are inlined into the loop over the steps, each with its own copy of the step's values.  (Called, a function saves the half of the
// registers that it uses and a caller may have use for: for an assignment 200 KB of a compute unit per call, out to memory and back.  k = d = 100,
// W = 512: 9300 us a run with all of them called, 8720 with the assignment inlined, 8610 with Eq. 4 and the update.)  The screened kernel of eight
// chunks keeps 160 vector registers in scratch memory even so, that of five 61, most of them what split_listed() needs.  Items that
// are called pass their arguments in vector registers; what is uniform is read back into scalar ones.
typedef SPLIT_ARG SplitRun *SplitRunPtr;
__device__ __forceinline__ int split_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ SplitRunPtr split_uniform(u64 p) { return (SplitRunPtr)split_uniform64(p); }
__device__ __noinline__ inline void split_long_call(u64 run, int worker, int share)
{
    SplitRunPtr r = split_uniform(run);
    const SplitStep now = split_shared().now;
    split_assign_long_item(r->a, now, split_uniform(worker), split_uniform(share), split_lds + SPLIT_LDS_SHARED);
}
__device__ __noinline__ inline void split_sums_call(u64 run, int worker, int share, int chunk)
{
    SplitRunPtr r = split_uniform(run);
    const SplitStep now = split_shared().now;
    split_sums_item(r->a, now, split_uniform(worker), split_uniform(share), split_uniform(chunk), split_lds + SPLIT_LDS_SHARED);
}
// Screened, as long as that decides enough; the item without it is called, not inlined, because ordinary data never need it.
template <int NC>
__device__ __noinline__ void split_assign_call(u64 run, int worker, int first)
{
    SplitRunPtr r = split_uniform(run);
    const SplitStep now = split_shared().now;
    split_assign_item<NC, false>(r->a, now, split_uniform(worker), 0, split_lds + SPLIT_LDS_SHARED, split_uniform(first));
}
template <int NC>
__device__ __forceinline__ void split_screen_call(u64 run, const SplitStep &now, int worker)
{
    SplitRunPtr r = split_uniform(run);
    const int off = split_uniform(split_shared().unscreened), first = off > 0 ? 0 : split_screen_item<NC>(r->a, now, worker, 0, split_lds + SPLIT_LDS_SHARED);
    __syncthreads();                            // (everybody has read it)
    if (threadIdx.x == 0) split_shared().unscreened = off > 0 ? off - 1 : first >= 0 ? SPLIT_UNSCREENED : 0;
    if (first >= 0) split_assign_call<NC>(run, worker, first);
}
template <bool CELLS>
__device__ __forceinline__ void split_gate_call(u64 run, int worker, int blk)
{
    SplitRunPtr r = split_uniform(run);
    const SplitStep now = split_shared().now;
    split_gate_item<false, CELLS>(r->p, r->u, r->a, now, split_uniform(worker), split_uniform(blk), split_shared().red);
}
template <int MODE, bool KEPT, bool REST, bool CELLS>
__device__ __forceinline__ void split_update_call(u64 run, int worker, int blk)
{
    SplitRunPtr r = split_uniform(run);
    const SplitStep now = split_shared().now;
    split_update_item<MODE, KEPT, REST, CELLS>(r->p, r->u, r->a, now, split_uniform(worker), split_uniform(blk), split_shared());
}

// Phases form.  WHAT: 0..4 modes of the update, 5 Eq. 4, 6 gradient sums, 9 assignment of long rows whose operands fit the LDS, 10 + NC assignment (10: longer rows)
template <int WHAT>
__global__ __launch_bounds__(SPLIT_THREADS) __attribute__((amdgpu_waves_per_eu(WHAT >= 13 || WHAT == 9 || WHAT == 10 ? 2 : 3)))
void split_phase_kernel(SplitLaunch args)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    (void)args;
    typedef SPLIT_ARG SplitLaunch *LaunchPtr;
    LaunchPtr l = (LaunchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    SplitStep now;
    now.slot = l->now.slot; now.slot_next = l->now.slot_next; now.slot_after = l->now.slot_after;
    now.merge = l->now.merge; now.send = l->now.send; now.round = l->now.round;
    now.read_parity = l->now.read_parity; now.send_parity = l->now.send_parity; now.local = 0;
    now.state = l->now.state; now.dump = l->now.dump; now.row0 = l->now.row0; now.row0_next = -1; now.batch = 0;
    for (int n = 0; n < MAX_BUFFERS; ++n) now.shift[n] = l->now.shift[n];
    const int W = l->run.p.W, worker = blockIdx.x % W, rest = blockIdx.x / W;
    if constexpr (WHAT >= 11) {
        split_assign_item<WHAT - 10, false>(l->run.a, now, worker, rest, lds + SPLIT_LDS_SHARED);
    } else if constexpr (WHAT == 10) {
        split_assign_long_item(l->run.a, now, worker, rest, lds + SPLIT_LDS_SHARED);
    } else if constexpr (WHAT == 9) {
        split_assign_wide_item(l->run.a, now, worker, rest, lds + SPLIT_LDS_SHARED);
    } else if constexpr (WHAT == 6) {
        const int ncol = l->run.a.ncol;
        split_sums_item(l->run.a, now, worker, rest / ncol, rest % ncol, lds + SPLIT_LDS_SHARED);
    } else if constexpr (WHAT == 5) {
        split_gate_item<false, false>(l->run.p, l->run.u, l->run.a, now, worker, rest, reinterpret_cast<SplitShared *>(lds)->red);
    } else {
        split_update_item<WHAT, false, false, false>(l->run.p, l->run.u, l->run.a, now, worker, rest, *reinterpret_cast<SplitShared *>(lds));
    }
}
template <int WHAT>
hipError_t split_launch_phase(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s)
{
    const hipError_t e = hipFuncSetAttribute((const void *)split_phase_kernel<WHAT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_phase_kernel<WHAT>, dim3(blocks), dim3(threads), lds, s, l);
    return hipGetLastError();
}

// Bounded wait for a flag another workgroup writes, by one thread; about half a microsecond per poll.  What a workgroup may
// spend on one wait follows the longest a round of its neighbour can take (SplitRun::wait_polls), and once a wait has
// expired it waits for nothing any more.  (A budget for all the waits of a launch ran out where one worker's samples all
// had to be decided in fp64.)
__device__ inline bool split_wait_flag(const int *flag, int want, bool at_least, int &budget)
{
    while (budget > 0) {
        const int v = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (at_least ? v >= want : v == want) return true;
        __builtin_amdgcn_s_sleep(8);
        --budget;
    }
    return false;
}

// Whether all the workgroups of a launch have a place on the device, by one thread of each: they wait for each other's messages
// later, and one that finds no place (another stream's kernel holds it) would let the others' waits expire.  All of them
// or none: the word ends as `expected` or with SPLIT_NOBODY in it, whichever comes first, and nothing has been touched yet.
__device__ inline bool split_all_arrived(int *word, int expected, int polls)
{
    int v = __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    while (v < expected) {
        if (polls-- > 0) {
            __builtin_amdgcn_s_sleep(8);
            v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (__hip_atomic_compare_exchange_strong(word, &v, v | SPLIT_NOBODY, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            return false;
        }
    }
    return v == expected;
}

// Local form.  NC: chunks of 16 columns of a row, 0: long rows.  Workgroup g has the workers g, g + grid, ...; every wait
// is for an event of an earlier round, and a workgroup does a step of all its workers before the next step of any, so
// the waits cannot form a cycle.
// KEPT: one worker per workgroup, whose operands, offsets, sums and counts stay in the LDS from step to step, the next mini-batch
// arrives there during a step, and the items are inlined: such steps are bound by latency, of calls, copies of the step and
// round trips to the L2 as much as of the memory (500 x 7 samples, 12 centroids, 1/count: 15.1 us per step, 14.2 without the round trips,
// 13.1 with the mini-batch there, 12.2 inlined).
// OTHER: the other assignment of its row length, wide for NC = 0, screened else.
template <int NC, bool KEPT, bool INV_COUNT, bool OTHER>
__global__ __launch_bounds__(SPLIT_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_local_kernel(SplitRun args)
{
    (void)args;
    SplitRunPtr r = (SplitRunPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const u64 run = (u64)r;
    SplitShared &sh = split_shared();
    SplitStep now;
    now.merge = now.send = now.round = now.read_parity = now.send_parity = 0;
    now.local = 1;
    now.slot = 0; now.slot_next = 1; now.slot_after = 2;
    now.state = nullptr; now.dump = nullptr; now.row0 = 0; now.row0_next = -1; now.batch = 0;
    for (int n = 0; n < MAX_BUFFERS; ++n) now.shift[n] = 0;
    const int W = r->p.W;
    const bool det = r->p.mode == ASGD_MODE_DETERMINISTIC;
    constexpr bool CELLS = NC != 0 && !OTHER;           // sums may be formed along with the assignment
    // (the test hook is a budget for all the waits of the launch)
    int budget = r->p.wait_polls > 0 ? r->p.wait_polls : r->wait_polls;
    auto wait = [&](const int *flag, int want, bool at_least) {            // (thread 0)
        if (budget <= 0) return;
        if (!split_wait_flag(flag, want, at_least, budget))
            __hip_atomic_store(r->p.error_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        else if (r->p.wait_polls == 0) budget = r->wait_polls;
    };
    if (r->sync) {
        if (threadIdx.x == 0) {
            sh.delta = split_all_arrived(r->arrived, r->expected, SPLIT_ARRIVAL_POLLS);
            if (!sh.delta) __hip_atomic_store(r->p.error_flag, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __syncthreads();
        if (!sh.delta) return;
    }
    if (threadIdx.x == 0) {
        sh.now = now;
        sh.unscreened = 0;
    }
    __syncthreads();
    if constexpr (KEPT) {
        if (r->t0 < r->t1) split_batch_fetch(r->a, blockIdx.x, r->t0 % r->p.S * r->p.b, split_lds + SPLIT_LDS_SHARED + r->a.off_batch);
    }
    for (int i = blockIdx.x; i < W; i += gridDim.x) {
        split_update_call<0, KEPT, false, false>(run, i, 0);
        __syncthreads();
        if constexpr (KEPT) {
            unsigned char *smem = split_lds + SPLIT_LDS_SHARED;
            const int d = r->a.d, n = r->a.k * (r->a.vec4 ? d : (d + 1) & ~1);
            for (int j = threadIdx.x; j < r->a.dpad; j += blockDim.x) reinterpret_cast<float *>(smem + r->a.off_ms)[j] = r->a.ms[j];
            for (int e = threadIdx.x; e < n; e += blockDim.x) reinterpret_cast<u64 *>(smem + r->a.off_cells)[e] = 0;
            for (int c = threadIdx.x; c < r->a.k; c += blockDim.x) reinterpret_cast<int *>(smem + r->a.off_cnt)[c] = 0;
        }
        split_update_call<1, KEPT, OTHER && NC != 0, false>(run, i, 0);
    }
    int te = r->te0;
    long long t = r->t0, round = r->round0, s = t % r->p.S;
    for (; t < r->t1; ++t) {
        const int old = now.slot;
        now.slot = now.slot_next; now.slot_next = now.slot_after; now.slot_after = old;
        if (r->p.E > 0) {
            now.round = (int)round;
            now.merge = t > 0 && te == 0;
            now.send = W > 1 && te + 1 == r->p.E;
            now.read_parity = det ? (int)((round - 1) & 1) : 0;
            now.send_parity = det ? (int)(round & 1) : 0;
            if (now.send && det)
                for (int n = 0; n < MAX_BUFFERS; ++n)
                    if (n < r->p.nb) now.shift[n] = shift_deterministic(r->p.seed, round, W, n);
            if (++te == r->p.E) { te = 0; ++round; }
        }
        now.state = r->u.state + (size_t)now.slot * W;
        now.row0 = s * r->p.b;
        now.dump = r->p.dump ? r->p.dump + (size_t)(t - r->p.t_dump0) * W * r->p.b : nullptr;
        if (++s == r->p.S) s = 0;
        now.row0_next = t + 1 < r->t1 ? s * r->p.b : -1;
        now.batch = (int)((t - r->t0) & 1);
        if constexpr (!KEPT) {
            __syncthreads();
            if (threadIdx.x == 0) sh.now = now;
            __syncthreads();
        }
        for (int i = blockIdx.x; i < W; i += gridDim.x) {
            if constexpr (KEPT) {
                split_assign_item<NC, true>(r->a, now, i, 0, split_lds + SPLIT_LDS_SHARED);
            } else if constexpr (NC == 0 && !OTHER) {
                split_long_call(run, i, 0);
            } else {
                const SplitStep then = sh.now;
                if constexpr (NC == 0) split_assign_wide_item(r->a, then, i, 0, split_lds + SPLIT_LDS_SHARED);
                else if constexpr (OTHER) split_screen_call<NC>(run, then, i);
                else split_assign_item<NC, false>(r->a, then, i, 0, split_lds + SPLIT_LDS_SHARED);
            }
            if (!KEPT && !r->a.fused)
                for (int q = 0; q < r->a.ncol; ++q) split_sums_call(run, i, 0, q);
            if (r->sync && now.merge) {
                // the messages of the last round (those sent before this launch are there)
                if (threadIdx.x == 0 && t > r->t0)
                    for (int n = 0; n < r->p.nb; ++n) {
                        const long long rs = now.round - 1;
                        const int sender = (i - shift_deterministic(r->p.seed, rs, W, n) + W) % W;
                        if (r->p.drop_unannounced || !message_dropped(r->p.seed, rs, sender, r->p.drop_thr, n))
                            wait(r->p.stamp + exchange_buffer(now.read_parity, r->p.nb, n, W, i), (int)rs, false);
                    }
                __syncthreads();
                if constexpr (!KEPT) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            if (now.merge) {
                if constexpr (KEPT) {
                    if (!split_gate_at_once(r->a, r->u)) split_gate_item<true, true>(r->p, r->u, r->a, now, i, 0, sh.red);
                } else {
                    if (CELLS && r->a.fused) split_gate_call<CELLS>(run, i, 0);
                    else split_gate_call<false>(run, i, 0);
                }
            }
            if (r->sync && now.send && now.round >= 2) {
                // a recipient's buffer still holds the message of round - 2 until it has passed merge point round - 1
                if (threadIdx.x == 0)
                    for (int n = 0; n < r->p.nb; ++n) {
                        const int q = i + now.shift[n];
                        wait(r->p.consumed + (q < W ? q : q - W), now.round - 1, true);
                    }
                __syncthreads();
            }
            if constexpr (KEPT) {
                split_update_item<INV_COUNT ? 3 : 2, true, false, true>(r->p, r->u, r->a, now, i, 0, sh);
            } else {
                auto update = [&](auto cells) {
                    if (r->p.lr_mode == ASGD_LR_INV_COUNT) split_update_call<3, KEPT, OTHER && NC != 0, decltype(cells)::value>(run, i, 0);
                    else split_update_call<2, KEPT, OTHER && NC != 0, decltype(cells)::value>(run, i, 0);
                };
                if (CELLS && r->a.fused) update(std::integral_constant<bool, CELLS>{});
                else update(std::false_type{});
            }
            if (r->sync && now.merge) {
                __syncthreads();
                // (thread 0 has emptied the stamps: they have arrived before the sender may write them again)
                if (threadIdx.x == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (threadIdx.x == 0) __hip_atomic_store(r->p.consumed + i, now.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <int NC, bool KEPT, bool INV_COUNT, bool OTHER>
hipError_t split_launch_local_form(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    const void *kern = (const void *)split_local_kernel<NC, KEPT, INV_COUNT, OTHER>;
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    SplitRun rr = r;
    void *args[] = {&rr};
    if (r.sync && r.p.cooperative) return hipLaunchCooperativeKernel(kern, dim3(blocks), dim3(threads), args, lds, s);
    split_local_kernel<NC, KEPT, INV_COUNT, OTHER><<<dim3(blocks), dim3(threads), lds, s>>>(rr);
    return hipGetLastError();
}
template <int NC>
hipError_t split_launch_local(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s)
{
    if constexpr (NC != 0 && NC <= SPLIT_KEPT_CHUNKS) {
        if (r.a.kept)
            return r.p.lr_mode == ASGD_LR_INV_COUNT ? split_launch_local_form<NC, true, true, false>(r, blocks, threads, lds, s)
                                                    : split_launch_local_form<NC, true, false, false>(r, blocks, threads, lds, s);
    }
    if constexpr (NC != 1) {
        if (NC == 0 ? r.a.wide : r.a.stages) return split_launch_local_form<NC, false, false, true>(r, blocks, threads, lds, s);
    }
    return split_launch_local_form<NC, false, false, false>(r, blocks, threads, lds, s);
}

}  // namespace asgd
