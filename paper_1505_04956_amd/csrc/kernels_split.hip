// Step kernels for any row length, second part: long rows, gradient sums of large states, merge and update, and the
// launches of a range of steps.
#include <string.h>

#include "split_steps.h"

namespace asgd {

hipError_t launch_split_assign_1(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_2(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_3(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_4(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_5(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_6(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_7(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_8(const SplitArgs &a, int blocks, int threads, unsigned lds, hipStream_t s);

namespace {

constexpr int SPLIT_SAMPLE_ROWS = 1024;     // rows looked at for the middle of the data
constexpr unsigned SPLIT_LDS = 150 * 1024;

// ---- once per call of the library: middle of the data, scale of the samples, scales of the fixed-point sums ----
// m_j: mean of up to SPLIT_SAMPLE_ROWS rows spread over the data (any value is a valid reference; one near the middle
// keeps |x - m| small).  One workgroup of 16 waves per 64 columns, eight rows per wave in flight.
__global__ __launch_bounds__(1024) void split_middle_kernel(const float *x, long long rows, int d, float *m)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
    const int n = (int)min(rows, (long long)SPLIT_SAMPLE_ROWS);
    const long long step = rows / n;
    float s = 0.0f;
    for (int q0 = wave; q0 < n; q0 += 128) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = x[(size_t)(min(q0 + 16 * u, n - 1) * step) * d + (j < d ? j : 0)];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += q0 + 16 * u < n ? v[u] : 0.0f;
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j < d) {
        s = 0.0f;
        for (int q = 0; q < 16; ++q) s += red[q][lane];
        m[j] = s / (float)n;
    }
}
// sx: power of two with max_j (max|x_j| + |m_j|) * sx in [2^13, 2^14); ms = -m * sx; scale of column j of the sums: 2^e
// with max|x_j| 2^e < 2^50 and b max|x_j| 2^e < 2^62
__global__ void split_scales_kernel(const float *xabsmax, float *m, int d, int dpad, int b, float *ms, float *xmeta, double *colscale)
{
    __shared__ float red[256];
    const int tid = threadIdx.x;
    float a = 0.0f;
    for (int j = tid; j < d; j += 256) a = fmaxf(a, xabsmax[j] + fabsf(m[j]));
    red[tid] = a;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (tid < off) red[tid] = fmaxf(red[tid], red[tid + off]);
        __syncthreads();
    }
    int q = 0;
    if (red[0] > 0.0f) (void)frexpf(red[0], &q);
    const float sx = ldexpf(1.0f, max(-100, min(100, 14 - q)));
    if (tid == 0) xmeta[0] = sx;
    for (int j = tid; j < dpad; j += 256) ms[j] = split_slot_used(j, d) ? -m[split_column(j, d)] * sx : 0.0f;
    for (int j = tid; j < d; j += 256) {
        int e = 0, bits = 1;
        (void)frexpf(xabsmax[j], &e);                  // |x_j| < 2^e
        while ((1LL << bits) < (long long)b) ++bits;   // b <= 2^bits
        const int sh = min(50, 62 - bits) - (xabsmax[j] > 0.0f ? e : 0);
        colscale[j] = ldexp(1.0, sh);
        colscale[d + j] = ldexp(1.0, -sh);
    }
}

// ---- assignment for rows of more than 128 columns ----
// The operands of the samples do not fit the registers: for every pair of row blocks the samples' columns are read
// again (from a cache) and split again, eight chunks of 16 columns per stage of the state's operands.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_assign_long_kernel(SplitArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int worker = blockIdx.x % a.W, share = blockIdx.x / a.W;
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int nw = blockDim.x >> 6, npair = (a.nblk + 1) / 2, ncg = a.dpad / 128, nstage = npair * ncg;
    float *hs = reinterpret_cast<float *>(smem + a.off_hs);
    float *ms = reinterpret_cast<float *>(smem + a.off_ms);
    const unsigned char *frag = a.frag + (size_t)worker * a.frag_bytes;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)a.row0) * a.d;
    const float sx = a.xmeta[0];
    for (int c = tid; c < a.kpad; c += blockDim.x) hs[c] = a.hs[(size_t)worker * a.kpad + c];
    for (int j = tid; j < a.dpad; j += blockDim.x) ms[j] = a.ms[j];
    __syncthreads();

    int rechecks = 0;
    const int span = nw * 64;
    for (int g0 = n_lo; g0 < n_hi; g0 += span) {
        const int g = g0 + wave * 64;
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
        __syncthreads();
        split_stage(frag, smem, SPLIT_STAGE / SPLIT_PIECE);
        sfloatx16 acc[2][2];                  // [block of the pair][tile of samples]
        int rp = 0, cg = 0;
        for (int st = 0; st < nstage; ++st) {
            split_stage_wait();
            if (st + 1 < nstage)
                split_stage(frag + (size_t)(st + 1) * SPLIT_STAGE, smem + ((st + 1) & 1) * SPLIT_STAGE, SPLIT_STAGE / SPLIT_PIECE);
            if (active) {
                if (cg == 0) {
                    split_init_acc(acc[0][0], hs, 2 * rp, half);
                    acc[0][1] = acc[0][0];
                    split_init_acc(acc[1][0], hs, 2 * rp + 1, half);
                    acc[1][1] = acc[1][0];
                }
                const half8 *A = reinterpret_cast<const half8 *>(smem + (st & 1) * SPLIT_STAGE) + lane;
                // (columns past d: the last stage is zero there; their loads are clamped)
                const bool last = cg + 1 == ncg;
                auto chunks = [&](auto tail) {
                    constexpr bool TAIL = decltype(tail)::value;
                    // four chunks' columns in flight while four are multiplied (with one, the loop was a chain of
                    // cache latencies)
                    constexpr int PF = 4;
                    float v[PF][2][8];
#pragma unroll
                    for (int q = 0; q < PF; ++q)
#pragma unroll
                        for (int m = 0; m < 2; ++m) split_load8<TAIL>(v[q][m], row[m], cg * 128 + q * 16 + 8 * half, a.d);
#pragma unroll
                    for (int ch = 0; ch < 8; ++ch) {
                        const int col = cg * 128 + ch * 16 + 8 * half;
                        half8 bh[2], bl[2];
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            float q = 0.0f;
                            split_convert<TAIL>(v[ch % PF][m], sx, ms, col, a.d, bh[m], bl[m], q);
                            n2[m] += rp == 0 ? q : 0.0f;
                        }
                        if (ch + PF < 8) {
#pragma unroll
                            for (int m = 0; m < 2; ++m) split_load8<TAIL>(v[ch % PF][m], row[m], col + PF * 16, a.d);
                        }
#pragma unroll
                        for (int blk = 0; blk < 2; ++blk) {
                            const half8 ah = A[ch * 256 + blk * 128], al = A[ch * 256 + blk * 128 + 64];
#pragma unroll
                            for (int m = 0; m < 2; ++m) {
                                acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[m], acc[blk][m], 0, 0, 0);
                                acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[m], acc[blk][m], 0, 0, 0);
                                acc[blk][m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[m], acc[blk][m], 0, 0, 0);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                if (last) chunks(std::true_type());
                else chunks(std::false_type());
                if (last) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        split_insert(top[m], acc[0][m], 2 * rp, big);
                        split_insert(top[m], acc[1][m], 2 * rp + 1, big);
                    }
                }
            }
            if (++cg == ncg) { cg = 0; ++rp; }
        }
        if (active) split_finish_group(a, top, n2, worker, g, n_hi, xb, half, nullptr, nullptr, nullptr, rechecks);
    }
    split_count_rechecks(a, worker, rechecks);
}

// ---- gradient sums of a (worker, share, group of dc columns) where the cells of a whole state do not fit LDS ----
// 64-bit fixed-point cells as in the fused form; a wave takes 64 / dc rows at a time.
__global__ __launch_bounds__(512) void split_sums_kernel(SplitArgs a, int dc, int ncol)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u64 *cells = reinterpret_cast<u64 *>(smem);
    int *cnt = reinterpret_cast<int *>(smem + (size_t)a.k * dc * sizeof(u64));
    // (workgroups of one worker are a multiple of eight apart when W is: they share an L2)
    const int worker = blockIdx.x % a.W, rest = blockIdx.x / a.W, chunk = rest % ncol, share = rest / ncol;
    const int n_lo = share * a.share_len, n_hi = min(a.b, n_lo + a.share_len);
    const int tid = threadIdx.x, d = a.d;
    for (int e = tid; e < a.k * dc; e += blockDim.x) cells[e] = 0;
    for (int c = tid; c < a.k; c += blockDim.x) cnt[c] = 0;
    __syncthreads();
    const int col = tid % dc, j = chunk * dc + col, R = blockDim.x / dc;
    const bool ok = j < d;
    const float *xb = a.x + ((size_t)worker * a.H + (size_t)a.row0) * d + (ok ? j : 0);
    const int *idx = a.idx + (size_t)worker * a.b;
    const double s = a.colscale[ok ? j : 0];
    for (int n0 = n_lo + tid / dc; n0 < n_hi; n0 += 8 * R) {
        float v[8];
        int c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int n = min(n0 + u * R, n_hi - 1);
            c[u] = idx[n];
            v[u] = xb[(size_t)n * d];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (n0 + u * R < n_hi) {
                split_add(cells + c[u] * dc + col, split_term(v[u], s));
                if (col == 0) atomicAdd(&cnt[c[u]], 1);
            }
    }
    __syncthreads();
    float *out = a.part + ((size_t)share * a.W + worker) * a.k * d;
    for (int e = tid; e < a.k * dc; e += blockDim.x) {
        const int c = e / dc, jj = chunk * dc + e - c * dc;
        if (jj < d) out[(size_t)c * d + jj] = split_sum(cells[e], cnt[c], a.colscale[d + jj]);
    }
    if (chunk == 0) {
        int *oc = a.cntpart + ((size_t)share * a.W + worker) * a.k;
        for (int c = tid; c < a.k; c += blockDim.x) oc[c] = cnt[c];
    }
}

// ---- merge, update, send and the operands of the next assignment ----
// A worker's rows are dealt to `parts` workgroups.  What they need to know of the whole state goes through device
// memory between launches: the three sums of Eq. 4 (partial sums per workgroup, added in order), the largest |v| and
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
    int slot, slot_next, slot_after;       // step modulo 3
    int merge, send, round;                // of this step: merge point, messages go out, round number
    int read_parity, send_parity;
    int shift[MAX_BUFFERS];                // deterministic schedule of the round
};

// scale that takes the largest |v| to [2^9, 2^10): 2^6 below the largest fp16 number, should the state grow
__device__ __forceinline__ float split_state_scale(unsigned vabs)
{
    int q = 0;
    const float v = __uint_as_float(vabs);
    if (v > 0.0f && v < 3.0e38f) (void)frexpf(v, &q);
    return ldexpf(1.0f, max(-100, min(100, 10 - q)));
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
__device__ __forceinline__ int split_count(const SplitUpdate &u, int W, int k, int i, int c)
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
__device__ __forceinline__ void split_sums8(float (&sm)[8], const SplitUpdate &u, int W, int k, int i, int c, int j0, int d)
{
    split_row8(sm, u.part + ((size_t)i * k + c) * d, j0, d);
    for (int s0 = 1; s0 < u.shares; s0 += 4) {
        float v[4][8];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_row8(v[q], u.part + (((size_t)min(s0 + q, u.shares - 1) * W + i) * k + c) * d, j0, d);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) sm[e] += s0 + q < u.shares ? v[q][e] : 0.0f;
    }
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
                                            const StepParams &p, double &lhs, double &rhs, double &nrm)
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
__global__ __launch_bounds__(256) void split_gate_kernel(StepParams p, SplitUpdate u)
{
    __shared__ double red[4];
    const int i = blockIdx.x % p.W, blk = blockIdx.x / p.W, k = p.k, d = p.d;
    const int lane_g = threadIdx.x & (u.g - 1), ngrp = 256 / u.g, grp = threadIdx.x / u.g;
    const size_t kd = (size_t)k * d;
    const int det = p.mode == ASGD_MODE_DETERMINISTIC;
    SplitMail mail;
    mail.has = 0;
    for (int n = 0; n < MAX_BUFFERS; ++n) {
        mail.round[n] = -1;
        if (n >= p.nb) continue;
        const int st = p.stamp[exchange_buffer(u.read_parity, p.nb, n, p.W, i)];
        if (det ? (st == u.round - 1) : (st >= 0)) mail.has |= 1 << n;
        mail.round[n] = st;
    }
    if (blk == 0 && threadIdx.x == 0) u.mail[i] = mail;
    if (p.parts > 1) return;
    const float *w = p.w + (size_t)i * kd;
    for (int n = 0; n < p.nb; ++n) {
        double lhs = 0.0, rhs = 0.0, nrm = 0.0;
        if (mail.has >> n & 1) {
            const float *ext = p.slot + exchange_buffer(u.read_parity, p.nb, n, p.W, i) * kd;
            for (int c = blk * ngrp + grp; c < k; c += u.blocks * ngrp) {
                const int cn = split_count(u, p.W, k, i, c);
                for (int j0 = lane_g * 8; j0 < d; j0 += u.g * 8) {
                    float wv[8], sm[8], ev[8];
                    split_row8(wv, w + (size_t)c * d, j0, d);
                    split_row8(ev, ext + (size_t)c * d, j0, d);
                    split_sums8(sm, u, p.W, k, i, c, j0, d);
                    split_gate8(wv, sm, ev, cn, j0, p, lhs, rhs, nrm);
                }
            }
        }
        lhs = split_block_sum(lhs, red); rhs = split_block_sum(rhs, red); nrm = split_block_sum(nrm, red);
        if (threadIdx.x == 0) u.gate[((size_t)i * p.nb + n) * u.blocks + blk] = SplitGate{lhs, rhs, nrm};
    }
}

// MODE 0: size of the states; 1: their operands; 2: a step; 3: a step with the 1/count step size (no exchange there);
// 4: a step with partial messages.
// (A template, and everything that is the same for all workers comes from the host: a launch this short is mostly the
// fetch of its own code - as one kernel with 64-bit divisions for the round numbers it took 22 us for 256 states of
// 12 x 7, three times the gate kernel's time for more work.)
template <int MODE>
__global__ __launch_bounds__(256) void split_update_kernel(StepParams p, SplitUpdate u)
{
    __shared__ int s_delta;
    __shared__ unsigned s_max[2][4];
    constexpr bool STEP = MODE >= 2, INV_COUNT = MODE == 3, ROWWISE = MODE == 4;
    const int i = blockIdx.x % p.W, blk = blockIdx.x / p.W, tid = threadIdx.x, k = p.k, d = p.d;
    const int lane_g = tid & (u.g - 1), ngrp = 256 / u.g, grp = tid / u.g;
    const size_t kd = (size_t)k * d;
    float *w = p.w + (size_t)i * kd;
    unsigned char *frag = u.frag + (size_t)i * u.frag_bytes;
    float *hs = u.hs + (size_t)i * u.kpad;
    SplitState *st_now = u.state + (size_t)u.slot * p.W + i, *st_next = u.state + (size_t)u.slot_next * p.W + i,
               *st_after = u.state + (size_t)u.slot_after * p.W + i;
    const float sx = u.xmeta[0];
    const float sw = MODE == 0 ? 1.0f : split_state_scale(st_now->vabs);

    SplitMail mail;
    mail.has = 0;
    int delta_mask = 0;
    if (STEP && !INV_COUNT && u.merge) {
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
            s_delta = delta_mask;
            if (blk == 0) {
                long long *cnp = p.counters + (size_t)i * CNT_STRIDE;
                if (received) {
                    cnp[CNT_RECEIVED] += received;
                    cnp[CNT_ACCEPTED] += __builtin_popcount(delta_mask);
                    cnp[CNT_PARZEN_NEAR] += near;
                }
                for (int n = 0; n < p.nb; ++n) p.stamp[exchange_buffer(u.read_parity, p.nb, n, p.W, i)] = -1;
            }
        }
        __syncthreads();
        delta_mask = s_delta;
    }
    if (blk == 0 && tid == 0) {
        if (MODE != 0) st_next->sw = sw;
        st_after->vabs = st_after->n2 = 0;               // (nobody looks at it in this launch)
    }
    auto peer_of = [&](int n) -> int {                   // recipient of copy n of this worker's message, -1: lost on the way
        if (p.drop_thr && message_dropped(p.seed, u.round, i, p.drop_thr, n)) return -1;
        if (p.mode != ASGD_MODE_DETERMINISTIC) return peer_free(p.seed, u.round, i, p.W, n);
        const int q = i + u.shift[n];
        return q < p.W ? q : q - p.W;
    };

    // ---- Eq. 6 (one buffer: Eq. 7), Alg. 5, update and send; operands of the new state ----
    const int units = u.dpad / 8, nch = u.dpad / 16;
    unsigned vabs = 0, n2max = 0;
    const float inv_all = 1.0f / (float)(__builtin_popcount(delta_mask) + 1);
    int nz = 0, accd = 0, near_row = 0;
    const int rows = MODE == 1 ? u.kpad : k;             // padding rows are written once
    for (int c = blk * ngrp + grp; c < rows; c += u.blocks * ngrp) {
        const bool real = MODE != 1 || c < k;
        const int cn = STEP ? split_count(u, p.W, k, i, c) : 0;
        int rowmask = delta_mask;
        float inv = inv_all;
        if (ROWWISE) {
            // partial messages: lambda, Eq. 4 and Eq. 6 row by row
            rowmask = 0;
            for (int n = 0; n < p.nb; ++n) {
                if (!(mail.has >> n & 1) || !row_travels(c, mail.round[n], i, n, p.parts)) continue;
                const float *ext = p.slot + exchange_buffer(u.read_parity, p.nb, n, p.W, i) * kd;
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
        float sq = 0.0f;
        for (int un = lane_g; un < units; un += u.g) {
            const int j0 = un * 8;
            const int lo_e = j0 + 8 <= d ? 0 : (d >= 8 ? 8 - (d - j0) : 0), hi_e = d >= 8 || j0 + 8 <= d ? 8 : d - j0;   // slots in use
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.0f;
            if (real && j0 < d) {
                float wn[8], mid[8];
                split_row8(wn, w + (size_t)c * d, j0, d);
                split_row8(mid, u.m, j0, d);
                if (STEP) {
                    float sm[8];
                    split_sums8(sm, u, p.W, k, i, c, j0, d);
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
                                split_row8(ev, p.slot + exchange_buffer(u.read_parity, p.nb, n, p.W, i) * kd + (size_t)c * d, j0, d);
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
                    if (!INV_COUNT && u.send)
                        for (int n = 0; n < p.nb; ++n) {
                            const int peer = peer_of(n);
                            if (peer >= 0 && (!ROWWISE || c % p.parts == message_part(u.round, peer, n, p.parts)))
                                split_put8(p.slot + exchange_buffer(u.send_parity, p.nb, n, p.W, peer) * kd + (size_t)c * d, wn, j0, d);
                        }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = e >= lo_e && e < hi_e ? wn[e] - mid[e] : 0.0f;
                    sq = fmaf(v[e], v[e], sq);
                    vabs = max(vabs, __float_as_uint(v[e]) & 0x7fffffffu);
                }
            }
            if (MODE != 0) {
                half8 hi, lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float y = v[e] * sw;
                    hi[e] = (_Float16)y;
                    lo[e] = (_Float16)(y - (float)hi[e]);
                }
                half8 *dst = reinterpret_cast<half8 *>(frag + ((((size_t)(c >> 6) * nch + (j0 >> 4)) * 2 + ((c >> 5) & 1)) * 2) * SPLIT_PIECE) +
                             (c & 31) + 32 * ((j0 >> 3) & 1);
                dst[0] = hi;
                dst[64] = lo;
            }
        }
        for (int off = u.g / 2; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        n2max = max(n2max, __float_as_uint(sq) & 0x7fffffffu);
        if (MODE != 0 && lane_g == 0) hs[c] = real ? -0.5f * sq * sx * sw : SPLIT_PAD_SCORE;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        vabs = max(vabs, (unsigned)__shfl_xor((int)vabs, off, 64));
        n2max = max(n2max, (unsigned)__shfl_xor((int)n2max, off, 64));
        if (ROWWISE) { nz |= __shfl_xor(nz, off, 64); accd |= __shfl_xor(accd, off, 64); near_row |= __shfl_xor(near_row, off, 64); }
    }
    if ((tid & 63) == 0) {
        s_max[0][tid >> 6] = vabs;
        s_max[1][tid >> 6] = n2max;
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
    if (tid < 2) {
        // mode 0 prepares the slot that mode 1 reads, mode 1 the one the first step reads
        SplitState *dst = MODE == 0 ? st_now : st_next;
        unsigned *at = tid == 0 ? &dst->vabs : &dst->n2;
        const unsigned v = max(max(s_max[tid][0], s_max[tid][1]), max(s_max[tid][2], s_max[tid][3]));
        if (u.blocks == 1) *at = v;
        else atomicMax(at, v);
    }
    if (STEP && !INV_COUNT && u.send && blk == 0 && tid == 0) {
        for (int n = 0; n < p.nb; ++n) {
            const int peer = peer_of(n);
            if (peer >= 0) p.stamp[exchange_buffer(u.send_parity, p.nb, n, p.W, peer)] = u.round;
        }
        p.counters[(size_t)i * CNT_STRIDE + CNT_SENT] += 1;
    }
}

}  // namespace

// ---- host side ----
bool split_kernel_supports(int k, int d, int b) { return k >= 2 && k <= 8192 && d <= 8192 && b <= (1 << 20); }

namespace {

struct SplitPlan {
    int nch, dpad, nblk, kpad, npair;
    size_t frag_bytes;
    bool longrow, fused, resident;
    int waves, shares, share_len;
    unsigned off_cells, off_cnt, off_hs, off_ms, off_args, lds;
    int dc, ncol, sum_shares, sum_len;      // sums in a launch of their own: columns per workgroup, shares
    unsigned lds_sums;
    int g, upd_blocks;             // update: lanes per row, workgroups per worker
};

unsigned round16(size_t v) { return (unsigned)((v + 15) / 16 * 16); }

SplitPlan make_plan(const StepParams &p)
{
    SplitPlan q;
    memset(&q, 0, sizeof(q));
    q.longrow = p.d > 128;
    q.dpad = q.longrow ? (p.d + 127) / 128 * 128 : (p.d + 15) / 16 * 16;
    q.nch = q.dpad / 16;
    q.nblk = (p.k + 31) / 32;
    q.npair = (q.nblk + 1) / 2;
    q.kpad = q.npair * 64;
    q.frag_bytes = (size_t)q.npair * q.nch * 4 * SPLIT_PIECE;
    const size_t cells = (size_t)p.k * p.d * sizeof(u64) + (size_t)p.k * sizeof(int);
    const size_t fixed = (size_t)q.kpad * 4 + (size_t)q.dpad * 4 + 8 * 64 * 4 + 64;
    const size_t stage2 = q.longrow ? 2 * SPLIT_STAGE : (size_t)2 * q.nch * 4 * SPLIT_PIECE;
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
    unsigned o = round16(q.resident ? q.frag_bytes : stage2);
    q.off_cells = o;
    if (q.fused) o += round16((size_t)p.k * p.d * sizeof(u64));
    q.off_cnt = o;
    if (q.fused) o += round16((size_t)p.k * sizeof(int));
    q.off_hs = o;  o += round16((size_t)q.kpad * 4);
    q.off_ms = o;  o += round16((size_t)q.dpad * 4);
    q.off_args = o; o += 8 * 64 * 4;
    q.lds = o;
    // waves of a workgroup and shares of a mini-batch: enough workgroups for the 256 compute units first, then as
    // many waves per workgroup as share the staged operands
    const int groups = (p.b + 63) / 64;
    int nw = q.lds <= 50 * 1024 ? 4 : 8;
    while (nw > 1 && (long long)p.W * ((groups + nw - 1) / nw) < 256) nw /= 2;
    q.waves = nw;
    const int max_shares = (groups + nw - 1) / nw;
    // (two waves per SIMD at more than 32 columns, three up to 32: as many workgroups as are resident at once)
    const int want = 256 * (q.nch <= 2 && q.lds <= 50 * 1024 ? 12 : 8) / nw;
    int shares = (want + p.W - 1) / p.W;
    if (shares > max_shares) shares = max_shares;
    if (shares > 64) shares = 64;
    q.share_len = (groups + shares - 1) / shares * 64;
    q.shares = (p.b + q.share_len - 1) / q.share_len;
    if (!q.fused) {
        int dc = 64;
        while (dc > 8 && (size_t)p.k * (dc * 8 + 4) > 72 * 1024) dc /= 2;
        while (dc > 1 && (size_t)p.k * (dc * 8 + 4) > SPLIT_LDS) dc /= 2;
        q.dc = dc;
        q.ncol = (p.d + dc - 1) / dc;
        q.lds_sums = round16((size_t)p.k * (dc * 8 + 4));
        // (every share writes and the update reads the sums of a whole state: no more than fill the device)
        int ss = 512 / (p.W * q.ncol);
        if (ss > groups / 8) ss = groups / 8;
        if (ss < 1) ss = 1;
        q.sum_len = (groups + ss - 1) / ss * 64;
        q.sum_shares = (p.b + q.sum_len - 1) / q.sum_len;
    } else {
        q.sum_shares = q.shares;
        q.sum_len = q.share_len;
    }
    int g = 1;
    while (g < q.dpad / 8 && g < 64) g *= 2;
    q.g = g;
    // workgroups of 256 threads per worker: enough for four on every compute unit, as long as each has rows to do
    q.upd_blocks = (1024 + p.W - 1) / p.W;
    const int row_groups = (p.k + 256 / g - 1) / (256 / g);
    if (q.upd_blocks > row_groups) q.upd_blocks = row_groups;
    return q;
}

struct Scratch { size_t frag, hs, state, gate, mail, m, ms, xmeta, colscale, part, cntpart, idx, bytes; };
Scratch scratch_layout(const StepParams &p, const SplitPlan &q)
{
    Scratch s;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) / 256 * 256; return at; };
    s.frag = take(q.frag_bytes * p.W);
    s.hs = take((size_t)q.kpad * p.W * 4);
    s.state = take((size_t)3 * p.W * sizeof(SplitState));
    s.gate = take((size_t)p.W * p.nb * q.upd_blocks * sizeof(SplitGate));
    s.mail = take((size_t)p.W * sizeof(SplitMail));
    s.m = take((size_t)p.d * 4);
    s.ms = take((size_t)q.dpad * 4);
    s.xmeta = take(16);
    s.colscale = take((size_t)p.d * 16);
    s.part = take((size_t)q.sum_shares * p.W * p.k * p.d * 4);
    s.cntpart = take((size_t)q.sum_shares * p.W * p.k * 4);
    s.idx = take(q.fused ? 0 : (size_t)p.W * p.b * 4);
    s.bytes = o;
    return s;
}

}  // namespace

size_t split_scratch_bytes(const StepParams &p) { return scratch_layout(p, make_plan(p)).bytes; }

hipError_t launch_split_steps(const StepParams &p, long long t0, long long t1, void *scratch, hipStream_t s, int *launches)
{
    const SplitPlan q = make_plan(p);
    const Scratch l = scratch_layout(p, q);
    unsigned char *base = static_cast<unsigned char *>(scratch);
    SplitArgs a;
    memset(&a, 0, sizeof(a));
    a.x = p.x; a.w = p.w;
    a.frag = base + l.frag; a.frag_bytes = q.frag_bytes;
    a.hs = (float *)(base + l.hs);
    a.ms = (float *)(base + l.ms); a.xmeta = (float *)(base + l.xmeta); a.colscale = (double *)(base + l.colscale);
    a.part = (float *)(base + l.part); a.cntpart = (int *)(base + l.cntpart);
    a.idx = q.fused ? nullptr : (int *)(base + l.idx);
    a.counters = p.counters;
    a.H = p.H;
    a.k = p.k; a.d = p.d; a.b = p.b; a.W = p.W; a.kpad = q.kpad; a.nblk = q.nblk; a.dpad = q.dpad;
    a.shares = q.shares; a.share_len = q.share_len; a.resident = q.resident; a.fused = q.fused;
    a.vec4 = p.d % 4 == 0 && ((uintptr_t)p.x & 15u) == 0;
    a.off_cells = q.off_cells; a.off_cnt = q.off_cnt; a.off_hs = q.off_hs; a.off_ms = q.off_ms; a.off_args = q.off_args;
    SplitUpdate u;
    u.frag = base + l.frag; u.hs = (float *)(base + l.hs);
    u.state = (SplitState *)(base + l.state); u.gate = (SplitGate *)(base + l.gate); u.mail = (SplitMail *)(base + l.mail);
    u.m = (float *)(base + l.m); u.xmeta = a.xmeta; u.part = a.part; u.cntpart = a.cntpart;
    u.frag_bytes = q.frag_bytes; u.kpad = q.kpad; u.dpad = q.dpad; u.shares = q.sum_shares; u.g = q.g; u.blocks = q.upd_blocks;

    hipLaunchKernelGGL(split_middle_kernel, dim3((p.d + 63) / 64), dim3(1024), 0, s, p.x, p.H * p.W, p.d, (float *)(base + l.m));
    hipLaunchKernelGGL(split_scales_kernel, dim3(1), dim3(256), 0, s, p.xabsmax, (float *)(base + l.m), p.d, q.dpad, p.b,
                       (float *)(base + l.ms), (float *)(base + l.xmeta), (double *)(base + l.colscale));
    hipError_t e = hipMemsetAsync(u.state, 0, (size_t)3 * p.W * sizeof(SplitState), s);
    if (e != hipSuccess) return e;
    auto set_slot = [&](int slot) { u.slot = slot; u.slot_next = (slot + 1) % 3; u.slot_after = (slot + 2) % 3; };
    const int det = p.mode == ASGD_MODE_DETERMINISTIC;
    u.merge = u.send = u.round = u.read_parity = u.send_parity = 0;
    set_slot(0);
    const dim3 upd_grid(p.W * q.upd_blocks);
    hipLaunchKernelGGL(split_update_kernel<0>, upd_grid, dim3(256), 0, s, p, u);
    hipLaunchKernelGGL(split_update_kernel<1>, upd_grid, dim3(256), 0, s, p, u);
    *launches += 4;
    e = hipGetLastError();
    if (e == hipSuccess && q.longrow)
        e = hipFuncSetAttribute((const void *)split_assign_long_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)q.lds);
    if (e == hipSuccess && !q.fused)
        e = hipFuncSetAttribute((const void *)split_sums_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)q.lds_sums);
    for (long long t = t0; t < t1 && e == hipSuccess; ++t) {
        set_slot((int)((1 + (t - t0)) % 3));
        if (p.E > 0) {
            const long long r = t / p.E;
            u.round = (int)r;
            u.merge = t > 0 && t % p.E == 0;
            u.send = p.W > 1 && (t + 1) % p.E == 0;
            u.read_parity = det ? (int)((r - 1) & 1) : 0;
            u.send_parity = det ? (int)(r & 1) : 0;
            for (int n = 0; n < MAX_BUFFERS; ++n) u.shift[n] = u.send && n < p.nb ? shift_deterministic(p.seed, r, p.W, n) : 0;
        }
        a.state = u.state + (size_t)u.slot * p.W;
        a.row0 = (t % p.S) * p.b;
        a.dump = p.dump ? p.dump + (size_t)(t - p.t_dump0) * p.W * p.b : nullptr;
        const int blocks = p.W * q.shares, threads = 64 * q.waves;
        if (q.longrow) {
            hipLaunchKernelGGL(split_assign_long_kernel, dim3(blocks), dim3(threads), q.lds, s, a);
            e = hipGetLastError();
        } else {
            switch (q.nch) {
                case 1: e = launch_split_assign_1(a, blocks, threads, q.lds, s); break;
                case 2: e = launch_split_assign_2(a, blocks, threads, q.lds, s); break;
                case 3: e = launch_split_assign_3(a, blocks, threads, q.lds, s); break;
                case 4: e = launch_split_assign_4(a, blocks, threads, q.lds, s); break;
                case 5: e = launch_split_assign_5(a, blocks, threads, q.lds, s); break;
                case 6: e = launch_split_assign_6(a, blocks, threads, q.lds, s); break;
                case 7: e = launch_split_assign_7(a, blocks, threads, q.lds, s); break;
                default: e = launch_split_assign_8(a, blocks, threads, q.lds, s); break;
            }
        }
        if (e != hipSuccess) break;
        if (!q.fused) {
            SplitArgs as = a;
            as.shares = q.sum_shares;
            as.share_len = q.sum_len;
            hipLaunchKernelGGL(split_sums_kernel, dim3(p.W * q.sum_shares * q.ncol), dim3(512), q.lds_sums, s, as, q.dc, q.ncol);
            ++*launches;
        }
        if (u.merge) {
            hipLaunchKernelGGL(split_gate_kernel, upd_grid, dim3(256), 0, s, p, u);
            ++*launches;
        }
        if (p.lr_mode == ASGD_LR_INV_COUNT) hipLaunchKernelGGL(split_update_kernel<3>, upd_grid, dim3(256), 0, s, p, u);
        else if (p.parts > 1) hipLaunchKernelGGL(split_update_kernel<4>, upd_grid, dim3(256), 0, s, p, u);
        else hipLaunchKernelGGL(split_update_kernel<2>, upd_grid, dim3(256), 0, s, p, u);
        *launches += 2;
        e = hipGetLastError();
    }
    return e;
}

}  // namespace asgd
