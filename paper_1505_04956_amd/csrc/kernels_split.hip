// Step kernel for any row length, host side: preparation of a call, sizes of the work items, launch.
#include <string.h>

#include "split_quant_screen.h"
#include "split_steps.h"

namespace asgd {

hipError_t launch_split_quant_0(const SplitQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_split_quant_1(const SplitQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_1(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_2(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_3(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_4(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_5(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_6(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_7(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_screen_quant_8(const ScreenQuant &a, int blocks, unsigned lds, hipStream_t s);
hipError_t launch_split_local_0(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_0(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_1(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_1(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_2(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_2(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_3(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_3(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_4(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_4(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_5(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_5(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_6(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_6(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_7(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_7(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_local_8(const SplitRun &r, int blocks, int threads, unsigned lds, hipStream_t s);
hipError_t launch_split_assign_8(const SplitLaunch &l, int blocks, int threads, unsigned lds, hipStream_t s);


namespace {

constexpr int SPLIT_SAMPLE_ROWS = 1024;     // rows looked at for the middle of the data

// ---- once per set of samples: middle of the data, scale of the samples, scales of the fixed-point sums ----
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
        for (int u = 0; u < 8; ++u) s += q0 + 16 * u < n ? v[u] * (1.0f / (float)n) : 0.0f;     // (the sum could overflow)
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && j < d) {
        s = 0.0f;
        for (int q = 0; q < 16; ++q) s += red[q][lane];
        m[j] = s;
    }
}
// sx: power of two with max_j (max|x_j| + |m_j|) * sx in [2^13, 2^14); ms = -m * sx; scale of column j of the sums: 2^e
// with max|x_j| 2^e < 2^50 and b max|x_j| 2^e < 2^62
__global__ void split_scales_kernel(const float *xabsmax, float *m, int d, int dpad, int b, float *ms, float *xmeta, double *colscale)
{
    __shared__ float red[256];
    const int tid = threadIdx.x;
    float a = 0.0f;
    for (int j = tid; j < d; j += 256) a = fmaxf(a, fminf(xabsmax[j] + fabsf(m[j]), 3.4e38f));
    red[tid] = a;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (tid < off) red[tid] = fmaxf(red[tid], red[tid + off]);
        __syncthreads();
    }
    int q = 0;
    if (red[0] > 0.0f) (void)frexpf(red[0], &q);
    const float sx = ldexpf(1.0f, max(-120, min(126, 14 - q)));
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

}  // namespace

// ---- host side ----
// (k: the cells of one column and the counts have to fit the LDS, 20 bytes a centroid; d: the middle of the data by slot)
bool split_kernel_supports(int k, int d, int b) { return k >= 2 && k <= 7680 && d <= 8192 && b <= (1 << 20); }

namespace {

// What depends on the samples only, computed once after they are loaded.
struct Data { size_t m, ms, xmeta, colscale, bytes; };
Data data_layout(int d)
{
    Data s;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) / 256 * 256; return at; };
    s.m = take((size_t)d * 4);
    s.ms = take((size_t)split_padded_row(d) * 4);
    s.xmeta = take(16);
    s.colscale = take((size_t)d * 16);
    s.bytes = o;
    return s;
}

struct Scratch { size_t frag, hs, state, arrived, gate, mail, part, cntpart, idx, bytes; };
Scratch scratch_layout(const StepParams &p, const SplitPlan &q)
{
    Scratch s;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) / 256 * 256; return at; };
    s.frag = take(q.frag_bytes * p.W);
    s.hs = take((size_t)q.kpad * p.W * 4);
    s.state = take((size_t)3 * p.W * sizeof(SplitState));
    s.arrived = take(sizeof(int));            // (cleared with the states before it)
    s.gate = take((size_t)p.W * p.nb * q.upd_blocks * sizeof(SplitGate));
    s.mail = take((size_t)p.W * sizeof(SplitMail));
    s.part = take((size_t)q.sum_shares * p.W * p.k * p.d * 4);
    s.cntpart = take((size_t)q.sum_shares * p.W * p.k * 4);
    s.idx = take(q.fused ? 0 : (size_t)p.W * p.b * 4);
    s.bytes = o;
    return s;
}

}  // namespace

// Kept workers: what a step needs besides messages is in the LDS when it begins, and it never needs a launch, also
// with a message every step.  Microseconds per step of long calls, W = 256 (phases where E < 4, else the local form that is not kept; kept): k = 12,
// d = 7: b = 100, E = 0 15.0, 11.2; b = 500, E = 0 17.5, 13.5; E = 2 26.5, 18.4; b = 2000, E = 4 52.9, 30.7; k = 64, d = 32, b = 500, E = 1 33.4, 24.6;
// k = 100, d = 60, b = 120, E = 1 45.9, 37.5; k = 500, d = 8, b = 256, E = 1 47.5, 37.0; k = 400, d = 10, b = 1000, E = 2 59.6, 47.5.
// (Where they do not fill the device, phases cut their mini-batches: k = 12, d = 7, b = 2000, W = 32 24.9, 29.6.)
static bool split_kept(const StepParams &p)
{
    return p.parts == 1 && !p.phases_only && 4LL * p.W >= 3LL * SPLIT_CUS && split_plan(p.k, p.d, p.b, p.W, true).kept;
}

// Local form: kept workers, or workers that fill the device, one workgroup of eight waves each
// (three quarters of them at least: fewer are better off with phases, which cut their mini-batches), and exchange every fourth step
// at most (every message costs its sender a write-back and its recipient an invalidation of the L2, which phases get from the end
// of a launch: k = 64, d = 32, b = 500, E = 1: 105 us per step local, 33 us in phases).  Two rounds of workers and more take longer
// than phases (512 workers, E = 8: k = 12, d = 8, b = 600: 47 us per step local, 34 in phases; k = d = 100, b = 2000, ten epochs a
// call: 245 and 227): only for the caller that promises one launch per call (the matrix-core kernel: asgd_run_epochs()).
bool split_local_form(const StepParams &p)
{
    const int rounds = (p.W + SPLIT_CUS - 1) / SPLIT_CUS;
    int dev = 0, cus = 0;                  // (a partition of a device may have fewer compute units: not resident at once)
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    const bool exchange = p.E > 0 && p.W > 1;
    if (p.phases_only || cus < SPLIT_CUS || p.parts > 1 || (exchange && p.mode != ASGD_MODE_DETERMINISTIC)) return false;
    return split_kept(p) || (4LL * p.W >= 3LL * rounds * SPLIT_CUS && (rounds == 1 || p.one_launch) && (!exchange || p.E >= 4));
}

size_t split_scratch_bytes(const StepParams &p) { return scratch_layout(p, split_plan(p.k, p.d, p.b, p.W, split_local_form(p))).bytes; }

size_t split_data_bytes(int d) { return data_layout(d).bytes; }

hipError_t launch_split_data(const StepParams &p, void *data, hipStream_t s)
{
    const Data l = data_layout(p.d);
    unsigned char *base = static_cast<unsigned char *>(data);
    hipLaunchKernelGGL(split_middle_kernel, dim3((p.d + 63) / 64), dim3(1024), 0, s, p.x, p.H * p.W, p.d, (float *)(base + l.m));
    hipLaunchKernelGGL(split_scales_kernel, dim3(1), dim3(256), 0, s, p.xabsmax, (float *)(base + l.m), p.d, split_padded_row(p.d), p.b,
                       (float *)(base + l.ms), (float *)(base + l.xmeta), (double *)(base + l.colscale));
    return hipGetLastError();
}

hipError_t launch_split_steps(const StepParams &p, long long t0, long long t1, const void *data, void *scratch, hipStream_t s, int *launches)
{
    const bool local = split_local_form(p);
    const SplitPlan q = split_plan(p.k, p.d, p.b, p.W, local);
    const Scratch l = scratch_layout(p, q);
    unsigned char *base = static_cast<unsigned char *>(scratch);
    SplitArgs a;
    memset(&a, 0, sizeof(a));
    a.x = p.x; a.w = p.w;
    a.frag = base + l.frag; a.frag_bytes = q.frag_bytes;
    a.hs = (float *)(base + l.hs);
    const Data dl = data_layout(p.d);
    const unsigned char *from = static_cast<const unsigned char *>(data);
    a.ms = (const float *)(from + dl.ms); a.xmeta = (const float *)(from + dl.xmeta); a.colscale = (const double *)(from + dl.colscale);
    a.part = (float *)(base + l.part); a.cntpart = (int *)(base + l.cntpart);
    a.idx = q.fused ? nullptr : (int *)(base + l.idx);
    a.counters = p.counters;
    a.H = p.H;
    a.k = p.k; a.d = p.d; a.b = p.b; a.W = p.W; a.kpad = q.kpad; a.nblk = q.nblk; a.dpad = q.dpad;
    a.shares = q.shares; a.share_len = q.share_len; a.sum_shares = q.sum_shares; a.sum_len = q.sum_len;
    a.dc = q.dc; a.ncol = q.ncol; a.resident = q.resident; a.fused = q.fused; a.wide = q.wide;
    a.vec4 = p.d % 4 == 0 && ((uintptr_t)p.x & 15u) == 0;
    a.kept = q.kept; a.off_batch = q.off_batch; a.batch_bytes = q.batch_bytes;
    a.off_cells = q.off_cells; a.off_cnt = q.off_cnt; a.off_hs = q.off_hs; a.off_ms = q.off_ms; a.off_args = q.off_args;
    a.stage_pairs = q.stage_pairs; a.stages = q.stages; a.off_list = q.off_list;
    SplitUpdate u;
    u.frag = base + l.frag; u.hs = (float *)(base + l.hs);
    u.state = (SplitState *)(base + l.state); u.gate = (SplitGate *)(base + l.gate); u.mail = (SplitMail *)(base + l.mail);
    u.m = (const float *)(from + dl.m); u.xmeta = a.xmeta; u.part = a.part; u.cntpart = a.cntpart;
    u.frag_bytes = q.frag_bytes; u.kpad = q.kpad; u.dpad = q.dpad; u.shares = q.sum_shares; u.g = q.g; u.blocks = q.upd_blocks;

    hipError_t e = hipMemsetAsync(base + l.state, 0, l.gate - l.state, s);
    if (e != hipSuccess) return e;
    SplitLaunch l2;
    memset(&l2, 0, sizeof(l2));
    SplitRun &r = l2.run;
    r.p = p; r.a = a; r.u = u;
    const int det = p.mode == ASGD_MODE_DETERMINISTIC;
    if (local) {
        r.t0 = t0; r.t1 = t1;
        r.round0 = p.E > 0 ? t0 / p.E : 0;
        r.te0 = p.E > 0 ? (int)(t0 % p.E) : 0;
        r.sync = det && p.E > 0 && p.W > 1 && !p.no_waits;
        r.arrived = (int *)(base + l.arrived);
        r.expected = q.grid + (p.refuse_one_launch == 2 ? 1 : 0);            // (test hook: one that never comes)
        // A round of a neighbour: E steps of all its workers, of which every sample may have to be decided in fp64 against all
        // centroids.  That was measured at up to 0.3 ns per element of b k d (1.2 where k d is small next to the 8 us of
        // a step); four times as much is allowed.
        const double step = 4e-3 * p.b * (double)p.k * p.d + 4096.0;
        const double polls = (double)(1 << 18) + step * (double)p.E * ((p.W + q.grid - 1) / q.grid);
        r.wait_polls = (int)(polls < (double)(1 << 29) ? polls : (double)(1 << 29));
        switch (q.longrow ? 0 : q.nch) {
            case 0: e = launch_split_local_0(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 1: e = launch_split_local_1(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 2: e = launch_split_local_2(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 3: e = launch_split_local_3(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 4: e = launch_split_local_4(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 5: e = launch_split_local_5(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 6: e = launch_split_local_6(r, q.grid, 64 * q.waves, q.lds, s); break;
            case 7: e = launch_split_local_7(r, q.grid, 64 * q.waves, q.lds, s); break;
            default: e = launch_split_local_8(r, q.grid, 64 * q.waves, q.lds, s); break;
        }
        *launches += 1;
        return e;
    }
    SplitStep &now = l2.now;
    auto set_slot = [&](int slot) { now.slot = slot; now.slot_next = (slot + 1) % 3; now.slot_after = (slot + 2) % 3; };
    const int upd = p.W * q.upd_blocks;
    const unsigned small_lds = SPLIT_LDS_SHARED;
    set_slot(0);
    e = split_launch_phase<0>(l2, upd, 256, small_lds, s);
    if (e == hipSuccess) e = split_launch_phase<1>(l2, upd, 256, small_lds, s);
    *launches += 2;
    for (long long t = t0; t < t1 && e == hipSuccess; ++t) {
        set_slot((int)((1 + (t - t0)) % 3));
        if (p.E > 0) {
            const long long rd = t / p.E;
            now.round = (int)rd;
            now.merge = t > 0 && t % p.E == 0;
            now.send = p.W > 1 && (t + 1) % p.E == 0;
            now.read_parity = det ? (int)((rd - 1) & 1) : 0;
            now.send_parity = det ? (int)(rd & 1) : 0;
            for (int n = 0; n < MAX_BUFFERS; ++n) now.shift[n] = now.send && n < p.nb ? shift_deterministic(p.seed, rd, p.W, n) : 0;
        }
        now.state = u.state + (size_t)now.slot * p.W;
        now.row0 = (t % p.S) * p.b;
        now.dump = p.dump ? p.dump + (size_t)(t - p.t_dump0) * p.W * p.b : nullptr;
        switch (q.longrow ? 0 : q.nch) {
            case 0: e = launch_split_assign_0(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 1: e = launch_split_assign_1(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 2: e = launch_split_assign_2(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 3: e = launch_split_assign_3(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 4: e = launch_split_assign_4(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 5: e = launch_split_assign_5(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 6: e = launch_split_assign_6(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            case 7: e = launch_split_assign_7(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
            default: e = launch_split_assign_8(l2, p.W * q.shares, 64 * q.waves, q.lds, s); break;
        }
        ++*launches;
        if (e == hipSuccess && !q.fused) {
            e = split_launch_phase<6>(l2, p.W * q.sum_shares * q.ncol, SPLIT_THREADS, q.lds_sums, s);
            ++*launches;
        }
        if (e == hipSuccess && now.merge) {
            e = split_launch_phase<5>(l2, upd, 256, small_lds, s);
            ++*launches;
        }
        if (e != hipSuccess) break;
        if (p.lr_mode == ASGD_LR_INV_COUNT) e = split_launch_phase<3>(l2, upd, 256, small_lds, s);
        else if (p.parts > 1) e = split_launch_phase<4>(l2, upd, 256, small_lds, s);
        else e = split_launch_phase<2>(l2, upd, 256, small_lds, s);
        ++*launches;
    }
    return e;
}

// ---- Eq. 8 ----
bool split_quant_supports(int k, int d) { return k >= 2 && k <= 8192 && d <= 8192; }

// One workgroup per pair of row blocks.  As the start of split_quant_kernel: m from nine rows, the scale of the state from the middle
// of their sizes, h_c = -|v_c|^2/2 in scaled units, rows 2^10 times as large left out.
__global__ __launch_bounds__(SPLITQ_THREADS) void splitq_operands_kernel(ScreenQuant a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ float most_of[16], red[4][8];
    float *m = reinterpret_cast<float *>(smem);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int k = a.q.k, d = a.q.d, dpad = a.q.dpad, nch = dpad / 16;
    const float *w = a.q.w;
    // this workgroup's rows, sixteen lanes per row at most, so twice 32 of them at most
    int g = 1;
    while (g < dpad / 8) g *= 2;
    const int lane_g = tid & (g - 1), slot = 8 * lane_g;
    float raw[2][8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c = min((int)blockIdx.x * 64 + tid / g + q * (SPLITQ_THREADS / g), k - 1);
        split_load8<true>(raw[q], w + (size_t)c * d, slot < d ? slot : 0, d);
    }
    for (int j = tid; j < dpad; j += SPLITQ_THREADS) {
        const float mid = splitq_middle_of(w, k, d, j);
        m[j] = mid;
        if (blockIdx.x == 0) a.m[j] = mid;
    }
    __syncthreads();
    auto size_of = [&](float v, int slot) { return __float_as_uint(v - m[slot]) & 0x7fffffffu; };
    auto largest = [&](unsigned v) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, 64));
        return __uint_as_float(min(v, 0x7f800000u));
    };
    // largest |v_cj| of the nine rows, and the largest finite one of SCREENQ_ROWS samples; all loads of a wave in flight (one row after the
    // other: 8 us of 17)
    constexpr int ROWS = SCREENQ_ROWS / 8;
    float nine[9], typical, far = 0.0f;
    {
        unsigned own = 0, last = 0;
        for (int slot = lane; slot < dpad; slot += 64) {
            if (!split_slot_used(slot, d)) continue;
            const int j = split_column(slot, d);
            float xv[ROWS];
            const float wv = w[(size_t)(wave * k / 9) * d + j], w8 = w[(size_t)(8 * k / 9) * d + j];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) xv[r] = a.q.x[(size_t)((8 * r + wave) * a.q.N / SCREENQ_ROWS) * d + j];
            own = max(own, size_of(wv, slot));
            last = max(last, size_of(w8, slot));
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const float v = __uint_as_float(size_of(xv[r], slot));
                if (v < INFINITY) far = fmaxf(far, v);
            }
        }
        const float own_most = largest(own), last_most = largest(last), far_most = largest(__float_as_uint(far));
        if (lane == 0) {
            most_of[wave] = own_most;
            if (wave == 0) most_of[8] = last_most;
            red[0][wave] = far_most;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 9; ++r) nine[r] = most_of[r];
    typical = splitq_middle(nine);
#pragma unroll
    for (int r = 0; r < 8; ++r) far = fmaxf(far, red[0][r]);
    __syncthreads();
    if (!(typical > 0.0f && typical < INFINITY)) {
        // (at m itself: the largest of all the rows)
        float most = 0.0f;
        for (int c = wave; c < k; c += 8) {
            unsigned row = 0;
            for (int slot = lane; slot < dpad; slot += 64)
                if (split_slot_used(slot, d)) row = max(row, size_of(w[(size_t)c * d + split_column(slot, d)], slot));
            const float v = largest(row);
            if (v < INFINITY) most = fmaxf(most, v);
        }
        if (lane == 0) red[0][wave] = most;
        __syncthreads();
        typical = 0.0f;
#pragma unroll
        for (int r = 0; r < 8; ++r) typical = fmaxf(typical, red[0][r]);
        __syncthreads();
    }
    const int sw_exp = splitq_exponent(typical, SPLITQ_TYPICAL);
    const float sw = ldexpf(1.0f, sw_exp);
    if (blockIdx.x == 0 && tid == 0) {
        const int e = splitq_exponent(far, SCREENQ_SAMPLE), r = far > 0.0f ? min(e - sw_exp, SPLITQ_RATIO_MAX) : 0;
        ScreenqHead h;
        h.sw = sw; h.sw_exp = sw_exp;
        h.ratio = ldexpf(1.0f, max(r, SPLITQ_RATIO_MIN));
        h.direct = r < SPLITQ_RATIO_MIN || r + sw_exp < -126 || r + sw_exp > 126 ? 1.0f : 0.0f;
        *reinterpret_cast<ScreenqHead *>(a.head) = h;
    }
    float vmin = INFINITY, vmax = 0.0f, vfar = INFINITY, rest = 0.0f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int c0 = tid / g + q * (SPLITQ_THREADS / g), c = blockIdx.x * 64 + c0;
        if (c0 >= 64) continue;                               // (the same for all lanes of a row)
        float v[8], sq = 0.0f, r2 = 0.0f;
        unsigned vb = 0;
        half8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c < k && slot < d && split_slot_used(slot + e, d) ? raw[q][e] - m[slot + e] : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = slot < dpad ? v[e] * sw : 0.0f;
            sq = fmaf(y, y, sq);
            vb = max(vb, slot < dpad ? __float_as_uint(v[e]) & 0x7fffffffu : 0u);
            hi[e] = (_Float16)y;
            const float left = y - (float)hi[e];
            lo[e] = (_Float16)left;
            r2 = fmaf(left, left, r2);
        }
        for (int off = g / 2; off > 0; off >>= 1) {
            sq += __shfl_xor(sq, off, 64);
            r2 += __shfl_xor(r2, off, 64);
            vb = max(vb, (unsigned)__shfl_xor((int)vb, off, 64));
        }
        const float most = __uint_as_float(min(vb, 0x7f800000u));
        const bool scored = c < k && most * sw < (float)(1 << SPLITQ_LIMIT);
        if (!scored) {
#pragma unroll
            for (int e = 0; e < 8; ++e) hi[e] = lo[e] = (_Float16)0.0f;
        }
        if (slot < dpad) {
            const size_t at = ((((size_t)blockIdx.x * nch + (slot >> 4)) * 2 + (c0 >> 5)) * 64 + (c0 & 31) + 32 * ((slot >> 3) & 1)) * 16;
            *reinterpret_cast<half8 *>(a.hi + at) = hi;
            *reinterpret_cast<half8 *>(a.lo + at) = lo;
        }
        if (lane_g == 0) a.hs[c] = scored ? -0.5f * sq : SPLIT_PAD_SCORE;
        if (scored) {
            vmin = fminf(vmin, sq);
            vmax = fmaxf(vmax, sq);
            rest = fmaxf(rest, r2);
        } else if (c < k && most < INFINITY) {
            vfar = fminf(vfar, sq < 1.0e37f ? sq : 1.0e37f);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        vmin = fminf(vmin, __shfl_xor(vmin, off, 64));
        vmax = fmaxf(vmax, __shfl_xor(vmax, off, 64));
        vfar = fminf(vfar, __shfl_xor(vfar, off, 64));
        rest = fmaxf(rest, __shfl_xor(rest, off, 64));
    }
    if (lane == 0) { red[0][wave] = vmin; red[1][wave] = vmax; red[2][wave] = vfar; red[3][wave] = rest; }
    __syncthreads();
    if (tid < 4) {
        float v = red[tid][0];
        for (int r = 1; r < 8; ++r) v = (tid & 1) ? fmaxf(v, red[tid][r]) : fminf(v, red[tid][r]);
        a.sizes[4 * blockIdx.x + tid] = v;
    }
}

// Screening for rows of 8 to 128 columns, whatever k is (the operands of a state, that is; see also launch_quant_error_split); microseconds with
// three products for all samples, and screened: 4e6 samples, k = 12, d = 9: 164, 100; k = 37, d = 75: 529, 333; k = 1000, d = 9: 917, 515; k =
// 1000, d = 32: 1040, 546; k = 100, d = 20: 303, 181; 2e6 samples, k = 512, d = 128: 1227, 478; 20000 samples, k = 512, d = 125: 105, 38.  Also
// where prototypes lie close together and many samples stay undecided (k = 1000, d = 9, sigma 0.3: 886, 439).  Shorter rows are loaded one by one,
// longer ones do not fit the registers.
static bool quant_screens(int k, int d) { return split_quant_supports(k, d) && d >= 8 && d <= 128; }
struct QuantOperands { size_t head, m, sizes, hs, hi, lo, bytes; };
static QuantOperands quant_operands(int k, int d)
{
    const size_t npair = (size_t)(k + 63) / 64, dpad = split_padded_row(d);
    QuantOperands l;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) / 256 * 256; return at; };
    l.head = take(sizeof(ScreenqHead));
    l.m = take(dpad * 4);
    l.sizes = take(npair * 16);
    l.hs = take(npair * 64 * 4);
    l.hi = take(npair * 64 * dpad * 2);
    l.lo = take(npair * 64 * dpad * 2);
    l.bytes = o;
    return l;
}
size_t quant_operand_bytes(int k, int d) { return quant_screens(k, d) ? quant_operands(k, d).bytes : 0; }

hipError_t launch_quant_error_split(const float *x, long long N, int d, int k, const float *w, double *partials, void *operands, int *nblocks_out,
                                    bool nan_is_inf, hipStream_t s)
{
    SplitQuant a;
    a.x = x; a.w = w; a.N = N; a.partials = partials; a.k = k; a.d = d;
    a.dpad = split_padded_row(d);
    a.nblk = (k + 31) / 32;
    const int npair = (a.nblk + 1) / 2, chunks = d > 128 ? 8 : a.dpad / 16, nblocks = SPLIT_CUS;
    *nblocks_out = nblocks;                       // one workgroup per compute unit
    a.kpad = npair * 64;
    a.nan_is_inf = nan_is_inf;
    // (Short rows, few rows and samples: the launch for the state and a wave's pass over its few undecided samples do not pay.  Microseconds without
    // and with them: k = 100, d = 9: 20000 samples 19, 20, 120000 20, 22; k = 150 22, 23; k = 300 27, 26 and 28, 29; d = 16: k = 31, 120000 samples 17, 17;
    // k = 1000, 60000 samples 54, 47.  Longer rows: k = 31, d = 20: 1000 samples 17, 14, 120000 18, 16; k = 300, d = 32: 60000 samples 31, 19.  Data with many
    // undecided samples, one column a thousand times as wide as the others: k = 100, d = 9 61, 25; k = 4000, d = 32, 5000 samples 2720, 372, the fp32 matrix
    // kernel 254.)
    if (quant_screens(k, d) && !(d <= 16 && k < 300 && N <= 120000)) {
        ScreenQuant c;
        c.q = a;
        const QuantOperands l = quant_operands(k, d);
        unsigned char *base = static_cast<unsigned char *>(operands);
        c.head = (float *)(base + l.head); c.m = (float *)(base + l.m); c.sizes = (float *)(base + l.sizes); c.hs = (float *)(base + l.hs);
        c.hi = base + l.hi; c.lo = base + l.lo;
        hipLaunchKernelGGL(splitq_operands_kernel, dim3(npair), dim3(SPLITQ_THREADS), a.dpad * 4, s, c);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        unsigned o = split_round16((size_t)a.kpad * 4);
        c.off_ms = o; o += split_round16((size_t)a.dpad * 4);
        c.off_list = o; o += SCREENQ_WAVES * (SCREENQ_LIST * 4 + SCREENQ_QUEUE);
        c.off_stage = o = (o + 1023) / 1024 * 1024;
        const unsigned pair = chunks * 2 * SPLIT_PIECE;
        // The samples stay in the registers for their distances, with fewer tiles per wave, or come a second time: the first as long as the matrix
        // work is small next to the memory (microseconds kept and not, 2e6 samples; d = 128: k = 16 253, 320, 128 260, 309, 192 389, 374, 512 539, 478; d = 80:
        // k = 256 251, 269, 1024 491, 484; d = 64: k = 512 283, 276; up to 32 columns the tiles stay four: k = 1000, d = 20 534, 545).
        c.keep = chunks <= 2 || k <= (chunks <= 6 ? 384 : 160);
        c.pairs_per_stage = (int)((SPLIT_LDS_ALL / 2 - 256 - o) / (2 * pair));      // (at least one: 32 KB of offsets and 32 KB of operands at most)
        if (c.pairs_per_stage > npair) c.pairs_per_stage = npair;
        o += 2 * c.pairs_per_stage * pair;
        *nblocks_out = 2 * SPLIT_CUS;
        switch (chunks) {
            case 1: return launch_screen_quant_1(c, 2 * SPLIT_CUS, o, s);
            case 2: return launch_screen_quant_2(c, 2 * SPLIT_CUS, o, s);
            case 3: return launch_screen_quant_3(c, 2 * SPLIT_CUS, o, s);
            case 4: return launch_screen_quant_4(c, 2 * SPLIT_CUS, o, s);
            case 5: return launch_screen_quant_5(c, 2 * SPLIT_CUS, o, s);
            case 6: return launch_screen_quant_6(c, 2 * SPLIT_CUS, o, s);
            case 7: return launch_screen_quant_7(c, 2 * SPLIT_CUS, o, s);
            default: return launch_screen_quant_8(c, 2 * SPLIT_CUS, o, s);
        }
    }
    const size_t all = (size_t)npair * chunks * 4 * SPLIT_PIECE, two = (size_t)2 * chunks * 4 * SPLIT_PIECE;
    a.resident = d <= 128 && all + (size_t)(a.kpad + a.dpad) * 4 <= SPLIT_LDS;
    unsigned o = (unsigned)(a.resident ? all : two);
    a.off_hs = o; o += split_round16((size_t)a.kpad * 4);
    a.off_m = o;  o += split_round16((size_t)a.dpad * 4);
    return d > 128 ? launch_split_quant_0(a, nblocks, o, s) : launch_split_quant_1(a, nblocks, o, s);
}

}  // namespace asgd
