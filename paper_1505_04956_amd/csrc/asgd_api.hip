// Host side of the C ABI declared in asgd.h: argument checks, device memory of a context,
// splitting of a run into launches, timing, copies to and from the host.
#include <math.h>
#include <new>
#include <string.h>
#include <vector>

#include "asgd_internal.h"
#include "launch_cuts.h"

using namespace asgd;

struct asgd_ctx {
    int k = 0, d = 0, W = 0, b = 0;
    float lr = 0.f;
    int E = 0;
    uint64_t seed = 1;
    int mode = ASGD_MODE_DETERMINISTIC;
    int parzen = 1;
    int lr_mode = ASGD_LR_CONST;
    double drop_rate = 0.0;
    int kernel_opt = ASGD_KERNEL_AUTO;
    int tune = 0;
    int nb = 1;                 // external buffers per worker
    int parts = 1;              // partial messages: parts of a state (1 = whole states)
    size_t slot_bytes_one = 0;  // bytes of both parities of ONE buffer per worker
    int cooperative = 1;
    int wait_polls = 0;
    int drop_unannounced = 0;
    int refuse_one_launch = 0;

    int device = 0;
    hipStream_t stream = nullptr;
    bool loaded = false;
    const float *x = nullptr;
    long long N = 0, H = 0, S = 0;
    long long t = 0;

    float *w = nullptr, *slot = nullptr, *acc = nullptr, *xabsmax = nullptr, *mean = nullptr;
    SeenSteps seen;                // streaming kernel: mini-batches it has looked at (flag_host[3]: and met an element beyond the
                                   // limits it forms of xsample)
    int *marks = nullptr;          // ... and, once it has looked at all, which ones hold such an element, allocated on first use
    size_t marks_bytes = 0;
    int marks_state = 0;           // 0: not made for the loaded samples, 1: made, -1: cannot be
    bool xabsmax_valid = false;    // xabsmax and flag_host[1], [2] are those of the loaded samples
    float *xsample = nullptr;      // streaming kernel only: column maxima over a part of the samples, and scratch (behind qpart)
    bool xsample_clear = false;    // its counter of workgroups is zero
    float *xnorm2max = nullptr;    // matrix-core kernel only, allocated on first use
    size_t slot_bytes = 0;         // size of the exchange buffers (both parities, all workers)
    int *shift_tab = nullptr;      // schedule table of the small-state kernel, grown on demand
    long long shift_cap = 0;
    long long tab_r0 = 0, tab_n = 0;   // rounds [tab_r0, tab_r0 + tab_n) the table holds, for tab_seed and tab_W
    uint64_t tab_seed = 0;
    int tab_W = 0;
    bool xnorm2max_valid = false;
    int *stamp = nullptr, *consumed = nullptr, *cnt = nullptr, *assign_tmp = nullptr;
    // Error flag of the kernels (an expired bounded wait), in pinned host memory that the device writes directly: the
    // host clears and reads it around a run without a memset or a copy on the stream (each is a separate operation
    // of several microseconds, which counts when a run is one launch of less than a millisecond).
    int *flag_host = nullptr;      // [0] error flag; set while loading: [1] a sample is not finite, [2] a column's typical
                                   // element is far smaller than its largest
    void *split_scratch = nullptr; // matrix-core form of the shape-agnostic kernel, allocated on first use
    size_t split_bytes = 0;
    void *split_data = nullptr;    // what its kernels need to know of the samples, allocated on first use
    bool split_data_valid = false;
    void *load_scratch = nullptr;  // partial maxima of asgd_load_shards(), kept: taking 3 MB and giving them back was 80 us a call
    long long *ncum = nullptr, *counters = nullptr;
    double *qpart = nullptr, *qout = nullptr;
    int32_t *dump = nullptr;
    size_t dump_cap = 0;

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    double last_ms = 0.0;
    int last_kernel = 0, last_launches = 0, last_form = ASGD_FORM_NONE;
    long long passed_t = -1;    // step up to which `consumed` holds what a one-launch run needs (-1: unknown)
    int fill_kernel = 0;        // kernel whose message format the exchange buffers were last emptied for
    bool desynced = false;      // a bounded wait expired in the last run: states and buffers are not those of any step
    // messages handed over by asgd_set_exchange(), kept until the next run knows which kernel's format they take
    std::vector<float> pending_values;
    std::vector<int32_t> pending_rounds;
    bool pending = false;
    int hip_err = 0;
};

namespace {

// device memory the step kernels with fp16-split operands may take besides the context's own (a state's operands are
// padded to 64 rows and 16 columns, which for a great many tiny states is a multiple of their size)
constexpr size_t SPLIT_SCRATCH_MAX = (size_t)32 << 30;

#define HIP_TRY(ctx, call)                              \
    do {                                                \
        hipError_t e__ = (call);                        \
        if (e__ != hipSuccess) {                        \
            (ctx)->hip_err = (int)e__;                  \
            return e__ == hipErrorOutOfMemory ? ASGD_ENOMEM : ASGD_EHIP; \
        }                                               \
    } while (0)

size_t kd_of(const asgd_ctx *c) { return (size_t)c->k * c->d; }

void free_all(asgd_ctx *c)
{
    void *ptrs[] = {c->w, c->slot, c->acc, c->xabsmax, c->mean, c->stamp, c->consumed, c->cnt, c->assign_tmp,
                    c->ncum, c->counters, c->qpart, c->qout, c->xnorm2max, c->shift_tab, c->split_scratch, c->split_data, c->load_scratch, c->marks};
    for (void *q : ptrs)
        if (q) (void)hipFree(q);
    if (c->flag_host) (void)hipHostFree(c->flag_host);
    if (c->ev0) (void)hipEventDestroy(c->ev0);
    if (c->ev1) (void)hipEventDestroy(c->ev1);
}

StepParams make_params(const asgd_ctx *c)
{
    StepParams p;
    memset(&p, 0, sizeof(p));
    p.x = c->x; p.w = c->w; p.slot = c->slot; p.stamp = c->stamp; p.consumed = c->consumed; p.ncum = c->ncum;
    p.counters = c->counters; p.acc = c->acc; p.cnt = c->cnt; p.assign_tmp = c->assign_tmp;
    p.dump = c->dump; p.xabsmax = c->xabsmax; p.error_flag = c->flag_host;
    p.H = c->H; p.S = c->S; p.t_dump0 = c->t; p.seed = c->seed;
    p.k = c->k; p.d = c->d; p.W = c->W; p.b = c->b; p.E = c->E; p.eps = c->lr; p.nb = c->nb; p.parts = c->parts;
    p.parzen = c->parzen; p.lr_mode = c->lr_mode; p.mode = c->mode;
    p.drop_thr = (uint32_t)llround(c->drop_rate * (double)(1u << 24));
    p.tune = c->tune;
    p.cooperative = c->cooperative;
    p.wait_polls = c->wait_polls;
    p.drop_unannounced = c->drop_unannounced;
    p.refuse_one_launch = c->refuse_one_launch;
    return p;
}

// Empties the exchange buffers for the kernel that is going to use them.  Small-state kernel: all bits set = stamp -1
// inside its (value, stamp) pairs.  The other kernels look at `stamp` before they read a buffer; with partial messages
// rows of a buffer stay unwritten, which a free-running recipient may look at: those start as zeros = empty rows.
int clear_exchange(asgd_ctx *c, int kernel)
{
    const int fill = (c->parts > 1 && kernel != ASGD_KERNEL_SMALL) ? 0 : 0xFF;
    if (fill == 0 || small_kernel_supports(c->k, c->d, c->b)) HIP_TRY(c, hipMemsetAsync(c->slot, fill, c->slot_bytes, c->stream));
    HIP_TRY(c, hipMemsetAsync(c->stamp, 0xFF, exchange_buffers_total(c->nb, c->W) * sizeof(int), c->stream));   // -1
    c->fill_kernel = kernel;
    return ASGD_OK;
}

// ---- messages in flight, in a format of their own -------------------------------------------------------------
// Logical content of the exchange buffers: values[n][i] = the k x d rows waiting in buffer n of worker i (rows that a
// partial message does not carry: zeros), rounds[n][i] = the round it was sent in, -1 = nothing waiting.  The
// kernels hold this in two device formats: plain rows + a stamp per buffer (shape-agnostic and matrix-core kernels),
// or (value, stamp) pairs in padded rows (small-state kernel).  Conversion runs on the host, in chunks of workers.

// parity of the buffers that hold what the next merge point reads, and the round those messages carry (-1: none can)
void inflight(const asgd_ctx *c, int *parity, long long *round)
{
    const bool det = c->mode == ASGD_MODE_DETERMINISTIC;
    *parity = 0;
    *round = -1;
    if (c->E <= 0 || c->W < 2 || c->t <= 0) return;
    if (!det) { *round = c->t / c->E - 1; return; }       // newest round that has sent; older stamps count too
    if (c->t % c->E != 0) return;                           // inside a round nothing is in flight
    *round = c->t / c->E - 1;
    *parity = (int)(*round & 1);
}

bool row_in_part(const asgd_ctx *c, int row, long long round, int worker, int n)
{
    return row_travels(row, round, worker, n, c->parts);
}

enum { EXCHANGE_CHUNK_BYTES = 32 << 20 };

int export_exchange(asgd_ctx *c, int kernel, float *values, int32_t *rounds)
{
    const size_t kd = kd_of(c), W = (size_t)c->W;
    const bool det = c->mode == ASGD_MODE_DETERMINISTIC;
    int par;
    long long r_want;
    inflight(c, &par, &r_want);
    for (size_t q = 0; q < (size_t)c->nb * W; ++q) rounds[q] = -1;
    memset(values, 0, (size_t)c->nb * W * kd * sizeof(float));
    if (r_want < 0 || kernel == 0) return ASGD_OK;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const bool small = kernel == ASGD_KERNEL_SMALL;
    const size_t msg_bytes = small ? small_kernel_message_bytes(c->k, c->d) : kd * sizeof(float);
    const size_t per_chunk = EXCHANGE_CHUNK_BYTES / msg_bytes > 0 ? EXCHANGE_CHUNK_BYTES / msg_bytes : 1;
    std::vector<unsigned char> stage;
    std::vector<int> stamps, row_round;
    try {
        stage.resize((per_chunk < W ? per_chunk : W) * msg_bytes);
        stamps.resize(W);
        row_round.resize((size_t)c->k);
    } catch (...) {
        return ASGD_ENOMEM;
    }
    for (int n = 0; n < c->nb; ++n) {
        const size_t buf0 = exchange_buffer(par, c->nb, n, c->W, 0);
        if (!small)
            HIP_TRY(c, hipMemcpy(stamps.data(), c->stamp + buf0, W * sizeof(int), hipMemcpyDeviceToHost));
        for (size_t i0 = 0; i0 < W; i0 += per_chunk) {
            const size_t cnt = W - i0 < per_chunk ? W - i0 : per_chunk;
            HIP_TRY(c, hipMemcpy(stage.data(), (const unsigned char *)c->slot + (buf0 + i0) * msg_bytes, cnt * msg_bytes,
                                 hipMemcpyDeviceToHost));
            for (size_t q = 0; q < cnt; ++q) {
                const size_t i = i0 + q;
                float *out = values + ((size_t)n * W + i) * kd;
                long long st = -1;
                if (small) {
                    small_kernel_unpack_message(c->k, c->d, stage.data() + q * msg_bytes, out, row_round.data());
                    for (int row = 0; row < c->k; ++row)
                        if (row_round[row] > st) st = row_round[row];
                } else {
                    st = stamps[i];
                    if (st >= 0) memcpy(out, stage.data() + q * msg_bytes, kd * sizeof(float));
                }
                const bool there = det ? st == r_want : st >= 0;
                for (int row = 0; row < c->k; ++row) {
                    const bool keep = there && row_in_part(c, row, st, (int)i, n) && (!small || row_round[row] == st);
                    if (!keep) memset(out + (size_t)row * c->d, 0, (size_t)c->d * sizeof(float));
                }
                rounds[(size_t)n * W + i] = there ? (int32_t)st : -1;
            }
        }
    }
    return ASGD_OK;
}

// Writes the messages into the (freshly emptied) buffers in the format of `kernel`.
int import_exchange(asgd_ctx *c, int kernel, const float *values, const int32_t *rounds)
{
    const size_t kd = kd_of(c), W = (size_t)c->W;
    int par;
    long long r_want;
    inflight(c, &par, &r_want);
    if (r_want < 0) return ASGD_OK;
    const bool small = kernel == ASGD_KERNEL_SMALL;
    const size_t msg_bytes = small ? small_kernel_message_bytes(c->k, c->d) : kd * sizeof(float);
    const size_t per_chunk = EXCHANGE_CHUNK_BYTES / msg_bytes > 0 ? EXCHANGE_CHUNK_BYTES / msg_bytes : 1;
    std::vector<unsigned char> stage;
    std::vector<int> stamps, row_round;
    try {
        stage.resize((per_chunk < W ? per_chunk : W) * msg_bytes);
        stamps.resize(W);
        row_round.resize((size_t)c->k);
    } catch (...) {
        return ASGD_ENOMEM;
    }
    const int fill = (c->parts > 1 && !small) ? 0 : 0xFF;              // what clear_exchange() left in an empty buffer
    for (int n = 0; n < c->nb; ++n) {
        const size_t buf0 = exchange_buffer(par, c->nb, n, c->W, 0);
        for (size_t i0 = 0; i0 < W; i0 += per_chunk) {
            const size_t cnt = W - i0 < per_chunk ? W - i0 : per_chunk;
            for (size_t q = 0; q < cnt; ++q) {
                const size_t i = i0 + q;
                const long long st = rounds[(size_t)n * W + i];
                const float *in = values + ((size_t)n * W + i) * kd;
                unsigned char *dst = stage.data() + q * msg_bytes;
                stamps[i] = (int)st;
                if (small) {
                    for (int row = 0; row < c->k; ++row)
                        row_round[row] = (st >= 0 && row_in_part(c, row, st, (int)i, n)) ? (int)st : -1;
                    small_kernel_pack_message(c->k, c->d, in, row_round.data(), dst);
                } else if (st >= 0) {
                    memcpy(dst, in, kd * sizeof(float));
                } else {
                    memset(dst, fill, msg_bytes);
                }
            }
            HIP_TRY(c, hipMemcpy((unsigned char *)c->slot + (buf0 + i0) * msg_bytes, stage.data(), cnt * msg_bytes,
                                 hipMemcpyHostToDevice));
        }
        if (!small)
            HIP_TRY(c, hipMemcpy(c->stamp + buf0, stamps.data(), W * sizeof(int), hipMemcpyHostToDevice));
    }
    return ASGD_OK;
}

// Per-dimension max |x| over the rows the workers own (inputs of the rounding-error bounds that decide when an assignment is
// recomputed exactly, and of the scales of fixed-point sums), and whether they are finite and of ordinary size.
// Synchronises the stream.
int take_absmax_scratch(asgd_ctx *c)
{
    const size_t bytes = absmax_scratch_bytes(c->d);
    if (bytes && !c->load_scratch) HIP_TRY(c, hipMalloc(&c->load_scratch, bytes));
    return ASGD_OK;
}
int take_absmax(asgd_ctx *c)
{
    const int rc = take_absmax_scratch(c);
    if (rc != ASGD_OK) return rc;
    c->flag_host[1] = c->flag_host[2] = 0;
    HIP_TRY(c, launch_absmax(c->x, c->H * c->W, c->d, c->xabsmax, c->flag_host + 1, c->flag_host + 2, c->load_scratch, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->xabsmax_valid = true;
    return ASGD_OK;
}

// Whether a run of the streaming kernel need not compare its terms with the limits (within_limits): all samples were looked at while
// loading; or in an epoch since, and no element was beyond them, or those mini-batches are marked (p->marks).  The stream is idle.
// (Where the list is full, or mini-batches are so short that the table would take a sixteenth of the samples' room, later
// epochs compare like the first.)
int take_limits(asgd_ctx *c, const SeenSteps &seen, StepParams *p)
{
    p->within_limits = 0;
    p->marks = nullptr;
    if (sample_is_all(c->H * c->W, c->d)) p->within_limits = 2;
    else if (seen.all(c->S)) {
        if (c->flag_host[3] != 0 && c->marks_state == 0) {
            int n = 0;
            const size_t bytes = (size_t)c->W * c->S * sizeof(int);
            HIP_TRY(c, hipMemcpy(&n, p->found, sizeof(int), hipMemcpyDeviceToHost));
            c->marks_state = -1;
            if (n <= FOUND_MAX && (double)c->b * c->d >= 16.0) {
                if (bytes > c->marks_bytes) {
                    if (c->marks) (void)hipFree(c->marks);
                    c->marks = nullptr;
                    c->marks_bytes = 0;
                    if (hipMalloc((void **)&c->marks, bytes) == hipSuccess) c->marks_bytes = bytes;
                    else (void)hipGetLastError();
                }
                if (c->marks) {
                    HIP_TRY(c, launch_marks(p->found, c->d, c->S, c->W, c->marks, c->stream));
                    c->marks_state = 1;
                }
            }
        }
        p->within_limits = c->flag_host[3] == 0 || c->marks_state == 1;
        if (c->flag_host[3] != 0 && p->within_limits) p->marks = c->marks;
    }
    return ASGD_OK;
}

// Whether the fp16-split step kernels are faster than the fp32 matrix kernel (the default variant of
// ASGD_KERNEL_MFMA).  The former take 14 to 20 us per step whatever its size, the latter a step of one workgroup per worker.
// Microseconds per step of long calls, fp32 and split:
//   mini-batches of 512 and more: W = 4, k = 12, d = 8: b = 512 20, 17; b = 2000 50, 26; W = 32, k = 64, d = 32, b = 512: 24, 23;
//     k = d = 100: W = 4 72, 45; W = 256 84, 79 (150 samples: W = 32, k = 64, d = 32: 14, 21).  A call of one step: 0.94 to 1.7
//     times as fast.  Not where the workers fill the device and exchange (one launch with waits on either side) and steps are
//     short (W = 256, b = 512: k = 64, d = 32: 34, 37; k = 12, d = 8: 27.6, 28, both with workers that are not kept; the split
//     kernels keep them now and are the faster ones here, E = 8 29.2, 20.8 and 25.4, 12.2, but the line has not been moved);
//   k > 256, any mini-batch: a state that does not fit the LDS as fp32 is streamed (k = 1000, d = 64, b = 16, W = 4: 125, 56); one
//     that does: k = 300, d = 16, b = 64: W = 4 29, 27; W = 200 39, 34; k = 500, d = 24: W = 200 52, 51, but W = 4 42, 48;
//   exchange at every step, 100 workers and more: always (fp32 waits for messages every step: W = 150, k = 12, d = 8, b = 100: 33,
//     24; W = 256, k = 64, d = 32, b = 60: 68, 25; calls of one step 1.2 to 1.8 times as fast);
//   more than 256 workers where the fp32 kernel keeps two of them on a compute unit: only long steps (k = d = 100, W = 512,
//     b = 600: 121, 155; b = 2000: in milliseconds per epoch of 19 steps, two epochs 5.1, 4.9, a first one 5.5, 5.1, ten late in a run,
//     when few samples lie between centroids and the two workers of a compute unit have drifted apart, 4.60, 4.65); otherwise
//     always (k = 500, d = 24, W = 300, E = 1: 200, 83).
bool mfma_split_pays(const asgd_ctx *c)
{
    const bool exchange = c->E > 0 && c->W > 1, often = exchange && c->E < 4;
    const double size = (double)c->b * c->k * c->d;
    if (c->W > 256) return often || !mfma_kernel_two_per_cu(c->k, c->d, c->b) || size >= 1.5e7;
    if (often && c->W >= 100) return true;
    if (c->k > 256) return c->W >= 64 || (double)c->k * c->d <= 8192.0 || !mfma_state_resident(c->k, c->d, c->b) || c->b >= 512;
    return c->b >= 512 && !(exchange && c->W >= 192 && size < 2.0e6);
}

}  // namespace

extern "C" {

const char *asgd_strerror(int code)
{
    switch (code) {
        case ASGD_OK: return "success";
        case ASGD_EINVAL: return "invalid argument";
        case ASGD_ENOMEM: return "out of memory";
        case ASGD_ESTATE: return "call out of order";
        case ASGD_EHIP: return "HIP runtime error";
        case ASGD_ESYNC: return "bounded wait inside a kernel expired";
        default: return "unknown error code";
    }
}

int64_t asgd_schedule_peer_n(uint64_t seed, int64_t r, int64_t i, int64_t W, int64_t n)
{
    if (W < 2 || W > 0x7fffffff || i < 0 || i >= W || r < 0 || n < 0 || n >= W - 1) return -1;
    return peer_deterministic(seed, r, (int)i, (int)W, (int)n);
}

int64_t asgd_schedule_peer(uint64_t seed, int64_t r, int64_t i, int64_t W)
{
    if (W < 2 || i < 0 || i >= W || r < 0) return -1;
    return peer_deterministic(seed, r, (int)i, (int)W);
}

int asgd_create(asgd_ctx **out, int k, int d, int W, int b, float lr)
{
    if (!out || k < 1 || d < 1 || W < 1 || b < 1 || !(lr > 0.0f) || !isfinite(lr)) return ASGD_EINVAL;
    if ((double)k * d > (double)(1 << 28) || (double)W * k * d > 4e10) return ASGD_EINVAL;
    asgd_ctx *c = new (std::nothrow) asgd_ctx();
    if (!c) return ASGD_ENOMEM;
    c->k = k; c->d = d; c->W = W; c->b = b; c->lr = lr;
    int rc = ASGD_OK;
    auto fail = [&](hipError_t e) {
        c->hip_err = (int)e;
        rc = (e == hipErrorOutOfMemory) ? ASGD_ENOMEM : ASGD_EHIP;
    };
    hipError_t e = hipGetDevice(&c->device);
    if (e != hipSuccess) { delete c; return ASGD_EHIP; }
    const size_t kd = kd_of(c), Wz = (size_t)W;
    {
        const size_t plain = kd * sizeof(float), own = small_kernel_message_bytes(k, d);
        c->slot_bytes_one = exchange_buffers_total(1, W) * (plain > own ? plain : own);
        c->slot_bytes = c->slot_bytes_one;
    }
    const bool small = small_kernel_supports(k, d, b);
    struct { void **p; size_t bytes; } allocs[] = {
        {(void **)&c->w, Wz * kd * sizeof(float)},
        {(void **)&c->slot, c->slot_bytes},
        {(void **)&c->acc, Wz * kd * sizeof(float)},
        {(void **)&c->xabsmax, (size_t)d * sizeof(float)},
        {(void **)&c->mean, kd * sizeof(float)},
        {(void **)&c->stamp, exchange_buffers_total(1, W) * sizeof(int)},
        {(void **)&c->consumed, Wz * sizeof(int)},
        {(void **)&c->cnt, Wz * k * sizeof(int)},
        {(void **)&c->assign_tmp, Wz * (size_t)b * sizeof(int)},
        {(void **)&c->ncum, Wz * k * sizeof(long long)},
        {(void **)&c->counters, Wz * CNT_STRIDE * sizeof(long long)},
        {(void **)&c->qpart, (size_t)quant_partials_count() * sizeof(double) + (small ? sample_scratch_bytes(d) : quant_operand_bytes(k, d))},
        {(void **)&c->qout, sizeof(double)},
    };
    for (auto &a : allocs) {
        e = hipMalloc(a.p, a.bytes);
        if (e != hipSuccess) { fail(e); break; }
    }
    if (rc == ASGD_OK && small) c->xsample = reinterpret_cast<float *>(c->qpart + quant_partials_count());
    if (rc == ASGD_OK && (e = hipHostMalloc((void **)&c->flag_host, 4 * sizeof(int), hipHostMallocDefault)) != hipSuccess) fail(e);
    if (rc == ASGD_OK && (e = hipEventCreate(&c->ev0)) != hipSuccess) fail(e);
    if (rc == ASGD_OK && (e = hipEventCreate(&c->ev1)) != hipSuccess) fail(e);
    if (rc != ASGD_OK) {
        free_all(c);
        delete c;
        return rc;
    }
    *out = c;
    return ASGD_OK;
}

void asgd_destroy(asgd_ctx *ctx)
{
    if (!ctx) return;
    if (ctx->stream || ctx->loaded) (void)hipStreamSynchronize(ctx->stream);
    free_all(ctx);
    delete ctx;
}

int asgd_last_hip_error(asgd_ctx *ctx) { return ctx ? ctx->hip_err : 0; }

int asgd_set_option(asgd_ctx *ctx, int key, double value)
{
    if (!ctx || !isfinite(value)) return ASGD_EINVAL;
    ctx->passed_t = -1;
    switch (key) {
        case ASGD_OPT_EXCHANGE_EVERY:
            if (value < 0 || value > 2e9 || value != floor(value)) return ASGD_EINVAL;
            ctx->E = (int)value;
            return ASGD_OK;
        case ASGD_OPT_SEED:
            if (value < 0 || value > 9007199254740992.0 || value != floor(value)) return ASGD_EINVAL;
            ctx->seed = (uint64_t)value;
            return ASGD_OK;
        case ASGD_OPT_MODE:
            if (value != ASGD_MODE_DETERMINISTIC && value != ASGD_MODE_FREE_RUNNING) return ASGD_EINVAL;
            ctx->mode = (int)value;
            return ASGD_OK;
        case ASGD_OPT_PARZEN:
            if (value != 0 && value != 1) return ASGD_EINVAL;
            ctx->parzen = (int)value;
            return ASGD_OK;
        case ASGD_OPT_LR_MODE:
            if (value != ASGD_LR_CONST && value != ASGD_LR_INV_COUNT) return ASGD_EINVAL;
            ctx->lr_mode = (int)value;
            return ASGD_OK;
        case ASGD_OPT_DROP_RATE:
            if (value < 0.0 || value > 1.0) return ASGD_EINVAL;
            ctx->drop_rate = value;
            return ASGD_OK;
        case ASGD_OPT_KERNEL:
            if (value != ASGD_KERNEL_AUTO && value != ASGD_KERNEL_GENERIC && value != ASGD_KERNEL_SMALL &&
                value != ASGD_KERNEL_MFMA)
                return ASGD_EINVAL;
            ctx->kernel_opt = (int)value;
            return ASGD_OK;
        case ASGD_OPT_COOPERATIVE:
            if (value != 0 && value != 1) return ASGD_EINVAL;
            ctx->cooperative = (int)value;
            return ASGD_OK;
        case ASGD_OPT_BUFFERS: {
            if (value < 1 || value > MAX_BUFFERS || value != floor(value)) return ASGD_EINVAL;
            if (ctx->t != 0) return ASGD_ESTATE;
            const int nb = (int)value;
            if (nb == ctx->nb) return ASGD_OK;
            HIP_TRY(ctx, hipSetDevice(ctx->device));
            HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
            float *slot = nullptr;
            int *stamp = nullptr;
            hipError_t e = hipMalloc((void **)&slot, (size_t)nb * ctx->slot_bytes_one);
            if (e == hipSuccess) e = hipMalloc((void **)&stamp, exchange_buffers_total(nb, ctx->W) * sizeof(int));
            if (e != hipSuccess) {
                if (slot) (void)hipFree(slot);
                HIP_TRY(ctx, e);
            }
            (void)hipFree(ctx->slot);
            (void)hipFree(ctx->stamp);
            ctx->slot = slot;
            ctx->stamp = stamp;
            ctx->slot_bytes = (size_t)nb * ctx->slot_bytes_one;
            ctx->nb = nb;
            return clear_exchange(ctx, ASGD_KERNEL_SMALL);
        }
        case ASGD_OPT_PARTS:
            if (value < 1 || value > ctx->k || value != floor(value)) return ASGD_EINVAL;
            if (ctx->t != 0) return ASGD_ESTATE;
            ctx->parts = (int)value;
            ctx->fill_kernel = 0;          // the first run empties the buffers for its kernel
            return ASGD_OK;
        case ASGD_OPT_WAIT_POLLS:
            if (value < 0 || value > (double)(1 << 24) || value != floor(value)) return ASGD_EINVAL;
            ctx->wait_polls = (int)value;
            return ASGD_OK;
        case ASGD_OPT_DROP_UNANNOUNCED:
            if (value != 0 && value != 1) return ASGD_EINVAL;
            ctx->drop_unannounced = (int)value;
            return ASGD_OK;
        case ASGD_OPT_REFUSE_ONE_LAUNCH:
            if (value < 0 || value > 2 || value != floor(value)) return ASGD_EINVAL;
            ctx->refuse_one_launch = (int)value;
            return ASGD_OK;
        case ASGD_OPT_TUNE:
            if (value < 0 || value > 1000 || value != floor(value)) return ASGD_EINVAL;
            ctx->tune = (int)value;
            return ASGD_OK;
        default:
            return ASGD_EINVAL;
    }
}

int asgd_load_shards(asgd_ctx *ctx, const float *x_dev, int64_t N, void *hip_stream)
{
    if (!ctx || !x_dev || N < 1) return ASGD_EINVAL;
    if (((uintptr_t)x_dev & 7u) != 0 || ctx->d > 65536) return ASGD_EINVAL;
    const long long H = N / ctx->W;
    if (H < ctx->k || H < ctx->b) return ASGD_EINVAL;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    // The streaming kernel makes do with maxima over a part of the samples; those over all of them are formed by the first run
    // of another kernel.
    const bool whole = !(ctx->xsample && ctx->lr_mode == ASGD_LR_CONST && (ctx->kernel_opt == ASGD_KERNEL_AUTO || ctx->kernel_opt == ASGD_KERNEL_SMALL));
    if (whole) {                          // (no memory: the context keeps the samples it has)
        const int rc = take_absmax_scratch(ctx);
        if (rc != ASGD_OK) return rc;
    }
    ctx->x = x_dev; ctx->N = N; ctx->H = H; ctx->S = H / ctx->b;
    ctx->stream = (hipStream_t)hip_stream;
    ctx->t = 0;
    ctx->passed_t = -1;
    ctx->desynced = false;
    ctx->pending = false;
    ctx->loaded = false;
    ctx->xnorm2max_valid = false;
    ctx->split_data_valid = false;
    ctx->xabsmax_valid = false;
    ctx->seen = SeenSteps();
    ctx->marks_state = 0;
    ctx->flag_host[3] = 0;
    LoadParams l;
    memset(&l, 0, sizeof(l));
    l.x = ctx->x; l.w = ctx->w; l.stamp = ctx->stamp; l.ncum = ctx->ncum; l.counters = ctx->counters;
    l.H = H; l.k = ctx->k; l.d = ctx->d; l.W = ctx->W;
    l.stamps = exchange_buffers_total(ctx->nb, ctx->W);
    if (small_kernel_supports(ctx->k, ctx->d, ctx->b)) {             // (the other kernels look at the stamps first)
        l.slot = reinterpret_cast<unsigned *>(ctx->slot);
        l.slot_words = ctx->slot_bytes / sizeof(unsigned);
    }
    if (ctx->xsample && !ctx->xsample_clear) {
        HIP_TRY(ctx, hipMemsetAsync(ctx->xsample, 0, (size_t)(ctx->d + 1) * sizeof(float), ctx->stream));
        ctx->xsample_clear = true;
    }
    HIP_TRY(ctx, launch_load(l, ctx->xsample, ctx->stream));
    ctx->fill_kernel = 0;
    if (whole) {
        const int rc = take_absmax(ctx);
        if (rc != ASGD_OK) return rc;
    }
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    ctx->loaded = true;
    return ASGD_OK;
}

int asgd_set_state(asgd_ctx *ctx, int worker, const float *w_host)
{
    if (!ctx || !w_host || worker < -2 || worker >= ctx->W) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    const size_t kdb = kd_of(ctx) * sizeof(float);
    if (worker >= 0) {
        HIP_TRY(ctx, hipMemcpy(ctx->w + (size_t)worker * kd_of(ctx), w_host, kdb, hipMemcpyHostToDevice));
    } else if (worker == -1) {
        // one copy over the bus, the rest on the device (a copy per worker took 9 us each)
        HIP_TRY(ctx, hipMemcpy(ctx->mean, w_host, kdb, hipMemcpyHostToDevice));
        HIP_TRY(ctx, launch_broadcast_state(ctx->mean, ctx->W, (int)kd_of(ctx), ctx->w, ctx->stream));
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    } else {
        HIP_TRY(ctx, hipMemcpy(ctx->w, w_host, kdb * ctx->W, hipMemcpyHostToDevice));
    }
    return ASGD_OK;
}

int asgd_set_step(asgd_ctx *ctx, int64_t t)
{
    if (!ctx || t < 0) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    ctx->t = t;
    ctx->passed_t = -1;
    ctx->desynced = false;
    ctx->pending = false;
    ctx->last_kernel = 0;       // the buffers are empty: no format to carry over
    int rc = clear_exchange(ctx, ASGD_KERNEL_SMALL);
    if (rc != ASGD_OK) return rc;
    ctx->fill_kernel = 0;
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    return ASGD_OK;
}

int asgd_get_exchange(asgd_ctx *ctx, float *values_host, size_t values_bytes, int32_t *rounds_host, size_t rounds_bytes)
{
    if (!ctx || !values_host || !rounds_host) return ASGD_EINVAL;
    if (!ctx->loaded || ctx->desynced) return ASGD_ESTATE;
    const size_t nmsg = (size_t)ctx->nb * ctx->W;
    if (values_bytes < nmsg * kd_of(ctx) * sizeof(float) || rounds_bytes < nmsg * sizeof(int32_t)) return ASGD_EINVAL;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    if (ctx->pending) {          // handed over and not yet used by a run: give the same messages back
        memcpy(values_host, ctx->pending_values.data(), nmsg * kd_of(ctx) * sizeof(float));
        memcpy(rounds_host, ctx->pending_rounds.data(), nmsg * sizeof(int32_t));
        return ASGD_OK;
    }
    return export_exchange(ctx, ctx->last_kernel, values_host, rounds_host);
}

int asgd_set_exchange(asgd_ctx *ctx, const float *values_host, const int32_t *rounds_host)
{
    if (!ctx || !values_host || !rounds_host) return ASGD_EINVAL;
    if (!ctx->loaded || ctx->desynced) return ASGD_ESTATE;
    const size_t nmsg = (size_t)ctx->nb * ctx->W;
    int par;
    long long r_want;
    inflight(ctx, &par, &r_want);
    const bool det = ctx->mode == ASGD_MODE_DETERMINISTIC;
    for (size_t q = 0; q < nmsg; ++q) {
        const long long st = rounds_host[q];
        if (st < -1 || st > r_want || (det && st >= 0 && st != r_want)) return ASGD_EINVAL;   // no such message can wait here
    }
    try {
        ctx->pending_values.assign(values_host, values_host + nmsg * kd_of(ctx));
        ctx->pending_rounds.assign(rounds_host, rounds_host + nmsg);
    } catch (...) {
        return ASGD_ENOMEM;
    }
    ctx->pending = true;
    ctx->passed_t = -1;
    return ASGD_OK;
}

int asgd_set_assign_dump(asgd_ctx *ctx, int32_t *assign_dev, size_t capacity)
{
    if (!ctx) return ASGD_EINVAL;
    ctx->dump = assign_dev;
    ctx->dump_cap = assign_dev ? capacity : 0;
    return ASGD_OK;
}

int asgd_run_steps(asgd_ctx *ctx, int64_t steps)
{
    if (!ctx || steps < 0) return ASGD_EINVAL;
    if (!ctx->loaded || ctx->desynced) return ASGD_ESTATE;
    if (ctx->lr_mode == ASGD_LR_INV_COUNT && ctx->E != 0) return ASGD_EINVAL;
    if (ctx->dump && (double)steps * ctx->W * ctx->b > (double)ctx->dump_cap) return ASGD_EINVAL;
    HIP_TRY(ctx, hipSetDevice(ctx->device));

    int kernel = ctx->kernel_opt;
    if (ctx->W > 1 && ctx->E > 0 && ctx->nb > ctx->W - 1) return ASGD_EINVAL;       // a message has nb different recipients
    const bool small_ok = small_kernel_supports(ctx->k, ctx->d, ctx->b) && ctx->lr_mode == ASGD_LR_CONST &&
                          ((ctx->nb == 1 && ctx->parts == 1) || ((ctx->tune >> 2) & 3) != 1);   // several buffers, partial messages: not in the private-rows shape
    // Partial messages in the matrix-core kernel are limited to the sizes its parity tests cover: the one batch of
    // full-size runs of that combination ended with a device fault whose cause was never found, so larger runs of
    // it are refused (an explicit choice of the kernel) or go to the shape-agnostic kernel (automatic choice).
    const bool mfma_parts_ok = ctx->parts == 1 || (double)ctx->W * ctx->k * ctx->d <= (double)ASGD_MFMA_PARTS_MAX_STATE;
    const bool mfma_ok = mfma_kernel_supports(ctx->k, ctx->d, ctx->b, ctx->x) && ctx->lr_mode == ASGD_LR_CONST && mfma_parts_ok;
    if (kernel == ASGD_KERNEL_AUTO) {
        // the streaming kernel for the small shapes it is built for; else the matrix-core kernel wherever its
        // layout rules allow (measured faster than the shape-agnostic kernel down to k = d = 4); else the latter
        kernel = small_ok ? ASGD_KERNEL_SMALL : (mfma_ok ? ASGD_KERNEL_MFMA : ASGD_KERNEL_GENERIC);
    }
    if (kernel == ASGD_KERNEL_SMALL && !small_ok) return ASGD_EINVAL;
    if (kernel == ASGD_KERNEL_MFMA && !mfma_ok) return ASGD_EINVAL;

    // (before the exchange buffers are touched: it may find no memory, and the messages are still there for another attempt)
    if (kernel != ASGD_KERNEL_SMALL && !ctx->xabsmax_valid && steps > 0) {
        const int rc = take_absmax(ctx);
        if (rc != ASGD_OK) return rc;
    }

    // The kernels keep a message in flight in different formats.  Messages handed over by asgd_set_exchange(), and
    // those a run of another kernel left behind, are written into the buffers in the format of this run's kernel.
    const bool switched = ctx->last_kernel != 0 && kernel != ctx->last_kernel && ctx->E > 0 && ctx->W > 1 && ctx->t > 0;
    if (ctx->pending || switched) {
        if (!ctx->pending) {
            try {
                ctx->pending_values.resize((size_t)ctx->nb * ctx->W * kd_of(ctx));
                ctx->pending_rounds.resize((size_t)ctx->nb * ctx->W);
            } catch (...) {
                return ASGD_ENOMEM;
            }
            const int rc = export_exchange(ctx, ctx->last_kernel, ctx->pending_values.data(), ctx->pending_rounds.data());
            if (rc != ASGD_OK) return rc;
        }
        int rc = clear_exchange(ctx, kernel);
        if (rc != ASGD_OK) return rc;
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        rc = import_exchange(ctx, kernel, ctx->pending_values.data(), ctx->pending_rounds.data());
        if (rc != ASGD_OK) return rc;
        ctx->pending = false;
        std::vector<float>().swap(ctx->pending_values);
        std::vector<int32_t>().swap(ctx->pending_rounds);
        ctx->passed_t = -1;
    } else if (ctx->parts > 1 && ctx->fill_kernel != kernel) {
        // Partial messages: the fill of the never-written rows of the exchange buffers depends on the kernel's
        // message format.  (No message is in flight here: first run after load / set_step.)
        const int rc = clear_exchange(ctx, kernel);
        if (rc != ASGD_OK) return rc;
    }

    StepParams p = make_params(ctx);
    SeenSteps seen = ctx->seen;
    if (kernel == ASGD_KERNEL_SMALL) {
        p.xabsmax = ctx->xsample;
        p.beyond_flag = ctx->flag_host + 3;
        p.found = sample_found(ctx->xsample, ctx->d);
        if (steps > 0) seen.begin(ctx->t, ctx->S);
        p.note_until = seen.from + ctx->S;
        const int rc = take_limits(ctx, seen, &p);
        if (rc != ASGD_OK) return rc;
    }
    const long long t_end = ctx->t + steps;
    if (kernel == ASGD_KERNEL_SMALL && ctx->mode == ASGD_MODE_DETERMINISTIC && ctx->E > 0 && ctx->W > 1 && steps > 0) {
        // cyclic shifts of the rounds this call touches: the round before the first step up to the last step's
        const long long r_lo = ctx->t / ctx->E > 0 ? ctx->t / ctx->E - 1 : 0;
        const long long r_hi = (t_end - 1) / ctx->E;
        if (r_hi - r_lo + 1 > (long long)1 << 30) return ASGD_EINVAL;
        const bool held = ctx->tab_n > 0 && ctx->tab_seed == ctx->seed && ctx->tab_W == ctx->W && r_lo >= ctx->tab_r0 &&
                          r_hi < ctx->tab_r0 + ctx->tab_n;
        if (!held) {
            // some rounds ahead as well, so that a run of many short calls computes the table once in a while
            long long n = r_hi - r_lo + 1;
            if (n < 4096) n = 4096;
            if (n > ctx->shift_cap) {
                if (ctx->shift_tab) (void)hipFree(ctx->shift_tab);
                ctx->shift_tab = nullptr;
                ctx->shift_cap = 0;
                ctx->tab_n = 0;
                HIP_TRY(ctx, hipMalloc((void **)&ctx->shift_tab, (size_t)n * sizeof(int)));
                ctx->shift_cap = n;
            }
            HIP_TRY(ctx, launch_schedule_table(ctx->seed, r_lo, (int)n, ctx->W, ctx->shift_tab, ctx->stream));
            ctx->tab_r0 = r_lo; ctx->tab_n = n; ctx->tab_seed = ctx->seed; ctx->tab_W = ctx->W;
        }
        p.shift_tab = ctx->shift_tab;
        p.shift_r0 = ctx->tab_r0;
    }
    // The step kernels with fp16-split operands: the matrix-core form of the shape-agnostic kernel, and in the default
    // variant also what the matrix-core kernel runs (three products on the fp16 matrix instructions take a fifth of the
    // time of the fp32 ones).  Free-running mode of the latter stays with the kernel whose workers drift freely.
    // Shape-agnostic: ASGD_OPT_TUNE bit 0 asks for one workgroup per worker, bit 1 for the matrix-core form whatever
    // the size.  A step of the former takes 0.14 us per sample of the mini-batch or more, one of the latter 14 us or more and a
    // call 25 us once (W = 4, k = 3, d = 2: b = 96 14.3 and 16.0 us per step, a call of one step 31 and 39; b = 128 18.8 and 15.8,
    // 38 and 39; k = 12, d = 7: b = 20 10.3 and 13.9, b = 96 19.5 and 15.7, 37 and 39; k = 20, d = 21, b = 20: 34 and 15, 50 and 38).
    // The split kernels' gradient sums are in fixed point with one scale per column: exact to 2^-51 of its largest element, which
    // is more than fp32 sums give unless a column's typical element is far smaller (one huge element, a marker for a missing
    // value): those go to the kernels with fp32 sums.  (More than 256 workers of the matrix-core kernel, two on
    // a compute unit: its sums are in 32-bit fixed point, the split kernels' are the finer ones.)
    bool split = false;
    const bool wide = ctx->flag_host[2] != 0 &&
                      !(kernel == ASGD_KERNEL_MFMA && ctx->W > 256 && mfma_kernel_two_per_cu(ctx->k, ctx->d, ctx->b));
    if (ctx->flag_host[1] == 0 && !wide && split_kernel_supports(ctx->k, ctx->d, ctx->b) && steps > 0) {
        if (kernel == ASGD_KERNEL_GENERIC)
            split = (ctx->tune & 2) || (!(ctx->tune & 1) && (ctx->b >= 128 || (double)ctx->b * ctx->k * ctx->d >= 6000.0));
        else if (kernel == ASGD_KERNEL_MFMA) {
            split = ctx->tune == 0 && ctx->parts == 1 && (ctx->mode == ASGD_MODE_DETERMINISTIC || ctx->E == 0 || ctx->W < 2) && mfma_split_pays(ctx);
            p.one_launch = 1;
        }
    }
    p.phases_only = kernel == ASGD_KERNEL_GENERIC && (ctx->tune & 4);
    // device memory of the split kernels' launches; none: the kernels that need none
    auto take_scratch = [&]() -> bool {
        const size_t need = split_scratch_bytes(p);
        if (need > SPLIT_SCRATCH_MAX) return false;
        if (need <= ctx->split_bytes) return true;
        if (ctx->split_scratch) (void)hipFree(ctx->split_scratch);
        ctx->split_scratch = nullptr;
        ctx->split_bytes = 0;
        if (hipMalloc(&ctx->split_scratch, need) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        ctx->split_bytes = need;
        return true;
    };
    auto take_data = [&]() -> hipError_t {
        hipError_t e = hipSuccess;
        if (!ctx->split_data) e = hipMalloc(&ctx->split_data, split_data_bytes(ctx->d));
        if (e == hipSuccess && !ctx->split_data_valid) {
            e = launch_split_data(p, ctx->split_data, ctx->stream);
            ctx->split_data_valid = e == hipSuccess;
        }
        return e;
    };
    auto take_norms = [&]() -> hipError_t {
        hipError_t e = hipSuccess;
        if (!ctx->xnorm2max) e = hipMalloc((void **)&ctx->xnorm2max, sizeof(float));
        if (e == hipSuccess && !ctx->xnorm2max_valid) {
            e = launch_rownorm2max(ctx->x, ctx->H * ctx->W, ctx->d, ctx->xnorm2max, ctx->stream);
            ctx->xnorm2max_valid = e == hipSuccess;
        }
        return e;
    };
    if (split) split = take_scratch();
    if (split) {
        const hipError_t e = take_data();
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            split = false;
        } else {
            HIP_TRY(ctx, e);
        }
    }
    if (kernel == ASGD_KERNEL_MFMA && !split) HIP_TRY(ctx, take_norms());
    // Deterministic mode: a worker may only read the message of round r-1 once its sender has
    // finished that round.  Either the whole run is one launch of co-resident workgroups that wait
    // for each other's stamps (small-state and matrix-core kernels, when the workers all fit the
    // device), or a launch never crosses a multiple of E, so that the message was written by an
    // earlier launch on the same stream.
    const bool rounds = (ctx->mode == ASGD_MODE_DETERMINISTIC && ctx->E > 0 && ctx->W > 1);
    auto first_epoch_end = [&](long long from) -> long long {        // step at which a launch from `from` on is cut, or t_end
        if (kernel != ASGD_KERNEL_SMALL || p.within_limits) return t_end;
        const long long cut = first_epoch_cut(t_end, seen.from, ctx->S, rounds ? ctx->E : 0, (double)ctx->W * ctx->b * ctx->d);
        return cut > from ? cut : t_end;
    };
    auto ran_to = [&](long long t, bool cut) -> int {                 // a launch up to step t has been enqueued
        if (kernel != ASGD_KERNEL_SMALL) return ASGD_OK;
        seen.ran(t);
        if (!cut) return ASGD_OK;
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        return take_limits(ctx, seen, &p);
    };
    int launches = 0;
    *ctx->flag_host = 0;         // (no kernel of this context is in flight: every run ends with a wait for the stream)
    HIP_TRY(ctx, hipEventRecord(ctx->ev0, ctx->stream));
    long long t_done = ctx->t;           // steps [ctx->t, t_done) have been launched
    const bool split_local = split && split_local_form(p);
    const bool one_launch = split_local || (!split && ((kernel == ASGD_KERNEL_SMALL && (ctx->tune & 3) != 3) || (kernel == ASGD_KERNEL_MFMA && !(ctx->tune & 4))));
    // The split kernels' one launch costs 45 us more than a plain one (cooperative, and its workgroups make sure that all have a
    // place): a call of less than two rounds is one plain launch per round instead, the same bits (k = 64, d = 32, W = 256,
    // b = 512, one step: 93 us, 50).
    if (rounds && one_launch && steps > 0 && !(split_local && steps / ctx->E < 2)) {
        // every worker has passed the merge points before the first step of this run
        const long long r0 = ctx->t / ctx->E;
        const int passed = (int)((ctx->t % ctx->E) != 0 ? r0 : (r0 > 0 ? r0 - 1 : 0));
        // (a one-launch run leaves exactly these values behind: no need to write them again for the run that follows it)
        if (ctx->passed_t != ctx->t)
            HIP_TRY(ctx, hipMemsetD32Async((hipDeviceptr_t)ctx->consumed, passed, (size_t)ctx->W, ctx->stream));
        while (t_done < t_end) {
            const long long cut = first_epoch_end(t_done), tb = one_launch_end(t_done, t_end, cut, ctx->E);
            int one = 0;
            hipError_t e = ctx->refuse_one_launch == 1 ? hipErrorCooperativeLaunchTooLarge
                           : split_local ? launch_split_steps(p, t_done, tb, ctx->split_data, ctx->split_scratch, ctx->stream, &one)
                           : (kernel == ASGD_KERNEL_SMALL) ? launch_small_steps(p, t_done, tb, ctx->stream, true)
                                                         : launch_mfma_steps(p, t_done, tb, ctx->xnorm2max, ctx->stream, true);
            if (e == hipSuccess && split_local) {
                // (the next launch may only begin if this one has not been called off)
                HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
                if (*ctx->flag_host == 2) {
                    *ctx->flag_host = 0;
                    e = hipErrorCooperativeLaunchTooLarge;
                }
            }
            if (e == hipSuccess) {
                ++launches;
                const bool waited = tb == cut && cut < t_end;
                const int rc = ran_to(tb, waited);
                if (rc != ASGD_OK) return rc;
                t_done = tb;
                ctx->passed_t = tb;
                if ((split_local || waited) && *ctx->flag_host) break;       // an expired wait: nothing more may run on these states
            } else if (e == hipErrorCooperativeLaunchTooLarge || e == hipErrorNotSupported) {
                (void)hipGetLastError();     // the rest (or all of it): one launch per round
                break;
            } else {
                HIP_TRY(ctx, e);
            }
        }
    }
    const int form = !split ? ASGD_FORM_FP32 : split_local ? ASGD_FORM_SPLIT_LAUNCH : ASGD_FORM_SPLIT_PHASES;
    if (*ctx->flag_host) t_done = t_end;
    p.no_waits = 1;
    while (split && t_done < t_end) {
        long long tb = t_end;
        if (split_local && rounds) {
            const long long next = (t_done / ctx->E + 1) * (long long)ctx->E;
            if (next < tb) tb = next;
        }
        HIP_TRY(ctx, launch_split_steps(p, t_done, tb, ctx->split_data, ctx->split_scratch, ctx->stream, &launches));
        ctx->passed_t = -1;
        t_done = tb;
    }
    for (long long ta = t_done; ta < t_end;) {
        long long tb = t_end;
        if (rounds) {
            const long long next = (ta / ctx->E + 1) * (long long)ctx->E;
            if (next < tb) tb = next;
        } else {
            tb = first_epoch_end(ta);
        }
        hipError_t e = (kernel == ASGD_KERNEL_SMALL) ? launch_small_steps(p, ta, tb, ctx->stream, false)
                       : (kernel == ASGD_KERNEL_MFMA)
                           ? launch_mfma_steps(p, ta, tb, ctx->xnorm2max, ctx->stream, false)
                           : launch_generic_steps(p, ta, tb, ctx->stream);
        HIP_TRY(ctx, e);
        ++launches;
        const int rc = ran_to(tb, !rounds && tb < t_end);
        if (rc != ASGD_OK) return rc;
        ta = tb;
        ctx->passed_t = -1;
    }
    HIP_TRY(ctx, hipEventRecord(ctx->ev1, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    float ms = 0.f;
    HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev0, ctx->ev1));
    ctx->last_ms = ms;
    ctx->last_kernel = kernel;
    ctx->last_launches = launches;
    if (steps > 0) ctx->last_form = form;
    if (*ctx->flag_host) {
        // A bounded wait inside a kernel expired: some worker went on without a message it was owed, so the states are
        // not those of any step of the deterministic run.  The step counter stays where it was and the context refuses
        // further runs until asgd_load_shards() or asgd_set_state() + asgd_set_step() put it back on a known footing.
        ctx->passed_t = -1;
        ctx->desynced = true;
        return ASGD_ESYNC;
    }
    ctx->seen = seen;
    ctx->t = t_end;
    return ASGD_OK;
}

int asgd_run_epochs(asgd_ctx *ctx, int epochs)
{
    if (!ctx || epochs < 0) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    return asgd_run_steps(ctx, (int64_t)epochs * ctx->S);
}

int asgd_get_state(asgd_ctx *ctx, int worker, float *out_host, size_t out_bytes)
{
    if (!ctx || !out_host || worker < -1 || worker >= ctx->W) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    const size_t kdb = kd_of(ctx) * sizeof(float);
    const size_t need = worker >= 0 ? kdb : kdb * ctx->W;
    if (out_bytes < need) return ASGD_EINVAL;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    const float *src = worker >= 0 ? ctx->w + (size_t)worker * kd_of(ctx) : ctx->w;
    HIP_TRY(ctx, hipMemcpy(out_host, src, need, hipMemcpyDeviceToHost));
    return ASGD_OK;
}

int asgd_get_mean_state(asgd_ctx *ctx, float *out_host, size_t out_bytes)
{
    if (!ctx || !out_host) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    const size_t kdb = kd_of(ctx) * sizeof(float);
    if (out_bytes < kdb) return ASGD_EINVAL;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    HIP_TRY(ctx, launch_mean_state(ctx->w, ctx->W, (int)kd_of(ctx), ctx->mean, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    HIP_TRY(ctx, hipMemcpy(out_host, ctx->mean, kdb, hipMemcpyDeviceToHost));
    return ASGD_OK;
}

int asgd_quant_error(asgd_ctx *ctx, int worker, double *out)
{
    if (!ctx || !out || worker < -1 || worker >= ctx->W) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    const float *w = ctx->w + (size_t)(worker >= 0 ? worker : 0) * kd_of(ctx);
    if (worker == -1) {
        HIP_TRY(ctx, launch_mean_state(ctx->w, ctx->W, (int)kd_of(ctx), ctx->mean, ctx->stream));
        w = ctx->mean;
    }
    HIP_TRY(ctx, launch_quant_error(ctx->x, ctx->N, ctx->d, ctx->k, w, ctx->qpart, ctx->qout, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    HIP_TRY(ctx, hipMemcpy(out, ctx->qout, sizeof(double), hipMemcpyDeviceToHost));
    return ASGD_OK;
}

int asgd_get_worker_counters(asgd_ctx *ctx, int64_t *sent, int64_t *received, int64_t *accepted)
{
    if (!ctx) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    std::vector<long long> h;
    try {
        h.resize((size_t)ctx->W * CNT_STRIDE);
    } catch (...) {
        return ASGD_ENOMEM;
    }
    HIP_TRY(ctx, hipMemcpy(h.data(), ctx->counters, h.size() * sizeof(long long), hipMemcpyDeviceToHost));
    for (int i = 0; i < ctx->W; ++i) {
        if (sent) sent[i] = h[(size_t)i * CNT_STRIDE + CNT_SENT];
        if (received) received[i] = h[(size_t)i * CNT_STRIDE + CNT_RECEIVED];
        if (accepted) accepted[i] = h[(size_t)i * CNT_STRIDE + CNT_ACCEPTED];
    }
    return ASGD_OK;
}

int asgd_last_run_ms(asgd_ctx *ctx, double *out)
{
    if (!ctx || !out) return ASGD_EINVAL;
    *out = ctx->last_ms;
    return ASGD_OK;
}

int asgd_last_run_form(asgd_ctx *ctx, int32_t *out)
{
    if (!ctx || !out) return ASGD_EINVAL;
    *out = ctx->last_form;
    return ASGD_OK;
}

int asgd_get_stats(asgd_ctx *ctx, asgd_stats *out)
{
    if (!ctx || !out) return ASGD_EINVAL;
    if (!ctx->loaded) return ASGD_ESTATE;
    HIP_TRY(ctx, hipSetDevice(ctx->device));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    std::vector<long long> h;
    try {
        h.resize((size_t)ctx->W * CNT_STRIDE);
    } catch (...) {
        return ASGD_ENOMEM;
    }
    HIP_TRY(ctx, hipMemcpy(h.data(), ctx->counters, h.size() * sizeof(long long), hipMemcpyDeviceToHost));
    memset(out, 0, sizeof(*out));
    for (int i = 0; i < ctx->W; ++i) {
        out->sent += h[(size_t)i * CNT_STRIDE + CNT_SENT];
        out->received += h[(size_t)i * CNT_STRIDE + CNT_RECEIVED];
        out->accepted += h[(size_t)i * CNT_STRIDE + CNT_ACCEPTED];
        out->parzen_near_ties += h[(size_t)i * CNT_STRIDE + CNT_PARZEN_NEAR];
        out->exact_rechecks += h[(size_t)i * CNT_STRIDE + CNT_RECHECK];
    }
    out->steps = ctx->t;
    out->samples = ctx->t * (long long)ctx->W * ctx->b;
    out->last_run_ms = ctx->last_ms;
    out->kernel = ctx->last_kernel;
    out->launches = ctx->last_launches;
    return ASGD_OK;
}

}  // extern "C"
