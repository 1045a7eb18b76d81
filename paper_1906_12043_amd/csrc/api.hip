// Host side of libcocod: argument validation, layout planning, the state machine of
// one CoCoD-SGD round (Algorithm 1: Step I and Step II in parallel, then line 6)
// and the stream/event choreography that makes the two steps overlap on one GPU.
// No arithmetic on model data happens here; every step of the round is a kernel.
#include "../../include/cocod.h"
#include "internal.hpp"

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using cocod::Chunk;

struct cocod_ctx {
    cocod_config cfg{};                 // copy of the caller's config (host array pointers cleared)
    std::vector<uint64_t> tensor_numel, tensor_offset, bucket_begin;
    uint64_t padded_d = 0;
    std::vector<Chunk> chunks;
    Chunk *d_chunks = nullptr;          // device copy of the chunk table (owned)
    float *d_weights = nullptr;         // device copy of p_i (owned), nullptr = uniform
    float *d_sigma_w = nullptr;         // device copy of the per-worker noise scale (owned), nullptr = cfg.noise_sigma
    double *d_reduce = nullptr;         // scratch of the diagnostics' reductions (owned, allocated on first use)
    double *host_result = nullptr;      // their two results, pinned host memory that the last kernel writes (owned, with d_reduce)
    double *static_scratch = nullptr;   // this GPU's copy of the library's static scratch array (not owned)
    float *mlp_ws = nullptr;            // MLP kind: work space (owned); mlp holds the pointers carved from it
    cocod::MlpParams mlp{};
    // MLP kind: two mini-batch buffers.  A local step draws the NEXT step's batch into the other one while
    // its output layer runs, so that only the first step after anything else draws its own up front.
    float *mlp_X[2] = {nullptr, nullptr};
    int32_t *mlp_y[2] = {nullptr, nullptr};
    uint32_t compute_units = 0;         // of the device the context was created on
    uint32_t batch_buf = 0;             // buffer the next eager step takes its batch from
    uint32_t batch_last = 0;            // buffer the most recent step took its batch from
    uint64_t batch_ready_step = ~0ull;  // mlp_X[batch_buf] holds the batch of this step index (~0: of none)
    hipEvent_t ev_snap = nullptr;       // compute stream reached the point where the models are stored
    hipEvent_t ev_mean = nullptr;       // mean of the stored models is complete
    hipStream_t s_compute = nullptr, s_avg = nullptr;
    float *live = nullptr;              // buffer holding the current models
    float *spare = nullptr;             // the other model buffer
    const float *snap = nullptr;        // stored models x_t^i of the open round (aliases one of the two)
    bool averaging = false;             // a round is open
    bool store_pending = false;         // next local step must write out of place (keeps the stored models intact)
    bool mean_pending = false;          // the open round's mean has not been enqueued yet (every schedule but OVERLAP)
    int schedule = COCOD_SCHED_OVERLAP;
    uint64_t step = 0;                  // global step counter t
    bool dry = false;
    bool timing = false;                // bracket step launches with start/stop events
    std::vector<hipEvent_t> t_start, t_stop;   // event pool for step timing (owned)
    std::vector<char> t_kind;           // per timed launch: 0 plain step, 1 step with line 6, 2 step that forms the mean
    size_t t_used = 0, t_limit = 0;     // steps timed since the last read, steps to time (the pool may hold more events)
    // replayable rounds: one instantiated graph per (k, variant, schedule, which buffer is live)
    struct RoundGraph { int k; int fused_tail; int schedule; bool live_is_A; uint32_t batch_buf; bool batch_ready; hipGraphExec_t exec; };
    std::vector<RoundGraph> graphs;     // owned
    // Device copies of t that captured kernels read (owned): a round that starts with xA live reads word 0 and its last step
    // leaves t + k in word 1, which the next round (xB live) reads, and so on.
    uint32_t *d_step = nullptr;
    uint64_t d_step_value[2] = {~0ull, ~0ull};   // what they hold once the work queued on the compute stream has run
    bool capturing = false;             // enqueue_step runs under stream capture: step relative to the word of the round
    uint64_t capture_base = 0;          // value of `step` when the capture began
    uint32_t capture_steps = 0;         // steps of the round
    uint32_t capture_word = 0;          // word it reads
    std::string err;
};

namespace {

// Scratch of cocod_consensus_distance_noalloc: block partials of the reduction, in device memory that
// exists from the moment the library is loaded, so the call never allocates.  One copy per GPU, held
// until the process ends; every call on a GPU shares that GPU's copy.  In host code the array's name
// is only a handle: the device address comes from hipGetSymbolAddress (scratch_for_current_device).
constexpr uint32_t kNoAllocMaxChunks = 1u << 18;                       // 2^18 chunks of 1024 = 268 M parameters per worker
static __device__ __align__(256) double scratch[2 + kNoAllocMaxChunks];   // result words, then one partial per chunk (2 MiB)

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[kMaxDevices] = {};                               // device address of `scratch`, per device

// Device address of this GPU's copy of `scratch`; looked up once per device, with that device current.
hipError_t scratch_for_current_device(double **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        double *ptr = nullptr;
        e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

thread_local std::string g_err;         // errors that have no context to live in

int fail(cocod_ctx *ctx, int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (ctx) ctx->err = buf; else g_err = buf;
    return code;
}

int hip_fail(cocod_ctx *ctx, hipError_t e, const char *what)
{
    return fail(ctx, COCOD_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define COCOD_HIP(ctx, call)                                             \
    do {                                                                 \
        hipError_t e_ = (call);                                          \
        if (e_ != hipSuccess) return hip_fail((ctx), e_, #call);         \
    } while (0)

// Block order of a line-6 step whose mean exceeds the cache: panels of this many tiles (4 MiB of the mean;
// every worker streams 4 MiB of each of its arrays per panel).  Measured at W = 16, d = 138 M: 9.9 ms per
// launch, against 10.6 ms with the worker fastest for every single tile and 11.4 ms on the (tiles, workers)
// grid, where the mean comes from memory once per worker.
constexpr uint32_t kPanelTiles = 16384;

// A mean vector up to this size is expected to stay in the 256 MB last-level cache while the W
// workers of a line-6 step read it one after the other.
constexpr uint64_t kMeanCacheBytes = 128ull << 20;
// Steps access a state (both model buffers, v, h, c: 20 bytes per worker-parameter) up to this size without the
// streaming hint: the next step or round finds it in the last-level cache.  Rounds, hint / no hint in us, one context and
// three in turn, at W = 8, d = 250 k (40 MB counted so), W = 16, d = 400 k (128 MB), 700 k (224 MB), 1 M (320 MB), 2 M (640 MB):
//   quadratic, k = 8 (one launch): 17.8/18.9 and 11.6/11.0; 42.0/42.4 and 40.1/39.2; 69/68 and 68/70; 98/96 and 97/102;
//     193/199 and 199/207.  k = 1: 12.6/12.4 and 12.0/10.8; 32.0/29.7 and 30.0/29.5; 51.8/48.3 and 52.3/53.1; 73/75 and
//     73/79; 142/156 and 144/159.  Without momentum, k = 2: 10.5/10.5 and 9.7/9.0; 24/23 and 21/20; 38.8/35.8 and
//     37.2/36.4; 54/55 and 53/56; 102/109 and 103/114.
//   the caller's gradient, k = 8 (eight launches): 62/49 and 53/52; 182/168 and 174/162; 304/279 and 302/281; 429/397 and
//     428/439; 835/908 and 868/955.
// The count is the same for every kind of context; those without momentum or with the caller's gradient hold less.  With a
// 16-bit gradient, k = 8, 40 / 128 / 224 MB: 74/62, 182/169, 290/269, without momentum 63/61, 122/112, 187/168.
constexpr uint64_t kCachedStateBytes = 224ull << 20;
// Local steps per launch with the built-in quadratic gradient.  The gradient of a coordinate depends on nothing but that
// coordinate, so a wave takes its tile through several steps in registers: 24 bytes per parameter once, not per step (a real
// gradient needs the whole model between two steps: one launch per step there).  Measured at W = 16, d = 11.2 M, one
// launch: 1 step 656 us, 2 656, 3 657, 4 673, 8 1005, 16 1703; from five steps on the generator and
// the arithmetic bound it (87 us a step), so more than 16 would only make launches long.  Without momentum 1 step 424 us, 2
// 432, 4 538; a round of the overlapped schedule with line 6 inside the last step at k = 2 1638 -> 835 us, at W = 12,
// d = 3.0 M, k = 4 with line 6 apart 668 -> 241, Local SGD at W = 21, d = 4.0 M, k = 2 777 -> 458.
constexpr int kMaxStepsPerLaunch = 16;
// A launch of several steps that forms the mean itself holds all workers' rows of a tile in one block of at most sixteen waves, one
// block or two to a compute unit, so with fewer blocks than compute units the others have no part in the steps.  A unit
// takes 8 element steps a nanosecond; where the steps would wait longer than 10 us for the idle units, the mean stays a
// kernel of its own (which costs a round 2 to 8 us) and the steps spread over the chip.  Rounds with line 6 inside, one launch
// per step / all in the mean's launch / mean apart, us: W = 64, d = 1500, k = 8 37 / 46 / 9.1, k = 16 62 / 85 / 11; W = 131,
// d = 6000, k = 8 46 / 48 / 17; W = 48, d = 14 000, k = 8 42 / 36 / 11; on the other side of the line W = 24, d = 6000, k = 2 11 / 8.1 / 7.3,
// W = 17, d = 60 000, k = 4 25 / 11.6 / 9.9, W = 131, d = 30 000, k = 2 37 / 25 / 27, W = 16, d = 14 000, k = 8 28 / 8.5 / 7.9.
// With enough blocks the launch is taken whatever W is, for it is always faster than one launch per step; against the mean apart
// and one launch for the steps, round of k = 2 / 4 / 8 / 16, us: W = 4, d = 32 M 511 / 533 / 748 / 1249 against 591 / 610 / 845 / 1357,
// W = 16, d = 8 M 548 / 580 / 786 / 1264 against 585 / 605 / 833 / 1351, W = 17, d = 7.5 M 623 / 724 / 941 / 1489 against 584 / 604 / 832 /
// 1355, W = 32, d = 4 M 572 / 597 / 796 / 1289 against 566 / 577 / 820 / 1339, W = 64, d = 2 M 582 / 593 / 841 / 1445 against 564 / 576 / 817 /
// 1340, W = 131, d = 977 k 573 / 589 / 824 / 1378 against 557 / 570 / 812 / 1332; rows off the lines, k = 2, W = 4 609 against 616, W = 16 629
// against 609, W = 64 636 against 572.
// With line 6 apart, W = 64, d = 1500, k = 8 38 / 48 / 18; W = 131, d = 14 000, k = 2 28 / 23 / 33, k = 4, already apart, 40 / 33 / 35.
constexpr uint64_t kIdleElementSteps = 80000;     // per compute unit
// Models of all workers up to this size are averaged on the one branch of a replayed round: reading them takes a few
// microseconds, fork and join between two branches more, and above all when several contexts replay rounds at a time.
// Perceptron rounds of k = 2, two branches / one, three contexts in turn (one context alone): W = 4, 768-192-10 (2.4 MB of
// models) 54 / 42 us (78 / 61; three contexts in turn take anything from 24 to 42 on one branch, process by process), 768-768-10
// (9.5 MB) 70 / 69 (109 / 98), W = 8, 2048-512-10 (34 MB) 175 / 179 (213 / 205), W = 16, 3072-1024-10 (202 MB) 575 / 581
// (609 / 607).  Rounds of the quadratic gradient, whose steps are one launch behind the mean,
// are the same either way.
constexpr uint64_t kGraphBranchBytes = 16ull << 20;
// one grid dimension holds fewer than 2^32 threads
constexpr uint64_t kMaxThreadsPerGridDim = 1ull << 32;
// the mean-forming steps launch up to four 1024-thread blocks per chunk in one grid dimension
constexpr uint64_t kMaxChunksMeanStep = 1ull << 20;

inline uint64_t round_up4(uint64_t n) { return (n + 3u) & ~static_cast<uint64_t>(3u); }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Layout of a parameter list: tensors in order, each start rounded up to a chunk (1024 elements =
// 4 KiB: measured 10 % faster streaming than 16-byte alignment, because every full chunk of the step
// kernel then covers whole 4 KiB blocks of memory); the end of the list rounded up to 4 elements.
// Buckets are maximal runs of tensors whose padded extent fits bucket_bytes.
int plan(uint64_t d, uint32_t n_tensors, const uint64_t *numel, uint64_t bucket_bytes,
         std::vector<uint64_t> &sizes, std::vector<uint64_t> &offsets, std::vector<uint64_t> &bucket_begin,
         uint64_t &padded_d)
{
    if (d == 0) return fail(nullptr, COCOD_ERR_INVALID, "d must be >= 1");
    if (d >= (1ull << 34)) return fail(nullptr, COCOD_ERR_INVALID, "d must be < 2^34 (generator counter width)");
    sizes.clear(); offsets.clear(); bucket_begin.clear();
    if (n_tensors <= 1) {
        if (n_tensors == 1 && numel && numel[0] != d)
            return fail(nullptr, COCOD_ERR_INVALID, "tensor_numel[0] != d");
        sizes.push_back(d);
    } else {
        if (!numel) return fail(nullptr, COCOD_ERR_INVALID, "tensor_numel is NULL with n_tensors > 1");
        uint64_t sum = 0;
        for (uint32_t t = 0; t < n_tensors; ++t) {
            if (numel[t] == 0) return fail(nullptr, COCOD_ERR_INVALID, "tensor %u is empty", t);
            if (numel[t] > d) return fail(nullptr, COCOD_ERR_INVALID, "tensor %u larger than d", t);
            sum += numel[t];
            sizes.push_back(numel[t]);
        }
        if (sum != d) return fail(nullptr, COCOD_ERR_INVALID, "tensor sizes sum to %llu, d is %llu",
                                  (unsigned long long)sum, (unsigned long long)d);
    }
    uint64_t at = 0;
    for (uint64_t n : sizes) {
        at = (at + cocod::kChunkElems - 1) / cocod::kChunkElems * cocod::kChunkElems;
        offsets.push_back(at);
        at += n;
    }
    padded_d = round_up4(at);
    // fewer than 2^24 chunks: the chunk table addresses memory in 32-bit quad offsets, and four single-wave
    // blocks (or one 256-thread block) per chunk must stay below 2^32 threads in one grid dimension
    if (padded_d > (1ull << 34) - cocod::kChunkElems)
        return fail(nullptr, COCOD_ERR_INVALID, "the padded parameter list holds %llu elements, more than 2^34 - 1024",
                    (unsigned long long)padded_d);
    const uint64_t cap = bucket_bytes / sizeof(float);
    bucket_begin.push_back(0);
    uint64_t bucket_start = 0;
    for (size_t t = 1; t < sizes.size(); ++t) {
        const uint64_t end_with_t = round_up4(offsets[t] + sizes[t]);
        if (cap != 0 && end_with_t - bucket_start > cap) {   // tensor t does not fit: it opens a new bucket
            bucket_begin.push_back(offsets[t]);
            bucket_start = offsets[t];
        }
    }
    bucket_begin.push_back(padded_d);
    return COCOD_OK;
}

bool overlap(const void *a, uint64_t a_bytes, const void *b, uint64_t b_bytes)
{
    if (!a || !b) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}

int validate(const cocod_config *cfg, uint64_t padded_d)
{
    const unsigned known_flags = COCOD_FLAG_DRY_RUN;
    if (cfg->flags & ~known_flags) return fail(nullptr, COCOD_ERR_INVALID, "unknown flag bits 0x%x", cfg->flags & ~known_flags);
    if (cfg->W == 0 || cfg->W > 65535u) return fail(nullptr, COCOD_ERR_INVALID, "W must be in 1..65535");
    if (cfg->grad != COCOD_GRAD_QUADRATIC && cfg->grad != COCOD_GRAD_MLP && cfg->grad != COCOD_GRAD_EXTERNAL)
        return fail(nullptr, COCOD_ERR_INVALID, "unknown gradient kind %u", cfg->grad);
    if (cfg->stride < padded_d || (cfg->stride & 3u))
        return fail(nullptr, COCOD_ERR_INVALID, "stride %llu must be a multiple of 4 and >= padded size %llu",
                    (unsigned long long)cfg->stride, (unsigned long long)padded_d);
    if (!std::isfinite(cfg->lr)) return fail(nullptr, COCOD_ERR_INVALID, "lr is not finite");
    if (!(cfg->momentum >= 0.0f && cfg->momentum < 1.0f)) return fail(nullptr, COCOD_ERR_INVALID, "momentum must be in [0,1)");
    if (!(cfg->weight_decay >= 0.0f) || !std::isfinite(cfg->weight_decay)) return fail(nullptr, COCOD_ERR_INVALID, "weight_decay must be finite and >= 0");
    if (!(cfg->noise_sigma >= 0.0f) || !std::isfinite(cfg->noise_sigma)) return fail(nullptr, COCOD_ERR_INVALID, "noise_sigma must be finite and >= 0");
    if (!cfg->xA || !cfg->xB || !cfg->mean) return fail(nullptr, COCOD_ERR_INVALID, "xA, xB and mean must not be NULL");
    if (cfg->momentum != 0.0f && !cfg->v) return fail(nullptr, COCOD_ERR_INVALID, "v must not be NULL when momentum != 0");
    if (cfg->grad == COCOD_GRAD_QUADRATIC && (!cfg->h || !cfg->c))
        return fail(nullptr, COCOD_ERR_INVALID, "h and c must not be NULL for the quadratic gradient");
    const void *ptrs[] = { cfg->xA, cfg->xB, cfg->v, cfg->mean, cfg->h, cfg->c };
    const char *names[] = { "xA", "xB", "v", "mean", "h", "c" };
    for (int i = 0; i < 6; ++i)
        if (!aligned16(ptrs[i])) return fail(nullptr, COCOD_ERR_INVALID, "%s is not 16-byte aligned", names[i]);
    const uint64_t big = static_cast<uint64_t>(cfg->W) * cfg->stride * sizeof(float);
    const uint64_t sizes[] = { big, big, big, cfg->stride * sizeof(float), big, big };
    for (int i = 0; i < 6; ++i)
        for (int j = i + 1; j < 6; ++j)
            if (overlap(ptrs[i], sizes[i], ptrs[j], sizes[j]))
                return fail(nullptr, COCOD_ERR_INVALID, "%s and %s overlap", names[i], names[j]);
    if (cfg->weights) {
        double sum = 0.0;
        for (uint32_t i = 0; i < cfg->W; ++i) {
            if (!(cfg->weights[i] >= 0.0f) || !std::isfinite(cfg->weights[i]))
                return fail(nullptr, COCOD_ERR_INVALID, "weights[%u] must be finite and >= 0", i);
            sum += cfg->weights[i];
        }
        if (std::fabs(sum - 1.0) > 1e-4) return fail(nullptr, COCOD_ERR_INVALID, "weights sum to %g, not 1", sum);
    }
    if (cfg->noise_sigma_w)
        for (uint32_t i = 0; i < cfg->W; ++i)
            if (!(cfg->noise_sigma_w[i] >= 0.0f) || !std::isfinite(cfg->noise_sigma_w[i]))
                return fail(nullptr, COCOD_ERR_INVALID, "noise_sigma_w[%u] must be finite and >= 0", i);
    if (cfg->grad == COCOD_GRAD_MLP) {
        const uint64_t want = static_cast<uint64_t>(cfg->mlp_in) * cfg->mlp_hidden + cfg->mlp_hidden +
                              static_cast<uint64_t>(cfg->mlp_hidden) * cfg->mlp_out + cfg->mlp_out;
        if (cfg->d != want)
            return fail(nullptr, COCOD_ERR_INVALID, "d is %llu but the MLP has %llu parameters",
                        (unsigned long long)cfg->d, (unsigned long long)want);
        if (cfg->n_tensors > 1) return fail(nullptr, COCOD_ERR_INVALID, "the MLP parameters are one flat tensor");
        if (!cocod::mlp_shape_supported(cfg->mlp_in, cfg->mlp_hidden, cfg->mlp_out, cfg->mlp_batch))
            return fail(nullptr, COCOD_ERR_UNSUPPORTED,
                        "MLP shape: mlp_in and mlp_batch must be multiples of 128 (batch <= 1024), mlp_hidden a "
                        "multiple of 64, 1 <= mlp_out <= 16, mlp_hidden * (mlp_out rounded up to odd) <= 32768");
    }
    return COCOD_OK;
}

void release(cocod_ctx *ctx)
{
    if (!ctx->dry) {
        if (ctx->d_chunks) (void)hipFree(ctx->d_chunks);
        if (ctx->d_weights) (void)hipFree(ctx->d_weights);
        if (ctx->d_sigma_w) (void)hipFree(ctx->d_sigma_w);
        if (ctx->mlp_ws) (void)hipFree(ctx->mlp_ws);
        if (ctx->d_reduce) (void)hipFree(ctx->d_reduce);
        if (ctx->host_result) (void)hipHostFree(ctx->host_result);
        if (ctx->d_step) (void)hipFree(ctx->d_step);
        for (auto &g : ctx->graphs) (void)hipGraphExecDestroy(g.exec);
        if (ctx->ev_snap) (void)hipEventDestroy(ctx->ev_snap);
        if (ctx->ev_mean) (void)hipEventDestroy(ctx->ev_mean);
        for (hipEvent_t e : ctx->t_start) (void)hipEventDestroy(e);
        for (hipEvent_t e : ctx->t_stop) (void)hipEventDestroy(e);
    }
    delete ctx;
}

uint32_t step_state_is_cached(const cocod_ctx *ctx)
{
    return 20 * ctx->cfg.stride * static_cast<uint64_t>(ctx->cfg.W) <= kCachedStateBytes ? 1u : 0u;
}

// Step I arithmetic on `stream`, one launch per bucket.
int enqueue_mean(cocod_ctx *ctx, hipStream_t stream)
{
    for (size_t b = 0; b + 1 < ctx->bucket_begin.size(); ++b)
        COCOD_HIP(ctx, cocod::launch_wmean(stream, ctx->snap, ctx->cfg.stride, ctx->cfg.W, ctx->bucket_begin[b],
                                           ctx->bucket_begin[b + 1], ctx->d_weights, ctx->cfg.mean, step_state_is_cached(ctx)));
    return COCOD_OK;
}

// The overlapped schedule's mean has a branch of its own: the averaging stream, or in a replayed round, which need not use
// that stream, a branch of the graph where the mean is long enough to pay for the fork and the join.
bool on_avg_stream(const cocod_ctx *ctx)
{
    return ctx->s_avg != ctx->s_compute &&
           !(ctx->capturing && ctx->cfg.stride * sizeof(float) * ctx->cfg.W <= kGraphBranchBytes);
}

// Make the open round's mean available to line 6 on the compute stream: enqueue it there if no
// earlier call has (sequential schedules), or join the averaging stream (overlapped schedule).
int mean_before_line6(cocod_ctx *ctx)
{
    if (ctx->mean_pending) {
        const int rc = enqueue_mean(ctx, ctx->s_compute);
        if (rc != COCOD_OK) return rc;
        ctx->mean_pending = false;
    } else if (ctx->schedule == COCOD_SCHED_OVERLAP && on_avg_stream(ctx)) {
        COCOD_HIP(ctx, hipStreamWaitEvent(ctx->s_compute, ctx->ev_mean, 0));
    }
    return COCOD_OK;
}

}  // namespace

extern "C" {

int cocod_version(void) { return 1000; }

const char *cocod_last_error(const cocod_ctx *ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

int cocod_plan_layout(uint64_t d, uint32_t n_tensors, const uint64_t *tensor_numel, uint64_t bucket_bytes,
                      uint64_t *padded_d, uint64_t *tensor_offset, uint32_t *n_buckets, uint64_t *bucket_begin)
{
    if (!padded_d) return fail(nullptr, COCOD_ERR_INVALID, "padded_d is NULL");
    std::vector<uint64_t> sizes, offsets, buckets;
    uint64_t pd = 0;
    const int rc = plan(d, n_tensors, tensor_numel, bucket_bytes, sizes, offsets, buckets, pd);
    if (rc != COCOD_OK) return rc;
    *padded_d = pd;
    if (tensor_offset) std::memcpy(tensor_offset, offsets.data(), offsets.size() * sizeof(uint64_t));
    if (n_buckets) *n_buckets = static_cast<uint32_t>(buckets.size() - 1);
    if (bucket_begin) std::memcpy(bucket_begin, buckets.data(), buckets.size() * sizeof(uint64_t));
    return COCOD_OK;
}

int cocod_create(const cocod_config *cfg, cocod_ctx **out)
{
    if (out) *out = nullptr;
    if (!cfg || !out) return fail(nullptr, COCOD_ERR_INVALID, "cfg and out must not be NULL");
    if (cfg->struct_size != sizeof(cocod_config))
        return fail(nullptr, COCOD_ERR_INVALID, "struct_size %u does not match this library (%zu)", cfg->struct_size,
                    sizeof(cocod_config));
    cocod_ctx *ctx = new (std::nothrow) cocod_ctx;
    if (!ctx) return fail(nullptr, COCOD_ERR_NOMEM, "out of host memory");
    int rc = plan(cfg->d, cfg->n_tensors, cfg->tensor_numel, cfg->bucket_bytes, ctx->tensor_numel, ctx->tensor_offset,
                  ctx->bucket_begin, ctx->padded_d);
    if (rc == COCOD_OK) rc = validate(cfg, ctx->padded_d);
    if (rc != COCOD_OK) { delete ctx; return rc; }

    ctx->cfg = *cfg;
    ctx->cfg.tensor_numel = nullptr;
    ctx->dry = (cfg->flags & COCOD_FLAG_DRY_RUN) != 0;
    ctx->s_compute = static_cast<hipStream_t>(cfg->compute_stream);
    ctx->s_avg = static_cast<hipStream_t>(cfg->avg_stream);
    ctx->live = cfg->xA;
    ctx->spare = cfg->xB;

    uint64_t global = 0;
    for (size_t t = 0; t < ctx->tensor_numel.size(); ++t) {
        const uint64_t span = cocod::kChunkElems;
        for (uint64_t off = 0; off < ctx->tensor_numel[t]; off += span) {
            const uint64_t left = ctx->tensor_numel[t] - off;
            Chunk ck{};
            ck.mem_quad = static_cast<uint32_t>((ctx->tensor_offset[t] + off) / 4);
            ck.glob_off = global + off;
            ck.n = static_cast<uint16_t>(left < span ? left : span);
            ck.after = static_cast<uint8_t>(left - ck.n < cocod::kLineElems ? left - ck.n : cocod::kLineElems);
            ck.first = off == 0;
            ctx->chunks.push_back(ck);
        }
        global += ctx->tensor_numel[t];
    }
    // Launch limits.  A grid dimension holds fewer than 2^32 THREADS.  The (tiles, workers) grid of the local
    // step has up to four single-wave blocks per chunk in x (fewer than 2^24 chunks: checked with the layout) and W <= 65535
    // in y (checked above); the orders that put more into ONE dimension (panels of a line-6 step, 1024-thread
    // blocks of the mean-forming steps) are only used below that limit (see enqueue_step).  The total is capped
    // as well, so that block counts stay inside 32-bit arithmetic everywhere.
    if (ctx->chunks.size() * static_cast<uint64_t>(cfg->W) > 0x7fffffffull) {
        delete ctx;
        return fail(nullptr, COCOD_ERR_INVALID, "W * d is too large for one launch (more than 2^31 chunks of 1024 elements)");
    }

    std::vector<float> weights;
    if (cfg->weights) weights.assign(cfg->weights, cfg->weights + cfg->W);
    ctx->cfg.weights = nullptr;
    std::vector<float> sigma_w;
    if (cfg->noise_sigma_w && cfg->grad == COCOD_GRAD_QUADRATIC) sigma_w.assign(cfg->noise_sigma_w, cfg->noise_sigma_w + cfg->W);
    ctx->cfg.noise_sigma_w = nullptr;

    if (!ctx->dry) {
        hipError_t e = hipMalloc(reinterpret_cast<void **>(&ctx->d_chunks), ctx->chunks.size() * sizeof(Chunk));
        if (e == hipSuccess)
            e = hipMemcpy(ctx->d_chunks, ctx->chunks.data(), ctx->chunks.size() * sizeof(Chunk), hipMemcpyHostToDevice);
        if (e == hipSuccess && !weights.empty()) {
            e = hipMalloc(reinterpret_cast<void **>(&ctx->d_weights), weights.size() * sizeof(float));
            if (e == hipSuccess)
                e = hipMemcpy(ctx->d_weights, weights.data(), weights.size() * sizeof(float), hipMemcpyHostToDevice);
        }
        if (e == hipSuccess && !sigma_w.empty()) {
            e = hipMalloc(reinterpret_cast<void **>(&ctx->d_sigma_w), sigma_w.size() * sizeof(float));
            if (e == hipSuccess)
                e = hipMemcpy(ctx->d_sigma_w, sigma_w.data(), sigma_w.size() * sizeof(float), hipMemcpyHostToDevice);
        }
        if (e == hipSuccess) {
            int dev = 0, cus = 0;
            e = hipGetDevice(&dev);
            if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
            ctx->compute_units = cus > 0 ? static_cast<uint32_t>(cus) : 0u;
        }
        if (e == hipSuccess && cfg->grad == COCOD_GRAD_MLP) {      // one work-space block, carved below
            const size_t wb = static_cast<size_t>(cfg->W) * cfg->mlp_batch;
            const size_t n_x = wb * cfg->mlp_in, n_h = wb * cfg->mlp_hidden, n_z = wb * cocod::mlp_dz_pitch();
            const uint32_t splits = cocod::mlp_forward_splits(cfg->W, cfg->mlp_in, cfg->mlp_hidden, cfg->mlp_batch, ctx->compute_units);
            e = hipMalloc(reinterpret_cast<void **>(&ctx->mlp_ws), (2 * n_x + (1 + splits) * n_h + n_z + 2 * wb) * sizeof(float));
            if (e == hipSuccess) {
                float *at = ctx->mlp_ws;
                ctx->mlp_X[0] = at; at += n_x;
                ctx->mlp_X[1] = at; at += n_x;
                ctx->mlp.fwd_splits = splits;
                ctx->mlp.H = at;  at += n_h;
                ctx->mlp.H_part = at; at += (splits - 1) * n_h;
                ctx->mlp.dA = at; at += n_h;
                ctx->mlp.dZ = at; at += n_z;
                ctx->mlp_y[0] = reinterpret_cast<int32_t *>(at); at += wb;
                ctx->mlp_y[1] = reinterpret_cast<int32_t *>(at);
                ctx->mlp.X = ctx->mlp_X[0];
                ctx->mlp.y = ctx->mlp_y[0];
            }
        }
        if (e == hipSuccess) e = scratch_for_current_device(&ctx->static_scratch);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_snap, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_mean, hipEventDisableTiming);
        if (e != hipSuccess) {
            const int code = (e == hipErrorOutOfMemory) ? COCOD_ERR_NOMEM : COCOD_ERR_HIP;
            fail(nullptr, code, "cocod_create: %s", hipGetErrorString(e));
            release(ctx);
            return code;
        }
    }
    *out = ctx;
    return COCOD_OK;
}

int cocod_destroy(cocod_ctx *ctx)
{
    if (!ctx) return COCOD_OK;
    int rc = COCOD_OK;
    if (!ctx->dry) {
        hipError_t e = hipStreamSynchronize(ctx->s_avg);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->s_compute);
        if (e != hipSuccess) rc = hip_fail(nullptr, e, "cocod_destroy");
    }
    release(ctx);
    return rc;
}

int cocod_sync(cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (ctx->dry) return COCOD_OK;
    COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_avg));
    COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_compute));
    return COCOD_OK;
}

// Panel order of the kernels that apply line 6 (see kPanelTiles): 4 * chunks * W single-wave blocks plus the
// padding of the last panel must fit one grid dimension.
static uint32_t panel_tiles_for(const cocod_ctx *ctx)
{
    return ctx->padded_d * sizeof(float) > kMeanCacheBytes &&
           (4 * ctx->chunks.size() + kPanelTiles) * static_cast<uint64_t>(ctx->cfg.W) * 64 < kMaxThreadsPerGridDim
               ? kPanelTiles : 0u;
}

// The next launch, of `steps` steps and with line 6 or without, can also form the round's mean itself: under the schedule that
// folds Step I into Step II the round's first launch reads exactly the stored models.
static bool step_forms_mean(const cocod_ctx *ctx, uint32_t steps, bool with_line6)
{
    if (ctx->schedule != COCOD_SCHED_HEAD || !ctx->mean_pending || !ctx->store_pending ||
        ctx->cfg.grad != COCOD_GRAD_QUADRATIC || ctx->chunks.size() >= kMaxChunksMeanStep) return false;
    const uint64_t quads = static_cast<uint64_t>(cocod::local_step_mean_quads_per_lane(ctx->cfg.W, with_line6));
    if (quads == 0) return false;
    if (steps == 1) return true;
    const uint64_t blocks = ctx->chunks.size() * (4 / quads), idle = blocks < ctx->compute_units ? ctx->compute_units - blocks : 0;
    return steps * ctx->cfg.W * quads * 256 * idle <= kIdleElementSteps * ctx->compute_units;
}

// Step timing: the next local step is one of those that were asked for, a launch of its own with timestamps.
static bool next_step_is_timed(const cocod_ctx *ctx) { return ctx->timing && ctx->t_used < ctx->t_limit; }

// Local steps that the next launch takes, of `left` still to take.
static uint32_t steps_per_launch(const cocod_ctx *ctx, int left)
{
    if (ctx->cfg.grad != COCOD_GRAD_QUADRATIC || next_step_is_timed(ctx)) return 1u;
    return static_cast<uint32_t>(left < kMaxStepsPerLaunch ? left : kMaxStepsPerLaunch);
}

// Where the launch that ends a captured round leaves t for the next one (no other launch of the round reads that word).
static uint32_t *step_next_for(const cocod_ctx *ctx, uint32_t steps)
{
    const bool last = ctx->capturing && ctx->step - ctx->capture_base + steps == ctx->capture_steps;
    return last ? ctx->d_step + (ctx->capture_word ^ 1u) : nullptr;
}

// `steps` local steps on the compute stream in one launch (an MLP step: in its three); with_line6 fuses line 6 into the
// last one (of a round).
static int enqueue_step(cocod_ctx *ctx, uint32_t steps, bool with_line6, const void *g_ext = nullptr, bool g_bf16 = false)
{
    // Keep the stored models intact: the first step of an open round reads them and
    // writes the spare buffer, which then becomes the live one.
    float *dst = ctx->store_pending ? ctx->spare : ctx->live;
    if (!ctx->dry && ctx->cfg.grad == COCOD_GRAD_MLP && !g_ext) {
        cocod::MlpParams p = ctx->mlp;             // work-space pointers
        // Mini-batch buffers: steps alternate between the two, and the context remembers for which step
        // index the next one is already filled (a captured round is keyed by both facts as they stand at
        // its first step, and leaves them as the same eager calls would).
        const uint32_t buf = ctx->batch_buf;
        p.X = ctx->mlp_X[buf];
        p.y = ctx->mlp_y[buf];
        p.X_next = ctx->mlp_X[buf ^ 1u];
        p.y_next = ctx->mlp_y[buf ^ 1u];
        p.have_batch = ctx->batch_ready_step == ctx->step;
        p.W = ctx->cfg.W;
        p.n_in = ctx->cfg.mlp_in; p.n_hid = ctx->cfg.mlp_hidden; p.n_out = ctx->cfg.mlp_out; p.batch = ctx->cfg.mlp_batch;
        p.stride = ctx->cfg.stride;
        p.x_in = ctx->live;
        p.x_out = dst;
        p.v = ctx->cfg.v;
        p.lr = ctx->cfg.lr;
        p.momentum = ctx->cfg.momentum;
        p.weight_decay = ctx->cfg.weight_decay;
        p.key0 = static_cast<uint32_t>(ctx->cfg.seed);
        p.key1 = static_cast<uint32_t>(ctx->cfg.seed >> 32);
        p.step = static_cast<uint32_t>(ctx->capturing ? ctx->step - ctx->capture_base : ctx->step);
        p.step_base = ctx->capturing ? ctx->d_step + ctx->capture_word : nullptr;
        p.step_next = step_next_for(ctx, steps);
        p.round_steps = ctx->capture_steps;
        p.snap = with_line6 ? ctx->snap : nullptr;
        p.mean = ctx->cfg.mean;
        const bool timed = next_step_is_timed(ctx);
        COCOD_HIP(ctx, cocod::launch_mlp_step(ctx->s_compute, p, timed ? ctx->t_start[ctx->t_used] : nullptr,
                                              timed ? ctx->t_stop[ctx->t_used] : nullptr));
        ctx->batch_last = buf;
        ctx->batch_buf = buf ^ 1u;
        ctx->batch_ready_step = ctx->step + 1;
        if (timed) {
            ctx->t_kind[ctx->t_used] = with_line6 ? 1 : 0;
            ctx->t_used += 1;
        }
    } else if (!ctx->dry) {
        cocod::StepParams p{};
        p.table = ctx->d_chunks;
        p.n_chunks = static_cast<uint32_t>(ctx->chunks.size());
        p.W = ctx->cfg.W;
        p.steps = steps;
        p.stride = ctx->cfg.stride;
        p.x_in = ctx->live;
        p.x_out = dst;
        p.v = ctx->cfg.v;
        p.h = ctx->cfg.h;
        p.c = ctx->cfg.c;
        p.g = static_cast<const float *>(g_ext);
        p.g_bf16 = g_bf16 ? 1u : 0u;
        p.snap = with_line6 ? ctx->snap : nullptr;
        p.mean = ctx->cfg.mean;
        p.lr = ctx->cfg.lr;
        p.momentum = ctx->cfg.momentum;
        p.weight_decay = ctx->cfg.weight_decay;
        p.sigma = ctx->cfg.noise_sigma;
        p.sigma_w = ctx->d_sigma_w;
        p.key0 = static_cast<uint32_t>(ctx->cfg.seed);
        p.key1 = static_cast<uint32_t>(ctx->cfg.seed >> 32);
        p.step = static_cast<uint32_t>(ctx->capturing ? ctx->step - ctx->capture_base : ctx->step);
        p.step_base = ctx->capturing ? ctx->d_step + ctx->capture_word : nullptr;
        p.step_next = step_next_for(ctx, steps);
        p.round_steps = ctx->capture_steps;
        p.panel_tiles = panel_tiles_for(ctx);
        p.cached = step_state_is_cached(ctx);
        // Step I inside the round's first launch, with line 6 in the same one a whole round in one pass over the stored models
        // (where that does not apply, the mean stays pending and is formed just before line 6)
        const bool forms_mean = !g_ext && step_forms_mean(ctx, steps, with_line6);
        if (forms_mean) {
            p.mean_out = ctx->cfg.mean;
            p.weights = ctx->d_weights;
            ctx->mean_pending = false;
        }
        hipEvent_t t0 = nullptr, t1 = nullptr;
        if (next_step_is_timed(ctx)) {
            t0 = ctx->t_start[ctx->t_used];
            t1 = ctx->t_stop[ctx->t_used];
            ctx->t_kind[ctx->t_used] = with_line6 ? 1 : (forms_mean ? 2 : 0);
            ctx->t_used += 1;
        }
        COCOD_HIP(ctx, cocod::launch_local_step(ctx->s_compute, p, t0, t1));
    }
    if (ctx->store_pending) {
        ctx->spare = ctx->live;
        ctx->live = dst;
        ctx->store_pending = false;
    }
    ctx->step += steps;
    return COCOD_OK;
}

static int check_steps(cocod_ctx *ctx, int k)
{
    if (k < 0) return fail(ctx, COCOD_ERR_INVALID, "k must be >= 0, got %d", k);
    if (ctx->step + static_cast<uint64_t>(k) > 0xffffffffull)
        return fail(ctx, COCOD_ERR_INVALID, "step counter would exceed 2^32 - 1");
    return COCOD_OK;
}

static int need_builtin_gradient(cocod_ctx *ctx)
{
    if (ctx->cfg.grad == COCOD_GRAD_EXTERNAL)
        return fail(ctx, COCOD_ERR_INVALID, "this context has no built-in gradient: use cocod_external_step");
    return COCOD_OK;
}

static int external_step(cocod_ctx *ctx, const void *g, bool bf16, int close_round)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (!g || (bf16 ? reinterpret_cast<uintptr_t>(g) % 8 != 0 : !aligned16(g)))
        return fail(ctx, COCOD_ERR_INVALID, "g must be a device pointer aligned to %d bytes", bf16 ? 8 : 16);
    if (close_round && !ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_external_step: no round is open to close");
    int rc = check_steps(ctx, 1);
    if (rc != COCOD_OK) return rc;
    if (close_round && !ctx->dry) {      // the mean is consumed inside this step
        rc = mean_before_line6(ctx);
        if (rc != COCOD_OK) return rc;
    }
    rc = enqueue_step(ctx, 1, close_round != 0, g, bf16);
    if (rc == COCOD_OK && close_round) {
        ctx->averaging = false;
        ctx->mean_pending = false;
        ctx->snap = nullptr;
    }
    return rc;
}

int cocod_external_step(cocod_ctx *ctx, const float *g, int close_round)
{
    return external_step(ctx, g, false, close_round);
}

int cocod_external_step_bf16(cocod_ctx *ctx, const uint16_t *g, int close_round)
{
    return external_step(ctx, g, true, close_round);
}

int cocod_local_steps(cocod_ctx *ctx, int k)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    int rc = check_steps(ctx, k);
    if (rc == COCOD_OK && k > 0) rc = need_builtin_gradient(ctx);
    for (int left = k; left > 0 && rc == COCOD_OK;) {
        const uint32_t n = steps_per_launch(ctx, left);
        rc = enqueue_step(ctx, n, false);
        left -= static_cast<int>(n);
    }
    return rc;
}

int cocod_local_steps_end_apply(cocod_ctx *ctx, int k)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (!ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_local_steps_end_apply: no round is open");
    int rc = check_steps(ctx, k);
    if (rc != COCOD_OK) return rc;
    if (k == 0) return cocod_average_end_apply(ctx);
    rc = need_builtin_gradient(ctx);
    if (rc != COCOD_OK) return rc;
    for (int left = k; left > 0;) {
        const uint32_t n = steps_per_launch(ctx, left);
        left -= static_cast<int>(n);
        if (left == 0 && !ctx->dry && !step_forms_mean(ctx, n, true)) {
            // the mean must be complete before the last launch starts: it is consumed inside it
            rc = mean_before_line6(ctx);
            if (rc != COCOD_OK) return rc;
        }
        rc = enqueue_step(ctx, n, left == 0);
        if (rc != COCOD_OK) return rc;
    }
    ctx->averaging = false;
    ctx->mean_pending = false;
    ctx->snap = nullptr;
    return COCOD_OK;
}

int cocod_average_begin(cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_average_begin: a round is already open");
    ctx->snap = ctx->live;
    if (!ctx->dry && ctx->schedule == COCOD_SCHED_OVERLAP) {
        const bool two_streams = on_avg_stream(ctx);
        if (two_streams) {
            COCOD_HIP(ctx, hipEventRecord(ctx->ev_snap, ctx->s_compute));
            COCOD_HIP(ctx, hipStreamWaitEvent(ctx->s_avg, ctx->ev_snap, 0));
        }
        const int rc = enqueue_mean(ctx, two_streams ? ctx->s_avg : ctx->s_compute);
        if (rc != COCOD_OK) return rc;
        if (two_streams) COCOD_HIP(ctx, hipEventRecord(ctx->ev_mean, ctx->s_avg));
    }
    ctx->averaging = true;
    ctx->store_pending = true;
    ctx->mean_pending = ctx->schedule != COCOD_SCHED_OVERLAP;
    return COCOD_OK;
}

int cocod_average_end_apply(cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (!ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_average_end_apply: no round is open");
    if (!ctx->dry) {
        const size_t n_buckets = ctx->bucket_begin.size() - 1;
        if (ctx->mean_pending && ctx->schedule != COCOD_SCHED_SERIAL) {     // FUSED, or HEAD with no step to ride on
            for (size_t b = 0; b < n_buckets; ++b)
                COCOD_HIP(ctx, cocod::launch_mean_correct(ctx->s_compute, ctx->live, ctx->snap, ctx->cfg.stride, ctx->cfg.W,
                                                          ctx->bucket_begin[b], ctx->bucket_begin[b + 1], ctx->d_weights,
                                                          ctx->cfg.mean));
        } else {
            const int rc = mean_before_line6(ctx);                                // SERIAL: the mean; OVERLAP: the join
            if (rc != COCOD_OK) return rc;
            {                                                                      // line 6, one launch for the whole list
                cocod::StepParams p{};
                p.table = ctx->d_chunks;
                p.n_chunks = static_cast<uint32_t>(ctx->chunks.size());
                p.W = ctx->cfg.W;
                p.stride = ctx->cfg.stride;
                p.x_in = ctx->live;
                p.x_out = ctx->live;
                p.snap = ctx->snap;
                p.mean = ctx->cfg.mean;
                p.panel_tiles = panel_tiles_for(ctx);
                p.cached = step_state_is_cached(ctx);
                COCOD_HIP(ctx, cocod::launch_line6(ctx->s_compute, p));
            }
        }
    }
    ctx->averaging = false;
    ctx->store_pending = false;
    ctx->mean_pending = false;
    ctx->snap = nullptr;
    return COCOD_OK;
}

int cocod_average_apply_fused(cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    const bool opened_here = !ctx->averaging;
    if (opened_here) {                   // blocking average of the live models: the stored models ARE the live ones
        ctx->snap = ctx->live;
        ctx->averaging = true;
        ctx->mean_pending = true;
    }
    if (!ctx->dry) {
        // a mean already running on the averaging stream (overlapped schedule) writes the same values to
        // `mean`: let it finish first so that the two writers never overlap
        if (!ctx->mean_pending && ctx->schedule == COCOD_SCHED_OVERLAP && ctx->s_avg != ctx->s_compute)
            COCOD_HIP(ctx, hipStreamWaitEvent(ctx->s_compute, ctx->ev_mean, 0));
        for (size_t b = 0; b + 1 < ctx->bucket_begin.size(); ++b)
            COCOD_HIP(ctx, cocod::launch_mean_correct(ctx->s_compute, ctx->live, ctx->snap, ctx->cfg.stride, ctx->cfg.W,
                                                      ctx->bucket_begin[b], ctx->bucket_begin[b + 1], ctx->d_weights,
                                                      ctx->cfg.mean));
    }
    ctx->averaging = false;
    ctx->store_pending = false;
    ctx->mean_pending = false;
    ctx->snap = nullptr;
    return COCOD_OK;
}

// Record one round into a graph.  Nothing executes; the context's state is put back afterwards.
static int capture_round(cocod_ctx *ctx, int k, int fused_tail, hipGraphExec_t *exec)
{
    float *const live = ctx->live, *const spare = ctx->spare;
    const uint64_t step = ctx->step;
    const bool timing = ctx->timing;
    const uint32_t batch_buf = ctx->batch_buf, batch_last = ctx->batch_last;
    const uint64_t batch_ready_step = ctx->batch_ready_step;
    ctx->timing = false;
    ctx->capturing = true;
    ctx->capture_base = step;
    ctx->capture_steps = static_cast<uint32_t>(k);
    ctx->capture_word = live == ctx->cfg.xA ? 0u : 1u;
    hipError_t e = hipStreamBeginCapture(ctx->s_compute, hipStreamCaptureModeThreadLocal);
    int rc = e == hipSuccess ? COCOD_OK : hip_fail(ctx, e, "hipStreamBeginCapture");
    hipGraph_t graph = nullptr;
    if (rc == COCOD_OK) {
        rc = cocod_average_begin(ctx);
        if (rc == COCOD_OK) {
            if (fused_tail) {
                rc = cocod_local_steps_end_apply(ctx, k);
            } else {
                rc = cocod_local_steps(ctx, k);
                if (rc == COCOD_OK) rc = cocod_average_end_apply(ctx);
            }
        }
        e = hipStreamEndCapture(ctx->s_compute, &graph);          // always: leaves the stream usable
        if (rc == COCOD_OK && e != hipSuccess) rc = hip_fail(ctx, e, "hipStreamEndCapture");
    }
    ctx->live = live; ctx->spare = spare; ctx->snap = nullptr;
    ctx->averaging = false; ctx->store_pending = false; ctx->mean_pending = false;
    ctx->step = step;
    ctx->batch_buf = batch_buf; ctx->batch_last = batch_last; ctx->batch_ready_step = batch_ready_step;
    ctx->timing = timing;
    ctx->capturing = false;
    if (rc == COCOD_OK) {
        e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) rc = hip_fail(ctx, e, "hipGraphInstantiate");
    }
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
}

int cocod_graph_round(cocod_ctx *ctx, int k, int fused_tail)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_graph_round: a round is already open");
    int rc = check_steps(ctx, k);
    if (rc == COCOD_OK && k > 0) rc = need_builtin_gradient(ctx);
    if (rc != COCOD_OK) return rc;
    // stream capture cannot record the null stream (nor the legacy default stream handle)
    if (!ctx->s_compute || ctx->s_compute == hipStreamLegacy)
        return fail(ctx, COCOD_ERR_INVALID, "cocod_graph_round needs a compute stream of its own: the null stream cannot be captured");
    fused_tail = fused_tail != 0;
    if (ctx->dry) {                                  // state transitions only
        rc = cocod_average_begin(ctx);
        if (rc == COCOD_OK) rc = fused_tail ? cocod_local_steps_end_apply(ctx, k) : cocod_local_steps(ctx, k);
        if (rc == COCOD_OK && !fused_tail) rc = cocod_average_end_apply(ctx);
        return rc;
    }
    if (!ctx->d_step) COCOD_HIP(ctx, hipMalloc(reinterpret_cast<void **>(&ctx->d_step), 2 * sizeof(uint32_t)));
    const bool live_is_A = ctx->live == ctx->cfg.xA;
    const bool mlp = ctx->cfg.grad == COCOD_GRAD_MLP && k > 0;
    const uint32_t batch_buf = mlp ? ctx->batch_buf : 0u;                    // which mini-batch buffer the first step reads,
    const bool batch_ready = mlp && ctx->batch_ready_step == ctx->step;      // and whether its batch is already there
    hipGraphExec_t exec = nullptr;
    for (const auto &g : ctx->graphs)
        if (g.k == k && g.fused_tail == fused_tail && g.schedule == ctx->schedule && g.live_is_A == live_is_A &&
            g.batch_buf == batch_buf && g.batch_ready == batch_ready) exec = g.exec;
    if (!exec) {
        rc = capture_round(ctx, k, fused_tail, &exec);
        if (rc != COCOD_OK) return rc;
        ctx->graphs.push_back({k, fused_tail, ctx->schedule, live_is_A, batch_buf, batch_ready, exec});
    }
    const uint32_t word = live_is_A ? 0u : 1u;
    if (k > 0 && ctx->d_step_value[word] != ctx->step) {     // eager calls since the last replay moved t
        COCOD_HIP(ctx, cocod::launch_set_word(ctx->s_compute, ctx->d_step + word, static_cast<uint32_t>(ctx->step)));
        ctx->d_step_value[word] = ctx->step;
    }
    COCOD_HIP(ctx, hipGraphLaunch(exec, ctx->s_compute));
    if (k > 0) {                                     // what the round's calls would have done to the host state
        float *t = ctx->live; ctx->live = ctx->spare; ctx->spare = t;
        ctx->step += static_cast<uint64_t>(k);
        ctx->d_step_value[word ^ 1u] = ctx->step;
        if (mlp) {                                   // k steps alternated the batch buffers; the last drew the next batch
            ctx->batch_last = (batch_buf + static_cast<uint32_t>(k - 1)) & 1u;
            ctx->batch_buf = ctx->batch_last ^ 1u;
            ctx->batch_ready_step = ctx->step;
        }
    }
    return COCOD_OK;
}

int cocod_set_schedule(cocod_ctx *ctx, int schedule)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (schedule != COCOD_SCHED_OVERLAP && schedule != COCOD_SCHED_SERIAL && schedule != COCOD_SCHED_FUSED &&
        schedule != COCOD_SCHED_HEAD)
        return fail(ctx, COCOD_ERR_INVALID, "unknown schedule %d", schedule);
    if (ctx->averaging) return fail(ctx, COCOD_ERR_STATE, "cocod_set_schedule: not while a round is open");
    ctx->schedule = schedule;
    return COCOD_OK;                     // graphs are keyed by schedule: nothing to drop
}

int cocod_set_lr(cocod_ctx *ctx, float lr)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (!std::isfinite(lr)) return fail(ctx, COCOD_ERR_INVALID, "lr is not finite");
    if (lr != ctx->cfg.lr && !ctx->graphs.empty()) {     // captured kernels carry the old step size
        COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_compute));
        for (auto &g : ctx->graphs) (void)hipGraphExecDestroy(g.exec);
        ctx->graphs.clear();
    }
    ctx->cfg.lr = lr;
    return COCOD_OK;
}

int cocod_get_step(const cocod_ctx *ctx, uint64_t *step)
{
    if (!ctx || !step) return fail(nullptr, COCOD_ERR_INVALID, "ctx and step must not be NULL");
    *step = ctx->step;
    return COCOD_OK;
}

int cocod_set_step(cocod_ctx *ctx, uint64_t step)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (step > 0xffffffffull) return fail(ctx, COCOD_ERR_INVALID, "step must be < 2^32");
    ctx->step = step;
    return COCOD_OK;
}

int cocod_live_model(const cocod_ctx *ctx, float **x_live)
{
    if (!ctx || !x_live) return fail(nullptr, COCOD_ERR_INVALID, "ctx and x_live must not be NULL");
    *x_live = ctx->live;
    return COCOD_OK;
}

int cocod_is_averaging(const cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    return ctx->averaging ? 1 : 0;
}

int cocod_get_plan(const cocod_ctx *ctx, uint64_t *padded_d, uint32_t *n_chunks, uint32_t *n_buckets)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (padded_d) *padded_d = ctx->padded_d;
    if (n_chunks) *n_chunks = static_cast<uint32_t>(ctx->chunks.size());
    if (n_buckets) *n_buckets = static_cast<uint32_t>(ctx->bucket_begin.size() - 1);
    return COCOD_OK;
}

int cocod_step_timing(cocod_ctx *ctx, int max_launches)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (max_launches < 0 || max_launches > (1 << 20)) return fail(ctx, COCOD_ERR_INVALID, "max_launches out of range");
    ctx->timing = false;
    ctx->t_used = 0;
    ctx->t_limit = 0;
    if (ctx->dry) return COCOD_OK;
    while (ctx->t_kind.size() < static_cast<size_t>(max_launches)) {
        hipEvent_t a = nullptr, b = nullptr;
        COCOD_HIP(ctx, hipEventCreate(&a));
        ctx->t_start.push_back(a);
        COCOD_HIP(ctx, hipEventCreate(&b));
        ctx->t_stop.push_back(b);
        ctx->t_kind.push_back(0);
    }
    ctx->timing = max_launches > 0;
    ctx->t_limit = static_cast<size_t>(max_launches);
    return COCOD_OK;
}

int cocod_step_timing_read(cocod_ctx *ctx, double total_ms[3], uint32_t launches[3])
{
    if (!ctx || !total_ms || !launches) return fail(nullptr, COCOD_ERR_INVALID, "ctx, total_ms and launches must not be NULL");
    total_ms[0] = total_ms[1] = total_ms[2] = 0.0;
    launches[0] = launches[1] = launches[2] = 0;
    if (ctx->dry) return COCOD_OK;
    COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_compute));
    for (size_t i = 0; i < ctx->t_used && i < ctx->t_stop.size(); ++i) {
        float ms = 0.0f;
        COCOD_HIP(ctx, hipEventElapsedTime(&ms, ctx->t_start[i], ctx->t_stop[i]));
        const int kind = ctx->t_kind[i];
        total_ms[kind] += ms;
        launches[kind] += 1;
    }
    ctx->t_used = 0;
    return COCOD_OK;
}

// Scratch of the diagnostics, on first use: block partials of two reductions, and the pinned words that receive the
// results (a copy of 8 bytes to ordinary host memory costs 10 us on the way to the caller).
static int diagnostics_scratch(cocod_ctx *ctx)
{
    if (!ctx->d_reduce)
        COCOD_HIP(ctx, hipMalloc(reinterpret_cast<void **>(&ctx->d_reduce), ctx->chunks.size() * 2 * sizeof(double)));
    if (!ctx->host_result)
        COCOD_HIP(ctx, hipHostMalloc(reinterpret_cast<void **>(&ctx->host_result), 2 * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent));
    return COCOD_OK;
}

int cocod_consensus_distance(cocod_ctx *ctx, double *result)
{
    if (!ctx || !result) return fail(nullptr, COCOD_ERR_INVALID, "ctx and result must not be NULL");
    *result = 0.0;
    if (ctx->dry) return COCOD_OK;
    const uint32_t n_chunks = static_cast<uint32_t>(ctx->chunks.size());
    const int rc = diagnostics_scratch(ctx);
    if (rc != COCOD_OK) return rc;
    COCOD_HIP(ctx, cocod::launch_consensus_distance(ctx->s_compute, ctx->d_chunks, n_chunks, ctx->live, ctx->cfg.stride,
                                                    ctx->cfg.W, ctx->d_weights, ctx->d_reduce, ctx->host_result));
    COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_compute));
    *result = ctx->host_result[0];
    return COCOD_OK;
}

int cocod_consensus_distance_noalloc(cocod_ctx *ctx, double *result_device)
{
    if (!ctx || !result_device) return fail(nullptr, COCOD_ERR_INVALID, "ctx and result_device must not be NULL");
    if (reinterpret_cast<uintptr_t>(result_device) % sizeof(double) != 0)
        return fail(ctx, COCOD_ERR_INVALID, "result_device must be 8-byte aligned");
    const uint64_t n_chunks = ctx->chunks.size();
    if (n_chunks > kNoAllocMaxChunks)
        return fail(ctx, COCOD_ERR_UNSUPPORTED,
                    "cocod_consensus_distance_noalloc: %llu chunks of 1024 parameters exceed the static scratch (%u chunks); "
                    "use cocod_consensus_distance", (unsigned long long)n_chunks, kNoAllocMaxChunks);
    if (ctx->dry) return COCOD_OK;
    // Every partial the final pass reads is written by this call's first pass: nothing has to start at zero.
    double *const partial = ctx->static_scratch + 2;
    COCOD_HIP(ctx, cocod::launch_consensus_distance(ctx->s_compute, ctx->d_chunks, static_cast<uint32_t>(n_chunks), ctx->live,
                                                    ctx->cfg.stride, ctx->cfg.W, ctx->d_weights, partial, result_device));
    return COCOD_OK;
}

int cocod_quadratic_objective(cocod_ctx *ctx, double *f_at_mean, double *grad_norm_sq_at_mean)
{
    if (!ctx || !f_at_mean || !grad_norm_sq_at_mean)
        return fail(nullptr, COCOD_ERR_INVALID, "ctx, f_at_mean and grad_norm_sq_at_mean must not be NULL");
    *f_at_mean = *grad_norm_sq_at_mean = 0.0;
    if (ctx->cfg.grad != COCOD_GRAD_QUADRATIC) return fail(ctx, COCOD_ERR_INVALID, "not a quadratic-gradient context");
    if (ctx->dry) return COCOD_OK;
    const uint32_t n_chunks = static_cast<uint32_t>(ctx->chunks.size());
    const int rc = diagnostics_scratch(ctx);
    if (rc != COCOD_OK) return rc;
    COCOD_HIP(ctx, cocod::launch_quadratic_objective(ctx->s_compute, ctx->d_chunks, n_chunks, ctx->live, ctx->cfg.h, ctx->cfg.c,
                                                     ctx->cfg.stride, ctx->cfg.W, ctx->d_weights, ctx->d_reduce,
                                                     ctx->host_result));
    COCOD_HIP(ctx, hipStreamSynchronize(ctx->s_compute));
    *f_at_mean = ctx->host_result[0];
    *grad_norm_sq_at_mean = ctx->host_result[1];
    return COCOD_OK;
}

int cocod_mlp_workspace(const cocod_ctx *ctx, float **X, float **H, float **dA, float **dZ, int32_t **y, uint32_t *dz_pitch)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (ctx->cfg.grad != COCOD_GRAD_MLP) return fail(nullptr, COCOD_ERR_INVALID, "not an MLP-gradient context");
    if (X) *X = ctx->mlp_X[ctx->batch_last];
    if (H) *H = ctx->mlp.H;
    if (dA) *dA = ctx->mlp.dA;
    if (dZ) *dZ = ctx->mlp.dZ;
    if (y) *y = ctx->mlp_y[ctx->batch_last];
    if (dz_pitch) *dz_pitch = static_cast<uint32_t>(cocod::mlp_dz_pitch());
    return COCOD_OK;
}

int cocod_fill_quadratic(cocod_ctx *ctx)
{
    if (!ctx) return fail(nullptr, COCOD_ERR_INVALID, "ctx is NULL");
    if (ctx->cfg.grad != COCOD_GRAD_QUADRATIC) return fail(ctx, COCOD_ERR_INVALID, "not a quadratic-gradient context");
    if (ctx->dry) return COCOD_OK;
    COCOD_HIP(ctx, cocod::launch_fill_quadratic(ctx->s_compute, ctx->d_chunks, static_cast<uint32_t>(ctx->chunks.size()),
                                                ctx->cfg.W, ctx->cfg.stride, ctx->padded_d,
                                                const_cast<float *>(ctx->cfg.h), const_cast<float *>(ctx->cfg.c),
                                                static_cast<uint32_t>(ctx->cfg.seed),
                                                static_cast<uint32_t>(ctx->cfg.seed >> 32)));
    return COCOD_OK;
}

int cocod_debug_copy(void *stream, const float *src, float *dst, uint64_t n)
{
    if (n == 0) return COCOD_OK;
    if (!src || !dst) return fail(nullptr, COCOD_ERR_INVALID, "src and dst must not be NULL");
    if ((n & 3u) || !aligned16(src) || !aligned16(dst))
        return fail(nullptr, COCOD_ERR_INVALID, "n must be a multiple of 4 and the pointers 16-byte aligned");
    const hipError_t e = cocod::launch_copy(static_cast<hipStream_t>(stream), src, dst, n / 4);
    if (e != hipSuccess) return hip_fail(nullptr, e, "cocod_debug_copy");
    return COCOD_OK;
}

int cocod_debug_normals(void *stream, uint64_t seed, uint32_t tag, uint32_t worker, uint32_t step, uint64_t j0,
                        uint64_t n, int fast, float *out)
{
    if (n == 0) return COCOD_OK;
    if (!out) return fail(nullptr, COCOD_ERR_INVALID, "out is NULL");
    if (j0 + n > (1ull << 34)) return fail(nullptr, COCOD_ERR_INVALID, "index range exceeds 2^34");
    const hipError_t e = cocod::launch_debug_normals(static_cast<hipStream_t>(stream), static_cast<uint32_t>(seed),
                                                     static_cast<uint32_t>(seed >> 32), tag, worker, step, j0, n, fast, out);
    if (e != hipSuccess) return hip_fail(nullptr, e, "cocod_debug_normals");
    return COCOD_OK;
}

}  // extern "C"
