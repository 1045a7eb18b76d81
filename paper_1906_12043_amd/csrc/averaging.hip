// Step I and line 6 of Algorithm 1 (CoCoD-SGD) on one GPU.
//
//   wmean         mean_j = sum_i p_i snap_ij           (the paper's all-reduce between workers)
//   mean_correct  the mean and line 6, x_ij = mean_j + (x_ij - snap_ij), in one pass (sequential
//                 schedule, nothing to overlap)
// (Line 6 on its own is a mode of the local-step kernel: a row-wise stream like the step itself.)
//
// Models are worker-major [W][stride], so the reduction runs along the SLOW axis:
// a thread owns one 16-byte column quad and walks the W rows with independent
// 16-byte loads; consecutive lanes own consecutive quads, so every wave load is
// 1 KiB contiguous.  The sum is taken in worker order 0..W-1 in fp32, which fixes
// the result bit for bit regardless of launch shape or schedule.
// In mean_correct the same thread then serves all W workers of its column for line 6, so each stored
// model is read once (12 + 4/W bytes per parameter).
#include "internal.hpp"
#include "mean_sum.hpp"

#include <type_traits>

namespace cocod {
namespace {

// Single-wave blocks.  Beside a local step made of single-wave blocks the workgroup dispatcher then gives
// the mean a fair share of the chip: measured at W = 16, d = 11.2 M the mean takes 0.20 ms next to the
// step with 64-thread blocks, 0.33 ms with 128 and 0.79 ms (the whole step) with 256 or 1024.  Alone the
// averaging kernels run at the same rate for every block size.
constexpr uint32_t kAvgThreads = 64;
constexpr uint32_t kXcds = 8;  // accelerator complex dies of the MI355X, each with its own L2
constexpr int kRowBatch = 8;   // independent row loads in flight per thread

typedef float f4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ void st4(float *p, const float4 &a) { *reinterpret_cast<float4 *>(p) = a; }
// models are streamed once per kernel and exceed the caches: non-temporal hint
__device__ __forceinline__ float4 ld4_stream(const float *p)
{
    const f4v t = __builtin_nontemporal_load(reinterpret_cast<const f4v *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void st4_stream(float *p, const float4 &a)
{
    __builtin_nontemporal_store(f4v{a.x, a.y, a.z, a.w}, reinterpret_cast<f4v *>(p));
}

// Ordered weighted sum over the rows of one column quad.  CACHED: ordinary loads, where the models are read again soon.
template <bool WEIGHTED, bool CACHED>
__device__ __forceinline__ float4 column_mean(const float *col, uint64_t stride, uint32_t W, const float *weights)
{
    auto load = [](const float *p) { return CACHED ? ld4(p) : ld4_stream(p); };
    MeanSum acc;
    acc.clear();
    uint32_t i = 0;
    for (; i + kRowBatch <= W; i += kRowBatch) {
        float4 r[kRowBatch];
        #pragma unroll
        for (int b = 0; b < kRowBatch; ++b) r[b] = load(col + static_cast<uint64_t>(i + b) * stride);
        #pragma unroll
        for (int b = 0; b < kRowBatch; ++b)
            acc.add<WEIGHTED>(WEIGHTED ? weights[i + b] : 1.0f, r[b].x, r[b].y, r[b].z, r[b].w);
    }
    for (; i < W; ++i) {
        const float4 r = load(col + static_cast<uint64_t>(i) * stride);
        acc.add<WEIGHTED>(WEIGHTED ? weights[i] : 1.0f, r.x, r.y, r.z, r.w);
    }
    acc.finish<WEIGHTED>(W);
    return make_float4(acc.s[0], acc.s[1], acc.s[2], acc.s[3]);
}

// CACHED: a state that stays in the last-level cache (step_state_is_cached): the step beside or behind reads the same models.
// Rounds of k = 2 with line 6 in the last step, mean in front of the steps, one context, streaming / ordinary loads: W = 8, d = 250 k
// 13.1 / 12.7 us, d = 1 M 41.8 / 39.4, W = 16, d = 700 k 49.3 / 48.6; three contexts in turn 11.8 / 11.1, 39.0 / 38.6, 54.3 / 53.3.
// The caller's fp32 gradient, mean beside the first step, k = 1: W = 8, d = 1 M 55.3 / 52.8, three contexts 37.2 / 37.4; W = 16,
// d = 400 k 46.2 / 44.2, 36.7 / 36.7; d = 700 k 62.1 / 59.7, 49.0 / 49.9; mean in front of the step W = 8, d = 250 k 10.8 / 10.1, 10.8 / 9.7,
// W = 16, d = 700 k 43.3 / 41.8, 43.9 / 45.1; k = 2 and k = 8 the same or up to 4 % faster.  So where three contexts together are far
// beyond the cache a round of one step loses 2 %, and one by itself gains 4.  Perceptron rounds, mean beside the forward product,
// k = 1 and 2: W = 16, 768-512-10 83.9 / 82.8, 128.2 / 126.5, three contexts 65.8 / 65.0, 110.8 / 109.2; from a graph, k = 2, W = 4,
// 768-768-10 98.0 / 95.2, 67.9 / 66.2.
template <bool WEIGHTED, bool CACHED>
__global__ __launch_bounds__(kAvgThreads) void wmean_kernel(const float *snap, uint64_t stride, uint32_t W,
                                                            uint64_t begin, uint64_t n_quads,
                                                            const float *weights, float *mean)
{
    // Line 6 waits for this kernel while the local step beside it has no one waiting: its waves issue first
    // (0.20 -> 0.18 ms next to the step; the round's time does not change).
    __builtin_amdgcn_s_setprio(3);
    const uint64_t quad = static_cast<uint64_t>(blockIdx.x) * kAvgThreads + threadIdx.x;
    if (quad >= n_quads) return;
    const uint64_t e = begin + quad * 4;
    st4(mean + e, column_mean<WEIGHTED, CACHED>(snap + e, stride, W, weights));
}

__device__ __forceinline__ void correct_column(float *xcol, const float *scol, const float4 m, uint64_t stride, uint32_t W)
{
    constexpr int B = 4;
    uint32_t i = 0;
    for (; i + B <= W; i += B) {
        float4 xr[B], sr[B];
        #pragma unroll
        for (int b = 0; b < B; ++b) {
            xr[b] = ld4_stream(xcol + static_cast<uint64_t>(i + b) * stride);
            sr[b] = ld4_stream(scol + static_cast<uint64_t>(i + b) * stride);
        }
        #pragma unroll
        for (int b = 0; b < B; ++b) {
            float4 o;
            o.x = m.x + (xr[b].x - sr[b].x); o.y = m.y + (xr[b].y - sr[b].y);
            o.z = m.z + (xr[b].z - sr[b].z); o.w = m.w + (xr[b].w - sr[b].w);
            st4_stream(xcol + static_cast<uint64_t>(i + b) * stride, o);
        }
    }
    for (; i < W; ++i) {
        const float4 xr = ld4_stream(xcol + static_cast<uint64_t>(i) * stride);
        const float4 sr = ld4_stream(scol + static_cast<uint64_t>(i) * stride);
        float4 o;
        o.x = m.x + (xr.x - sr.x); o.y = m.y + (xr.y - sr.y);
        o.z = m.z + (xr.z - sr.z); o.w = m.w + (xr.w - sr.w);
        st4_stream(xcol + static_cast<uint64_t>(i) * stride, o);
    }
}

// R > 0: W <= R and the column's stored models stay in registers between the two passes, so each is read from
// memory once (12 + 4/W bytes per parameter).  R == 0: any W, the stored models are read a second time for line 6.
// V: elements per thread, a column quad or (above 32 workers, to keep the rows in 128 registers) a column pair.
// SAME: the models ARE the stored models (the blocking average of Local SGD): x is not read again, 8 + 4/W bytes.
// LINES: every row starts on a 128-byte line.  Off the lines a wave's kilobyte of a row leaves half a line at both ends;
// there the stores are ordinary ones and an XCD owns a contiguous run of columns, so that neighbouring waves'
// halves meet in its L2.
// Memory bounds all of it.  Blocking average, before (rows read up to three times) and now: W = 16, d = 11.2 M 380 -> 255 us
// (5.6 TB/s of 8 bytes), W = 21, d = 4.0 M 183 -> 128, W = 64, d = 5.6 M 784 -> 546; the same off the lines 457 -> 315,
// 220 -> 132, 967 -> 636 (with streaming stores in plain block order 320, 151, 785).  Open round, W = 21: 245 -> 180 us, W = 64:
// 1076 -> 829.  On the lines the plain order with streaming stores is the faster one (W = 16: 247 us against 290).
constexpr int mean_correct_waves(int R) { return R == 0 || R <= 8 ? 8 : R <= 16 ? 4 : 3; }    // per SIMD: the rows of a thread and a batch of x fit
template <bool WEIGHTED, int R, int V, bool SAME, bool LINES>
__global__ __launch_bounds__(kAvgThreads, mean_correct_waves(R)) void mean_correct_kernel(float *x, const float *snap, uint64_t stride,
                                                                   uint32_t W, uint64_t begin, uint64_t n_groups,
                                                                   const float *weights, float *mean)
{
    #pragma clang fp contract(off)
    uint32_t block = blockIdx.x;
    if (!LINES) {
        const uint32_t run = gridDim.x / kXcds;                // what does not divide stays in place at the end
        if (block < run * kXcds) block = (block % kXcds) * run + block / kXcds;
    }
    const uint64_t group = static_cast<uint64_t>(block) * kAvgThreads + threadIdx.x;
    if (group >= n_groups) return;
    const uint64_t e = begin + group * V;
    if constexpr (R == 0) {
        const float4 m = column_mean<WEIGHTED, false>(snap + e, stride, W, weights);
        st4(mean + e, m);
        correct_column(x + e, snap + e, m, stride, W);
    } else {
        typedef float fv __attribute__((ext_vector_type(V)));
        fv s[R];
        #pragma unroll
        for (int i = 0; i < R; ++i)                            // guards, not breaks: the loops must unroll fully or s[] goes to scratch
            if (static_cast<uint32_t>(i) < W)
                s[i] = __builtin_nontemporal_load(reinterpret_cast<const fv *>(snap + e + static_cast<uint64_t>(i) * stride));
        MeanSumN<V> acc;
        acc.clear();
        #pragma unroll
        for (int i = 0; i < R; ++i)                            // same order and operations as column_mean
            if (static_cast<uint32_t>(i) < W) {
                #pragma unroll
                for (int c = 0; c < V; ++c) acc.template add_one<WEIGHTED>(c, WEIGHTED ? weights[i] : 1.0f, s[i][c]);
            }
        acc.template finish<WEIGHTED>(W);
        fv m;
        #pragma unroll
        for (int c = 0; c < V; ++c) m[c] = acc.s[c];
        *reinterpret_cast<fv *>(mean + e) = m;
        auto put = [&](int i, const fv xr) {
            fv *to = reinterpret_cast<fv *>(x + e + static_cast<uint64_t>(i) * stride);
            if (LINES) __builtin_nontemporal_store(m + (xr - s[i]), to);
            else       *to = m + (xr - s[i]);
        };
        auto get = [&](int i) { return __builtin_nontemporal_load(reinterpret_cast<const fv *>(x + e + static_cast<uint64_t>(i) * stride)); };
        constexpr int B = 4;                                   // rows of x in flight
        #pragma unroll
        for (int i0 = 0; i0 < R; i0 += B) {
            if (SAME || static_cast<uint32_t>(i0 + B) > W) {
                #pragma unroll
                for (int i = i0; i < i0 + B; ++i)
                    if (static_cast<uint32_t>(i) < W) put(i, SAME ? s[i] : get(i));
            } else {
                fv xr[B];
                #pragma unroll
                for (int b = 0; b < B; ++b) xr[b] = get(i0 + b);
                #pragma unroll
                for (int b = 0; b < B; ++b) put(i0 + b, xr[b]);
                __builtin_amdgcn_sched_barrier(0);             // or the loads of all batches are hoisted into registers
            }
        }
    }
}

// ---- consensus distance: sum_i p_i || xbar - x_i ||^2 with xbar = sum_i p_i x_i ---------------------
// (the quantity bounded by Lemma 2 of the paper).  A scalar, so this is where wave and LDS reductions
// belong: per thread a column quad or pair, then a butterfly over the wave, the four wave sums through LDS, one double
// per block; a second one-block kernel adds the block partials in a fixed order, so the result is deterministic.
__device__ __forceinline__ double wave_sum_f64(double v)
{
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// R > 0: up to R workers a thread holds V columns of every row in registers and reads each model once; R == 0: any W,
// two passes over the rows.  (This kernel alone, W = 64, d = 2.8 M: two passes 202 us, the second one mostly from memory
// again, as the rows of the blocks in flight are far more than L2 holds; column pairs in registers 123 us = 5.8 TB/s.
// W = 21, d = 4.0 M: 101 -> 53 us; W = 1, d = 10 M, where registers for 16 rows cost occupancy: 16 -> 12.)
template <bool WEIGHTED, int R, int V>
__global__ __launch_bounds__(kStepThreads, R > 16 ? 3 : 4) void consensus_partial_kernel(const Chunk *table, const float *x, uint64_t stride,
                                                                                                 uint32_t W, const float *weights, double *partial)
{
    __shared__ double wave_part[kStepThreads / 64];
    const Chunk ck = table[blockIdx.x];
    const float uniform = 1.0f / static_cast<float>(W);
    double local = 0.0;
    auto columns = [&](uint32_t e) {
        const float *col = x + static_cast<uint64_t>(ck.mem_quad) * 4 + e;
        float acc[V], m[V];
        #pragma unroll
        for (int c = 0; c < V; ++c) acc[c] = 0.0f;
        auto add_row = [&](uint32_t i, const auto &r) {
            const float pw = WEIGHTED ? weights[i] : uniform;
            #pragma unroll
            for (int c = 0; c < V; ++c) acc[c] += pw * (r[c] - m[c]) * (r[c] - m[c]);
        };
        typedef float fv __attribute__((ext_vector_type(V)));
        if constexpr (R > 0) {
            fv r[R];                                          // every row is requested at once (the guards are uniform over the grid)
            #pragma unroll
            for (int i = 0; i < R; ++i)
                if (static_cast<uint32_t>(i) < W) r[i] = __builtin_nontemporal_load(reinterpret_cast<const fv *>(col + static_cast<uint64_t>(i) * stride));
            MeanSumN<V> ms;
            ms.clear();
            #pragma unroll
            for (int i = 0; i < R; ++i)
                if (static_cast<uint32_t>(i) < W) {
                    #pragma unroll
                    for (int c = 0; c < V; ++c) ms.template add_one<WEIGHTED>(c, WEIGHTED ? weights[i] : 1.0f, r[i][c]);
                }
            ms.template finish<WEIGHTED>(W);
            #pragma unroll
            for (int c = 0; c < V; ++c) m[c] = ms.s[c];
            #pragma unroll
            for (int i = 0; i < R; ++i)
                if (static_cast<uint32_t>(i) < W) add_row(i, r[i]);
        } else {
            static_assert(V == 4, "column quads");
            const float4 mean = column_mean<WEIGHTED, true>(col, stride, W, weights);
            m[0] = mean.x; m[1] = mean.y; m[2] = mean.z; m[3] = mean.w;
            uint32_t i = 0;
            for (; i + kRowBatch <= W; i += kRowBatch) {
                fv r[kRowBatch];
                #pragma unroll
                for (int b = 0; b < kRowBatch; ++b) r[b] = *reinterpret_cast<const fv *>(col + static_cast<uint64_t>(i + b) * stride);
                #pragma unroll
                for (int b = 0; b < kRowBatch; ++b) add_row(i + b, r[b]);
            }
            for (; i < W; ++i) add_row(i, *reinterpret_cast<const fv *>(col + static_cast<uint64_t>(i) * stride));
        }
        #pragma unroll
        for (int c = 0; c < V; ++c)                           // alignment pads of a tensor's tail quad do not count
            if (e + c < ck.n) local += static_cast<double>(acc[c]);
    };
    if (threadIdx.x * V < ck.n) columns(threadIdx.x * V);
    if (V * kStepThreads < kChunkElems)
        for (uint32_t e = (kStepThreads + threadIdx.x) * V; e < ck.n; e += kStepThreads * V) columns(e);
    local = wave_sum_f64(local);
    if (threadIdx.x % 64 == 0) wave_part[threadIdx.x / 64] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (uint32_t w = 0; w < kStepThreads / 64; ++w) s += wave_part[w];
        partial[blockIdx.x] = s;
    }
}

// block b adds the b-th run of n block partials into out[b] (one block is a chain of load latencies: sixteen waves, four
// loads in flight each: n = 2735 6.3 -> 5.8 us, n = 9766 about 16 -> 8 us)
constexpr uint32_t kFinalThreads = 1024;
__global__ __launch_bounds__(kFinalThreads) void consensus_final_kernel(const double *partial, uint32_t n, double *out)
{
    __shared__ double wave_part[kFinalThreads / 64];
    partial += static_cast<uint64_t>(blockIdx.x) * n;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint32_t i = threadIdx.x; i < n; i += 4 * kFinalThreads) {
        #pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (i + u * kFinalThreads < n) sum[u] += partial[i + u * kFinalThreads];
    }
    const double local = wave_sum_f64((sum[0] + sum[1]) + (sum[2] + sum[3]));
    if (threadIdx.x % 64 == 0) wave_part[threadIdx.x / 64] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        #pragma unroll
        for (uint32_t w = 0; w < kFinalThreads / 64; ++w) s += wave_part[w];
        out[blockIdx.x] = s;
    }
}

// ---- the objective of the paper's problem definition at the averaged model ------------------------
// f(xbar) = sum_i p_i f_i(xbar) with the workers' quadratics f_i(x) = 1/2 sum_j h_ij (x_j - c_ij)^2 and
// xbar = sum_i p_i x_i, and || grad f(xbar) ||^2 (the quantity whose running mean Theorem 1 bounds),
// grad f(xbar)_j = sum_i p_i h_ij (xbar_j - c_ij).  Same reduction structure as the consensus distance;
// partial holds two runs of gridDim.x doubles (objective, squared gradient norm).
template <bool WEIGHTED>
__global__ __launch_bounds__(kStepThreads) void objective_partial_kernel(const Chunk *table, const float *x, const float *h,
                                                                         const float *c, uint64_t stride, uint32_t W,
                                                                         const float *weights, double *partial)
{
    __shared__ double wave_part[2][kStepThreads / 64];
    const Chunk ck = table[blockIdx.x];
    const uint32_t e = threadIdx.x * 4;
    double f_local = 0.0, g_local = 0.0;
    if (e < ck.n) {
        const uint64_t at = static_cast<uint64_t>(ck.mem_quad) * 4 + e;
        const float uniform = 1.0f / static_cast<float>(W);
        const float4 m = column_mean<WEIGHTED, true>(x + at, stride, W, weights);
        float4 f = make_float4(0.f, 0.f, 0.f, 0.f), g = make_float4(0.f, 0.f, 0.f, 0.f);
        auto add_row = [&](uint32_t i, const float4 &hr, const float4 &cr) {
            const float pw = WEIGHTED ? weights[i] : uniform;
            const float4 dl = make_float4(m.x - cr.x, m.y - cr.y, m.z - cr.z, m.w - cr.w);
            g.x += pw * hr.x * dl.x; g.y += pw * hr.y * dl.y; g.z += pw * hr.z * dl.z; g.w += pw * hr.w * dl.w;
            f.x += pw * hr.x * dl.x * dl.x; f.y += pw * hr.y * dl.y * dl.y;
            f.z += pw * hr.z * dl.z * dl.z; f.w += pw * hr.w * dl.w * dl.w;
        };
        uint32_t i = 0;
        for (; i + kRowBatch <= W; i += kRowBatch) {              // h and c are read once: streamed, a batch of rows in flight
            float4 hr[kRowBatch], cr[kRowBatch];
            #pragma unroll
            for (int b = 0; b < kRowBatch; ++b) {
                hr[b] = ld4_stream(h + at + static_cast<uint64_t>(i + b) * stride);
                cr[b] = ld4_stream(c + at + static_cast<uint64_t>(i + b) * stride);
            }
            #pragma unroll
            for (int b = 0; b < kRowBatch; ++b) add_row(i + b, hr[b], cr[b]);
        }
        for (; i < W; ++i)
            add_row(i, ld4_stream(h + at + static_cast<uint64_t>(i) * stride), ld4_stream(c + at + static_cast<uint64_t>(i) * stride));
        const uint32_t keep = ck.n - e;                   // alignment pads of a tensor's tail quad do not count
        f_local = static_cast<double>(f.x);              g_local = static_cast<double>(g.x) * g.x;
        if (keep > 1) { f_local += static_cast<double>(f.y); g_local += static_cast<double>(g.y) * g.y; }
        if (keep > 2) { f_local += static_cast<double>(f.z); g_local += static_cast<double>(g.z) * g.z; }
        if (keep > 3) { f_local += static_cast<double>(f.w); g_local += static_cast<double>(g.w) * g.w; }
        f_local *= 0.5;
    }
    f_local = wave_sum_f64(f_local);
    g_local = wave_sum_f64(g_local);
    if (threadIdx.x % 64 == 0) { wave_part[0][threadIdx.x / 64] = f_local; wave_part[1][threadIdx.x / 64] = g_local; }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0.0;
        for (uint32_t w = 0; w < kStepThreads / 64; ++w) s += wave_part[threadIdx.x][w];
        partial[static_cast<uint64_t>(threadIdx.x) * gridDim.x + blockIdx.x] = s;
    }
}

inline uint32_t blocks_for(uint64_t n_quads) { return static_cast<uint32_t>((n_quads + kAvgThreads - 1) / kAvgThreads); }

}  // namespace

hipError_t launch_wmean(hipStream_t stream, const float *snap, uint64_t stride, uint32_t W, uint64_t begin,
                        uint64_t end, const float *weights, float *mean, bool cached)
{
    const uint64_t n_quads = (end - begin) / 4;
    if (n_quads == 0) return hipSuccess;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks_for(n_quads)), dim3(kAvgThreads), 0, stream, snap, stride, W, begin, n_quads, weights, mean);
        return hipGetLastError();
    };
    if (cached) return weights ? launch(wmean_kernel<true, true>) : launch(wmean_kernel<false, true>);
    return weights ? launch(wmean_kernel<true, false>) : launch(wmean_kernel<false, false>);
}

hipError_t launch_mean_correct(hipStream_t stream, float *x, const float *snap, uint64_t stride, uint32_t W,
                               uint64_t begin, uint64_t end, const float *weights, float *mean)
{
    const uint64_t n_quads = (end - begin) / 4;
    if (n_quads == 0) return hipSuccess;
    auto launch = [&](auto kernel, uint32_t v) {
        hipLaunchKernelGGL(kernel, dim3(blocks_for((end - begin) / v)), dim3(kAvgThreads), 0, stream, x, snap, stride, W, begin,
                           (end - begin) / v, weights, mean);
        return hipGetLastError();
    };
    auto rows = [&](auto weighted, auto same, auto lines) {
        constexpr bool WT = decltype(weighted)::value, SAME = decltype(same)::value, LINES = decltype(lines)::value;
        if (W <= 8) return launch(mean_correct_kernel<WT, 8, 4, SAME, LINES>, 4);
        if (W <= 16) return launch(mean_correct_kernel<WT, 16, 4, SAME, LINES>, 4);
        if (W <= 32) return launch(mean_correct_kernel<WT, 32, 4, SAME, LINES>, 4);
        if (W <= 64) return launch(mean_correct_kernel<WT, 64, 2, SAME, LINES>, 2);
        return launch(mean_correct_kernel<WT, 0, 4, false, true>, 4);
    };
    using T = std::true_type;
    using F = std::false_type;
    const bool lines = W == 1 || ((reinterpret_cast<uintptr_t>(x + begin) | stride * sizeof(float)) & 127u) == 0;
    auto with_rows = [&](auto weighted, auto same) { return lines ? rows(weighted, same, T{}) : rows(weighted, same, F{}); };
    if (x == snap) return weights ? with_rows(T{}, T{}) : with_rows(F{}, T{});
    return weights ? with_rows(T{}, F{}) : with_rows(F{}, F{});
}

hipError_t launch_consensus_distance(hipStream_t stream, const Chunk *table, uint32_t n_chunks, const float *x,
                                     uint64_t stride, uint32_t W, const float *weights, double *partial, double *out)
{
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(n_chunks), dim3(kStepThreads), 0, stream, table, x, stride, W, weights, partial); };
    auto rows = [&](auto weighted) {
        constexpr bool WT = decltype(weighted)::value;
        if (W <= 8) launch(consensus_partial_kernel<WT, 8, 4>);
        else if (W <= 16) launch(consensus_partial_kernel<WT, 16, 4>);
        else if (W <= 32) launch(consensus_partial_kernel<WT, 32, 4>);
        else if (W <= 64) launch(consensus_partial_kernel<WT, 64, 2>);
        else launch(consensus_partial_kernel<WT, 0, 4>);
    };
    if (weights) rows(std::true_type{}); else rows(std::false_type{});
    hipLaunchKernelGGL(consensus_final_kernel, dim3(1), dim3(kFinalThreads), 0, stream, partial, n_chunks, out);
    return hipGetLastError();
}

hipError_t launch_quadratic_objective(hipStream_t stream, const Chunk *table, uint32_t n_chunks, const float *x,
                                      const float *h, const float *c, uint64_t stride, uint32_t W, const float *weights,
                                      double *partial, double *out)
{
    if (weights) hipLaunchKernelGGL((objective_partial_kernel<true>), dim3(n_chunks), dim3(kStepThreads), 0, stream, table, x, h, c, stride, W, weights, partial);
    else         hipLaunchKernelGGL((objective_partial_kernel<false>), dim3(n_chunks), dim3(kStepThreads), 0, stream, table, x, h, c, stride, W, weights, partial);
    hipLaunchKernelGGL(consensus_final_kernel, dim3(2), dim3(kFinalThreads), 0, stream, partial, n_chunks, out);
    return hipGetLastError();
}

}  // namespace cocod
