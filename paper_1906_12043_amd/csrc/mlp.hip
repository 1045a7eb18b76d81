// Step II of Algorithm 1 (CoCoD-SGD) with a REAL mini-batch gradient: every worker is a two-layer
// perceptron  A = X W1 + b1, H = relu(A), Z = H W2 + b2, loss = mean softmax cross-entropy,
// on a fresh seeded mini-batch per (worker, step); all W workers advance in the same launches.
//
// One local step = three launches on the compute stream (four for a step whose mini-batch no earlier
// step has drawn: gen_batch in front):
//   gemm<FWD>      X W1, in K splits                           [B x in] x [in x hid]
//   head           H = relu(X W1 + b1), Z = H W2 + b2, softmax, dZ = (P - onehot)/B, dA = (dZ W2^T) * [H > 0]
//                  (sixteen samples per block, fp32 matrix instructions)
//   gemm<BWD>      dW1 = X^T dA with the momentum-SGD update of W1 fused into the epilogue
//                  (the 12.6 MB gradient of W1 never goes to memory)   [in x B] x [B x hid]; its first blocks
//                  update W2, b2, b1 (dW2 = H^T dZ, db2, db1 = colsum(dA)), and every block draws a share of the
//                  NEXT step's X and labels from the counter-based generator into the other of two batch buffers
//
// The two big contractions (98 % of the flops) run on the 16-bit matrix instructions at fp32 accuracy: every fp32
// operand is split exactly into three bf16 values (8 + 8 + 8 bits), and six of the nine partial products are formed with
// fp32 accumulation; the three left out are below 2^-24 of the product together.  The leading products and the small ones
// have accumulators of their own, so the long chain of additions has one rounding per 16 products.  Against 64 bits
// (W = 16, 3072-1024-10, batch 128) H = relu(X W1 + b1) is off by 2.4e-7 and dW1 by 5.9e-8 of their norms; the fp32 matrix
// instruction gave 1.0e-6 and 1.46e-7.  Columns far below the others, sums of one term and operands down to the
// smallest fp32 numbers are as exact.  (fp16 pairs with three products are half the matrix work, forward 61 us against 93,
// backward 143 against 160 at that shape, but hold 22 bits and need scales: a sum of one term was off by up to 2^-11, a
// column of dA 2^-45 of the largest was lost.)
// The fp32 instruction peaks at 157 TFLOP/s; six bf16 products per fp32 product cost two fifths of its time.
//
// GEMM kernel: 256 threads, four waves, each with 32 columns of the block's tile and all of its rows (128 forward,
// 64 backward).  A (the mini-batch) goes through LDS in slices of K = 32, two buffers and one barrier per slice: loaded as
// fp32, split in registers on its way into LDS, read back as 16-byte operand pieces by every wave.  B (W1 or dA) belongs to
// one wave alone: eight consecutive k of a column per lane, straight from memory into the operand registers.  (With both
// operands in LDS the backward product's reads took longer than its multiplies: W = 6, 1024-2048-10, batch 512, 115 us
// against 108, the forward one 102 against 88.)  No transposed copy is ever written.
#include "internal.hpp"
#include "philox.hpp"

#include <hip/hip_ext.h>

#include <type_traits>

namespace cocod {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

constexpr int kBK = 32;               // K slice staged through LDS
constexpr int kShapeM = 128, kShapeN = 64;   // shape contract: n_in, batch multiples of 128; n_hid of 64
constexpr int kMaxOut = 16;
constexpr uint32_t kXcds = 8;                // accelerator complex dies of the MI355X
constexpr uint64_t kMaxHiddenOut = 32768;    // and n_hid * (n_out rounded up to odd) is at most this

struct Offsets { uint64_t W1, b1, W2, b2; };
__host__ __device__ inline Offsets offsets_of(const MlpParams &p)
{
    Offsets o;
    o.W1 = 0;
    o.b1 = static_cast<uint64_t>(p.n_in) * p.n_hid;
    o.W2 = o.b1 + p.n_hid;
    o.b2 = o.W2 + static_cast<uint64_t>(p.n_hid) * p.n_out;
    return o;
}

// g = G + lambda x ; v = mu v + g ; x' = x - gamma v   (same update as the quadratic step)
__device__ __forceinline__ void sgd_update(const MlpParams &p, uint64_t row, uint64_t e, float G)
{
    const uint64_t at = row + e;              // worker's row of the model buffers, element in it
    const float x = p.x_in[at];
    float g = G + p.weight_decay * x;
    if (p.momentum != 0.0f) {
        const float v = p.momentum * p.v[at] + g;
        p.v[at] = v;
        g = v;
    }
    float x_new = x - p.lr * g;
    if (p.snap) x_new = p.mean[e] + (x_new - p.snap[at]);     // line 6 (last step of a round)
    p.x_out[at] = x_new;
}

// ---- mini-batch ---------------------------------------------------------------------------------
// X[b][f] = normal(stream X, worker, step, flat index b*n_in + f);
// y[b] = (word * n_out) >> 32 from stream Y at index b.
// One 256-thread group's share (thread tid of group `block`) of a worker's mini-batch for local step
// `step`: 256 quads of X, and in group 0 the labels.
__device__ __forceinline__ void gen_batch_block(const MlpParams &p, uint32_t block, uint32_t tid, uint32_t worker, uint32_t step,
                                                float *X_all, int32_t *y_all)
{
    const uint64_t n_quads = static_cast<uint64_t>(p.batch) * p.n_in / 4;
    const uint64_t q = static_cast<uint64_t>(block) * 256 + tid;
    if (q < n_quads) {
        const Normals4 z = box_muller_fast(philox4x32_10(static_cast<uint32_t>(q), step, worker, kTagMlpX, p.key0, p.key1));
        float *X = X_all + static_cast<uint64_t>(worker) * p.batch * p.n_in;
        *reinterpret_cast<f4 *>(X + q * 4) = f4{z.z[0], z.z[1], z.z[2], z.z[3]};
    }
    if (block == 0 && tid < p.batch / 4) {
        const Words4 r = philox4x32_10(tid, step, worker, kTagMlpY, p.key0, p.key1);
        #pragma unroll
        for (int i = 0; i < 4; ++i)
            y_all[static_cast<uint64_t>(worker) * p.batch + tid * 4 + i] =
                static_cast<int32_t>((static_cast<uint64_t>(r.w[i]) * p.n_out) >> 32);
    }
}

__host__ __device__ inline uint32_t gen_batch_blocks(const MlpParams &p)
{
    return static_cast<uint32_t>((static_cast<uint64_t>(p.batch) * p.n_in / 4 + 255) / 256);
}

__global__ __launch_bounds__(256) void gen_batch_kernel(const MlpParams p)
{
    const uint32_t step = p.step_base ? *p.step_base + p.step : p.step;
    gen_batch_block(p, blockIdx.x, threadIdx.x, blockIdx.y, step, p.X, p.y);
}

// ---- output layer -----------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v)
{
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Output layer, forward and backward, for sixteen samples of one worker per block:
//   H = relu(sum of the forward product's K splits + b1), Z = H W2 + b2, softmax (row maximum subtracted),
//   dZ = (P - onehot(y)) / batch, dA = (dZ W2^T) * [H > 0].
// Memory is touched a row at a time: a wave takes one sample's row in 1 KiB pieces and puts it into LDS, and dA leaves
// the same way (reading the rows straight into the products' operand layout, 64 bytes from each of 16 rows 4 KiB
// apart, took 25 us instead of 17 us at W = 16, 3072-1024-10, batch 128, four K splits).  Both products run on the fp32 matrix
// instruction 16x16x4; a wave owns every sixteenth block of 16 hidden units, and a lane's four consecutive units of
// one sample are at once the A operand of Z = H W2 (quarter j of a block's 16 k in instruction j) and the result
// of dA^T = W2 dZ^T, so one LDS tile serves H, both products, the relu mask and dA.
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int kHeadSamples = 16;       // per block
constexpr int kHeadWaves = 16;
constexpr uint32_t kHeadChunk = 2048;  // hidden units held in LDS at a time (132 KB); more pass through it chunk by chunk
constexpr int kHeadGroup = 4;          // 1 KiB pieces of a row, and
constexpr int kHeadTerms = 2;          //   terms of H (K splits beside the first, bias) that are requested together
__host__ __device__ inline uint32_t head_pitch(uint32_t n_hid) { return (n_hid < kHeadChunk ? n_hid : kHeadChunk) + 4; }

__global__ __launch_bounds__(64 * kHeadWaves) void head_kernel(const MlpParams p)
{
    static_assert(kHeadWaves == kHeadSamples, "one wave per row");
    extern __shared__ __attribute__((aligned(16))) float tile[];                // [kHeadSamples][head_pitch]: a chunk of H, then of dA
    __shared__ float zs[kHeadWaves][kHeadSamples][kMaxOut];
    __shared__ float dzs[kHeadSamples][kMaxOut + 1];
    const uint32_t worker = blockIdx.y, group = blockIdx.x, pitch = head_pitch(p.n_hid);
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t s16 = lane % 16, g = lane / 16;
    const Offsets o = offsets_of(p);
    const float *theta = p.x_in + static_cast<uint64_t>(worker) * p.stride;
    const float *W2 = theta + o.W2;
    const uint64_t sample = static_cast<uint64_t>(worker) * p.batch + group * kHeadSamples + wave;     // the wave's row
    float *Hrow = p.H + sample * p.n_hid;
    const uint64_t part = static_cast<uint64_t>(p.W) * p.batch * p.n_hid;      // one K split of the forward product
    const float *Prow = p.H_part + sample * p.n_hid;
    // the softmax's thread per sample and class
    const uint32_t smp = (threadIdx.x / kMaxOut) % kHeadSamples, c = threadIdx.x % kMaxOut;
    const uint64_t row = static_cast<uint64_t>(worker) * p.batch + group * kHeadSamples + smp;
    const bool real = c < p.n_out;
    const int label = p.y[row];
    const float b2 = real ? theta[o.b2 + c] : 0.0f;

    // operands of W2 for kHeadGroup blocks of a wave, requested ahead of the barriers that their use stands behind
    float w2[kHeadGroup][4];
    auto load_w2_rows = [&](uint32_t c0, uint32_t blk0, uint32_t n_blocks) {           // k = hidden unit, column = class
        #pragma unroll
        for (int i = 0; i < kHeadGroup; ++i) {
            const uint32_t blk = blk0 + kHeadWaves * i;
            #pragma unroll
            for (int j = 0; j < 4; ++j)
                w2[i][j] = blk < n_blocks && s16 < p.n_out ? W2[static_cast<uint64_t>(c0 + 16 * blk + 4 * g + j) * p.n_out + s16] : 0.0f;
        }
    };
    auto load_w2_classes = [&](uint32_t c0, uint32_t blk0, uint32_t n_blocks) {        // row = hidden unit, k = class
        #pragma unroll
        for (int i = 0; i < kHeadGroup; ++i) {
            const uint32_t blk = blk0 + kHeadWaves * i;
            #pragma unroll
            for (int q = 0; q < 4; ++q)
                w2[i][q] = blk < n_blocks && 4 * q + g < p.n_out ? W2[static_cast<uint64_t>(c0 + 16 * blk + s16) * p.n_out + 4 * q + g] : 0.0f;
        }
    };

    f4v zq[4] = {};                                            // one chain of additions per quarter j: shorter and independent
    for (uint32_t c0 = 0; c0 < p.n_hid; c0 += kHeadChunk) {
        const uint32_t width = p.n_hid - c0 < kHeadChunk ? p.n_hid - c0 : kHeadChunk;
        if (c0 != 0) __syncthreads();                          // the chunk before has been multiplied
        for (uint32_t n0 = 4 * lane; n0 < width; n0 += 256 * kHeadGroup) {
            f4 h[kHeadGroup];
            #pragma unroll
            for (int i = 0; i < kHeadGroup; ++i) {
                const uint32_t n = n0 + 256 * i;
                h[i] = n < width ? *reinterpret_cast<const f4 *>(Hrow + c0 + n) : f4{0.f, 0.f, 0.f, 0.f};
            }
            for (uint32_t t0 = 1; t0 <= p.fwd_splits; t0 += kHeadTerms) {      // the other K splits in order, then the bias
                f4 q[kHeadTerms][kHeadGroup];
                #pragma unroll
                for (int s = 0; s < kHeadTerms; ++s) {
                    const float *src = t0 + s < p.fwd_splits ? Prow + (t0 + s - 1) * part : theta + o.b1;
                    #pragma unroll
                    for (int i = 0; i < kHeadGroup; ++i) {
                        const uint32_t n = n0 + 256 * i;
                        q[s][i] = t0 + s <= p.fwd_splits && n < width ? *reinterpret_cast<const f4 *>(src + c0 + n) : f4{0.f, 0.f, 0.f, 0.f};
                    }
                }
                #pragma unroll
                for (int s = 0; s < kHeadTerms; ++s)
                    #pragma unroll
                    for (int i = 0; i < kHeadGroup; ++i) h[i] += q[s][i];
            }
            #pragma unroll
            for (int i = 0; i < kHeadGroup; ++i) {
                const uint32_t n = n0 + 256 * i;
                if (n < width) {
                    f4 a = h[i];
                    a.x = fmaxf(a.x, 0.f); a.y = fmaxf(a.y, 0.f); a.z = fmaxf(a.z, 0.f); a.w = fmaxf(a.w, 0.f);
                    *reinterpret_cast<f4 *>(Hrow + c0 + n) = a;
                    *reinterpret_cast<f4 *>(tile + wave * pitch + n) = a;
                }
            }
        }
        const uint32_t n_blocks = width / 16;
        load_w2_rows(c0, wave, n_blocks);
        __syncthreads();
        for (uint32_t blk0 = wave; blk0 < n_blocks; blk0 += kHeadWaves * kHeadGroup) {
            if (blk0 != wave) load_w2_rows(c0, blk0, n_blocks);
            #pragma unroll
            for (int i = 0; i < kHeadGroup; ++i) {
                const uint32_t blk = blk0 + kHeadWaves * i;
                if (blk < n_blocks) {                          // wave-uniform
                    const f4 h = *reinterpret_cast<const f4 *>(tile + s16 * pitch + 16 * blk + 4 * g);
                    #pragma unroll
                    for (int j = 0; j < 4; ++j) zq[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(h[j], w2[i][j], zq[j], 0, 0, 0);
                }
            }
        }
    }
    load_w2_classes(0, wave, (p.n_hid < kHeadChunk ? p.n_hid : kHeadChunk) / 16);
    const f4v z = (zq[0] + zq[1]) + (zq[2] + zq[3]);
    #pragma unroll
    for (int r = 0; r < 4; ++r) zs[wave][4 * g + r][s16] = z[r];
    __syncthreads();
    if (threadIdx.x < kHeadSamples * kMaxOut) {                // one thread per sample and class
        float q[4] = {0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int w = 0; w < kHeadWaves; ++w) q[w % 4] += zs[w][smp][c];
        float a = (q[0] + q[1]) + (q[2] + q[3]);
        a = real ? a + b2 : -INFINITY;
        float zmax = a;
        #pragma unroll
        for (int off = 8; off > 0; off >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, off, 16));
        const float e = real ? expf(a - zmax) : 0.0f;
        float denom = e;
        #pragma unroll
        for (int off = 8; off > 0; off >>= 1) denom += __shfl_xor(denom, off, 16);
        const float dz = real ? (e / denom - (label == static_cast<int>(c) ? 1.0f : 0.0f)) * (1.0f / static_cast<float>(p.batch)) : 0.0f;
        dzs[smp][c] = dz;
        p.dZ[row * kMaxOut + c] = dz;
    }
    __syncthreads();
    float dz[kMaxOut / 4];
    #pragma unroll
    for (int q = 0; q < kMaxOut / 4; ++q) dz[q] = dzs[s16][4 * q + g];
    const uint32_t steps = (p.n_out + 3) / 4;
    float *dArow = p.dA + sample * p.n_hid;
    for (uint32_t c0 = 0; c0 < p.n_hid; c0 += kHeadChunk) {
        const uint32_t width = p.n_hid - c0 < kHeadChunk ? p.n_hid - c0 : kHeadChunk;
        if (p.n_hid > kHeadChunk) {                            // H did not stay in LDS (the wave's own row: same lanes wrote it)
            for (uint32_t n = 4 * lane; n < width; n += 256)
                *reinterpret_cast<f4 *>(tile + wave * pitch + n) = *reinterpret_cast<const f4 *>(Hrow + c0 + n);
            __syncthreads();
        }
        const uint32_t n_blocks = width / 16;
        for (uint32_t blk0 = wave; blk0 < n_blocks; blk0 += kHeadWaves * kHeadGroup) {
            if (c0 != 0 || blk0 != wave) load_w2_classes(c0, blk0, n_blocks);
            #pragma unroll
            for (int i = 0; i < kHeadGroup; ++i) {
                const uint32_t blk = blk0 + kHeadWaves * i;
                if (blk < n_blocks) {                          // wave-uniform
                    f4 *at = reinterpret_cast<f4 *>(tile + s16 * pitch + 16 * blk + 4 * g);
                    const f4 h = *at;
                    f4v d = {0.f, 0.f, 0.f, 0.f};
                    #pragma unroll
                    for (int q = 0; q < kMaxOut / 4; ++q)
                        if (static_cast<uint32_t>(q) < steps) d = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[i][q], dz[q], d, 0, 0, 0);
                    *at = f4{h.x > 0.0f ? d[0] : 0.0f, h.y > 0.0f ? d[1] : 0.0f, h.z > 0.0f ? d[2] : 0.0f, h.w > 0.0f ? d[3] : 0.0f};
                }
            }
        }
        __syncthreads();
        for (uint32_t n = 4 * lane; n < width; n += 256) {
            const f4 a = *reinterpret_cast<const f4 *>(tile + wave * pitch + n);
            *reinterpret_cast<f4 *>(dArow + c0 + n) = a;
        }
        if (c0 + kHeadChunk < p.n_hid) __syncthreads();
    }
}

// Gradients of the small parameters and their update, as blocks of the backward product's launch (in a launch of their
// own they were a chain of memory round trips of 16 us on one block per compute unit; beside the update of W1 they are
// not seen).  A block owns 64 hidden units (rows of W2, and b1): dW2 = H^T dZ on the fp32 matrix instruction 16x16x4,
// each of the four waves over a quarter of the batch, db1 = colsum(dA); the waves' sums meet in LDS in a fixed order.
// Block 0 of a worker also owns b2 and the alignment pads.
constexpr uint32_t kSmallUnits = 64;
constexpr int kSmallWaves = 4, kSmallSteps = 4;                // waves per block; matrix instructions' worth of samples requested together
struct SmallUpdateLds { float part[kSmallWaves][kSmallUnits][kMaxOut + 1]; float b2[16][kMaxOut]; };
__host__ __device__ inline uint32_t small_blocks(const MlpParams &p) { return p.n_hid / kSmallUnits * p.W; }

__device__ __forceinline__ void small_update_block(const MlpParams &p, uint32_t block, SmallUpdateLds &lds)
{
    const uint32_t own_blocks = p.n_hid / kSmallUnits;
    const uint32_t worker = block / own_blocks, own = block % own_blocks;
    const uint32_t t = threadIdx.x, wave = t / 64, lane = t % 64, s16 = lane % 16, g = lane / 16;
    const Offsets o = offsets_of(p);
    const uint64_t base = static_cast<uint64_t>(worker) * p.stride;
    const uint32_t per = p.batch / kSmallWaves;                // samples of a wave: a multiple of 32
    const uint64_t sample = static_cast<uint64_t>(worker) * p.batch + wave * per + g;
    const float *H = p.H + sample * p.n_hid + own * kSmallUnits + s16, *dA = p.dA + sample * p.n_hid + own * kSmallUnits + s16;
    const float *dZ = p.dZ + sample * kMaxOut + s16;
    f4v d[4] = {};
    float gb[4] = {0.f, 0.f, 0.f, 0.f};
    for (uint32_t s0 = 0; s0 < per; s0 += 4 * kSmallSteps) {
        float h[kSmallSteps][4], a[kSmallSteps][4], z[kSmallSteps];
        #pragma unroll
        for (int s = 0; s < kSmallSteps; ++s) {
            const uint64_t at = s0 + 4 * s;
            z[s] = dZ[at * kMaxOut];
            #pragma unroll
            for (int b = 0; b < 4; ++b) { h[s][b] = H[at * p.n_hid + 16 * b]; a[s][b] = dA[at * p.n_hid + 16 * b]; }
        }
        #pragma unroll
        for (int s = 0; s < kSmallSteps; ++s)
            #pragma unroll
            for (int b = 0; b < 4; ++b) {
                d[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(h[s][b], z[s], d[b], 0, 0, 0);
                gb[b] += a[s][b];
            }
    }
    #pragma unroll
    for (int b = 0; b < 4; ++b) {
        #pragma unroll
        for (int r = 0; r < 4; ++r) lds.part[wave][16 * b + 4 * g + r][s16] = d[b][r];
        gb[b] += __shfl_xor(gb[b], 16, 64);
        gb[b] += __shfl_xor(gb[b], 32, 64);
        if (g == 0) lds.part[wave][16 * b + s16][kMaxOut] = gb[b];
    }
    if (own == 0) {                                            // db2[c]: thread (r, c) takes the samples r, r + 16, ...
        float sum = 0.0f;
        for (uint32_t b = t / kMaxOut; b < p.batch; b += 16) sum += p.dZ[(static_cast<uint64_t>(worker) * p.batch + b) * kMaxOut + t % kMaxOut];
        lds.b2[t / kMaxOut][t % kMaxOut] = sum;
    }
    __syncthreads();
    for (uint32_t e = t; e < kSmallUnits * p.n_out; e += 64 * kSmallWaves) {        // this block's rows of W2: contiguous
        const uint32_t n = e / p.n_out, c = e % p.n_out;
        float G = lds.part[0][n][c];
        #pragma unroll
        for (int w = 1; w < kSmallWaves; ++w) G += lds.part[w][n][c];
        sgd_update(p, base, o.W2 + static_cast<uint64_t>(own) * kSmallUnits * p.n_out + e, G);
    }
    if (t < kSmallUnits) {
        float G = lds.part[0][t][kMaxOut];
        #pragma unroll
        for (int w = 1; w < kSmallWaves; ++w) G += lds.part[w][t][kMaxOut];
        sgd_update(p, base, o.b1 + own * kSmallUnits + t, G);
    }
    if (own == 0 && wave == kSmallWaves - 1) {
        if (lane < p.n_out) {
            float G = lds.b2[0][lane];
            #pragma unroll
            for (int r = 1; r < 16; ++r) G += lds.b2[r][lane];
            sgd_update(p, base, o.b2 + lane, G);
        }
        const uint64_t d_end = o.b2 + p.n_out;                // pads after the last parameter travel along
        if (p.x_out != p.x_in && lane < ((d_end + 3) & ~3ull) - d_end) p.x_out[base + d_end + lane] = p.x_in[base + d_end + lane];
    }
}

// ---- the two big contractions ---------------------------------------------------------------------
// kBwdTail: the backward product of a round's last step (line 6 in its epilogue); kBwdOnly: of its only step, whose input models are
// the stored ones
enum { kFwd = 0, kBwd = 1, kBwdTail = 2, kBwdOnly = 3 };

typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef __bf16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 h8 __attribute__((ext_vector_type(8)));

// Eight values as three bf16 vectors: the value rounded to 8 bits, the remainder rounded to 8 bits, and what is left, at
// most 8 bits.  Exact where the last bit of the value is a normal bf16, 2^-126: B is scaled so that this holds for the
// smallest fp32 number, and values below 2^104 still have room above.  (X needs no scale: normals of 24-bit uniforms, zero
// or above 1e-12.)
constexpr float kScale = 0x1p24f, kUnscale = 0x1p-24f;
struct Planes { u4 p[3]; };
__device__ __forceinline__ unsigned int pack_bf16(float a, float b)
{
    typedef float v2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned int, __builtin_convertvector(v2{a, b}, h2));
}
template <bool SCALED>
__device__ __forceinline__ Planes split8(const float (&a)[8])
{
    Planes out;
    #pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x0 = SCALED ? a[2 * i] * kScale : a[2 * i], x1 = SCALED ? a[2 * i + 1] * kScale : a[2 * i + 1];
        #pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            const unsigned int pair = pack_bf16(x0, x1);
            out.p[pl][i] = pair;
            x0 -= __uint_as_float(pair << 16);
            x1 -= __uint_as_float(pair & 0xffff0000u);
        }
    }
    return out;
}

constexpr int kGemmThreads = 256;

// The planes of A's K slice in LDS, in the order in which the matrix instruction's lanes read them:
// [plane][32-row block][k octet][slot] pieces of 16 bytes (8 consecutive k of one row).  A fragment read is then 1 KiB
// contiguous per wave.  The slot of a row is chosen so that the eight lanes that write together also hit eight different
// 16-byte bank groups: a wave that stages one octet of 64 rows does so as it is, rows staged k-wise (four octets of one
// row in four lanes) rotate by the octet.
template <int ROWS>
struct OperandTile {
    u4 q[3][ROWS / 32][4][32];
};
template <int EPI>
__device__ __forceinline__ uint32_t slot_of(uint32_t r, uint32_t octet) { return EPI == kFwd ? (r + 2 * octet) & 31u : r; }

// BM x BN block tile, four waves, each 32 columns of BN and all of BM (half of it where BN is 64).
template <int EPI, int BM, int BN>
__global__ __launch_bounds__(kGemmThreads, 2) void mlp_gemm_kernel(const MlpParams p)
{
    constexpr int NWN = BN / 32, NWM = 4 / NWN, MB = BM / 32 / NWM;      // waves per direction, 32-row blocks per wave
    constexpr int CPITCH = BN + 4;
    constexpr bool LINE6 = EPI == kBwdTail || EPI == kBwdOnly;
    constexpr int OPERANDS = 2 * sizeof(OperandTile<BM>), TILE = EPI == kFwd ? 0 : BM * CPITCH * 4;
    static_assert(EPI == kFwd || BM == 64, "a lane stages one row");
    static_assert(EPI == kFwd || OPERANDS >= static_cast<int>(sizeof(SmallUpdateLds)), "the small update's sums fit");
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERANDS > TILE ? OPERANDS : TILE];
    OperandTile<BM> *ops = reinterpret_cast<OperandTile<BM> *>(smem);                              // two buffers
    float (*Ct)[CPITCH] = reinterpret_cast<float (*)[CPITCH]>(smem);                               // epilogue tile

    // Workgroups go to the 8 XCDs (each with its own L2) round-robin by linear id.  Renumber them so
    // that every XCD owns a CONTIGUOUS run of tiles (n fastest, then m, then K split, then worker): the tiles that
    // share an operand panel (all n-tiles of an m-tile share its X panel, all m-tiles of an n-tile its
    // W1 / dA panel) then meet in one L2 instead of fetching the panel once per XCD.
    const uint32_t splits = EPI == kFwd ? p.fwd_splits : 1u;
    const uint32_t nx = p.n_hid / BN, ny = (EPI == kFwd ? p.batch : p.n_in) / BM, total = nx * ny * p.W * splits;
    uint32_t linear = blockIdx.x;
    if (EPI != kFwd) {                                         // the launch's first blocks update the small parameters
        if (p.step_next && linear == 0 && threadIdx.x == 0) *p.step_next = *p.step_base + p.round_steps;
        if (linear < small_blocks(p)) {
            small_update_block(p, linear, *reinterpret_cast<SmallUpdateLds *>(smem));
            return;
        }
        linear -= small_blocks(p);
    }
    uint32_t bx, by, bz;
    if (LINE6 && ny % kXcds == 0) {
        // the mean is read by every worker: an XCD owns the same eighth of the rows of W1 for all of them
        // (222 -> 206 us at W = 16, 3072-1024-10; measured, like the two figures at the epilogue, with half the products)
        const uint32_t rows = ny / kXcds, r = linear / kXcds;
        bx = r % nx;
        by = (linear % kXcds) * rows + (r / nx) % rows;
        bz = r / (nx * rows);
    } else {
        const uint32_t logical = total % kXcds == 0 ? (linear % kXcds) * (total / kXcds) + linear / kXcds : linear;
        bx = logical % nx;
        by = (logical / nx) % ny;
        bz = logical / (nx * ny);
    }
    const uint32_t worker = bz / splits, split = bz % splits;
    const uint32_t m0 = by * BM, n0 = bx * BN;
    const Offsets o = offsets_of(p);
    const uint32_t t = threadIdx.x, wave = t / 64, lane = t % 64;
    const uint32_t ldb = p.n_hid;
    const float *Xw = p.X + static_cast<uint64_t>(worker) * p.batch * p.n_in;

    // Global -> registers, one K slice: 8 consecutive k of one row or column per piece.
    //   forward : A = X [batch][n_in], K-contiguous: lane t takes octet t % 4 of row t / 4 (+ 64)
    //   backward: A = X^T, read from X M-contiguous: wave w takes octet w, lane l row l of the tile
    //   B       : K-major (W1 rows, or dA rows), as the matrix instruction wants it: lane l has column l % 32 of its
    //             wave, octets l / 32 and 2 + l / 32
    constexpr int AP = BM / 64;                                // pieces of A per thread
    const uint32_t wm = wave / NWN, wn = wave % NWN;           // wave owns rows 32 MB wm .., columns 32 wn ..
    const float *a_src, *b_base, *b_src;
    uint32_t slice0 = 0, n_slices;                             // this block's K slices: an even number, at least two
    if (EPI == kFwd) {
        const uint32_t pairs = p.n_in / kBK / 2;
        slice0 = 2 * (pairs * split / splits);
        n_slices = 2 * (pairs * (split + 1) / splits) - slice0;
        a_src = Xw + static_cast<uint64_t>(m0 + t / 4) * p.n_in + (t % 4) * 8;
        b_base = p.x_in + static_cast<uint64_t>(worker) * p.stride + o.W1;                // W1 [n_in][n_hid]
    } else {
        n_slices = p.batch / kBK;
        a_src = Xw + static_cast<uint64_t>(wave) * 8 * p.n_in + m0 + lane;
        b_base = p.dA + static_cast<uint64_t>(worker) * p.batch * p.n_hid;                // dA [batch][n_hid]
    }
    // Columns of this block's tile.  The update streams x, v (and the stored model) in rows of BN floats, and rows that
    // start off a 128-byte line cost it 40 % (W = 16, 3072-1024-10: the stream alone takes 124 us on lines and 174 us
    // off them).  A worker's W1 starts wherever its row of the model buffer does, so the columns are counted from the
    // first one that lies on a line; the last tile wraps around to the columns before it.
    uint32_t first_col = n0;
    if (EPI != kFwd) {
        const uint64_t at = reinterpret_cast<uintptr_t>(p.x_out) / 4 + static_cast<uint64_t>(worker) * p.stride;
        first_col += static_cast<uint32_t>(-at & 31u);
    }
    auto column = [&](uint32_t c) { const uint32_t n = first_col + c; return n < p.n_hid ? n : n - p.n_hid; };
    b_src = b_base + static_cast<uint64_t>(lane / 32) * 8 * ldb + column(wn * 32 + lane % 32);

    float ra[AP][8], rb[2][8];
    auto load_slice = [&](uint32_t slice) {
        const uint64_t s = slice0 + slice;
        if (EPI == kFwd) {
            #pragma unroll
            for (int i = 0; i < AP; ++i) {
                const float *src = a_src + s * kBK + static_cast<uint64_t>(i) * 64 * p.n_in;
                const f4 lo = *reinterpret_cast<const f4 *>(src), hi = *reinterpret_cast<const f4 *>(src + 4);
                #pragma unroll
                for (int j = 0; j < 4; ++j) { ra[i][j] = lo[j]; ra[i][4 + j] = hi[j]; }
            }
        } else {
            #pragma unroll
            for (int j = 0; j < 8; ++j) ra[0][j] = a_src[(s * kBK + j) * p.n_in];
        }
        #pragma unroll
        for (int kb = 0; kb < 2; ++kb)
            #pragma unroll
            for (int j = 0; j < 8; ++j) rb[kb][j] = b_src[(s * kBK + 16 * kb + j) * ldb];
    };
    float largest = 0.0f;                                       // |b|, a NaN not counted
    Planes bp[2];
    auto stage_slice = [&](auto buffer) {                       // A -> LDS buffer, B -> operand registers
        constexpr int S = decltype(buffer)::value;
        #pragma unroll
        for (int i = 0; i < AP; ++i) {
            const uint32_t row = EPI == kFwd ? t / 4 + 64 * i : lane, oct = EPI == kFwd ? t % 4 : wave;
            const uint32_t slot = slot_of<EPI>(row % 32, oct);
            const Planes s = split8<false>(ra[i]);
            #pragma unroll
            for (int pl = 0; pl < 3; ++pl) ops[S].q[pl][row / 32][oct][slot] = s.p[pl];
        }
        #pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            #pragma unroll
            for (int j = 0; j < 8; j += 2) largest = fmaxf(fmaxf(largest, fabsf(rb[kb][j])), fabsf(rb[kb][j + 1]));
            bp[kb] = split8<true>(rb[kb]);
        }
    };

    // The product is formed transposed (W1 columns as the instruction's rows): a lane then holds four consecutive
    // columns of one row of the result.
    // (One accumulator for all six products: dW1 is off by 1.72e-7 instead of 5.9e-8 at W = 16, 3072-1024-10, batch 128.)
    f16v acc[MB], low[MB];                                      // leading products, the others
    auto multiply_slice = [&](auto buffer) {
        constexpr int S = decltype(buffer)::value;
        #pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const uint32_t oct = 2 * kb + lane / 32, r = lane % 32;
            const uint32_t slot = slot_of<EPI>(r, oct);
            h8 a[3][MB];
            #pragma unroll
            for (int i = 0; i < MB; ++i)
                #pragma unroll
                for (int pl = 0; pl < 3; ++pl) a[pl][i] = __builtin_bit_cast(h8, ops[S].q[pl][wm * MB + i][oct][slot]);
            constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
            #pragma unroll
            for (int q = 0; q < 6; ++q)
                #pragma unroll
                for (int i = 0; i < MB; ++i) {
                    f16v &to = q < 5 ? low[i] : acc[i];
                    to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(h8, bp[kb].p[PB[q]]), a[PA[q]][i], to, 0, 0, 0);
                }
        }
    };

    // Backward product: the epilogue updates this block's tile of W1 and its momentum.  Vector loads
    // return in order, so these loads must be the YOUNGEST in flight or every operand slice
    // behind them would wait for them: they are issued right after the loads of the last K slice
    // and land under the remaining multiplies.
    constexpr int EPI_ITERS = (BM * BN / 4) / kGemmThreads, ROWS_PER_PASS = kGemmThreads / (BN / 4);
    const uint32_t tile_row = t / (BN / 4), tile_col = (t % (BN / 4)) * 4;
    const uint64_t row_at = o.W1 + static_cast<uint64_t>(m0 + tile_row) * p.n_hid + column(tile_col);
    const uint64_t tile_at = static_cast<uint64_t>(worker) * p.stride + row_at;
    f4 x_old[EPI_ITERS], v_old[EPI_ITERS];
    auto prefetch_x = [&]() {
        #pragma unroll
        for (int it = 0; it < EPI_ITERS; ++it)
            x_old[it] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p.x_in + tile_at + static_cast<uint64_t>(it * ROWS_PER_PASS) * p.n_hid));
    };
    auto prefetch_v = [&]() {
        #pragma unroll
        for (int it = 0; it < EPI_ITERS; ++it) {
            const uint64_t at = tile_at + static_cast<uint64_t>(it * ROWS_PER_PASS) * p.n_hid;
            v_old[it] = p.momentum != 0.0f ? __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p.v + at)) : f4{0.f, 0.f, 0.f, 0.f};
        }
    };

    using Buffer0 = std::integral_constant<int, 0>;
    using Buffer1 = std::integral_constant<int, 1>;
    load_slice(0);
    if (EPI != kFwd && p.X_next) {
        // The NEXT local step's mini-batch is drawn here, a share per block, into the other batch buffer: vector
        // arithmetic under the latency of the first operand loads.
        const uint32_t step = p.step_base ? *p.step_base + p.step : p.step, per_worker = gen_batch_blocks(p);
        for (uint32_t id = linear; id < per_worker * p.W; id += total)
            gen_batch_block(p, id % per_worker, t, id / per_worker, step + 1, p.X_next, p.y_next);
    }
    #pragma unroll
    for (int i = 0; i < MB; ++i) { acc[i] = f16v{0}; low[i] = f16v{0}; }
    for (uint32_t s = 0; s + 2 < n_slices; s += 2) {          // one barrier per slice: waves stage one buffer while others multiply the other
        stage_slice(Buffer0{});
        load_slice(s + 1);
        __syncthreads();
        multiply_slice(Buffer0{});
        stage_slice(Buffer1{});
        load_slice(s + 2);
        __syncthreads();
        multiply_slice(Buffer1{});
    }
    stage_slice(Buffer0{});
    load_slice(n_slices - 1);
    if (EPI != kFwd) prefetch_x();
    __syncthreads();
    multiply_slice(Buffer0{});
    stage_slice(Buffer1{});
    if (EPI != kFwd) prefetch_v();
    __syncthreads();
    multiply_slice(Buffer1{});

    // undo the scale: lane l, register r of a 32 x 32 block is row l % 32, column 8 (r / 4) + 4 (l / 32) + r % 4
    bool mine = true;
    #pragma unroll
    for (int i = 0; i < MB; ++i)
        #pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float sum = acc[i][r] + low[i][r];
            mine &= fabsf(sum) < INFINITY;
            acc[i][r] = sum * kUnscale;
        }
    // A sum that is not finite comes from a NaN, and is NaN either way, or from an operand out of the planes' range: an
    // infinity (it splits into inf and NaN) or one so large that products overflow with the scale (below 2^64 none can:
    // |X| < 8, fewer than 2^37 terms).  Such a tile is formed with fp32 products throughout, which give inf, NaN or neither
    // just as the fp32 arithmetic of the rest of the step.  (The first vote is also the barrier behind which the operand
    // buffers are free.)
    if (__syncthreads_or(!mine) && __syncthreads_or(largest >= 0x1p64f)) {
        // (A pair of k and one block of rows at a time, such a step took 0.5 ms longer.)
        constexpr int kPairs = 8;                               // pairs of k requested together; slices come in pairs, 64 k
        const uint32_t k0 = slice0 * kBK + lane / 32, n = column(wn * 32 + lane % 32);
        const uint64_t lda = EPI == kFwd ? 1 : p.n_in, ldm = EPI == kFwd ? p.n_in : 1;
        const float *bk = b_base + static_cast<uint64_t>(k0) * ldb + n, *ak = Xw + (m0 + wm * MB * 32 + lane % 32) * ldm + k0 * lda;
        #pragma unroll
        for (int i = 0; i < MB; ++i) acc[i] = f16v{0};
        #pragma unroll 1
        for (uint32_t k = 0; k < n_slices * kBK; k += 2 * kPairs, bk += 2 * kPairs * static_cast<uint64_t>(ldb), ak += 2 * kPairs * lda) {
            float bq[kPairs], aq[MB][kPairs];
            #pragma unroll
            for (int q = 0; q < kPairs; ++q) {
                bq[q] = bk[2 * q * static_cast<uint64_t>(ldb)];
                #pragma unroll
                for (int i = 0; i < MB; ++i) aq[i][q] = ak[2 * q * lda + 32 * i * ldm];
            }
            #pragma unroll
            for (int q = 0; q < kPairs; ++q)
                #pragma unroll
                for (int i = 0; i < MB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(bq[q], aq[i][q], acc[i], 0, 0, 0);
        }
    }

    if (EPI == kFwd) {
        // raw sums of this K split; bias and relu follow where the splits are added (head_kernel)
        float *out = (split == 0 ? p.H : p.H_part + static_cast<uint64_t>(split - 1) * p.W * p.batch * p.n_hid) +
                     (static_cast<uint64_t>(worker) * p.batch + m0) * p.n_hid + n0;
        #pragma unroll
        for (int i = 0; i < MB; ++i)
            #pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f4 *>(out + static_cast<uint64_t>((wm * MB + i) * 32 + lane % 32) * p.n_hid + wn * 32 + 8 * g + 4 * (lane / 32)) =
                    f4{acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
        return;
    }
    // accumulators -> LDS tile (the operand buffers are dead: the vote above was a barrier), then the update over
    // the tile in row-major quads: BN/4 lanes cover one row
    #pragma unroll
    for (int i = 0; i < MB; ++i)
        #pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f4 *>(&Ct[(wm * MB + i) * 32 + lane % 32][wn * 32 + 8 * g + 4 * (lane / 32)]) =
                f4{acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
    // line 6: the stored model and the mean, into the registers that the accumulators have just left (stored model requested
    // with v, mean one quad at a time below: 203 us, like this 191, W = 16, 3072-1024-10).  A round's only step has read the
    // stored model already (read a second time: a round of one step 330 us instead of 307).
    f4 snap_old[EPI_ITERS], mean[EPI_ITERS];
    if (LINE6) {
        #pragma unroll
        for (int it = 0; it < EPI_ITERS; ++it) {
            const uint64_t down = static_cast<uint64_t>(it * ROWS_PER_PASS) * p.n_hid;
            snap_old[it] = EPI == kBwdOnly ? x_old[it] : __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p.snap + tile_at + down));
            mean[it] = *reinterpret_cast<const f4 *>(p.mean + row_at + down);
        }
    }
    __syncthreads();
    #pragma unroll
    for (int it = 0; it < EPI_ITERS; ++it) {
        const f4 val = *reinterpret_cast<const f4 *>(&Ct[tile_row + it * ROWS_PER_PASS][tile_col]);
        const uint64_t at = tile_at + static_cast<uint64_t>(it * ROWS_PER_PASS) * p.n_hid;
        f4 g = val + p.weight_decay * x_old[it];
        if (p.momentum != 0.0f) {
            g = p.momentum * v_old[it] + g;
            __builtin_nontemporal_store(g, reinterpret_cast<f4 *>(p.v + at));
        }
        f4 x_new = x_old[it] - p.lr * g;
        if (LINE6) x_new = mean[it] + (x_new - snap_old[it]);      // line 6 on the fresh model, same operation order as the separate kernel
        __builtin_nontemporal_store(x_new, reinterpret_cast<f4 *>(p.x_out + at));
    }
}

template <int EPI, int BM, int BN>
void launch_gemm(hipStream_t stream, const MlpParams &p, hipEvent_t start = nullptr, hipEvent_t stop = nullptr)
{
    const uint32_t M = (EPI == kFwd) ? p.batch : p.n_in;
    const dim3 grid(p.n_hid / BN * (M / BM) * p.W * (EPI == kFwd ? p.fwd_splits : 1u) + (EPI == kFwd ? 0u : small_blocks(p))), block(kGemmThreads);
    // the events, if any, take the kernel's own start / end timestamps (no marker of their own in the queue)
    if (start || stop) hipExtLaunchKernelGGL((mlp_gemm_kernel<EPI, BM, BN>), grid, block, 0, stream, start, stop, 0, p);
    else               hipLaunchKernelGGL((mlp_gemm_kernel<EPI, BM, BN>), grid, block, 0, stream, p);
}

}  // namespace

bool mlp_shape_supported(uint32_t n_in, uint32_t n_hid, uint32_t n_out, uint32_t batch)
{
    return n_in >= static_cast<uint32_t>(kShapeM) && n_in % kShapeM == 0 && n_hid >= static_cast<uint32_t>(kShapeN) &&
           n_hid % kShapeN == 0 && n_out >= 1 && n_out <= static_cast<uint32_t>(kMaxOut) &&
           batch >= static_cast<uint32_t>(kShapeM) && batch % kShapeM == 0 && batch <= 1024 &&
           static_cast<uint64_t>(n_hid) * (n_out | 1u) <= kMaxHiddenOut;
}

size_t mlp_dz_pitch() { return kMaxOut; }

// K splits of the forward product: the fewest that give every compute unit a block, at least four K slices each.
// More of them feed the chip better (W = 16, 3072-1024-10, batch 128, 128 tiles: the product alone takes 93 us at two
// splits, 74 at four) but every split writes and reads H once more and the kernels behind it slow down: round 595 us at
// two splits, 584 at four; W = 6, 1024-2048-10, batch 512, 384 tiles: 260 us at one split, 265 at two.
uint32_t mlp_forward_splits(uint32_t W, uint32_t n_in, uint32_t n_hid, uint32_t batch, uint32_t compute_units)
{
    const uint64_t tiles = static_cast<uint64_t>(W) * (batch / 128) * (n_hid / (n_hid % 128 == 0 ? 128 : 64));
    const uint64_t want = ((compute_units ? compute_units : 256u) + tiles - 1) / tiles;
    const uint64_t most = n_in / kBK / 4 < 8u ? n_in / kBK / 4 : 8u;
    return static_cast<uint32_t>(want < most ? want : most);
}

hipError_t launch_mlp_step(hipStream_t stream, const MlpParams &p, hipEvent_t start, hipEvent_t stop)
{
    const bool wide = p.n_hid % 128 == 0;      // 64 x 128 block tiles (fastest measured), else 64 x 64
    if (!p.have_batch) {                       // the step then begins with this kernel
        if (start) hipExtLaunchKernelGGL(gen_batch_kernel, dim3(gen_batch_blocks(p), p.W), dim3(256), 0, stream, start, nullptr, 0, p);
        else       hipLaunchKernelGGL(gen_batch_kernel, dim3(gen_batch_blocks(p), p.W), dim3(256), 0, stream, p);
        start = nullptr;
    }
    if (wide) launch_gemm<kFwd, 128, 128>(stream, p, start); else launch_gemm<kFwd, 128, 64>(stream, p, start);
    const size_t head_lds = kHeadSamples * head_pitch(p.n_hid) * sizeof(float);
    // more than the default 64 KB of dynamic LDS for wide hidden layers
    static const hipError_t lds_ok = hipFuncSetAttribute(reinterpret_cast<const void *>(head_kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         kHeadSamples * (kHeadChunk + 4) * sizeof(float));
    if (lds_ok != hipSuccess) return lds_ok;
    hipLaunchKernelGGL(head_kernel, dim3(p.batch / kHeadSamples, p.W), dim3(64 * kHeadWaves), head_lds, stream, p);
    if (!p.snap)               { if (wide) launch_gemm<kBwd, 64, 128>(stream, p, nullptr, stop); else launch_gemm<kBwd, 64, 64>(stream, p, nullptr, stop); }
    else if (p.snap != p.x_in) { if (wide) launch_gemm<kBwdTail, 64, 128>(stream, p, nullptr, stop); else launch_gemm<kBwdTail, 64, 64>(stream, p, nullptr, stop); }
    else                       { if (wide) launch_gemm<kBwdOnly, 64, 128>(stream, p, nullptr, stop); else launch_gemm<kBwdOnly, 64, 64>(stream, p, nullptr, stop); }
    return hipGetLastError();
}

}  // namespace cocod
