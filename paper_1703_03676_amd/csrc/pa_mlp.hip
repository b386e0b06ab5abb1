// Training and inference kernels of the learned temperature-step proposer
// (MLP 8 -> 64 -> 64 -> 1, ReLU; layout in pa_mlp_dev.h).
//
// Training is FP32 with a deterministic fixed-order gradient reduction: each
// block sums the gradient of its samples in matrix-core accumulators
// (k_backprop), and one thread per parameter sums the blocks in order
// (k_apply), so a training run is reproducible bit for bit.  SGD with momentum
// updates the FP32 master weights and refreshes the BF16 copy used for
// inference.  The loss is the mean squared error on the normalised target.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <random>
#include <string>
#include <vector>

#include "pa.h"
#include "pa_mlp_dev.h"

namespace pa {
namespace mlp {
namespace {

// ---------------------------------------------------------------------------
// Forward pass, deltas and gradient of the mean squared error
// L = (1/B) sum_s (y_s - t_s)^2, for the samples idx[0..B) (0..B without idx).
//
// Block b of the nblk blocks that B samples have takes the tiles of 16 samples
// b, b + nblk, ..., and leaves the sums over them in its part of the partials
// (one entry per parameter, then the sum of squared errors).  Its four waves
// own 16 hidden units each.  All contractions run on the FP32 matrix cores
// (v_mfma_f32_16x16x4: inputs and accumulation in FP32): lane l holds
// A[m = l % 16][k] and B[k][n = l % 16] for the k of its quarter q = l / 16 and
// D[m = 4 q + i][n], i = 0..3.  A contraction over 64 units gives quarter q the
// k of 16 q .. 16 q + 15, so its operands are contiguous.  The gradients of
// the block's tiles stay in the accumulators.
//
// Bound by latency (two dependent loads, about 40 matrix instructions, six
// barriers per tile), so a tile has a block of its own up to kMaxParts of them
// (tiles of 32 samples on eight waves halve the partials but took 8.2 us
// against 6.4).  One thread per parameter running over all samples kept 19
// blocks busy for 65 us at B = 256 and 138 us at B = 500; these blocks take
// 6.4 us at either, k_apply 3.5-4.7.  A training step of 256 samples took 92 us
// (five launches, an upload and a wait) and takes 10 in two launches.
// ---------------------------------------------------------------------------
constexpr int kTile = 16;                // samples per tile
constexpr int kPartStride = 4804;        // floats per block: parameters, squared error, padding
constexpr int kMaxParts = 64;            // blocks, so that k_apply stays short
constexpr int kLd = kHid + 4;            // row length of the tile's activations in LDS
static_assert(kPartStride > kParams, "one partial per parameter and one for the loss");

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sum over the 16 lanes of a quarter, and over the four quarters.
__device__ __forceinline__ float sum_quarter(float v)
{
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ float sum_quarters(float v)
{
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

__global__ __launch_bounds__(256) void k_backprop(const float* __restrict__ x_all, const float* __restrict__ t_all,
                                                  const int32_t* __restrict__ idx, int B,
                                                  const float* __restrict__ norm, const float* __restrict__ p, int blk0,
                                                  int nblk, float* __restrict__ parts)
{
    __shared__ __align__(16) float sh1[kTile][kLd], sd2[kTile][kLd], sd1[kTile][kLd];
    __shared__ float sx[kTile][kIn + 1], sy[4][kTile], sdy[kTile];
    const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
    const int n = lane & 15, q = lane >> 4;
    const int u = 16 * w + n;  // the hidden unit of this lane's column
    // weights of this lane, the same for every tile
    float w1[2], w2r[16], w2c[16];
#pragma unroll
    for (int i = 0; i < 2; ++i) w1[i] = p[kW1 + u * kIn + 4 * i + q];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        w2r[i] = p[kW2 + u * kHid + 16 * q + i];    // row u: layer 2
        w2c[i] = p[kW2 + (16 * q + i) * kHid + u];  // column u: its transpose, for the deltas of layer 1
    }
    const float b1 = p[kB1 + u], b2 = p[kB2 + u], w3 = p[kW3 + u], b3 = p[kB3];
    const float t_mean = norm[2 * kIn], t_std = norm[2 * kIn + 1];
    f4 gw2[4] = {}, gw1 = {};
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, sq = 0.0f;

    for (int s0 = (blk0 + (int)blockIdx.x) * kTile; s0 < B; s0 += nblk * kTile) {
        // layer 1: A = the tile's normalised features (row n of the tile, features q and 4 + q)
        const bool have = s0 + n < B;
        const int row = have ? (idx ? idx[s0 + n] : s0 + n) : 0;
        f4 z = {b1, b1, b1, b1};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = 4 * i + q;
            const float xn = have ? (x_all[(size_t)row * kIn + k] - norm[k]) / norm[kIn + k] : 0.0f;
            if (w == 0) sx[n][k] = xn;
            z = mfma4(xn, w1[i], z);
        }
        const float tn = (w == 0 && have) ? (t_all[row] - t_mean) / t_std : 0.0f;
        f4 h1, h2, d2, d1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h1[i] = z[i] > 0.0f ? z[i] : 0.0f;
            sh1[4 * q + i][u] = h1[i];
        }
        __syncthreads();
        // layer 2
        z = f4{b2, b2, b2, b2};
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const f4 a = *reinterpret_cast<const f4*>(&sh1[n][16 * q + i]);
#pragma unroll
            for (int k = 0; k < 4; ++k) z = mfma4(a[k], w2r[i + k], z);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h2[i] = z[i] > 0.0f ? z[i] : 0.0f;
            const float part = sum_quarter(w3 * h2[i]);
            if (n == 0) sy[w][4 * q + i] = part;
        }
        __syncthreads();
        // output and its delta
        if (w == 0 && lane < kTile) {
            const float d = b3 + sy[0][n] + sy[1][n] + sy[2][n] + sy[3][n] - tn;
            sdy[n] = have ? 2.0f * d / (float)B : 0.0f;
            if (have) sq += d * d;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float dy = sdy[4 * q + i];
            d2[i] = h2[i] > 0.0f ? dy * w3 : 0.0f;
            sd2[4 * q + i][u] = d2[i];
            gw3 += dy * h2[i];
            gb2 += d2[i];
        }
        if (w == 0 && lane < kTile) gb3 += sdy[n];
        __syncthreads();
        // deltas of layer 1
        z = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const f4 a = *reinterpret_cast<const f4*>(&sd2[n][16 * q + i]);
#pragma unroll
            for (int k = 0; k < 4; ++k) z = mfma4(a[k], w2c[i + k], z);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            d1[i] = h1[i] > 0.0f ? z[i] : 0.0f;
            sd1[4 * q + i][u] = d1[i];
            gb1 += d1[i];
        }
        __syncthreads();
        // gradient of W2: rows of this wave's units, all columns, over the 16 samples
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = sd2[4 * i + q][u];
#pragma unroll
            for (int c = 0; c < 4; ++c) gw2[c] = mfma4(a, sh1[4 * i + q][16 * c + n], gw2[c]);
        }
        // gradient of W1
#pragma unroll
        for (int i = 0; i < 4; ++i)
            gw1 = mfma4(sd1[4 * i + q][u], n < kIn ? sx[4 * i + q][n] : 0.0f, gw1);
        __syncthreads();  // the next tile reuses the tables
    }

    float* out = parts + (size_t)blockIdx.x * kPartStride;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[kW2 + (16 * w + 4 * q + i) * kHid + 16 * c + n] = gw2[c][i];
    if (n < kIn)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[kW1 + (16 * w + 4 * q + i) * kIn + n] = gw1[i];
    gb1 = sum_quarters(gb1);
    gb2 = sum_quarters(gb2);
    gw3 = sum_quarters(gw3);
    if (q == 0) {
        out[kB1 + u] = gb1;
        out[kB2 + u] = gb2;
        out[kW3 + u] = gw3;
    }
    gb3 = sum_quarter(gb3);
    sq = sum_quarter(sq);
    if (threadIdx.x == 0) {
        out[kB3] = gb3;
        out[kParams] = sq;
    }
}

// One thread per parameter: the partial sums of nparts blocks in order, after
// those of the blocks before them in carry (with `carried`).  If more blocks
// follow, the sum goes to carry; else either the gradient goes to `grad` (host
// memory), or SGD with momentum updates the FP32 master weights and their BF16
// copy.  The thread after the last parameter adds the loss of the minibatch to
// *loss, or starts it (`start`).
__global__ __launch_bounds__(64) void k_apply(const float* __restrict__ parts, int nparts, float* __restrict__ carry,
                                              int carried, int more, int B, float* __restrict__ grad,
                                              float* __restrict__ p, float* __restrict__ mom, float lr,
                                              float momentum, __hip_bfloat16* __restrict__ wb,
                                              float* __restrict__ loss, int start)
{
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (q > kParams) return;
    const bool update = !grad && !more && q < kParams;
    const float m0 = update ? mom[q] : 0.0f, p0 = update ? p[q] : 0.0f;
    float g = carried ? carry[q] : 0.0f;
#pragma unroll 8
    for (int k = 0; k < nparts; ++k) g += parts[(size_t)k * kPartStride + q];
    if (more) {
        carry[q] = g;
        return;
    }
    if (q == kParams) {
        const float l = g / (float)B;
        *loss = start ? l : *loss + l;
        return;
    }
    if (grad) {
        grad[q] = g;
        return;
    }
    const float m = momentum * m0 + g;
    mom[q] = m;
    const float v = p0 - lr * m;
    p[q] = v;
    wb[q] = __float2bfloat16(v);
}

__global__ void k_to_bf16(const float* __restrict__ p, __hip_bfloat16* __restrict__ wb)
{
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (q < kParams) wb[q] = __float2bfloat16(p[q]);
}

// Inference on raw features: BF16 weights and activations (bf16 = 1) or the
// FP32 master weights (bf16 = 0).  One block of 64 threads per sample.
__global__ __launch_bounds__(64) void k_infer(const float* __restrict__ x, const float* __restrict__ p,
                                              const __hip_bfloat16* __restrict__ wb, const float* __restrict__ norm,
                                              int bf16, float* __restrict__ y)
{
    __shared__ float h[kHid];
    const int s = (int)blockIdx.x, t = (int)threadIdx.x;
    if (bf16) {
        const float o = forward_bf16(x + s * kIn, wb, norm, h, t);
        if (t == 0) y[s] = o;
        return;
    }
    float a = p[kB1 + t];
    for (int k = 0; k < kIn; ++k) a += p[kW1 + t * kIn + k] * ((x[s * kIn + k] - norm[k]) / norm[kIn + k]);
    h[t] = a > 0.0f ? a : 0.0f;
    __syncthreads();
    float a2 = p[kB2 + t];
    for (int v = 0; v < kHid; ++v) a2 += p[kW2 + t * kHid + v] * h[v];
    const float h2 = a2 > 0.0f ? a2 : 0.0f;
    __syncthreads();
    h[t] = p[kW3 + t] * h2;
    __syncthreads();
    if (t == 0) {
        float o = p[kB3];
        for (int v = 0; v < kHid; ++v) o += h[v];
        y[s] = o * norm[2 * kIn + 1] + norm[2 * kIn];
    }
}

// Mean and standard deviation of each feature and of the target (FP64): one
// block per variable, its threads' strided sums added in a fixed tree.  (One
// thread per variable over all samples took 0.34-0.66 ms at n = 4096.)
constexpr int kNormThreads = 512;

__global__ __launch_bounds__(kNormThreads) void k_fit_norm(const float* __restrict__ x, const float* __restrict__ t,
                                                           int n, float* __restrict__ norm)
{
    __shared__ double sh[2][kNormThreads];
    const int v = (int)blockIdx.x, th = (int)threadIdx.x;
    double s = 0.0, s2 = 0.0;
    for (int i = th; i < n; i += kNormThreads) {
        const double z = (v < kIn) ? (double)x[(size_t)i * kIn + v] : (double)t[i];
        s += z;
        s2 += z * z;
    }
    sh[0][th] = s;
    sh[1][th] = s2;
    __syncthreads();
    for (int off = kNormThreads / 2; off >= 1; off >>= 1) {
        if (th < off) {
            sh[0][th] += sh[0][th + off];
            sh[1][th] += sh[1][th + off];
        }
        __syncthreads();
    }
    if (th != 0) return;
    const double mean = sh[0][0] / n;
    const double var = sh[1][0] / n - mean * mean;
    const double sd = var > 1e-24 ? sqrt(var) : 1.0;
    if (v < kIn) {
        norm[v] = (float)mean;
        norm[kIn + v] = (float)sd;
    } else {
        norm[2 * kIn] = (float)mean;
        norm[2 * kIn + 1] = (float)sd;
    }
}

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Workspace.  `work` holds the partial gradients of as many blocks as fit and,
// behind them, the sample order of the coming minibatches (its size is that of
// the activations and deltas of max_batch samples).  `grad` carries the sum
// over blocks that did not fit at once, and holds the partials of a single one.
struct Layout {
    size_t params, grad, mom, wb, norm, work, loss, idx, total;
    size_t work_floats;
};

Layout layout(int max_batch)
{
    Layout l;
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t at = o;
        o = align_up(o + b);
        return at;
    };
    const size_t B = (size_t)max_batch;
    l.params = take(kParams * 4);
    l.grad = take(kParams * 4);
    l.mom = take(kParams * 4);
    l.wb = take(kParams * 2);
    l.norm = take(kNorm * 4);
    l.work = take(B * kIn * 4);
    take(B * 4);
    for (int k = 0; k < 4; ++k) take(B * kHid * 4);
    take(B * 4);
    take(B * 4);
    l.work_floats = (o - l.work) / 4;
    l.loss = take(16);
    l.idx = take(B * 4);
    l.total = o;
    return l;
}
static_assert((kParams * 4 + kAlign - 1) / kAlign * kAlign >= kPartStride * sizeof(float), "grad holds one block");

}  // namespace
}  // namespace mlp
}  // namespace pa

using namespace pa::mlp;

struct pa_mlp {
    int max_batch;
    hipStream_t stream;
    Layout lo;
    uint8_t* ws;
    float *p, *grad, *mom, *norm, *work, *loss;
    __hip_bfloat16* wb;
    int32_t* idx;
    // one pinned block, from pa_mlp_create on: no later call allocates any
    float* h_out = nullptr;         // gradient and loss, written by k_apply
    void* h_out_dev = nullptr;      // device view of h_out
    float* h_loss = nullptr;        // losses of kLossRing epochs
    int32_t* h_order[2] = {nullptr, nullptr};  // sample orders on their way, in turn
    size_t order_cap = 0;           // samples each of them holds
    hipEvent_t order_read[2] = {nullptr, nullptr};  // the last upload from each
    bool broken;
    std::string last_error;
};

namespace {

pa_status mfail(pa_mlp* m, hipError_t e, const char* what)
{
    m->broken = true;
    m->last_error = std::string(what) + ": " + hipGetErrorString(e);
    return PA_EHIP;
}

#define MCHK(expr)                                           \
    do {                                                     \
        const hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return mfail(m, e_, #expr);    \
    } while (0)

// Blocks that B samples are split over: a function of B alone, and with it the
// order of every sum.  Up to two tiles stay in one block, whose partials need
// no room in `work`; from 33 samples on `work` holds at least one block
// (267 floats per sample of max_batch >= B).
int blocks_of(int B) { return B <= 2 * kTile ? 1 : std::min((B + kTile - 1) / kTile, kMaxParts); }
static_assert((2 * kTile + 1) * (4 * kHid + kIn + 3) > kPartStride, "work holds a block");

// Blocks whose partials fit `work` at once.
int blocks_at_once(const pa_mlp* m, int blocks)
{
    return blocks == 1 ? 1 : (int)std::min<size_t>((size_t)blocks, m->lo.work_floats / kPartStride);
}

// Gradient of the B samples idx[0..B) (0..B without idx) of d_x, d_t, and the
// update or, with `grad`, the gradient itself.  Two launches where the
// partials of all blocks fit the workspace (max_batch of about 1.13 B on, and
// B <= 32), else two for every set that fits.
pa_status grad_pass(pa_mlp* m, const float* d_x, const float* d_t, const int32_t* idx, int B, float* grad, float lr,
                    float momentum, float* loss, bool start)
{
    const int blocks = blocks_of(B), set = blocks_at_once(m, blocks);
    float* parts = blocks == 1 ? m->grad : m->work;
    for (int b0 = 0; b0 < blocks; b0 += set) {
        const int nb = std::min(set, blocks - b0);
        hipLaunchKernelGGL(k_backprop, dim3(nb), dim3(256), 0, m->stream, d_x, d_t, idx, B, m->norm, m->p, b0, blocks,
                           parts);
        MCHK(hipGetLastError());
        hipLaunchKernelGGL(k_apply, dim3((kParams + 1 + 63) / 64), dim3(64), 0, m->stream, parts, nb, m->grad,
                           b0 > 0 ? 1 : 0, b0 + nb < blocks ? 1 : 0, B, grad, m->p, m->mom, lr, momentum, m->wb, loss,
                           start ? 1 : 0);
        MCHK(hipGetLastError());
    }
    return PA_OK;
}

// Samples of one upload of the order (at least a minibatch), and epochs whose
// losses are read back together.
constexpr int kOrderChunk = 8192;
constexpr int kLossRing = 1024;

}  // namespace

extern "C" {

size_t pa_mlp_workspace_bytes(int32_t max_batch)
{
    if (max_batch < 1 || max_batch > (1 << 20)) return 0;
    return layout(max_batch).total;
}

pa_status pa_mlp_create(int32_t max_batch, uint64_t seed, void* d_workspace, size_t bytes, void* hip_stream,
                        pa_mlp** out)
{
    if (!out) return PA_EINVAL;
    *out = nullptr;
    if (max_batch < 1 || max_batch > (1 << 20) || !d_workspace || ((uintptr_t)d_workspace) % 256) return PA_EINVAL;
    const Layout lo = layout(max_batch);
    if (bytes < lo.total) return PA_ENOMEM;
    pa_mlp* m = new (std::nothrow) pa_mlp();
    if (!m) return PA_ENOMEM;
    m->max_batch = max_batch;
    m->stream = (hipStream_t)hip_stream;
    m->lo = lo;
    uint8_t* w = (uint8_t*)d_workspace;
    m->ws = w;
    m->p = (float*)(w + lo.params);
    m->grad = (float*)(w + lo.grad);
    m->mom = (float*)(w + lo.mom);
    m->wb = (__hip_bfloat16*)(w + lo.wb);
    m->norm = (float*)(w + lo.norm);
    m->work = (float*)(w + lo.work);
    m->loss = (float*)(w + lo.loss);
    m->idx = (int32_t*)(w + lo.idx);
    // He initialisation from the seed; biases zero; identity normalisation.
    std::vector<float> p(kParams, 0.0f), zero(kParams, 0.0f), norm(kNorm, 0.0f);
    std::mt19937_64 rng(seed);
    std::normal_distribution<double> nd(0.0, 1.0);
    for (int i = 0; i < kHid * kIn; ++i) p[kW1 + i] = (float)(nd(rng) * std::sqrt(2.0 / kIn));
    for (int i = 0; i < kHid * kHid; ++i) p[kW2 + i] = (float)(nd(rng) * std::sqrt(2.0 / kHid));
    for (int i = 0; i < kHid; ++i) p[kW3 + i] = (float)(nd(rng) * std::sqrt(1.0 / kHid));
    for (int k = 0; k < kIn; ++k) norm[kIn + k] = 1.0f;
    norm[2 * kIn + 1] = 1.0f;
    m->order_cap = (size_t)std::max(max_batch, kOrderChunk);
    const size_t pinned = (size_t)(kPartStride + kLossRing) * 4 + 2 * m->order_cap * 4;
    if (hipHostMalloc((void**)&m->h_out, pinned, hipHostMallocMapped) != hipSuccess) {
        delete m;
        return PA_ENOMEM;
    }
    m->h_loss = m->h_out + kPartStride;
    m->h_order[0] = reinterpret_cast<int32_t*>(m->h_loss + kLossRing);
    m->h_order[1] = m->h_order[0] + m->order_cap;
    *out = m;
    MCHK(hipHostGetDevicePointer(&m->h_out_dev, m->h_out, 0));
    for (int k = 0; k < 2; ++k) MCHK(hipEventCreateWithFlags(&m->order_read[k], hipEventDisableTiming));
    MCHK(hipMemcpyAsync(m->p, p.data(), kParams * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemcpyAsync(m->mom, zero.data(), kParams * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemcpyAsync(m->norm, norm.data(), kNorm * 4, hipMemcpyHostToDevice, m->stream));
    hipLaunchKernelGGL(k_to_bf16, dim3((kParams + 255) / 256), dim3(256), 0, m->stream, m->p, m->wb);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    return PA_OK;
}

pa_status pa_mlp_set_params(pa_mlp* m, const float* params, const float* norm)
{
    if (!m || (!params && !norm)) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    if (params) {
        MCHK(hipMemcpyAsync(m->p, params, kParams * 4, hipMemcpyHostToDevice, m->stream));
        hipLaunchKernelGGL(k_to_bf16, dim3((kParams + 255) / 256), dim3(256), 0, m->stream, m->p, m->wb);
        MCHK(hipGetLastError());
    }
    if (norm) MCHK(hipMemcpyAsync(m->norm, norm, kNorm * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return PA_OK;
}

pa_status pa_mlp_get_params(pa_mlp* m, float* params, float* norm)
{
    if (!m || (!params && !norm)) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    if (params) MCHK(hipMemcpyAsync(params, m->p, kParams * 4, hipMemcpyDeviceToHost, m->stream));
    if (norm) MCHK(hipMemcpyAsync(norm, m->norm, kNorm * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return PA_OK;
}

pa_status pa_mlp_fit_norm(pa_mlp* m, const float* d_x, const float* d_t, int32_t n)
{
    if (!m || !d_x || !d_t || n < 2) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    hipLaunchKernelGGL(k_fit_norm, dim3(kIn + 1), dim3(kNormThreads), 0, m->stream, d_x, d_t, n, m->norm);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    return PA_OK;
}

pa_status pa_mlp_forward(pa_mlp* m, const float* d_x, int32_t n, float* d_y, int32_t bf16)
{
    if (!m || !d_x || !d_y || n < 0) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    if (n == 0) return PA_OK;
    hipLaunchKernelGGL(k_infer, dim3(n), dim3(64), 0, m->stream, d_x, m->p, m->wb, m->norm, bf16 ? 1 : 0, d_y);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    return PA_OK;
}

pa_status pa_mlp_gradient(pa_mlp* m, const float* d_x, const float* d_t, int32_t n, float* grad, float* loss)
{
    if (!m || !d_x || !d_t || n < 1 || n > m->max_batch) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    float* out = (float*)m->h_out_dev;
    const pa_status st = grad_pass(m, d_x, d_t, nullptr, n, out, 0.0f, 0.0f, out + kParams, true);
    if (st != PA_OK) return st;
    MCHK(hipStreamSynchronize(m->stream));
    if (grad) std::memcpy(grad, m->h_out, kParams * 4);
    if (loss) *loss = m->h_out[kParams];
    return PA_OK;
}

pa_status pa_mlp_train(pa_mlp* m, const float* d_x, const float* d_t, int32_t n, int32_t batch, int32_t epochs,
                       float lr, float momentum, uint64_t seed, float* epoch_loss)
{
    if (!m || !d_x || !d_t || n < 1 || batch < 1 || batch > m->max_batch || epochs < 0 || !(lr > 0.0f)) return PA_EINVAL;
    if (m->broken) return PA_ESTATE;
    std::mt19937_64 rng(seed);
    const int nb = n / batch;  // full minibatches only
    if (nb < 1) return PA_EINVAL;
    const std::unique_ptr<int32_t[]> perm(new (std::nothrow) int32_t[(size_t)n]);
    if (!perm) return PA_ENOMEM;
    // device room for the sample order: behind the partial sums, or the index
    // buffer of one minibatch
    int32_t* order = m->idx;
    size_t room = (size_t)m->max_batch;
    const int blocks = blocks_of(batch);
    const size_t used = blocks == 1 ? 0 : (size_t)blocks_at_once(m, blocks) * kPartStride;
    if (m->lo.work_floats - used > room) {
        order = (int32_t*)(m->work + used);
        room = m->lo.work_floats - used;
    }
    const int per_upload = (int)std::min<size_t>((size_t)nb, std::min(room, m->order_cap) / (size_t)batch);
    // Everything is queued without a wait: the order goes through two pinned
    // buffers in turn, each rewritten only after its last upload has been read.
    int uploads = 0;
    for (int e = 0; e < epochs; ++e) {
        for (int i = 0; i < n; ++i) perm[(size_t)i] = i;
        std::shuffle(perm.get(), perm.get() + n, rng);
        for (int k = 0; k < nb; ++k) {
            const int at = k % per_upload;
            if (at == 0) {
                const size_t count = (size_t)std::min(per_upload, nb - k) * (size_t)batch;
                const int h = uploads & 1;
                if (uploads >= 2) MCHK(hipEventSynchronize(m->order_read[h]));
                ++uploads;
                std::memcpy(m->h_order[h], perm.get() + (size_t)k * batch, count * 4);
                MCHK(hipMemcpyAsync(order, m->h_order[h], count * 4, hipMemcpyHostToDevice, m->stream));
                MCHK(hipEventRecord(m->order_read[h], m->stream));
            }
            const pa_status st = grad_pass(m, d_x, d_t, order + (size_t)at * batch, batch, nullptr, lr, momentum,
                                           m->loss, k == 0);
            if (st != PA_OK) return st;
        }
        const int slot = e % kLossRing;
        MCHK(hipMemcpyAsync(&m->h_loss[slot], m->loss, 4, hipMemcpyDeviceToHost, m->stream));
        if (slot == kLossRing - 1 || e == epochs - 1) {
            MCHK(hipStreamSynchronize(m->stream));
            if (epoch_loss)
                for (int i = 0; i <= slot; ++i) epoch_loss[e - slot + i] = m->h_loss[i] / (float)nb;
        }
    }
    return PA_OK;
}

const char* pa_mlp_last_error(const pa_mlp* m) { return m ? m->last_error.c_str() : ""; }

pa_status pa_mlp_free(pa_mlp* m)
{
    if (!m) return PA_OK;
    for (int k = 0; k < 2; ++k) {
        if (m->order_read[k]) (void)hipEventDestroy(m->order_read[k]);
    }
    if (m->h_out) (void)hipHostFree(m->h_out);
    delete m;
    return PA_OK;
}

}  // extern "C"
