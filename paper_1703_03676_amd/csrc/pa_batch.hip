// Batched population annealing: many independent runs (each with its own L,
// R, seed, spin store and schedule) advanced one temperature step at a time.
//
// One step of the whole batch:
//   host    per run, in a thread pool: next beta (fixed, adaptive bisection or
//           learned proposal + exact overlap test), FP64 copy-count tables of
//           Eq. (resampling factors), Metropolis thresholds
//   copy    one upload of every run's step descriptor and tables
//   device  counts -> parent scatter -> sweep (one launch for all register-path
//           lattice sizes of a store, one per larger size) -> statistics,
//           written to host memory by the last block of every run, which the
//           host polls
//   host    commit each run (ln Z += ln Q, observables of Eq. (observables))
// The launches of a step are few and queued one by one: the first kernel runs
// while the later ones are queued.  (A captured graph of the same kernels took
// the host 28 us to launch before the first one started, and left 4-8 us
// between its nodes.  A step of 12 runs of L = 16, 32 and 64 with 1000 and 5000
// replicas: 271 us by the graph, a scan launch for every run, a stream wait and
// fences in every wave of the statistics; 247 us so.)
// Kernels read each run's step descriptor and its device-side population
// size, so launch shapes stay fixed while R_i changes.  A run whose resampling
// would exceed its capacity or die out is flagged on the device; its copy and
// sweep are skipped and its state stays at the last good step.
//
// Launch shapes of the sweep (waves per block) are chosen per launch by timing
// the candidates on the batch's own spare buffers at start-up.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "pa.h"
#include "pa_device.h"
#include "pa_reduce.h"
#include "pa_host.h"
#include "pa_mlp_dev.h"

namespace pa {
namespace batch {

using namespace pa::dev;

struct RunDev {
    uint8_t* spin[2];
    int32_t* E[2];
    int32_t* M[2];
    uint32_t* counts;
    uint32_t* parent;
    uint32_t* bsum;
    DevStats* stats;  // followed by the energy histogram
    uint32_t* hist;
    StatsPart* parts;  // per-block partial statistics
    DevMhr mhr;
    int32_t L, N, nbins, capacity, layout, R;
    uint32_t rep_bytes;
    uint32_t key0, key1;  // Philox key: the run's seed
    uint32_t tag;         // 16 * run_id: counter word 3 without the stream number
    uint32_t qcap;        // tie-queue limit of the LDS-path sweeps (SweepArgs::qcap)
    uint64_t host_off;    // the run's statistics block and histogram in the host's download area
};

struct StepDev {
    int32_t active;    // the run takes part in this step
    int32_t resample;  // resample before the sweeps
    int32_t init;      // draw the initial state instead of loading spins
    int32_t record;    // add this measurement to the multi-histogram accumulators
    int32_t cur;       // buffer holding the parents
    int32_t n_parent;  // R_{i-1}
    uint32_t step;     // resampling index i (RESAMPLE stream counter)
    uint32_t g0;       // sweep counter of the first sweep of this step
    int32_t nsweeps;
    uint32_t t2h, t2l, t4h, t4l;
    int32_t bmin, nwin;
    uint32_t tbl_off;  // offset in u32 of this run's tables in the table area
    uint32_t seq;      // number of the step, by which the host knows its publication
    double beta;        // inverse temperature after this step
    double last_dbeta;  // the step just taken (0: none)
};

// Features of the population after a step and the learned proposal for the
// next step (natural log of the step size).
struct FeatDev {
    float x[8];
    float prop;
    int32_t valid;
};

// Learned proposer as used by the batch: BF16 weights and normalisation.
struct ModelDev {
    int32_t set;
    int32_t pad[3];
    float norm[pa::mlp::kNorm];
    __hip_bfloat16 wb[pa::mlp::kParams];
};

struct ResultDev {
    uint32_t r_new;  // sum of the copy counts
    uint32_t err;    // 0 ok, 1 capacity exceeded, 2 no replica left
};

struct Item {
    int32_t run, blk;
};

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

// The buffer and population size the sweep and the statistics work on.
__device__ __forceinline__ bool post_resample(const StepDev& st, const ResultDev& rs, int* buf, int* n)
{
    if (st.resample) {
        if (rs.err) {
            *buf = st.cur;
            *n = st.n_parent;
            return false;
        }
        *buf = st.cur ^ 1;
        *n = (int)rs.r_new;
        return true;
    }
    *buf = st.cur;
    *n = st.n_parent;
    return true;
}

// Runs of more parents than this (kScanFreeBlocks blocks of b_counts) have their
// block sums scanned by b_scan; in the others every block of b_scatter sums
// those before it, which saves the launch.
__host__ __device__ constexpr bool scanned_run(int32_t capacity)
{
    return capacity > pa::kScanFreeBlocks * kBlock;
}

// Also clears the run's statistics for this step's population (the host has
// read the previous ones).
__global__ __launch_bounds__(kBlock) void b_counts(const Item* __restrict__ items, const RunDev* __restrict__ runs,
                                                   const StepDev* __restrict__ steps, const uint32_t* __restrict__ tbl)
{
    const Item it = items[blockIdx.x];
    const StepDev st = steps[it.run];
    if (!st.active || it.blk * kBlock >= st.n_parent) return;  // uniform per block
    const RunDev& rd = runs[it.run];
    const int j = it.blk * kBlock + (int)threadIdx.x;
    if (j == 0) {
        DevStats* s = rd.stats;
        s->emin = 0x7FFFFFFF;
        s->emax = (int32_t)0x80000000;
        s->r_new = 0;
        s->done = 0;
        s->sumE = s->sumE2 = s->sumAbsM = s->sumM2 = s->sumM4_lo = s->sumM4_hi = 0;
    }
    const int nblk = (st.n_parent + kBlock - 1) / kBlock;
    for (int b = j; b < rd.nbins; b += nblk * kBlock) rd.hist[b] = 0;
    if (!st.resample) return;
    uint32_t c = 0;
    if (j < st.n_parent) {
        const int b = ((rd.E[st.cur][j] + 2 * rd.N) >> 2) - st.bmin;
        const uint32_t x = pick(philox10((uint32_t)j >> 2, st.step, 0u, rd.tag | kStreamResample, rd.key0, rd.key1),
                                (uint32_t)j & 3u);
        if (b >= 0 && b < st.nwin) {
            const uint32_t base = tbl[st.tbl_off + 2 * b], thr = tbl[st.tbl_off + 2 * b + 1];
            c = base + (x <= thr ? 1u : 0u);
        }
        rd.counts[j] = c;
    }
    uint32_t total;
    block_exclusive_scan(c, &total);
    if (threadIdx.x == 0) rd.bsum[it.blk] = total;
}

// Size and status of a run's resampled population.
__device__ __forceinline__ ResultDev resampled(uint32_t total, int32_t capacity)
{
    return ResultDev{total, total > (uint32_t)capacity ? 1u : (total == 0u ? 2u : 0u)};
}

// One block per run that needs it (scanned_run): the exclusive scan of its
// block sums, total and status.
__global__ __launch_bounds__(1024) void b_scan(const RunDev* __restrict__ runs, const StepDev* __restrict__ steps,
                                               ResultDev* __restrict__ res)
{
    __shared__ uint32_t part[1024];
    const StepDev st = steps[blockIdx.x];
    if (!st.active || !st.resample || !scanned_run(runs[blockIdx.x].capacity)) return;
    uint32_t* bsum = runs[blockIdx.x].bsum;
    const int nblk = (st.n_parent + kBlock - 1) / kBlock;
    const int t = (int)threadIdx.x;
    const int per = (nblk + 1023) / 1024;
    const int lo = t * per, hi = min(nblk, lo + per);
    uint32_t s = 0;
    for (int i = lo; i < hi; ++i) s += bsum[i];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint32_t y = (t >= off) ? part[t - off] : 0u;
        __syncthreads();
        part[t] += y;
        __syncthreads();
    }
    uint32_t run = part[t] - s;
    for (int i = lo; i < hi; ++i) {
        const uint32_t v = bsum[i];
        bsum[i] = run;
        run += v;
    }
    if (t == 1023) res[blockIdx.x] = resampled(part[1023], runs[blockIdx.x].capacity);
}

// Parent of every child; children beyond the capacity (a refused step) are not
// written.
__global__ __launch_bounds__(kBlock) void b_scatter(const Item* __restrict__ items, const RunDev* __restrict__ runs,
                                                    const StepDev* __restrict__ steps,
                                                    ResultDev* __restrict__ res)
{
    __shared__ uint32_t wpart[kBlock / 64];
    const Item it = items[blockIdx.x];
    const StepDev st = steps[it.run];
    if (!st.active || !st.resample || it.blk * kBlock >= st.n_parent) return;
    const RunDev& rd = runs[it.run];
    const bool scanned = scanned_run(rd.capacity);
    const int lane = (int)(threadIdx.x & 63u);
    const int j = it.blk * kBlock + (int)threadIdx.x;
    const uint32_t c = (j < st.n_parent) ? rd.counts[j] : 0u;
    uint32_t base = 0;
    if (scanned) {
        base = rd.bsum[it.blk];
    } else {
        uint32_t before = 0;
        for (int i = (int)threadIdx.x; i < it.blk; i += kBlock) before += rd.bsum[i];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) before += (uint32_t)__shfl_xor((int)before, off);
        if (lane == 0) wpart[threadIdx.x >> 6] = before;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) base += wpart[w];
    }
    uint32_t total;
    const uint32_t off = base + block_exclusive_scan(c, &total);
    fill_parents(rd.parent, off, c, (uint32_t)(j - lane), (uint32_t)rd.capacity);
    if (!scanned && threadIdx.x == 0 && (it.blk + 1) * kBlock >= st.n_parent)
        res[it.run] = resampled(base + total, rd.capacity);
}

// Item blk covers 16-byte chunks [blk * kBlock, (blk + 1) * kBlock) of the run's new population.
__global__ __launch_bounds__(kBlock) void b_copy(const Item* __restrict__ items, const RunDev* __restrict__ runs,
                                                 const StepDev* __restrict__ steps, const ResultDev* __restrict__ res)
{
    const Item it = items[blockIdx.x];
    const StepDev st = steps[it.run];
    // a step with sweeps gathers its parents in b_sweep instead
    if (!st.active || !st.resample || res[it.run].err || st.nsweeps > 0) return;
    const RunDev& rd = runs[it.run];
    const uint32_t chunks = rd.rep_bytes / 16;
    const size_t total = (size_t)res[it.run].r_new * chunks;
    const size_t i = (size_t)it.blk * kBlock + threadIdx.x;
    if (i >= total) return;
    const uint32_t child = (uint32_t)(i / chunks), ch = (uint32_t)(i % chunks);
    const uint32_t p = rd.parent[child];
    const uint4* src = reinterpret_cast<const uint4*>(rd.spin[st.cur]);
    uint4* dst = reinterpret_cast<uint4*>(rd.spin[st.cur ^ 1]);
    dst[i] = src[(size_t)p * chunks + ch];
    if (ch == 0) {
        rd.E[st.cur ^ 1][child] = rd.E[st.cur][p];
        rd.M[st.cur ^ 1][child] = rd.M[st.cur][p];
    }
}

// Item blk covers waves [blk * wpb, (blk + 1) * wpb) of the run (wpb = blockDim.x / 64).
// L = kSmall: the register-path lattice sizes together, each block that of its
// run, so that the short launches of small lattices fill the GPU beside the
// larger ones instead of following them (12 runs of L = 16, 32 and 64: 47 us of
// separate launches per step beside 137 for L = 64 alone).
constexpr int kSmall = 0;

template <int L, bool INT8, int U>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(sweep_min_waves<L>(), 8))) void b_sweep(
    const Item* __restrict__ items, const RunDev* __restrict__ runs, const StepDev* __restrict__ steps,
    const ResultDev* __restrict__ res)
{
    extern __shared__ __align__(16) uint32_t lds_dyn[];
    const Item it = items[blockIdx.x];
    const StepDev st = steps[it.run];
    if (!st.active) return;
    int buf, n;
    if (!post_resample(st, res[it.run], &buf, &n)) return;  // failed resampling: no sweep
    const RunDev& rd = runs[it.run];
    SweepArgs a;
    a.n_dev = nullptr;
    // after a resampling, every child is loaded straight from its parent (the
    // replica copy and the sweep's load are one pass over the store)
    const bool gather = st.resample && st.nsweeps > 0;
    a.src = gather ? rd.spin[st.cur] : nullptr;
    a.parent = gather ? rd.parent : nullptr;
    a.spin = rd.spin[buf];
    a.E = rd.E[buf];
    a.M = rd.M[buf];
    a.n_rep = n;
    a.nsweeps = st.nsweeps;
    a.g0 = st.g0;
    a.key0 = rd.key0;
    a.key1 = rd.key1;
    a.tag = rd.tag;
    a.qcap = rd.qcap;
    a.acc = nullptr;  // the batch takes its statistics in b_stats
    a.acc_hist = nullptr;
    a.nbins = 0;
    a.t2h = st.t2h;
    a.t2l = st.t2l;
    a.t4h = st.t4h;
    a.t4l = st.t4l;
    a.init = st.init;
    const int wpb = (int)(blockDim.x >> 6);
    a.one_round = (int)gridDim.x * wpb <= sweep_resident_waves<(L == kSmall ? 64 : L)>() ? 1 : 0;
    constexpr bool HB = U == pa::kHeatbath, LCG = U == pa::kLcg;
    if constexpr (L == kSmall) {
        switch (rd.L) {  // uniform
        case 16: sweep_waves<16, INT8, HB, LCG>(a, it.blk * wpb, lds_dyn); break;
        case 32: sweep_waves<32, INT8, HB, LCG>(a, it.blk * wpb, lds_dyn); break;
        default: sweep_waves<64, INT8, HB, LCG>(a, it.blk * wpb, lds_dyn); break;
        }
    } else {
        sweep_waves<L, INT8, HB, LCG>(a, it.blk * wpb, lds_dyn);
    }
}

// Energy moments of a measured population from its histogram (FP64, fixed-order
// reduction over the first 64 threads), the proposer's features, and -- when a
// model is loaded -- the BF16 proposal for the next step:
//   x = (e/N, ln sigma_E, skew, excess kurtosis, beta, ln L, ln R, ln last step).
// Called by every thread of the block.
__device__ __forceinline__ void run_features(const RunDev& rd, const StepDev& st, int n, bool ok,
                                             const ModelDev* __restrict__ model, FeatDev* __restrict__ out)
{
    __shared__ double red[3][64];
    __shared__ float h[pa::mlp::kHid];
    __shared__ float xs[8];
    const DevStats* sp = rd.stats;
    const int t = (int)threadIdx.x;
    const double mean = (double)(int64_t)sp->sumE / (double)n;
    if (t < 64) {
        const int bmin = (sp->emin + 2 * rd.N) / 4, bmax = (sp->emax + 2 * rd.N) / 4;
        double a2 = 0.0, a3 = 0.0, a4 = 0.0;
        for (int b = bmin + t; b <= bmax; b += 64) {
            const uint32_t c = rd.hist[b];
            if (c == 0) continue;
            const double d = (double)(4 * b - 2 * rd.N) - mean;
            const double d2 = d * d;
            a2 += c * d2;
            a3 += c * d2 * d;
            a4 += c * d2 * d2;
        }
        red[0][t] = a2;
        red[1][t] = a3;
        red[2][t] = a4;
    }
    __syncthreads();
    for (int off = 32; off >= 1; off >>= 1) {
        if (t < off) {
            red[0][t] += red[0][t + off];
            red[1][t] += red[1][t + off];
            red[2][t] += red[2][t + off];
        }
        __syncthreads();
    }
    const double var = red[0][0] / n;
    const bool valid = ok && var > 0.0 && st.last_dbeta > 0.0;
    if (t == 0) {
        const double sd = var > 0.0 ? sqrt(var) : 1.0;
        xs[0] = (float)(mean / rd.N);
        xs[1] = (float)log(sd);
        xs[2] = (float)(red[1][0] / n / (sd * sd * sd));
        xs[3] = (float)(red[2][0] / n / (var * var) - 3.0);
        xs[4] = (float)st.beta;
        xs[5] = (float)log((double)rd.L);
        xs[6] = (float)log((double)rd.R);
        xs[7] = st.last_dbeta > 0.0 ? (float)log(st.last_dbeta) : 0.0f;
        for (int k = 0; k < 8; ++k) out->x[k] = xs[k];
        out->valid = valid ? 1 : 0;
        out->prop = 0.0f;
    }
    __syncthreads();
    if (valid && model->set) {  // uniform
        const float y = pa::mlp::forward_bf16(xs, model->wb, model->norm, h, t);
        if (t == 0) out->prop = y;
    }
}

// Statistics of every run's population, one block per chunk of kBlock replicas.
// The block of a run that finishes last (counted in its statistics block) sums
// the partials, computes the features, and writes the run's results, features,
// statistics block and the occupied window of its histogram to the host's
// download area, so that no further kernel and no copy follows.  (Separate
// kernels for the clearing, the sum and the features, and the copy of every
// histogram, took 24 us per step of 12 small runs; this one takes 15.)
__global__ __launch_bounds__(kBlock) void b_stats(const Item* __restrict__ items, const RunDev* __restrict__ runs,
                                                  const StepDev* __restrict__ steps, const ResultDev* __restrict__ res,
                                                  const ModelDev* __restrict__ model, uint8_t* host, size_t feats_off)
{
    const Item it = items[blockIdx.x];
    const StepDev st = steps[it.run];
    if (!st.active) return;
    const ResultDev rs = res[it.run];
    int buf, n;
    const bool ok = post_resample(st, rs, &buf, &n);
    if (it.blk * kBlock >= n) return;
    const RunDev& rd = runs[it.run];
    stats_block(rd.E[buf], rd.M[buf], n, rd.N, it.blk * kBlock, rd.hist, rd.nbins, st.record && ok, rd.mhr,
                &rd.parts[it.blk]);
    const int nparts = (n + kBlock - 1) / kBlock;
    if (!finishes_last(&rd.stats->done, (uint32_t)nparts)) return;  // uniform per block
    stats_final(rd.parts, nparts, rd.stats);
    __syncthreads();  // *rd.stats written by thread 0 is visible to the block
    const uint32_t* sw = reinterpret_cast<const uint32_t*>(rd.stats);
    uint32_t* hs = reinterpret_cast<uint32_t*>(host + rd.host_off);
    if (threadIdx.x < sizeof(DevStats) / 4 && threadIdx.x != 3) hs[threadIdx.x] = sw[threadIdx.x];
    if (threadIdx.x == 0) reinterpret_cast<ResultDev*>(host)[it.run] = rs;
    const int32_t emin = rd.stats->emin, emax = rd.stats->emax;
    if (emin >= -2 * rd.N && emax <= 2 * rd.N)
        for (int b = (emin + 2 * rd.N) / 4 + (int)threadIdx.x; b <= (emax + 2 * rd.N) / 4; b += kBlock)
            hs[sizeof(DevStats) / 4 + b] = rd.hist[b];
    run_features(rd, st, n, ok, model, reinterpret_cast<FeatDev*>(host + feats_off) + it.run);
    publish_seq(hs, st.seq);
}

__global__ void b_fill_u32(uint32_t* p, uint32_t value, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool lattice_supported(int L) { return L == 16 || L == 32 || L == 64 || L == 128 || L == 256; }

int32_t default_capacity(int32_t R) { return R + (int32_t)std::ceil(10.0 * std::sqrt((double)R)) + 64; }

bool valid_params(const pa_params& p)
{
    if (!lattice_supported(p.L) || p.R < 1) return false;
    if (p.layout != PA_SPIN_INT8 && p.layout != PA_SPIN_BITS) return false;
    if (p.flags & ~(uint32_t)(PA_FLAG_MHR | PA_FLAG_HEATBATH | PA_FLAG_LCG)) return false;
    if ((p.flags & PA_FLAG_HEATBATH) && (p.flags & PA_FLAG_LCG)) return false;
    if (p.run_id >= (1u << 28)) return false;
    const int64_t cap = p.capacity ? p.capacity : default_capacity(p.R);
    return cap >= p.R && cap <= ((int64_t)1 << 30);
}

bool valid_schedule(const pa_schedule& s)
{
    if (!(s.beta_f > 0.0) || !std::isfinite(s.beta_f) || s.theta < 0) return false;
    switch (s.mode) {
    case PA_STEP_FIXED: return s.dbeta > 0.0 && std::isfinite(s.dbeta);
    case PA_STEP_ADAPTIVE: return s.alpha_star > 0.0 && s.alpha_star < 1.0;
    case PA_STEP_LEARNED: return s.alpha_star > 0.0 && s.alpha_star < 1.0 && s.alpha_tol >= 0.0;
    case PA_STEP_FOLLOW: return true;  // the leader is checked against the whole batch
    default: return false;
    }
}

// Per-run placement inside the batch workspace.
struct RunLayout {
    size_t spin[2], E[2], M[2], counts, parent, bsum, parts, mhr;
    size_t stats_off;  // offset of the stats block inside the download area
    size_t tbl_words;  // table capacity in u32
    int32_t capacity, nbins, nblk;
    size_t rep_bytes;
};

struct BatchLayout {
    std::vector<RunLayout> runs;
    size_t rundev, steps, results, download, tables, items, model, total;
    size_t feats;           // offset of the features in the host's download area, behind the rest
    size_t download_bytes;  // results + all stats blocks and histograms, then the features
    size_t steps_bytes;     // step descriptors + table area
    size_t n_items;
};

struct Group {
    int L, layout;  // L: kSmall for the register-path sizes together
    int upd;  // update rule of its runs (pa::Update)
    int wpb;
    size_t item_off, n_items;
};

bool heatbath(const pa_params& p) { return (p.flags & PA_FLAG_HEATBATH) != 0; }

int update_of(const pa_params& p)
{
    if (p.flags & PA_FLAG_HEATBATH) return pa::kHeatbath;
    if (p.flags & PA_FLAG_LCG) return pa::kLcg;
    return pa::kMetropolis;
}

// Sweep group of a lattice size, and whether a run belongs to a group.
int group_size(int L) { return L <= 64 ? kSmall : L; }

bool in_group(const pa_params& p, const Group& g)
{
    return group_size(p.L) == g.L && p.layout == g.layout && update_of(p) == g.upd;
}

bool make_batch_layout(const pa_params* runs, int nruns, BatchLayout* bl)
{
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    bl->runs.resize((size_t)nruns);
    size_t dl = align_up(sizeof(ResultDev) * (size_t)nruns);
    size_t tbl = 0;
    for (int r = 0; r < nruns; ++r) {
        const pa_params& p = runs[r];
        if (!valid_params(p)) return false;
        RunLayout& rl = bl->runs[(size_t)r];
        const int64_t N = (int64_t)p.L * p.L;
        rl.capacity = p.capacity ? p.capacity : default_capacity(p.R);
        rl.nbins = (int32_t)N + 1;
        rl.nblk = (rl.capacity + kBlock - 1) / kBlock;
        rl.rep_bytes = (p.layout == PA_SPIN_INT8) ? (size_t)N : (size_t)N / 8;
        for (int b = 0; b < 2; ++b) {
            rl.spin[b] = take((size_t)rl.capacity * rl.rep_bytes);
            rl.E[b] = take((size_t)rl.capacity * 4);
            rl.M[b] = take((size_t)rl.capacity * 4);
        }
        rl.counts = take((size_t)rl.capacity * 4);
        rl.parent = take((size_t)rl.capacity * 4);
        rl.bsum = take((size_t)rl.nblk * 4 + 4);
        rl.parts = take(sizeof(StatsPart) * (size_t)rl.nblk);
        rl.mhr = (p.flags & PA_FLAG_MHR) ? take((size_t)rl.nbins * 40) : 0;
        rl.stats_off = dl;
        dl = align_up(dl + sizeof(DevStats) + (size_t)rl.nbins * 4);
        rl.tbl_words = (size_t)rl.nbins * 2;
        tbl += rl.tbl_words;
    }
    bl->feats = dl;
    bl->download_bytes = dl + sizeof(FeatDev) * (size_t)nruns;
    bl->steps_bytes = align_up(sizeof(StepDev) * (size_t)nruns) + tbl * 4;
    bl->rundev = take(sizeof(RunDev) * (size_t)nruns);
    bl->steps = take(bl->steps_bytes);
    bl->download = take(dl);
    bl->results = bl->download;  // results lead the download area
    bl->model = take(sizeof(ModelDev));
    // items: parents/statistics, copy chunks, and sweep items of every candidate shape
    size_t n_items = 0;
    for (int r = 0; r < nruns; ++r) {
        const RunLayout& rl = bl->runs[(size_t)r];
        const int64_t L = runs[r].L;
        const int64_t N = L * L, NW = N / 64, G = NW < 64 ? NW : 64, repw = 64 / G;
        const size_t chunks = rl.rep_bytes / 16;
        n_items += (size_t)rl.nblk;                                             // counts / scatter / stats
        n_items += ((size_t)rl.capacity * chunks + kBlock - 1) / kBlock;          // copy
        n_items += 2 * (size_t)((rl.capacity + repw - 1) / repw);                 // sweep, any shape (upper bound)
    }
    bl->n_items = n_items;
    bl->items = take(n_items * sizeof(Item));
    bl->tables = bl->steps + align_up(sizeof(StepDev) * (size_t)nruns);
    bl->total = o;
    return true;
}

// Minimal fork-join pool for the per-run host work.
class Pool {
public:
    explicit Pool(int n) : nthreads_(std::max(1, n)) {
        for (int i = 1; i < nthreads_; ++i) workers_.emplace_back([this, i] { loop(i); });
    }
    ~Pool() {
        {
            std::lock_guard<std::mutex> g(m_);
            stop_ = true;
            ++gen_;
        }
        cv_.notify_all();
        for (auto& t : workers_) t.join();
    }
    void parallel_for(int n, const std::function<void(int)>& fn) {
        if (nthreads_ == 1 || n <= 1) {
            for (int i = 0; i < n; ++i) fn(i);
            return;
        }
        {
            std::lock_guard<std::mutex> g(m_);
            fn_ = &fn;
            n_ = n;
            next_.store(0);
            pending_ = nthreads_ - 1;
            ++gen_;
        }
        cv_.notify_all();
        run_items();
        std::unique_lock<std::mutex> lk(m_);
        done_cv_.wait(lk, [this] { return pending_ == 0; });
        fn_ = nullptr;
    }

private:
    void run_items() {
        for (;;) {
            const int i = next_.fetch_add(1);
            if (i >= n_) break;
            (*fn_)(i);
        }
    }
    void loop(int) {
        uint64_t seen = 0;
        for (;;) {
            {
                std::unique_lock<std::mutex> lk(m_);
                cv_.wait(lk, [&] { return gen_ != seen; });
                seen = gen_;
                if (stop_) return;
            }
            run_items();
            {
                std::lock_guard<std::mutex> g(m_);
                if (--pending_ == 0) done_cv_.notify_one();
            }
        }
    }
    int nthreads_;
    std::vector<std::thread> workers_;
    std::mutex m_;
    std::condition_variable cv_, done_cv_;
    const std::function<void(int)>* fn_ = nullptr;
    int n_ = 0;
    std::atomic<int> next_{0};
    int pending_ = 0;
    uint64_t gen_ = 0;
    bool stop_ = false;
};

}  // namespace batch
}  // namespace pa

using namespace pa::batch;
using pa::DevMhr;
using pa::DevStats;
using pa::kBlock;
namespace host = pa::host;

struct RunHost {
    pa_params p;
    pa_schedule sched;
    int64_t R_cur = 0;
    int32_t step = 0;
    uint64_t sweeps = 0;
    double beta = 0.0, lnZ = 0.0, lnQ_last = 0.0;
    int cur = 0;
    pa_status status = PA_OK;
    bool finished = false;
    // pending step
    bool stepping = false;
    double beta_next = 0.0, lnQ_next = 0.0;
    std::vector<pa_obs> history;
    std::vector<double> m_beta, m_lnZ;
    std::vector<int64_t> m_R;
    std::vector<double> w;  // scratch
    DevStats h_stats;
    const uint32_t* h_hist = nullptr;
    FeatDev feat;
    double last_dbeta = 0.0;
    int32_t proposals = 0, accepted = 0;
    int64_t alpha_evals = 0;   // overlaps compared with the target to choose the temperatures
    double choose_s = 0.0;     // host seconds spent choosing them
    std::vector<float> pair_x, pair_t;  // (features, ln(step sigma_E)) from the bisection
};

struct pa_batch {
    int nruns = 0;
    BatchLayout lo;
    uint8_t* ws = nullptr;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    std::vector<RunHost> runs;
    std::vector<RunDev> rundev;
    RunDev* d_rundev = nullptr;
    StepDev* d_steps = nullptr;
    uint32_t* d_tables = nullptr;
    ResultDev* d_results = nullptr;
    ModelDev* d_model = nullptr;
    bool model_set = false;
    uint8_t* d_download = nullptr;
    Item* d_items = nullptr;
    // items: parents, copy, and sweep items per group
    size_t parent_off = 0, n_parent_items = 0, copy_off = 0, n_copy_items = 0;
    std::vector<Group> groups;
    uint8_t* h_steps = nullptr;     // pinned: step descriptors + tables
    uint8_t* h_download = nullptr;  // pinned: results, features and statistics, written by b_stats
    void* h_download_dev = nullptr; // device view of h_download
    bool any_scanned = false;       // some run's block sums need b_scan
    uint32_t seq = 0;               // number of the last step queued
    pa::batch::Pool* pool = nullptr;
    pa_batch_options opt{0};  // forced launch shape (0: autotuned)
    bool broken = false;
    std::string last_error;
};

namespace {

pa_status fail_hip(pa_batch* b, hipError_t e, const char* what)
{
    b->broken = true;
    b->last_error = std::string(what) + ": " + hipGetErrorString(e);
    return PA_EHIP;
}

#define BCHK(expr)                                            \
    do {                                                      \
        const hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) return fail_hip(b, e_, #expr);  \
    } while (0)

template <int L, bool INT8, int U>
hipError_t launch_group_t(const Item* items, size_t n, int wpb, const RunDev* rd, const StepDev* st,
                          const ResultDev* rs, hipStream_t s)
{
    size_t lds = 0;
    if constexpr (L != kSmall) lds = (size_t)pa::dev::Geo<L>::lds_words(wpb) * 4;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((b_sweep<L, INT8, U>), dim3((unsigned)n), dim3(64 * wpb), lds, s, items, rd, st, rs);
    return hipGetLastError();
}

template <int L, bool INT8>
hipError_t launch_group_u(int upd, const Item* items, size_t n, int wpb, const RunDev* rd, const StepDev* st,
                          const ResultDev* rs, hipStream_t s)
{
    switch (upd) {
    case pa::kMetropolis: return launch_group_t<L, INT8, pa::kMetropolis>(items, n, wpb, rd, st, rs, s);
    case pa::kHeatbath: return launch_group_t<L, INT8, pa::kHeatbath>(items, n, wpb, rd, st, rs, s);
    case pa::kLcg: return launch_group_t<L, INT8, pa::kLcg>(items, n, wpb, rd, st, rs, s);
    default: return hipErrorInvalidValue;
    }
}

template <int L>
hipError_t launch_group_l(bool i8, int upd, const Item* items, size_t n, int wpb, const RunDev* rd,
                          const StepDev* st, const ResultDev* rs, hipStream_t s)
{
    return i8 ? launch_group_u<L, true>(upd, items, n, wpb, rd, st, rs, s)
              : launch_group_u<L, false>(upd, items, n, wpb, rd, st, rs, s);
}

hipError_t launch_group(const Group& g, const Item* items, size_t n, int wpb, const RunDev* rd, const StepDev* st,
                        const ResultDev* rs, hipStream_t s)
{
    const bool i8 = g.layout == PA_SPIN_INT8;
    switch (g.L) {
    case kSmall: return launch_group_l<kSmall>(i8, g.upd, items, n, wpb, rd, st, rs, s);
    case 128: return launch_group_l<128>(i8, g.upd, items, n, wpb, rd, st, rs, s);
    case 256: return launch_group_l<256>(i8, g.upd, items, n, wpb, rd, st, rs, s);
    default: return hipErrorInvalidValue;
    }
}

int reps_per_wave(int L)
{
    switch (L) {
    case 16: return pa::dev::Geo<16>::RPWV;
    case 32: return pa::dev::Geo<32>::RPWV;
    case 64: return pa::dev::Geo<64>::RPWV;
    case 128: return pa::dev::Geo<128>::RPWV;
    default: return pa::dev::Geo<256>::RPWV;
    }
}

// LDS bytes of a sweep block of wpb waves.
size_t sweep_lds_bytes(int L, int wpb)
{
    switch (L) {
    case kSmall: return 0;
    case 128: return (size_t)pa::dev::Geo<128>::lds_words(wpb) * 4;
    default: return (size_t)pa::dev::Geo<256>::lds_words(wpb) * 4;
    }
}

// Sweep items of one group for a given number of waves per block.
// The group's blocks, those of the larger lattices (the longer ones) first.
std::vector<Item> sweep_items(const pa_batch* b, const Group& g, int wpb)
{
    std::vector<Item> it;
    for (int L = 256; L >= 16; L >>= 1)
        for (int r = 0; r < b->nruns; ++r) {
            const pa_params& p = b->runs[(size_t)r].p;
            if (p.L != L || !in_group(p, g)) continue;
            const int per_block = reps_per_wave(L) * wpb;
            const int cap = b->lo.runs[(size_t)r].capacity;
            const int nb = (cap + per_block - 1) / per_block;
            for (int k = 0; k < nb; ++k) it.push_back(Item{r, k});
        }
    return it;
}

// Enqueue the device part of one step, with or without the separate replica
// copy of runs that resample without sweeping.
pa_status enqueue_step(pa_batch* b, bool with_copy)
{
    const hipStream_t s = b->stream;
    const Item* items = b->d_items;
    if (b->n_parent_items) {
        hipLaunchKernelGGL(b_counts, dim3((unsigned)b->n_parent_items), dim3(kBlock), 0, s, items + b->parent_off,
                           b->d_rundev, b->d_steps, b->d_tables);
        BCHK(hipGetLastError());
    }
    if (b->any_scanned) {
        hipLaunchKernelGGL(b_scan, dim3((unsigned)b->nruns), dim3(1024), 0, s, b->d_rundev, b->d_steps, b->d_results);
        BCHK(hipGetLastError());
    }
    hipLaunchKernelGGL(b_scatter, dim3((unsigned)b->n_parent_items), dim3(kBlock), 0, s, items + b->parent_off,
                       b->d_rundev, b->d_steps, b->d_results);
    BCHK(hipGetLastError());
    if (with_copy && b->n_copy_items) {
        hipLaunchKernelGGL(b_copy, dim3((unsigned)b->n_copy_items), dim3(kBlock), 0, s, items + b->copy_off,
                           b->d_rundev, b->d_steps, b->d_results);
        BCHK(hipGetLastError());
    }
    for (const Group& g : b->groups)
        BCHK(launch_group(g, items + g.item_off, g.n_items, g.wpb, b->d_rundev, b->d_steps, b->d_results, s));
    hipLaunchKernelGGL(b_stats, dim3((unsigned)b->n_parent_items), dim3(kBlock), 0, s, items + b->parent_off,
                       b->d_rundev, b->d_steps, b->d_results, b->d_model, (uint8_t*)b->h_download_dev, b->lo.feats);
    BCHK(hipGetLastError());
    return PA_OK;
}

StepDev* host_steps(pa_batch* b) { return reinterpret_cast<StepDev*>(b->h_steps); }
uint32_t* host_tables(pa_batch* b)
{
    return reinterpret_cast<uint32_t*>(b->h_steps + (b->lo.tables - b->lo.steps));
}

// Runs one step after uploading the first `bytes` bytes of the step descriptors
// and packed tables, with the separate replica copy only if some run resamples
// without sweeping (its launch covers every run's capacity and costs tens of
// microseconds even when it has nothing to do).  Waits for the publication of
// every run that takes part.
pa_status run_step(pa_batch* b, size_t bytes, bool need_copy)
{
    if (++b->seq == 0u) b->seq = 1u;
    StepDev* sd = host_steps(b);
    for (int r = 0; r < b->nruns; ++r) sd[r].seq = b->seq;
    BCHK(hipMemcpyAsync(b->d_steps, b->h_steps, bytes, hipMemcpyHostToDevice, b->stream));
    const pa_status st = enqueue_step(b, need_copy);
    if (st != PA_OK) return st;
    int r = 0;
    const auto published = [&] {
        for (; r < b->nruns; ++r) {
            if (!sd[r].active) continue;
            const uint32_t* at = reinterpret_cast<const uint32_t*>(b->h_download + b->lo.runs[(size_t)r].stats_off) + 3;
            if (__atomic_load_n(at, __ATOMIC_ACQUIRE) != b->seq) return false;
        }
        return true;
    };
    if (!host::spin_for(published)) BCHK(hipStreamSynchronize(b->stream));
    return PA_OK;
}

void read_stats(pa_batch* b, int r)
{
    RunHost& h = b->runs[(size_t)r];
    const RunLayout& rl = b->lo.runs[(size_t)r];
    std::memcpy(&h.h_stats, b->h_download + rl.stats_off, sizeof(DevStats));
    h.h_hist = reinterpret_cast<const uint32_t*>(b->h_download + rl.stats_off + sizeof(DevStats));
    std::memcpy(&h.feat, b->h_download + b->lo.feats + sizeof(FeatDev) * (size_t)r,
                sizeof(FeatDev));
}

void record_measurement(RunHost& h)
{
    pa_obs o;
    host::observables(h.h_stats, h.R_cur, h.p.L * h.p.L, h.beta, h.lnZ, h.lnQ_last, &o);
    h.history.push_back(o);
    if (h.p.flags & PA_FLAG_MHR) {
        h.m_beta.push_back(h.beta);
        h.m_lnZ.push_back(h.lnZ);
        h.m_R.push_back(h.R_cur);
    }
}

// Next inverse temperature of a run, or false (with the run's status set).
// Learned mode: the proposal beta + exp(prop) is accepted when the exact
// overlap is within alpha_tol of the target (or it reaches beta_f with enough
// overlap); otherwise the bisection decides.  Every interior bisection root is
// logged as a training pair (features, ln(step sigma_E)).
bool choose_beta(RunHost& h, const host::Hist& hw, bool model_set, double* beta_next)
{
    const pa_schedule& s = h.sched;
    if (s.mode == PA_STEP_FIXED) {
        const int64_t nb = std::max<int64_t>(1, std::llround(s.beta_f / s.dbeta));
        const int64_t i = (int64_t)h.step + 1;
        *beta_next = (i >= nb) ? s.beta_f : (double)i * s.dbeta;
        if (*beta_next > s.beta_f) *beta_next = s.beta_f;
        return true;
    }
    if (s.mode == PA_STEP_LEARNED && model_set && h.feat.valid) {
        // the network predicts ln(dbeta sigma_E); x[1] = ln sigma_E
        const double d = std::exp((double)h.feat.prop - (double)h.feat.x[1]);
        if (std::isfinite(d) && d > 0.0) {
            const double bp = std::min(h.beta + d, s.beta_f);
            if (bp > h.beta) {
                const double a = host::overlap(hw, h.p.R, h.R_cur, bp - h.beta, h.w);
                h.alpha_evals += 1;
                h.proposals += 1;
                if (std::fabs(a - s.alpha_star) <= s.alpha_tol || (bp == s.beta_f && a >= s.alpha_star)) {
                    h.accepted += 1;
                    *beta_next = bp;
                    return true;
                }
            }
        }
    }
    if (!host::adapt_beta(hw, h.p.R, h.R_cur, h.beta, s.beta_f, s.alpha_star, beta_next, nullptr, h.w,
                          &h.alpha_evals)) {
        h.status = PA_EINVAL;
        return false;
    }
    if (*beta_next < s.beta_f && h.feat.valid) {
        h.pair_x.insert(h.pair_x.end(), h.feat.x, h.feat.x + 8);
        h.pair_t.push_back((float)(std::log(*beta_next - h.beta) + (double)h.feat.x[1]));
    }
    return true;
}

pa_status autotune(pa_batch* b);

}  // namespace

extern "C" {

size_t pa_batch_workspace_bytes(const pa_params* runs, int32_t nruns)
{
    if (!runs || nruns < 1) return 0;
    BatchLayout bl;
    return make_batch_layout(runs, nruns, &bl) ? bl.total : 0;
}

static pa_status batch_init(const pa_params* runs, const pa_schedule* sched, int32_t nruns,
                            const pa_batch_options* opt, void* d_workspace, size_t bytes, void* hip_stream,
                            pa_batch** out);

pa_status pa_batch_init(const pa_params* runs, const pa_schedule* sched, int32_t nruns, void* d_workspace,
                        size_t bytes, void* hip_stream, pa_batch** out)
{
    return pa_batch_init_ex(runs, sched, nruns, nullptr, d_workspace, bytes, hip_stream, out);
}

pa_status pa_batch_init_ex(const pa_params* runs, const pa_schedule* sched, int32_t nruns,
                           const pa_batch_options* opt, void* d_workspace, size_t bytes, void* hip_stream,
                           pa_batch** out)
{
    if (!out) return PA_EINVAL;
    *out = nullptr;
    if (opt) {
        const int w = opt->waves_per_block;
        if (!(w == 0 || w == 1 || w == 2 || w == 4 || w == 8)) return PA_EINVAL;
    }
    pa_batch* b = nullptr;
    const pa_status st = batch_init(runs, sched, nruns, opt, d_workspace, bytes, hip_stream, &b);
    if (st != PA_OK) {
        if (b && b->stream) (void)hipStreamSynchronize(b->stream);
        pa_batch_free(b);
        return st;
    }
    *out = b;
    return PA_OK;
}

static pa_status batch_init(const pa_params* runs, const pa_schedule* sched, int32_t nruns,
                            const pa_batch_options* opt, void* d_workspace, size_t bytes, void* hip_stream,
                            pa_batch** out)
{
    if (!runs || !sched || nruns < 1 || !d_workspace || ((uintptr_t)d_workspace) % kAlign) return PA_EINVAL;
    for (int r = 0; r < nruns; ++r) {
        if (sched[r].mode == PA_STEP_FOLLOW) {
            const int l = sched[r].leader;
            if (l < 0 || l >= nruns || l == r || sched[l].mode == PA_STEP_FOLLOW || sched[r].theta < 0) return PA_EINVAL;
        } else if (!valid_schedule(sched[r])) {
            return PA_EINVAL;
        }
    }
    BatchLayout bl;
    if (!make_batch_layout(runs, nruns, &bl)) return PA_EINVAL;
    if (bytes < bl.total) return PA_ENOMEM;
    pa_batch* b = new (std::nothrow) pa_batch();
    if (!b) return PA_ENOMEM;
    b->nruns = nruns;
    b->lo = bl;
    b->ws = (uint8_t*)d_workspace;
    if (opt) b->opt = *opt;
    *out = b;
    if (hip_stream) {
        b->stream = (hipStream_t)hip_stream;
    } else {
        BCHK(hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking));
        b->own_stream = true;
    }
    uint8_t* ws = b->ws;
    b->d_rundev = reinterpret_cast<RunDev*>(ws + bl.rundev);
    b->d_steps = reinterpret_cast<StepDev*>(ws + bl.steps);
    b->d_tables = reinterpret_cast<uint32_t*>(ws + bl.tables);
    b->d_download = ws + bl.download;
    b->d_results = reinterpret_cast<ResultDev*>(ws + bl.results);
    b->d_model = reinterpret_cast<ModelDev*>(ws + bl.model);
    b->d_items = reinterpret_cast<Item*>(ws + bl.items);
    b->runs.resize((size_t)nruns);
    b->rundev.resize((size_t)nruns);
    for (int r = 0; r < nruns; ++r) {
        const RunLayout& rl = bl.runs[(size_t)r];
        RunHost& h = b->runs[(size_t)r];
        h.p = runs[r];
        h.p.capacity = rl.capacity;
        h.sched = sched[r];
        if (h.sched.mode == PA_STEP_FOLLOW) h.sched.beta_f = sched[h.sched.leader].beta_f;
        RunDev& d = b->rundev[(size_t)r];
        std::memset(&d, 0, sizeof(d));
        for (int k = 0; k < 2; ++k) {
            d.spin[k] = ws + rl.spin[k];
            d.E[k] = reinterpret_cast<int32_t*>(ws + rl.E[k]);
            d.M[k] = reinterpret_cast<int32_t*>(ws + rl.M[k]);
        }
        d.counts = reinterpret_cast<uint32_t*>(ws + rl.counts);
        d.parent = reinterpret_cast<uint32_t*>(ws + rl.parent);
        d.bsum = reinterpret_cast<uint32_t*>(ws + rl.bsum);
        d.stats = reinterpret_cast<DevStats*>(b->d_download + rl.stats_off);
        d.hist = reinterpret_cast<uint32_t*>(b->d_download + rl.stats_off + sizeof(DevStats));
        d.parts = reinterpret_cast<pa::StatsPart*>(ws + rl.parts);
        if (h.p.flags & PA_FLAG_MHR) {
            uint64_t* m = reinterpret_cast<uint64_t*>(ws + rl.mhr);
            d.mhr = DevMhr{m, m + rl.nbins, m + 2 * (size_t)rl.nbins, m + 3 * (size_t)rl.nbins};
        }
        d.L = h.p.L;
        d.N = h.p.L * h.p.L;
        d.nbins = rl.nbins;
        d.capacity = rl.capacity;
        d.layout = h.p.layout;
        d.R = h.p.R;
        d.rep_bytes = (uint32_t)rl.rep_bytes;
        d.key0 = (uint32_t)h.p.seed;
        d.key1 = (uint32_t)(h.p.seed >> 32);
        d.tag = h.p.run_id << 4;
        d.qcap = 0xFFFFFFFFu;
        d.host_off = rl.stats_off;
    }
    if (hipHostMalloc((void**)&b->h_steps, bl.steps_bytes, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&b->h_download, bl.download_bytes, hipHostMallocMapped) != hipSuccess)
        return PA_ENOMEM;
    BCHK(hipHostGetDevicePointer(&b->h_download_dev, b->h_download, 0));
    std::memset(b->h_steps, 0, bl.steps_bytes);
    std::memset(b->h_download, 0, bl.download_bytes);
    {
        ModelDev md;
        std::memset(&md, 0, sizeof(md));
        BCHK(hipMemcpyAsync(b->d_model, &md, sizeof(md), hipMemcpyHostToDevice, b->stream));
        BCHK(hipStreamSynchronize(b->stream));
    }
    BCHK(hipMemcpyAsync(b->d_rundev, b->rundev.data(), sizeof(RunDev) * (size_t)nruns, hipMemcpyHostToDevice,
                        b->stream));
    for (int r = 0; r < nruns; ++r) {
        const RunDev& d = b->rundev[(size_t)r];
        if (d.mhr.H) {
            hipLaunchKernelGGL(b_fill_u32, dim3(256), dim3(kBlock), 0, b->stream, (uint32_t*)d.mhr.H, 0u,
                               (size_t)d.nbins * 10);
            BCHK(hipGetLastError());
        }
    }
    // static item tables: parents/statistics and copy chunks
    std::vector<Item> items;
    b->parent_off = 0;
    for (int r = 0; r < nruns; ++r)
        for (int k = 0; k < bl.runs[(size_t)r].nblk; ++k) items.push_back(Item{r, k});
    b->n_parent_items = items.size();
    b->copy_off = items.size();
    for (int r = 0; r < nruns; ++r) {
        const RunLayout& rl = bl.runs[(size_t)r];
        const size_t n = ((size_t)rl.capacity * (rl.rep_bytes / 16) + kBlock - 1) / kBlock;
        for (size_t k = 0; k < n; ++k) items.push_back(Item{r, (int32_t)k});
    }
    b->n_copy_items = items.size() - b->copy_off;
    // sweep groups, one per (lattice sizes of one launch, store, update)
    std::map<std::tuple<int, int, int>, int> seen;
    for (int r = 0; r < nruns; ++r) {
        const auto key = std::make_tuple(group_size(runs[r].L), runs[r].layout, update_of(runs[r]));
        if (!seen.count(key)) {
            seen[key] = (int)b->groups.size();
            b->groups.push_back(Group{group_size(runs[r].L), runs[r].layout, update_of(runs[r]), 1, 0, 0});
        }
    }
    b->pool = new (std::nothrow) Pool((int)std::min<unsigned>(16u, std::max(1u, std::thread::hardware_concurrency())));
    if (!b->pool) return PA_ENOMEM;
    // launch shapes, then the sweep items of the chosen shapes
    const size_t fixed_items = items.size();
    for (Group& g : b->groups) {
        g.item_off = items.size();
        const std::vector<Item> it = sweep_items(b, g, 1);
        items.insert(items.end(), it.begin(), it.end());
        g.n_items = it.size();
    }
    if (items.size() > bl.n_items) return PA_ENOMEM;
    BCHK(hipMemcpyAsync(b->d_items, items.data(), items.size() * sizeof(Item), hipMemcpyHostToDevice, b->stream));
    BCHK(hipStreamSynchronize(b->stream));
    pa_status st = autotune(b);
    if (st != PA_OK) return st;
    items.resize(fixed_items);
    for (Group& g : b->groups) {
        g.item_off = items.size();
        const std::vector<Item> it = sweep_items(b, g, g.wpb);
        items.insert(items.end(), it.begin(), it.end());
        g.n_items = it.size();
    }
    BCHK(hipMemcpyAsync(b->d_items, items.data(), items.size() * sizeof(Item), hipMemcpyHostToDevice, b->stream));
    for (int r = 0; r < nruns; ++r) b->any_scanned = b->any_scanned || scanned_run(bl.runs[(size_t)r].capacity);
    // initial state (Sec. 2.1 step 1) and the measurement at beta_0 = 0
    StepDev* sd = host_steps(b);
    for (int r = 0; r < nruns; ++r) {
        RunHost& h = b->runs[(size_t)r];
        StepDev& d = sd[r];
        std::memset(&d, 0, sizeof(d));
        d.active = 1;
        d.init = 1;
        d.record = (h.p.flags & PA_FLAG_MHR) ? 1 : 0;
        d.n_parent = h.p.R;
        host::sweep_thresholds(heatbath(h.p), 0.0, &d.t2h, &d.t2l, &d.t4h, &d.t4l);
        h.R_cur = h.p.R;
        h.lnZ = (double)(h.p.L * h.p.L) * std::log(2.0);
    }
    st = run_step(b, b->lo.tables - b->lo.steps, false);  // initial states: no resampling
    if (st != PA_OK) return st;
    for (int r = 0; r < nruns; ++r) {
        read_stats(b, r);
        record_measurement(b->runs[(size_t)r]);
    }
    return PA_OK;
}

pa_status pa_batch_step(pa_batch* b, int32_t* n_active)
{
    if (!b) return PA_EINVAL;
    if (b->broken) return PA_ESTATE;
    StepDev* sd = host_steps(b);
    uint32_t* tb = host_tables(b);
    // place of every run's tables: its occupied energy window, known before its
    // temperature
    std::vector<uint32_t> toff((size_t)b->nruns, 0u);
    uint32_t o = 0;
    for (int r = 0; r < b->nruns; ++r) {
        RunHost& h = b->runs[(size_t)r];
        h.stepping = false;
        if (h.finished || h.status != PA_OK) continue;
        toff[(size_t)r] = o;
        const int bmin = (h.h_stats.emin + 2 * h.p.L * h.p.L) / 4, bmax = (h.h_stats.emax + 2 * h.p.L * h.p.L) / 4;
        o += 2u * (uint32_t)(bmax - bmin + 1);
    }
    // tables of Eq. (resampling factors) and the step descriptor of a run
    const auto fill_step = [&](int r) {
        RunHost& h = b->runs[(size_t)r];
        StepDev& d = sd[r];
        std::memset(&d, 0, sizeof(d));
        if (!h.stepping) return;
        const host::Hist hw = host::hist_window(h.h_hist, h.h_stats, h.p.L * h.p.L);
        const double bn = h.beta_next;
        h.lnQ_next = host::resample_tables(hw, h.p.R, h.R_cur, bn - h.beta, tb + toff[(size_t)r], h.w);
        d.active = 1;
        d.resample = 1;
        d.record = (h.p.flags & PA_FLAG_MHR) ? 1 : 0;
        d.cur = h.cur;
        d.n_parent = (int32_t)h.R_cur;
        d.step = (uint32_t)(h.step + 1);
        d.g0 = (uint32_t)h.sweeps;
        d.nsweeps = h.sched.theta;
        host::sweep_thresholds(heatbath(h.p), bn, &d.t2h, &d.t2l, &d.t4h, &d.t4l);
        d.bmin = hw.bmin;
        d.nwin = hw.bmax - hw.bmin + 1;
        d.tbl_off = toff[(size_t)r];
        d.beta = bn;
        d.last_dbeta = bn - h.beta;
    };
    // per run: next beta, then its tables.  One pass of the thread pool, whose
    // wake-up and join cost about 40 us each: the temperatures, the tables and
    // the commit in passes of their own took 147 us per step of 12 runs.
    b->pool->parallel_for(b->nruns, [&](int r) {
        RunHost& h = b->runs[(size_t)r];
        if (h.sched.mode == PA_STEP_FOLLOW) return;
        if (!h.finished && h.status == PA_OK) {
            const host::Hist hw = host::hist_window(h.h_hist, h.h_stats, h.p.L * h.p.L);
            double bn = 0.0;
            const auto t0 = std::chrono::steady_clock::now();
            const bool ok = choose_beta(h, hw, b->model_set, &bn);
            h.choose_s += std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
            if (ok) {
                h.beta_next = bn;
                h.stepping = true;
            }
        }
        fill_step(r);
    });
    // followers take their leader's temperature of this step
    int any = 0, followers = 0;
    for (int r = 0; r < b->nruns; ++r) {
        RunHost& h = b->runs[(size_t)r];
        if (h.sched.mode == PA_STEP_FOLLOW) {
            ++followers;
            if (!h.finished && h.status == PA_OK) {
                const RunHost& l = b->runs[(size_t)h.sched.leader];
                if (l.stepping && l.step == h.step) {
                    h.beta_next = l.beta_next;
                    h.stepping = true;
                } else if (l.status != PA_OK || l.step != h.step) {
                    h.status = PA_ESTATE;  // the leader has stopped (or fell behind on an error)
                }
            }
        }
        any += h.stepping ? 1 : 0;
    }
    if (followers)
        b->pool->parallel_for(b->nruns, [&](int r) {
            if (b->runs[(size_t)r].sched.mode == PA_STEP_FOLLOW) fill_step(r);
        });
    if (any) {
        bool need_copy = false;
        for (int r = 0; r < b->nruns; ++r)
            need_copy = need_copy || (sd[r].active && sd[r].resample && sd[r].nsweeps == 0);
        const pa_status st = run_step(b, (b->lo.tables - b->lo.steps) + (size_t)o * 4, need_copy);
        if (st != PA_OK) return st;
        const ResultDev* res = reinterpret_cast<const ResultDev*>(b->h_download);
        for (int r = 0; r < b->nruns; ++r) {
            RunHost& h = b->runs[(size_t)r];
            if (!h.stepping) continue;
            h.stepping = false;
            if (res[r].err) {
                h.status = (res[r].err == 1) ? PA_ECAPACITY : PA_EEXTINCT;
                read_stats(b, r);  // statistics of the unchanged population
                continue;
            }
            h.cur ^= 1;
            h.R_cur = res[r].r_new;
            h.step += 1;
            h.sweeps += (uint64_t)h.sched.theta;
            h.last_dbeta = h.beta_next - h.beta;
            h.beta = h.beta_next;
            h.lnZ += h.lnQ_next;
            h.lnQ_last = h.lnQ_next;
            read_stats(b, r);
            record_measurement(h);
            if (h.beta >= h.sched.beta_f) h.finished = true;
        }
    }
    if (n_active) {
        int n = 0;
        for (const RunHost& h : b->runs) n += (!h.finished && h.status == PA_OK) ? 1 : 0;
        *n_active = n;
    }
    return PA_OK;
}

pa_status pa_batch_run(pa_batch* b)
{
    if (!b) return PA_EINVAL;
    int32_t n = 1;
    while (n > 0) {
        const pa_status st = pa_batch_step(b, &n);
        if (st != PA_OK) return st;
    }
    BCHK(hipStreamSynchronize(b->stream));
    return PA_OK;
}

pa_status pa_batch_run_status(const pa_batch* b, int32_t run)
{
    if (!b || run < 0 || run >= b->nruns) return PA_EINVAL;
    return b->runs[(size_t)run].status;
}

pa_status pa_batch_state(const pa_batch* b, int32_t run, pa_state_info* out)
{
    if (!b || !out || run < 0 || run >= b->nruns) return PA_EINVAL;
    const RunHost& h = b->runs[(size_t)run];
    out->R = h.R_cur;
    out->step = h.step;
    out->sweeps = h.sweeps;
    out->beta = h.beta;
    out->lnZ = h.lnZ;
    return PA_OK;
}

pa_status pa_batch_history(const pa_batch* b, int32_t run, pa_obs* out, int32_t cap, int32_t* n)
{
    if (!b || !n || run < 0 || run >= b->nruns || cap < 0 || (cap > 0 && !out)) return PA_EINVAL;
    const RunHost& h = b->runs[(size_t)run];
    *n = (int32_t)h.history.size();
    const size_t k = std::min<size_t>((size_t)cap, h.history.size());
    if (k) std::memcpy(out, h.history.data(), k * sizeof(pa_obs));
    return PA_OK;
}

pa_status pa_batch_reweight(pa_batch* b, int32_t run, const double* betas, int32_t nb, pa_obs* out)
{
    if (!b || run < 0 || run >= b->nruns || nb < 0 || (nb > 0 && (!betas || !out))) return PA_EINVAL;
    if (b->broken) return PA_ESTATE;
    const RunHost& h = b->runs[(size_t)run];
    const RunDev& d = b->rundev[(size_t)run];
    if (!(h.p.flags & PA_FLAG_MHR) || h.m_beta.empty()) return PA_EINVAL;
    const size_t nbins = (size_t)d.nbins;
    std::vector<uint64_t> acc(5 * nbins);
    BCHK(hipMemcpyAsync(acc.data(), d.mhr.H, acc.size() * 8, hipMemcpyDeviceToHost, b->stream));
    BCHK(hipStreamSynchronize(b->stream));
    const uint64_t* H = acc.data();
    host::reweight(d.N, H, H + nbins, H + 2 * nbins, H + 3 * nbins, h.m_beta, h.m_lnZ, h.m_R, betas, nb, out);
    return PA_OK;
}

pa_status pa_batch_download_population(pa_batch* b, int32_t run, int8_t* spins, int32_t* E, int32_t* M)
{
    if (!b || run < 0 || run >= b->nruns) return PA_EINVAL;
    if (b->broken) return PA_ESTATE;
    const RunHost& h = b->runs[(size_t)run];
    const RunDev& d = b->rundev[(size_t)run];
    const size_t n = (size_t)h.R_cur;
    if (E) BCHK(hipMemcpyAsync(E, d.E[h.cur], n * 4, hipMemcpyDeviceToHost, b->stream));
    if (M) BCHK(hipMemcpyAsync(M, d.M[h.cur], n * 4, hipMemcpyDeviceToHost, b->stream));
    if (spins) {
        if (h.p.layout == PA_SPIN_INT8) {
            BCHK(hipMemcpyAsync(spins, d.spin[h.cur], n * (size_t)d.N, hipMemcpyDeviceToHost, b->stream));
        } else {
            std::vector<uint32_t> words(n * (size_t)d.N / 32);
            BCHK(hipMemcpyAsync(words.data(), d.spin[h.cur], words.size() * 4, hipMemcpyDeviceToHost, b->stream));
            BCHK(hipStreamSynchronize(b->stream));
            host::bits_to_int8(words.data(), d.L, n, spins);
        }
    }
    BCHK(hipStreamSynchronize(b->stream));
    return PA_OK;
}

pa_status pa_batch_set_model(pa_batch* b, const float* params, const float* norm)
{
    if (!b || !params || !norm) return PA_EINVAL;
    if (b->broken) return PA_ESTATE;
    ModelDev md;
    std::memset(&md, 0, sizeof(md));
    md.set = 1;
    for (int k = 0; k < pa::mlp::kNorm; ++k) md.norm[k] = norm[k];
    for (int q = 0; q < pa::mlp::kParams; ++q) md.wb[q] = __float2bfloat16(params[q]);
    BCHK(hipMemcpyAsync(b->d_model, &md, sizeof(md), hipMemcpyHostToDevice, b->stream));
    BCHK(hipStreamSynchronize(b->stream));
    b->model_set = true;
    return PA_OK;
}

pa_status pa_batch_training_pairs(const pa_batch* b, float* x, float* t, int32_t cap, int32_t* n)
{
    if (!b || !n || cap < 0 || (cap > 0 && (!x || !t))) return PA_EINVAL;
    int32_t k = 0;
    for (const RunHost& h : b->runs) {
        for (size_t i = 0; i < h.pair_t.size(); ++i) {
            if (k < cap) {
                std::memcpy(x + (size_t)k * 8, h.pair_x.data() + i * 8, 8 * sizeof(float));
                t[k] = h.pair_t[i];
            }
            ++k;
        }
    }
    *n = k;
    return PA_OK;
}

pa_status pa_batch_features(const pa_batch* b, int32_t run, float* x, int32_t* valid, float* prop)
{
    if (!b || run < 0 || run >= b->nruns || !x || !valid || !prop) return PA_EINVAL;
    const FeatDev& f = b->runs[(size_t)run].feat;
    std::memcpy(x, f.x, sizeof(f.x));
    *valid = f.valid;
    *prop = f.prop;
    return PA_OK;
}

pa_status pa_batch_set_tie_queue_cap(pa_batch* b, int32_t cap)
{
    if (!b || cap < 0) return PA_EINVAL;
    if (b->broken) return PA_ESTATE;
    for (RunDev& d : b->rundev) d.qcap = (uint32_t)cap;
    BCHK(hipMemcpyAsync(b->d_rundev, b->rundev.data(), sizeof(RunDev) * b->rundev.size(), hipMemcpyHostToDevice,
                        b->stream));
    BCHK(hipStreamSynchronize(b->stream));
    return PA_OK;
}

pa_status pa_batch_waves_per_block(const pa_batch* b, int32_t run, int32_t* wpb)
{
    if (!b || !wpb || run < 0 || run >= b->nruns) return PA_EINVAL;
    const pa_params& p = b->runs[(size_t)run].p;
    for (const Group& g : b->groups)
        if (in_group(p, g)) {
            *wpb = g.wpb;
            return PA_OK;
        }
    return PA_EINVAL;
}

pa_status pa_batch_choice_stats(const pa_batch* b, int32_t run, int64_t* alpha_evals, double* host_seconds)
{
    if (!b || run < 0 || run >= b->nruns || !alpha_evals || !host_seconds) return PA_EINVAL;
    *alpha_evals = b->runs[(size_t)run].alpha_evals;
    *host_seconds = b->runs[(size_t)run].choose_s;
    return PA_OK;
}

pa_status pa_batch_learned_stats(const pa_batch* b, int32_t run, int32_t* proposals, int32_t* accepted)
{
    if (!b || run < 0 || run >= b->nruns || !proposals || !accepted) return PA_EINVAL;
    *proposals = b->runs[(size_t)run].proposals;
    *accepted = b->runs[(size_t)run].accepted;
    return PA_OK;
}

pa_status pa_batch_free(pa_batch* b)
{
    if (!b) return PA_OK;
    if (b->h_steps) (void)hipHostFree(b->h_steps);
    if (b->h_download) (void)hipHostFree(b->h_download);
    if (b->own_stream && b->stream) (void)hipStreamDestroy(b->stream);
    delete b->pool;
    delete b;
    return PA_OK;
}

}  // extern "C"

namespace {

// Picks waves per block for every sweep group by timing the sweep on the
// spare half of each run's ping-pong store: the spare buffers are overwritten
// by the first resampling, so tuning leaves no trace in the runs.  The timed
// launches draw a fresh state and do a few sweeps at beta = 0.44.
// Waves per block chosen by autotune, kept for the life of the process per
// (device architecture, store, update, lattice sizes with their waves): later
// batches of the same shape skip the timed search.
struct TuneKey {
    std::string arch;
    int layout, upd;
    host::LaunchMix mix;
    bool operator<(const TuneKey& o) const
    {
        return std::tie(arch, layout, upd, mix) < std::tie(o.arch, o.layout, o.upd, o.mix);
    }
};
std::mutex g_tune_mu;
std::map<TuneKey, int> g_tune_cache;

pa_status autotune(pa_batch* b)
{
    const int cands[] = {1, 2, 4, 8};
    StepDev* sd = host_steps(b);
    int dev = 0;
    BCHK(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    BCHK(hipGetDeviceProperties(&prop, dev));
    const std::string arch = prop.gcnArchName;
    hipEvent_t e0, e1;
    BCHK(hipEventCreate(&e0));
    BCHK(hipEventCreate(&e1));
    std::vector<Item> it;
    for (Group& g : b->groups) {
        if (b->opt.waves_per_block > 0) {
            // a forced shape; where its LDS does not fit, the largest smaller one that does
            int w = b->opt.waves_per_block;
            while (w > 1 && sweep_lds_bytes(g.L, w) > 65536) w >>= 1;
            g.wpb = w;
            continue;
        }
        host::LaunchMix mix;
        for (int r = 0; r < b->nruns; ++r) {
            const RunHost& h = b->runs[(size_t)r];
            if (in_group(h.p, g)) mix.add(h.p.L, (h.p.R + reps_per_wave(h.p.L) - 1) / reps_per_wave(h.p.L));
        }
        const TuneKey key{arch, g.layout, g.upd, mix.rounded()};
        {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            const auto f = g_tune_cache.find(key);
            if (f != g_tune_cache.end()) {
                g.wpb = f->second;
                continue;
            }
        }
        for (int r = 0; r < b->nruns; ++r) {
            StepDev& d = sd[r];
            std::memset(&d, 0, sizeof(d));
            const RunHost& h = b->runs[(size_t)r];
            if (!in_group(h.p, g)) continue;
            d.active = 1;
            d.init = 1;
            d.cur = 1;  // spare buffer
            d.n_parent = h.p.R;
            d.nsweeps = 4;
            d.g0 = 0x40000000u;
            host::sweep_thresholds(g.upd == pa::kHeatbath, 0.44, &d.t2h, &d.t2l, &d.t4h, &d.t4l);
        }
        BCHK(hipMemcpyAsync(b->d_steps, b->h_steps, b->lo.steps_bytes, hipMemcpyHostToDevice, b->stream));
        float best = 1e30f;
        int best_w = 1;
        for (int wpb : cands) {
            if (sweep_lds_bytes(g.L, wpb) > 65536) continue;  // at most 64 KB of LDS per block
            it = sweep_items(b, g, wpb);
            const size_t off = g.item_off;  // scratch slot: the group's own item range is large enough
            BCHK(hipMemcpyAsync(b->d_items + off, it.data(), it.size() * sizeof(Item), hipMemcpyHostToDevice,
                                b->stream));
            float t = 0.0f;
            for (int rep = 0; rep < 3; ++rep) {
                BCHK(hipEventRecord(e0, b->stream));
                BCHK(launch_group(g, b->d_items + off, it.size(), wpb, b->d_rundev, b->d_steps,
                                  b->d_results, b->stream));
                BCHK(hipEventRecord(e1, b->stream));
                BCHK(hipEventSynchronize(e1));
                float ms = 0.0f;
                BCHK(hipEventElapsedTime(&ms, e0, e1));
                if (rep > 0) t += ms;  // the first launch warms up
            }
            if (t < best) {
                best = t;
                best_w = wpb;
            }
        }
        g.wpb = best_w;
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune_cache[key] = best_w;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    std::memset(sd, 0, sizeof(StepDev) * (size_t)b->nruns);
    return PA_OK;
}

}  // namespace
