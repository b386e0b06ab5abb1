// Checkerboard Metropolis sweep kernel of the single-run path for gfx950
// (CDNA4): sweeps (Sec. 3 spin updates), the initial state (Sec. 2.1 step 1)
// and the recount of E and M.
//
// Spin representation inside the sweep: each colour of a replica is a set of
// 32-site words (canonical within-colour index q = (y L + x) >> 1, bit q & 31
// of word q >> 5; bit set = spin -1).  A wave owns whole replicas and keeps
// them on chip for all requested sweeps: in VGPRs for L <= 64 (vertical
// neighbours cross lanes by shuffle, horizontal ones are funnel shifts), in
// LDS for L >= 128; in small launches four lanes share a word (L <= 64) or four
// waves a replica (L >= 64).
// The Metropolis decision for all 32 sites of a word is
// bit-sliced: the uniform of each site is compared to the integer threshold
// one bit plane at a time (16 planes from four Philox blocks, high bit first).
// For L <= 64 the planes stop as soon as no site of the wave is undecided; for
// L >= 128 a lane decides 8 planes for several words and queues the sites
// still tied, which the wave then decides one per lane (pa_device.h).  A run
// created with PA_FLAG_HEATBATH uses the heat-bath update in the same scheme,
// one created with PA_FLAG_LCG the in-line LCG variant of the multi-spin-coded
// sweep (Sec. 4), each with its own kernel instantiations.
#include "pa_device.h"
#include "pa_launch.h"

namespace pa {
namespace {

using namespace pa::dev;

template <int L, bool INT8, int U, bool PRIO>
__global__ __launch_bounds__(sweep_block<L>())
__attribute__((amdgpu_waves_per_eu(sweep_min_waves<L>(), 8))) void sweep_kernel(SweepArgs a)
{
    using Gm = Geo<L>;
    constexpr int WPB = sweep_block<L>() / 64;
    __shared__ __align__(16) uint32_t lds[Gm::lds_words(WPB) > 0 ? Gm::lds_words(WPB) : 1];
    if (a.n_dev) a.n_rep = min(a.n_rep, (int32_t)*a.n_dev);
    sweep_waves<L, INT8, U == kHeatbath, U == kLcg, PRIO>(a, (int)blockIdx.x * WPB, lds);
}

template <int L, bool INT8, int U>
__global__ __launch_bounds__(64) void sweep_quads_kernel(SweepArgs a)
{
    if (a.n_dev) a.n_rep = min(a.n_rep, (int32_t)*a.n_dev);
    if ((int)blockIdx.x * quad_replicas<L>() >= a.n_rep) return;
    sweep_quads<L, INT8, U == kHeatbath>(a, (int)blockIdx.x);
}

// One replica per block of four waves: L = 64 by sweep_quads64, L >= 128 by the
// LDS path with the replica shared.  Few replicas leave most SIMDs empty and the
// others with one wave, whose time is its number of instructions; four waves
// each have a quarter of them, for a barrier per half sweep.
constexpr int kReplicaWaves = 4;

template <int L, bool INT8, int U>
__global__ __launch_bounds__(64 * kReplicaWaves) void sweep_shared_kernel(SweepArgs a)
{
    constexpr int W = kReplicaWaves;
    constexpr bool HB = U == kHeatbath;
    __shared__ __align__(16) uint32_t lds[L == 64 ? 128 + 2 * W : 2 * Geo<L>::NW + W * kTieQueueWords];
    if (a.n_dev) a.n_rep = min(a.n_rep, (int32_t)*a.n_dev);
    if ((int)blockIdx.x >= a.n_rep) return;
    if constexpr (L == 64) {
        sweep_quads64<INT8, HB>(a, blockIdx.x, lds);
    } else {
        const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        sweep_lds<L, INT8, HB, false, true, W>(a, blockIdx.x, lds, wv);
    }
}

// Replicas up to which a launch takes it, five to eight waves per SIMD.  Launches
// of 20 sweeps in us, one wave per replica and four:
//   L = 64:  R = 300 46, 27; 1000 47, 39; 1500 49, 49; 2500 54, 69
//   L = 128: R = 300 93, 62; 1000 94, 71; 1500 108, 82; 2500 126, 137
//   L = 256: R = 300 303, 121; 1000 311, 225; 1500 376, 266; 2500 456, 464
template <int L>
constexpr int shared_replicas()
{
    return L == 64 ? 1280 : 2048;
}

// Waves of sweep_quads up to which it is taken, four per SIMD (without the
// statistics in the epilogue, which it has none of).  Launches in ms, ordinary
// path and this one: L = 16, theta = 50: R = 1000 0.088, 0.029; 8000 0.090,
// 0.044; 16000 (4000 waves) 0.093, 0.078; 30000 0.103, 0.138.  L = 32, theta =
// 20: R = 100 0.038, 0.014; 2000 0.040, 0.025; 4000 0.041, 0.033; 8000 0.046,
// 0.057.
constexpr int kQuadWaves = 4096;

// Launches of the LCG update without wave priorities and with its comparisons in
// pairs (shift_in_pair): up to one wave per SIMD, which priorities cannot help,
// and, in the bit store of L = 16, launches whose last round would be a thin one
// (up to a quarter), since waves kept together leave all of it to the end.
// Launches of 20 sweeps in us, with priorities and without.  One wave per SIMD:
// L = 16, R = 300 24.6, 23.9, int8 24.8, 21.8; L = 64, R = 300 31.1, 30.4; L = 128,
// R = 300 124, 104; two: L = 64, R = 1400 40.2, 42.9.  A thin last round: L = 16,
// R = 145000 146, 138, R = 160000 160, 153, in the int8 store 151, 164; but L = 32,
// R = 36000 134, 141, and L = 64, R = 9000 135, 140.  A long queue: L = 16,
// R = 200000 188, 196; L = 64, R = 26000 382, 379.
template <int L, bool INT8>
bool lcg_without_priorities(int waves)
{
    constexpr int ALL = sweep_resident_waves<L>();
    return waves <= 1024 || (L == 16 && !INT8 && waves > ALL && waves <= ALL / 4 * 5);
}

template <int L, bool INT8, int U>
hipError_t launch_sweep_t(SweepArgs a, hipStream_t s)
{
    using Gm = Geo<L>;
    a.one_round = 1;
    if constexpr (L <= 32 && U != kLcg) {
        const int waves = (a.n_rep + quad_replicas<L>() - 1) / quad_replicas<L>();
        if (waves > 0 && waves <= kQuadWaves && !a.acc && !a.init && a.nsweeps > 0) {
            hipLaunchKernelGGL((sweep_quads_kernel<L, INT8, U>), dim3(waves), dim3(64), 0, s, a);
            return hipGetLastError();
        }
    }
    if constexpr (L >= 64 && U != kLcg) {
        if (a.n_rep > 0 && a.n_rep <= shared_replicas<L>() && !a.init && a.nsweeps > 0) {
            hipLaunchKernelGGL((sweep_shared_kernel<L, INT8, U>), dim3(a.n_rep), dim3(64 * kReplicaWaves), 0, s, a);
            return hipGetLastError();
        }
    }
    const int reps_per_block = (sweep_block<L>() / 64) * Gm::RPWV;
    const int blocks = (a.n_rep + reps_per_block - 1) / reps_per_block;
    if (blocks == 0) return hipSuccess;
    const int waves = blocks * (sweep_block<L>() / 64);
    a.one_round = waves <= sweep_resident_waves<L>() ? 1 : 0;
    if constexpr (U == kLcg) {
        if (lcg_without_priorities<L, INT8>(waves)) {
            hipLaunchKernelGGL((sweep_kernel<L, INT8, U, false>), dim3(blocks), dim3(sweep_block<L>()), 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((sweep_kernel<L, INT8, U, true>), dim3(blocks), dim3(sweep_block<L>()), 0, s, a);
    return hipGetLastError();
}

template <int L, bool INT8>
hipError_t launch_sweep_u(int update, const SweepArgs& a, hipStream_t s)
{
    switch (update) {
    case kMetropolis: return launch_sweep_t<L, INT8, kMetropolis>(a, s);
    case kHeatbath: return launch_sweep_t<L, INT8, kHeatbath>(a, s);
    case kLcg: return launch_sweep_t<L, INT8, kLcg>(a, s);
    default: return hipErrorInvalidValue;
    }
}

template <int L>
hipError_t launch_sweep_l(bool i8, int update, const SweepArgs& a, hipStream_t s)
{
    return i8 ? launch_sweep_u<L, true>(update, a, s) : launch_sweep_u<L, false>(update, a, s);
}

}  // namespace

hipError_t launch_sweep(int L, int layout, int update, const SweepArgs& a, hipStream_t s)
{
    const bool i8 = layout == 0;
    switch (L) {
    case 16: return launch_sweep_l<16>(i8, update, a, s);
    case 32: return launch_sweep_l<32>(i8, update, a, s);
    case 64: return launch_sweep_l<64>(i8, update, a, s);
    case 128: return launch_sweep_l<128>(i8, update, a, s);
    case 256: return launch_sweep_l<256>(i8, update, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace pa
