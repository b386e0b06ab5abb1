// Checkerboard Metropolis sweep kernel of the single-run path for gfx950
// (CDNA4): sweeps (Sec. 3 spin updates), the initial state (Sec. 2.1 step 1)
// and the recount of E and M.
//
// Spin representation inside the sweep: each colour of a replica is a set of
// 32-site words (canonical within-colour index q = (y L + x) >> 1, bit q & 31
// of word q >> 5; bit set = spin -1).  A wave owns whole replicas and keeps
// them on chip for all requested sweeps: in VGPRs for L <= 64 (vertical
// neighbours cross lanes by shuffle, horizontal ones are funnel shifts), in
// LDS for L >= 128.  The Metropolis decision for all 32 sites of a word is
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

template <int L, bool INT8, int U>
__global__ __launch_bounds__(sweep_block<L>())
__attribute__((amdgpu_waves_per_eu(sweep_min_waves<L>(), 8))) void sweep_kernel(SweepArgs a)
{
    using Gm = Geo<L>;
    constexpr int WPB = sweep_block<L>() / 64;
    __shared__ __align__(16) uint32_t lds[Gm::lds_words(WPB) > 0 ? Gm::lds_words(WPB) : 1];
    if (a.n_dev) a.n_rep = min(a.n_rep, (int32_t)*a.n_dev);
    sweep_waves<L, INT8, U == kHeatbath, U == kLcg>(a, (int)blockIdx.x * WPB, lds);
}

template <int L, bool INT8, int U>
__global__ __launch_bounds__(64) void sweep_quads_kernel(SweepArgs a)
{
    if (a.n_dev) a.n_rep = min(a.n_rep, (int32_t)*a.n_dev);
    if ((int)blockIdx.x * quad_replicas<L>() >= a.n_rep) return;
    sweep_quads<L, INT8, U == kHeatbath>(a, (int)blockIdx.x);
}

// Waves of sweep_quads up to which it is taken, four per SIMD (without the
// statistics in the epilogue, which it has none of).  Launches in ms, ordinary
// path and this one: L = 16, theta = 50: R = 1000 0.088, 0.029; 8000 0.090,
// 0.044; 16000 (4000 waves) 0.093, 0.078; 30000 0.103, 0.138.  L = 32, theta =
// 20: R = 100 0.038, 0.014; 2000 0.040, 0.025; 4000 0.041, 0.033; 8000 0.046,
// 0.057.
constexpr int kQuadWaves = 4096;

template <int L, bool INT8, int U>
hipError_t launch_sweep_t(SweepArgs a, hipStream_t s)
{
    using Gm = Geo<L>;
    if constexpr (L <= 32 && U != kLcg) {
        const int waves = (a.n_rep + quad_replicas<L>() - 1) / quad_replicas<L>();
        if (waves > 0 && waves <= kQuadWaves && !a.acc && !a.init && a.nsweeps > 0) {
            hipLaunchKernelGGL((sweep_quads_kernel<L, INT8, U>), dim3(waves), dim3(64), 0, s, a);
            return hipGetLastError();
        }
    }
    const int reps_per_block = (sweep_block<L>() / 64) * Gm::RPWV;
    const int blocks = (a.n_rep + reps_per_block - 1) / reps_per_block;
    if (blocks == 0) return hipSuccess;
    a.one_round = blocks * (sweep_block<L>() / 64) <= sweep_resident_waves<L>() ? 1 : 0;
    hipLaunchKernelGGL((sweep_kernel<L, INT8, U>), dim3(blocks), dim3(sweep_block<L>()), 0, s, a);
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
