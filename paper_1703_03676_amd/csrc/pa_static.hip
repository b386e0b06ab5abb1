// Population statistics for callers that cannot allocate memory: the
// observables of Eq. (observables), (free energy) and (entropy) of a population
// held in caller buffers, with the partial sums and the statistics block in a
// statically allocated device array instead of a run's workspace.  They need no
// energy histogram, so only the sums are taken: up to 4096 replicas in one
// launch of one block (R = 1000: 37.6 us per call with the reset and the full
// statistics, 31.7 us so).
//
// The array lives in this translation unit.  Host code never passes its name
// to a kernel: on the host the name is only a stand-in for the symbol.  The
// device address of each GPU's copy comes from hipGetSymbolAddress, taken once
// per device with that device current, and only that address reaches the
// kernels and the copies.
#include <mutex>

#include "pa.h"
#include "pa_host.h"
#include "pa_internal.h"
#include "pa_launch.h"

namespace {

using pa::DevStats;

// Layout of the array: statistics block, one partial per block of a large population.
constexpr size_t kOffParts = 256;
constexpr size_t kScratchBytes = kOffParts + (size_t)pa::kMomentBlocks * sizeof(DevStats);

static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
uint8_t* g_ptr[kMaxDevices];  // device address of `scratch` on each GPU (null until looked up)

// Device address of this GPU's scratch, looked up on first use with the device
// current (the caller's current device is the one the stream belongs to).
hipError_t scratch_ptr(uint8_t** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_ptr[dev] = static_cast<uint8_t*>(p);
    }
    *out = g_ptr[dev];
    return hipSuccess;
}

}  // namespace

extern "C" size_t pa_static_scratch_bytes(void) { return kScratchBytes; }

extern "C" pa_status pa_observables_static(int32_t L, int32_t R, const int32_t* d_E, const int32_t* d_M, double beta,
                                           double lnZ, double lnQ, void* hip_stream, pa_obs* out)
{
    if (!(L == 16 || L == 32 || L == 64 || L == 128 || L == 256)) return PA_EINVAL;
    if (R < 1 || R > PA_STATIC_MAX_R || !d_E || !d_M || !out) return PA_EINVAL;
    if (!std::isfinite(beta) || !std::isfinite(lnZ)) return PA_EINVAL;
    const int32_t N = L * L;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    uint8_t* base = nullptr;
    if (scratch_ptr(&base) != hipSuccess) return PA_EHIP;
    DevStats* st = reinterpret_cast<DevStats*>(base);
    DevStats* parts = reinterpret_cast<DevStats*>(base + kOffParts);
    if (pa::launch_moments(d_E, d_M, R, parts, st, s) != hipSuccess) return PA_EHIP;
    DevStats h;
    if (hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess) return PA_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return PA_EHIP;
    pa::host::observables(h, R, N, beta, lnZ, lnQ, out);
    return PA_OK;
}
