// Kernels of the interleaved spin store (PA_SPIN_INTERLEAVED): spin (x, y) of
// replica j is the signed byte at (y L + x) * stride + j, stride = the capacity
// rounded up to 64, so the same spin of all replicas is adjacent (Sec. 3, the
// replica-parallel setup).
//
// Sweeps do not work on these bytes: the population is packed into the 32-site
// words of the bit store, swept there by the bit-sliced kernels, and unpacked
// again (once per pa_sweep, once per pa_anneal whatever its number of steps),
// so the chain is theirs.  Site by site with a lane of its own per replica,
// each site pays its own uniform and five byte reads: 1661 us per launch at
// L = 64, R = 3001, theta = 5, against 16 us packed, with 9 us for pack_kernel
// and 12 us for unpack_kernel (12.3 MB of bytes).
#include "pa_device.h"
#include "pa_launch.h"

namespace pa {
namespace {

using namespace pa::dev;

// Site of within-colour index q of colour c: row y = q / (L/2), column
// x = 2 (q mod L/2) + ((y + c) & 1).
template <int L>
__device__ __forceinline__ int site_of(int c, int q)
{
    const int y = q / (L / 2), h = q - y * (L / 2);
    return y * L + 2 * h + ((y + c) & 1);
}

// Bound by memory: N bytes per replica on the interleaved side, N/8 on the
// other.  A wave takes 64 consecutive replicas, one per lane, so every byte
// instruction touches one 64-byte run of a site row, and a lane moves four
// words (128 sites) of one colour, so the words go as one 16-byte access; a
// launch has N/128 waves per 64 replicas, enough to fill the GPU from a few
// hundred replicas on.
constexpr int kWordsPerLane = 4;

template <int L>
__device__ __forceinline__ bool lane_words(int n, int* j, int* c, int* v)
{
    constexpr int GROUPS = Geo<L>::NW / kWordsPerLane;  // per colour
    const int group = (int)(blockIdx.y * (kBlock / 64) + (threadIdx.x >> 6));
    *j = (int)(blockIdx.x * 64 + (threadIdx.x & 63u));
    *c = group / GROUPS;
    *v = (group - *c * GROUPS) * kWordsPerLane;
    return *j < n && group < 2 * GROUPS;
}

template <int L>
__global__ __launch_bounds__(kBlock) void pack_kernel(const uint8_t* __restrict__ src, size_t stride, int n,
                                                      uint8_t* __restrict__ dst)
{
    int j, c, v;
    if (!lane_words<L>(n, &j, &c, &v)) return;
    uint32_t w[kWordsPerLane];
#pragma unroll
    for (int k = 0; k < kWordsPerLane; ++k) {
        w[k] = 0u;
#pragma unroll
        for (int b = 0; b < 32; ++b)
            w[k] |= (uint32_t)(src[(size_t)site_of<L>(c, 32 * (v + k) + b) * stride + (size_t)j] >> 7) << b;
    }
    uint32_t* rep = reinterpret_cast<uint32_t*>(dst + (size_t)j * Geo<L>::BITS_BYTES);
    *reinterpret_cast<uint4*>(rep + c * Geo<L>::NW + v) = make_uint4(w[0], w[1], w[2], w[3]);
}

template <int L>
__global__ __launch_bounds__(kBlock) void unpack_kernel(const uint8_t* __restrict__ src, size_t stride, int n,
                                                        uint8_t* __restrict__ dst)
{
    int j, c, v;
    if (!lane_words<L>(n, &j, &c, &v)) return;
    const uint32_t* rep = reinterpret_cast<const uint32_t*>(src + (size_t)j * Geo<L>::BITS_BYTES);
    const uint4 q = *reinterpret_cast<const uint4*>(rep + c * Geo<L>::NW + v);
    const uint32_t w[kWordsPerLane] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int k = 0; k < kWordsPerLane; ++k) {
#pragma unroll
        for (int b = 0; b < 32; ++b)  // +1 (0x01) or -1 (0xFF)
            dst[(size_t)site_of<L>(c, 32 * (v + k) + b) * stride + (size_t)j] =
                (uint8_t)(1u | (0u - ((w[k] >> b) & 1u)));
    }
}

template <int L>
dim3 lane_grid(int n)
{
    constexpr int GROUPS = 2 * Geo<L>::NW / kWordsPerLane, PER_BLOCK = kBlock / 64;
    static_assert(Geo<L>::NW % kWordsPerLane == 0, "whole 16-byte accesses");
    return dim3((unsigned)((n + 63) / 64), (unsigned)((GROUPS + PER_BLOCK - 1) / PER_BLOCK));
}

template <int L>
hipError_t launch_pack_l(bool pack, const uint8_t* src, uint32_t stride, int32_t n, uint8_t* dst, hipStream_t s)
{
    if (pack)
        hipLaunchKernelGGL(pack_kernel<L>, lane_grid<L>(n), dim3(kBlock), 0, s, src, (size_t)stride, n, dst);
    else
        hipLaunchKernelGGL(unpack_kernel<L>, lane_grid<L>(n), dim3(kBlock), 0, s, src, (size_t)stride, n, dst);
    return hipGetLastError();
}

hipError_t launch_pack_any(int L, bool pack, const uint8_t* src, uint32_t stride, int32_t n, uint8_t* dst,
                           hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    switch (L) {
    case 16: return launch_pack_l<16>(pack, src, stride, n, dst, s);
    case 32: return launch_pack_l<32>(pack, src, stride, n, dst, s);
    case 64: return launch_pack_l<64>(pack, src, stride, n, dst, s);
    case 128: return launch_pack_l<128>(pack, src, stride, n, dst, s);
    case 256: return launch_pack_l<256>(pack, src, stride, n, dst, s);
    default: return hipErrorInvalidValue;
    }
}

// Replica copy child <- parent[child] of the interleaved store, for child <
// min(*n_new, cap): threads take consecutive children of one chunk of sites,
// so each site row is read near the parents' columns and written as one
// contiguous run of bytes.
constexpr int kCopySites = 256;

__global__ __launch_bounds__(kBlock) void interleaved_copy_kernel(
    const int8_t* __restrict__ src, const int32_t* __restrict__ Es, const int32_t* __restrict__ Ms,
    const uint32_t* __restrict__ parent, const uint32_t* __restrict__ n_new, uint32_t cap, int32_t N, uint32_t stride,
    int8_t* __restrict__ dst, int32_t* __restrict__ Ed, int32_t* __restrict__ Md)
{
    const uint32_t nn = min(*n_new, cap);
    const uint32_t child = blockIdx.x * kBlock + threadIdx.x;
    if (child >= nn) return;
    const uint32_t p = parent[child];
    const int s0 = (int)blockIdx.y * kCopySites, s1 = min(s0 + kCopySites, N);
    for (int s = s0; s < s1; ++s) dst[(size_t)s * stride + child] = src[(size_t)s * stride + p];
    if (blockIdx.y == 0) {
        Ed[child] = Es[p];
        Md[child] = Ms[p];
    }
}

}  // namespace

hipError_t launch_pack(int L, const uint8_t* src, uint32_t stride, int32_t n, uint8_t* dst, hipStream_t s)
{
    return launch_pack_any(L, true, src, stride, n, dst, s);
}

hipError_t launch_unpack(int L, const uint8_t* src, uint32_t stride, int32_t n, uint8_t* dst, hipStream_t s)
{
    return launch_pack_any(L, false, src, stride, n, dst, s);
}

hipError_t launch_copy_interleaved(const uint8_t* src, const int32_t* Esrc, const int32_t* Msrc,
                                   const uint32_t* parent, const uint32_t* n_new, int32_t cap, int32_t N,
                                   uint32_t stride, uint8_t* dst, int32_t* Edst, int32_t* Mdst, hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    const dim3 grid((unsigned)((cap + kBlock - 1) / kBlock), (unsigned)((N + kCopySites - 1) / kCopySites));
    hipLaunchKernelGGL(interleaved_copy_kernel, grid, dim3(kBlock), 0, s, reinterpret_cast<const int8_t*>(src), Esrc,
                       Msrc, parent, n_new, (uint32_t)cap, N, stride, reinterpret_cast<int8_t*>(dst), Edst, Mdst);
    return hipGetLastError();
}

}  // namespace pa
