// Device building blocks of the sweep, shared by the single-run kernel
// (pa_sweep.hip) and the batched kernels (pa_batch.hip): Philox4x32-10,
// lattice geometry, the bit-sliced Metropolis sweep cores and the spin stores.
// The population reductions live in pa_reduce.h.
#pragma once
#include "pa_internal.h"


namespace pa {
namespace dev {

constexpr uint32_t kM0 = 0xD2511F53u;
constexpr uint32_t kM1 = 0xCD9E8D57u;
constexpr uint32_t kW0 = 0x9E3779B9u;
constexpr uint32_t kW1 = 0xBB67AE85u;

struct U4 {
    uint32_t x, y, z, w;
};

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32->64
// multiplies, xor of the high halves with the other words and the round key.
// The three-way xors are single v_bitop3 instructions (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ U4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                       uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)kM0 * c0;
        const uint64_t p1 = (uint64_t)kM1 * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += kW0;
        k1 += kW1;
    }
    return {c0, c1, c2, c3};
}

// The same function for counters whose words 1..3 are equal on every lane of
// the wave (only c0 differs).  In the first three rounds some products and
// xors then involve wave-uniform values only; written as plain xors with the
// uniform operands combined first, those parts compile to scalar
// instructions.  The arithmetic is that of philox10.
__device__ __forceinline__ U4 philox10u(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                        uint32_t k1)
{
    uint64_t p0, p1;
    uint32_t n0, n2;
    // first Philox round: c1, c2, c3 uniform
    p0 = (uint64_t)kM0 * c0;
    p1 = (uint64_t)kM1 * c2;
    n0 = ((uint32_t)(p1 >> 32) ^ c1) ^ k0;
    n2 = (uint32_t)(p0 >> 32) ^ (c3 ^ k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += kW0;
    k1 += kW1;
    // second Philox round: c0, c1 uniform
    p0 = (uint64_t)kM0 * c0;
    p1 = (uint64_t)kM1 * c2;
    n0 = (uint32_t)(p1 >> 32) ^ (c1 ^ k0);
    n2 = c3 ^ ((uint32_t)(p0 >> 32) ^ k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += kW0;
    k1 += kW1;
    // third Philox round: c3 uniform
    p0 = (uint64_t)kM0 * c0;
    p1 = (uint64_t)kM1 * c2;
    n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    n2 = (uint32_t)(p0 >> 32) ^ (c3 ^ k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += kW0;
    k1 += kW1;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        p0 = (uint64_t)kM0 * c0;
        p1 = (uint64_t)kM1 * c2;
        n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += kW0;
        k1 += kW1;
    }
    return {c0, c1, c2, c3};
}

// The register-path sweep evaluates Philox4x32-10 on counters (c0, c1, c2, c3)
// whose words c1 (sweep and colour), c2 (replica) and c3 (stream) are the same
// for every block of a half sweep, and the same on every lane of a wave that
// holds one replica.  The first round's new word 0, hi(M1 c2) ^ c1 ^ k0, then
// depends on none of c0, and so does the second round's product of it: both
// are taken once per half sweep (PhiloxHalf) instead of per block, with plain
// operations that stay scalar when their inputs are.  philox10_h is philox10
// with those values supplied; the arithmetic is the same.
struct PhiloxHalf {
    uint32_t a0;      // round 1: hi(M1 c2) ^ c1 ^ k0
    uint32_t a1;      // round 1: lo(M1 c2)
    uint32_t p0h, p0l;  // round 2: the product M0 a0
};

__device__ __forceinline__ PhiloxHalf philox_half(uint32_t c1, uint32_t c2, uint32_t k0)
{
    const uint64_t P1 = (uint64_t)kM1 * c2;
    PhiloxHalf h;
    h.a0 = ((uint32_t)(P1 >> 32) ^ c1) ^ k0;
    h.a1 = (uint32_t)P1;
    const uint64_t P0 = (uint64_t)kM0 * h.a0;
    h.p0h = (uint32_t)(P0 >> 32);
    h.p0l = (uint32_t)P0;
    return h;
}

// The keys of rounds 4 to 10 of the sweep's Philox blocks, each in a vector
// register of its own.  gfx950 issues instructions of two waves of a SIMD
// together only where their operands are all in vector registers (measured:
// a three-way xor takes 2.4 cycles that way and 4.2 with one scalar operand; a
// chain of Philox rounds 3.9 cycles per instruction at five waves per SIMD
// against 5.0 with the keys in scalar registers, the multiplier staying
// there).  The values go through an opaque move so that the compiler leaves
// them in vector registers.  Sweeps of 20000 replicas: L = 64 1.11 -> 0.98 ms
// (theta = 100), L = 32 0.085 -> 0.080 ms (theta = 20).
struct PhiloxKeys {
    uint32_t k0[7], k1[7];
};

__device__ __forceinline__ uint32_t in_vgpr(uint32_t x)
{
    uint32_t v;
    __asm__("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
    return v;
}

__device__ __forceinline__ PhiloxKeys philox_keys(uint32_t key0, uint32_t key1)
{
    PhiloxKeys k;
#pragma unroll
    for (uint32_t r = 0; r < 7u; ++r) {
        k.k0[r] = in_vgpr(key0 + (r + 3u) * kW0);
        k.k1[r] = in_vgpr(key1 + (r + 3u) * kW1);
    }
    return k;
}

__device__ __forceinline__ U4 philox10_h(uint32_t c0, uint32_t c3, const PhiloxHalf& h, uint32_t k0, uint32_t k1,
                                         const PhiloxKeys& K)
{
    // round 1 (word 0 and word 1 of its output are h.a0, h.a1)
    const uint64_t P0 = (uint64_t)kM0 * c0;
    const uint32_t a2 = (uint32_t)(P0 >> 32) ^ (c3 ^ k1);
    const uint32_t a3 = (uint32_t)P0;
    k0 += kW0;
    k1 += kW1;
    // round 2 (its product M0 a0 is h.p0h, h.p0l)
    const uint64_t P1 = (uint64_t)kM1 * a2;
    uint32_t x0 = (uint32_t)(P1 >> 32) ^ (h.a1 ^ k0);
    uint32_t x1 = (uint32_t)P1;
    uint32_t x2 = a3 ^ (h.p0h ^ k1);
    uint32_t x3 = h.p0l;
    k0 += kW0;
    k1 += kW1;
    // round 3 (word 3 of its input is h.p0l)
    {
        const uint64_t p0 = (uint64_t)kM0 * x0;
        const uint64_t p1 = (uint64_t)kM1 * x2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ (x1 ^ k0);
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ (x3 ^ k1);
        x1 = (uint32_t)p1;
        x3 = (uint32_t)p0;
        x0 = n0;
        x2 = n2;
    }
#pragma unroll
    for (int r = 0; r < 7; ++r) {
        const uint64_t p0 = (uint64_t)kM0 * x0;
        const uint64_t p1 = (uint64_t)kM1 * x2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), x1, K.k0[r]);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), x3, K.k1[r]);
        x1 = (uint32_t)p1;
        x3 = (uint32_t)p0;
        x0 = n0;
        x2 = n2;
    }
    return {x0, x1, x2, x3};
}

// Philox blocks of one half sweep on the register path, counter (c0, 2g + c, j,
// c3): the per-half-sweep values of philox_half are shared by every block.
struct HalfBlocks {
    PhiloxHalf h;
    uint32_t k0, k1;
    const PhiloxKeys& K;
    __device__ __forceinline__ U4 operator()(uint32_t c0, uint32_t c3) const
    {
        return philox10_h(c0, c3, h, k0, k1, K);
    }
};

__device__ __forceinline__ uint32_t pick(const U4& v, uint32_t i)
{
    return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

// Random-stream numbers: the low 4 bits of counter word 3, whose upper bits
// hold the run number (SweepArgs::tag = 16 * run), so every (seed, run,
// stream) has streams of its own.
constexpr uint32_t kStreamSweepHigh = 0;
constexpr uint32_t kStreamResample = 1;
constexpr uint32_t kStreamInit = 2;
constexpr uint32_t kStreamSweepLow = 3;
constexpr uint32_t kStreamLcgSeed = 4;

// Entries of a wave's tie queue on the LDS path (four words each, queue_ties).
constexpr int kTieQueue = 128;
constexpr int kTieQueueWords = 4 * kTieQueue;

template <int L>
struct Geo {
    static constexpr int N = L * L;
    static constexpr int HW = L / 2;                  // sites per row of one colour
    static constexpr int NW = N / 64;                 // 32-site words per colour
    static constexpr int G = NW < 64 ? NW : 64;       // lanes sharing one replica
    static constexpr int K = NW / G;                  // words per lane per colour
    static constexpr int REPW = 64 / G;               // replicas per wave
    static constexpr bool WIDE = HW >= 32;            // rows made of whole words
    static constexpr int WPR = WIDE ? HW / 32 : 1;    // words per row (wide)
    static constexpr int RL = WIDE ? K / WPR : 1;     // rows per lane (wide)
    static constexpr int RPW = WIDE ? 1 : 32 / HW;    // rows per word (narrow)
    static constexpr size_t BITS_BYTES = N / 8;       // bytes per replica, bit store
    static constexpr int RPWV = (K == 1) ? REPW : 1;  // replicas per wave
    // LDS path: a lane decides up to 8 of its K words before the words with
    // sites still tied are resolved through the wave's tie queue.
    static constexpr int SLOTS = (K == 1) ? 1 : (K < 8 ? K : 8);
    // LDS words of one wave on the LDS path: replica [2][NW], then the queue
    static constexpr int WAVE_LDS_WORDS = (K == 1) ? 0 : 2 * NW + kTieQueueWords;
    static constexpr int lds_words(int wpb) { return wpb * WAVE_LDS_WORDS; }
    static_assert(L % 16 == 0 && L >= 16 && L <= 256, "lattice size");
    static_assert(K >= 1 && NW % G == 0, "lane mapping");
};

// Segment masks for narrow rows (HW < 32): bit 0 / top bit of every row
// segment, and the segments of even rows inside a word.
template <int HW>
struct Seg {
    static constexpr uint32_t seg = (HW >= 32) ? 0xFFFFFFFFu : ((1u << (HW % 32)) - 1u);
    static constexpr uint32_t low()
    {
        uint32_t m = 0;
        for (int o = 0; o < 32; o += HW) m |= 1u << o;
        return m;
    }
    static constexpr uint32_t high() { return low() << (HW - 1); }
    static constexpr uint32_t even()
    {
        uint32_t m = 0;
        for (int o = 0; o < 32; o += 2 * HW) m |= seg << o;
        return m;
    }
};

// Value held by the lane `delta` positions away inside the same G-lane group.
template <int G>
__device__ __forceinline__ uint32_t from_lane(uint32_t v, int lane, int delta)
{
    const int base = lane & ~(G - 1);
    const int src = base + ((lane - base + delta + G) & (G - 1));
    return (uint32_t)__shfl((int)v, src);
}

// Value held by lane CTRL of the same four lanes.
template <int CTRL>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL * 0x55, 0xF, 0xF, true);
}

// Neighbour words (other colour) of one own word of colour C.
struct Nb {
    uint32_t up, dn, same, side;
};

// S lanes hold copies of the same word (sweep_quads), the next word being S lanes on.
template <int L, int C, int S = 1>
struct Neighbours {
    using Gm = Geo<L>;
    // boundary words fetched from the adjacent lanes, one set per half sweep
    uint32_t upb[Gm::WPR], dnb[Gm::WPR];
    int lane, gl;

    __device__ __forceinline__ Neighbours(const uint32_t (&oth)[Gm::K], int lane_, int gl_) : lane(lane_), gl(gl_)
    {
        if constexpr (Gm::WIDE) {
#pragma unroll
            for (int t = 0; t < Gm::WPR; ++t) {
                upb[t] = from_lane<Gm::G>(oth[(Gm::RL - 1) * Gm::WPR + t], lane, -1);
                dnb[t] = from_lane<Gm::G>(oth[t], lane, +1);
            }
        } else {
            upb[0] = from_lane<S * Gm::G>(oth[0], lane, -S);
            dnb[0] = from_lane<S * Gm::G>(oth[0], lane, +S);
        }
    }

    __device__ __forceinline__ Nb get(const uint32_t (&oth)[Gm::K], int k) const
    {
        Nb n;
        if constexpr (Gm::WIDE) {
            const int r = k / Gm::WPR, t = k % Gm::WPR;
            const int tp = (t + Gm::WPR - 1) % Gm::WPR, tn = (t + 1) % Gm::WPR;
            const uint32_t cur = oth[k];
            n.same = cur;
            n.up = (r > 0) ? oth[k - Gm::WPR] : upb[t];
            n.dn = (r < Gm::RL - 1) ? oth[k + Gm::WPR] : dnb[t];
            // (y + C) even: horizontal neighbour at h-1, else at h+1
            const uint32_t hm1 = __builtin_amdgcn_alignbit(cur, oth[r * Gm::WPR + tp], 31);
            const uint32_t hp1 = __builtin_amdgcn_alignbit(oth[r * Gm::WPR + tn], cur, 1);
            if constexpr (Gm::RL % 2 == 0) {
                n.side = (((r + C) & 1) == 0) ? hm1 : hp1;
            } else {
                const int y = gl * Gm::RL + r;
                n.side = (((y + C) & 1) == 0) ? hm1 : hp1;
            }
        } else {
            constexpr int HW = Gm::HW;
            using Sg = Seg<HW>;
            const uint32_t o = oth[0];
            n.same = o;
            n.up = __builtin_amdgcn_alignbit(o, upb[0], 32 - HW);
            n.dn = __builtin_amdgcn_alignbit(dnb[0], o, HW);
            const uint32_t rotl = ((o << 1) & ~Sg::low()) | ((o >> (HW - 1)) & Sg::low());
            const uint32_t rotr = ((o >> 1) & ~Sg::high()) | ((o << (HW - 1)) & Sg::high());
            n.side = (C == 0) ? ((rotl & Sg::even()) | (rotr & ~Sg::even()))
                              : ((rotr & Sg::even()) | (rotl & ~Sg::even()));
        }
        return n;
    }
};

// One bit plane of the bit-serial comparison "uniform < threshold", high bit
// first, for NG words together.  k = 2 sites (cls1) compare against T_2, k = 4
// sites against T_4.  acc holds the sites accepted so far and open those not
// rejected so far, so acc is a subset of open and open & ~acc are the sites
// still tied.  A threshold bit 1 accepts the tied sites whose plane bit is 0, a
// threshold bit 0 rejects those whose plane bit is 1; with
//   m = acc | (open & ~x)
// a plane therefore replaces acc (bit 1) or open (bit 0) by m: one operation
// per word where both classes have the same threshold bit and three where they
// differ (select by class into both masks).  tb holds the two threshold bits of
// the plane (bit 1: T_2, bit 0: T_4) and is uniform.  Its four cases are one
// block of assembly, arithmetic and branches only: written as a switch, the
// compiler joins the cases with five register moves per plane of four words
// (L = 128, R = 50000: 144 -> 131 vector instructions per word and half sweep,
// 1.68 -> 1.63 ms per launch of 20 sweeps).  The masks are early
// clobbers: the cases that select read the class again after writing them.
#define PA_PLANE_M(i, t) "v_bitop3_b32 %[" t "], %[a" i "], %[o" i "], %[x" i "] bitop3:0xf4\n\t"
#define PA_PLANE_SEL(d, i, p, q) "v_bitop3_b32 %[" d i "], %[c" i "], %[" p "], %[" q "] bitop3:0xca\n\t"
#define PA_PLANE_0(i) PA_PLANE_M(i, "o" i)
#define PA_PLANE_3(i) PA_PLANE_M(i, "a" i)
#define PA_PLANE_2(i, t) PA_PLANE_M(i, t) PA_PLANE_SEL("a", i, t, "a" i) PA_PLANE_SEL("o", i, "o" i, t)
#define PA_PLANE_1(i, t) PA_PLANE_M(i, t) PA_PLANE_SEL("a", i, "a" i, t) PA_PLANE_SEL("o", i, t, "o" i)
#define PA_PLANE_ASM(C0, C1, C2, C3)                                                                              \
    "s_cmp_lt_u32 %[tb], 2\n\t"                                                                                   \
    "s_cbranch_scc1 .Lpa_plane_low%=\n\t"                                                                         \
    "s_cmp_eq_u32 %[tb], 3\n\t"                                                                                   \
    "s_cbranch_scc1 .Lpa_plane_3%=\n\t" C2                                                                        \
    "s_branch .Lpa_plane_end%=\n"                                                                                 \
    ".Lpa_plane_low%=:\n\t"                                                                                       \
    "s_cmp_eq_u32 %[tb], 0\n\t"                                                                                   \
    "s_cbranch_scc1 .Lpa_plane_0%=\n\t" C1                                                                        \
    "s_branch .Lpa_plane_end%=\n"                                                                                 \
    ".Lpa_plane_3%=:\n\t" C3                                                                                      \
    "s_branch .Lpa_plane_end%=\n"                                                                                 \
    ".Lpa_plane_0%=:\n\t" C0                                                                                      \
    ".Lpa_plane_end%=:\n\t"

template <int NG>
__device__ __forceinline__ void open_plane(const uint32_t (&x)[NG], uint32_t tb, const uint32_t (&cls1)[NG],
                                           uint32_t (&acc)[NG], uint32_t (&open)[NG])
{
    static_assert(NG == 1 || NG == 2 || NG == 4, "words of a group");
    uint32_t t0;
    if constexpr (NG == 1) {
        __asm__(PA_PLANE_ASM(PA_PLANE_0("0"), PA_PLANE_1("0", "t0"), PA_PLANE_2("0", "t0"), PA_PLANE_3("0"))
                : [a0] "+&v"(acc[0]), [o0] "+&v"(open[0]), [t0] "=&v"(t0)
                : [x0] "v"(x[0]), [c0] "v"(cls1[0]), [tb] "s"(tb)
                : "scc");
    } else if constexpr (NG == 2) {
        __asm__(PA_PLANE_ASM(PA_PLANE_0("0") PA_PLANE_0("1"), PA_PLANE_1("0", "t0") PA_PLANE_1("1", "t0"),
                             PA_PLANE_2("0", "t0") PA_PLANE_2("1", "t0"), PA_PLANE_3("0") PA_PLANE_3("1"))
                : [a0] "+&v"(acc[0]), [o0] "+&v"(open[0]), [a1] "+&v"(acc[1]), [o1] "+&v"(open[1]), [t0] "=&v"(t0)
                : [x0] "v"(x[0]), [c0] "v"(cls1[0]), [x1] "v"(x[1]), [c1] "v"(cls1[1]), [tb] "s"(tb)
                : "scc");
    } else {
        __asm__(PA_PLANE_ASM(PA_PLANE_0("0") PA_PLANE_0("1") PA_PLANE_0("2") PA_PLANE_0("3"),
                             PA_PLANE_1("0", "t0") PA_PLANE_1("1", "t0") PA_PLANE_1("2", "t0") PA_PLANE_1("3", "t0"),
                             PA_PLANE_2("0", "t0") PA_PLANE_2("1", "t0") PA_PLANE_2("2", "t0") PA_PLANE_2("3", "t0"),
                             PA_PLANE_3("0") PA_PLANE_3("1") PA_PLANE_3("2") PA_PLANE_3("3"))
                : [a0] "+&v"(acc[0]), [o0] "+&v"(open[0]), [a1] "+&v"(acc[1]), [o1] "+&v"(open[1]), [a2] "+&v"(acc[2]),
                  [o2] "+&v"(open[2]), [a3] "+&v"(acc[3]), [o3] "+&v"(open[3]), [t0] "=&v"(t0)
                : [x0] "v"(x[0]), [c0] "v"(cls1[0]), [x1] "v"(x[1]), [c1] "v"(cls1[1]), [x2] "v"(x[2]),
                  [c2] "v"(cls1[2]), [x3] "v"(x[3]), [c3] "v"(cls1[3]), [tb] "s"(tb)
                : "scc");
    }
}

// The threshold bits of plane q (0: the highest of the 16 high bits) as
// open_plane takes them.
__device__ __forceinline__ uint32_t plane_bits(const SweepArgs& a, int q)
{
    const int bit = 15 - q;
    return (((a.t2h >> bit) & 1u) << 1) | ((a.t4h >> bit) & 1u);
}

// Metropolis acceptance mask of one 32-site word.  A site flips if at least two
// of its four neighbours are anti-aligned (k = s h <= 0), else if its uniform
// x (high 16 bits from the bit planes, low 16 bits drawn on a tie) is below
// the threshold of its class (one anti-aligned neighbour: k = 2; none: k = 4).
template <class BLK>
__device__ __forceinline__ uint32_t accept_mask(uint32_t w, const Nb& n, uint32_t v, const BLK& blk,
                                                const SweepArgs& a)
{
    const uint32_t d1 = w ^ n.up, d2 = w ^ n.dn, d3 = w ^ n.same, d4 = w ^ n.side;
    const uint32_t o12 = d1 | d2, a12 = d1 & d2, o34 = d3 | d4, a34 = d3 & d4;
    const uint32_t ge2 = a12 | a34 | (o12 & o34);
    const uint32_t any = o12 | o34;
    const uint32_t cls1[1] = {any & ~ge2};  // k = 2
    uint32_t acc[1] = {ge2}, open[1] = {0xFFFFFFFFu};  // open & ~acc: sites still tied with their threshold
    if (__builtin_expect((a.t2h | a.t4h) > 0xFFFFu, 0)) {  // a threshold is 2^32 (beta ~ 0): always accepted
        if (a.t2h > 0xFFFFu) acc[0] |= cls1[0];
        if (a.t4h > 0xFFFFu) acc[0] |= ~any;
    }
    if (__any(open[0] != acc[0])) {
        // blocks 0, 1 and 2 are computed together (three independent chains),
        // since the first eight planes leave some site of the wave tied almost
        // surely (the wave holds about 2000 sites that need a uniform)
        const U4 P0 = blk(4u * v, a.tag | kStreamSweepHigh);
        const U4 P1 = blk(4u * v + 1u, a.tag | kStreamSweepHigh);
        const U4 P2 = blk(4u * v + 2u, a.tag | kStreamSweepHigh);
        const uint32_t pl[12][1] = {{P0.x}, {P0.y}, {P0.z}, {P0.w}, {P1.x}, {P1.y},
                                    {P1.z}, {P1.w}, {P2.x}, {P2.y}, {P2.z}, {P2.w}};
#pragma unroll
        for (int q = 0; q < 12; ++q) open_plane<1>(pl[q], plane_bits(a, q), cls1, acc, open);
        if (__any(open[0] != acc[0])) {
            const U4 P = blk(4u * v + 3u, a.tag | kStreamSweepHigh);
            const uint32_t pq[4][1] = {{P.x}, {P.y}, {P.z}, {P.w}};
#pragma unroll
            for (int q = 0; q < 4; ++q) open_plane<1>(pq[q], plane_bits(a, 12 + q), cls1, acc, open);
        }
    }
    uint32_t tie = open[0] & ~acc[0];
    while (tie) {
        const int b = __builtin_ctz(tie);
        tie &= tie - 1u;
        const uint32_t q = 32u * v + (uint32_t)b;
        const U4 P = blk(q >> 3, a.tag | kStreamSweepLow);
        const uint32_t word = pick(P, (q >> 1) & 3u);
        const uint32_t lo = (q & 1u) ? (word & 0xFFFFu) : (word >> 16);
        const uint32_t tl = ((cls1[0] >> b) & 1u) ? a.t2l : a.t4l;
        if (lo < tl) acc[0] |= 1u << b;
    }
    return acc[0];
}

// Neighbour classes of the heat-bath update.  With a the number of
// anti-aligned neighbours, k = s h = 4 - 2a: neg holds the sites with k < 0
// (a >= 3), zero those with k = 0 (a = 2) and cls1 those with |k| = 2 (a = 1
// or 3); the remaining sites have |k| = 4.
struct HbClass {
    uint32_t neg, zero, cls1;
};

__device__ __forceinline__ HbClass hb_classes(uint32_t w, const Nb& n)
{
    const uint32_t d1 = w ^ n.up, d2 = w ^ n.dn, d3 = w ^ n.same, d4 = w ^ n.side;
    const uint32_t o12 = d1 | d2, a12 = d1 & d2, o34 = d3 | d4, a34 = d3 & d4;
    const uint32_t ge1 = o12 | o34;
    const uint32_t ge2 = a12 | a34 | (o12 & o34);
    const uint32_t ge3 = (a12 & o34) | (a34 & o12);
    const uint32_t all4 = a12 & a34;
    HbClass c;
    c.neg = ge3;
    c.zero = ge2 & ~ge3;
    c.cls1 = (ge1 & ~ge2) | (ge3 & ~all4);
    return c;
}

// Heat-bath flip mask of one 32-site word.  A site flips with probability
// 1 / (1 + e^{2 beta k}): iff its uniform x is below U_k, where U_2 and U_4 (at
// most 2^31) arrive in the threshold arguments, U_0 = 2^31 and
// U_{-k} = 2^32 - U_k.  For k < 0, "x < 2^32 - U_|k|" is "not (~x < U_|k|)",
// so those sites compare the complement of their uniform with U_|k| (the
// planes and the low half xored with neg) and take the opposite result.  The
// k = 0 sites are decided by the top bit of x alone.
template <class BLK>
__device__ __forceinline__ uint32_t heatbath_mask(uint32_t w, const Nb& n, uint32_t v, const BLK& blk,
                                                  const SweepArgs& a)
{
    const HbClass c = hb_classes(w, n);
    const uint32_t cls1[1] = {c.cls1};
    // blocks 0, 1 and 2 together (three independent chains), as in accept_mask
    const U4 P0 = blk(4u * v, a.tag | kStreamSweepHigh);
    const U4 P1 = blk(4u * v + 1u, a.tag | kStreamSweepHigh);
    const U4 P2 = blk(4u * v + 2u, a.tag | kStreamSweepHigh);
    const uint32_t pl[12] = {P0.x, P0.y, P0.z, P0.w, P1.x, P1.y, P1.z, P1.w, P2.x, P2.y, P2.z, P2.w};
    uint32_t acc[1] = {c.zero & ~pl[0]};  // U_0 = 2^31: x < U_0 iff its top bit is 0
    uint32_t open[1] = {acc[0] | ~c.zero};
#pragma unroll
    for (int q = 0; q < 12; ++q) {
        const uint32_t x[1] = {pl[q] ^ c.neg};
        open_plane<1>(x, plane_bits(a, q), cls1, acc, open);
    }
    if (__any(open[0] != acc[0])) {
        const U4 P = blk(4u * v + 3u, a.tag | kStreamSweepHigh);
        const uint32_t pq[4] = {P.x, P.y, P.z, P.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t x[1] = {pq[q] ^ c.neg};
            open_plane<1>(x, plane_bits(a, 12 + q), cls1, acc, open);
        }
    }
    uint32_t tie = open[0] & ~acc[0];
    while (tie) {
        const int b = __builtin_ctz(tie);
        tie &= tie - 1u;
        const uint32_t q = 32u * v + (uint32_t)b;
        const U4 P = blk(q >> 3, a.tag | kStreamSweepLow);
        const uint32_t word = pick(P, (q >> 1) & 3u);
        uint32_t lo = (q & 1u) ? (word & 0xFFFFu) : (word >> 16);
        if ((c.neg >> b) & 1u) lo ^= 0xFFFFu;
        const uint32_t tl = ((c.cls1 >> b) & 1u) ? a.t2l : a.t4l;
        if (lo < tl) acc[0] |= 1u << b;
    }
    return acc[0] ^ c.neg;
}

// In-line LCG variant of the multi-spin-coded sweep (Sec. 4): the generator
// r' = A r + C mod 2^32 (A = 1664525, C = 1013904223), seeded once per word
// and update by the base generator, supplies the 32 uniforms of the word.
// Site b takes the (b+1)-th output after the seed r_0, written in closed form
// as r_{b+1} = A^{b+1} r_0 + C (A^b + ... + 1) mod 2^32, so the 32 outputs
// are independent multiply-adds instead of a chain.
constexpr uint32_t kLcgA = 1664525u;
constexpr uint32_t kLcgC = 1013904223u;

constexpr uint32_t lcg_mul(int n)  // A^n mod 2^32
{
    uint32_t m = 1u;
    for (int i = 0; i < n; ++i) m *= kLcgA;
    return m;
}

constexpr uint32_t lcg_add(int n)  // C (A^{n-1} + ... + A + 1) mod 2^32
{
    uint32_t c = 0u;
    for (int i = 0; i < n; ++i) c = c * kLcgA + kLcgC;
    return c;
}

// acc = 2 acc + [x <= t]: the comparison writes a lane mask that the add
// takes as its carry-in (two VALU instructions; the compiler's own form is a
// compare, a select and a shift-or).  Arithmetic only, no memory access.
__device__ __forceinline__ uint32_t shift_in_le(uint32_t acc, uint32_t x, uint32_t t)
{
    uint64_t le, carry;
    __asm__("v_cmp_ge_u32_e64 %1, %4, %3\n\t"
            "v_addc_co_u32_e64 %0, %2, %0, %0, %1"
            : "+v"(acc), "=&s"(le), "=&s"(carry)
            : "v"(x), "s"(t));
    return acc;
}

// The same for two outputs and both thresholds as one block, the comparisons
// before the adds, so that no add waits for its own.  Between blocks of which one
// writes a register and the next reads it the compiler puts a wait state: about
// 50 in the 528 instructions of a sweep with a block per comparison.  They and
// the waits are lost time where a wave has its SIMD to itself, and free
// where others fill them; there the shorter blocks mix better with the
// multiplications (20 sweeps, with wave priorities, by these and by pairs: L = 64,
// R = 9800 149, 180 us; L = 16, R = 200000 188, 199).
__device__ __forceinline__ void shift_in_pair(uint32_t& m2, uint32_t& m4, uint32_t x, uint32_t y, uint32_t t2,
                                              uint32_t t4)
{
    uint64_t x2, x4, y2, y4;
    __asm__("v_cmp_ge_u32_e64 %[x2], %[t2], %[x]\n\t"
            "v_cmp_ge_u32_e64 %[x4], %[t4], %[x]\n\t"
            "v_cmp_ge_u32_e64 %[y2], %[t2], %[y]\n\t"
            "v_cmp_ge_u32_e64 %[y4], %[t4], %[y]\n\t"
            "v_addc_co_u32_e64 %[m2], %[x2], %[m2], %[m2], %[x2]\n\t"
            "v_addc_co_u32_e64 %[m4], %[x4], %[m4], %[m4], %[x4]\n\t"
            "v_addc_co_u32_e64 %[m2], %[y2], %[m2], %[m2], %[y2]\n\t"
            "v_addc_co_u32_e64 %[m4], %[y4], %[m4], %[m4], %[y4]"
            : [m2] "+&v"(m2), [m4] "+&v"(m4), [x2] "=&s"(x2), [x4] "=&s"(x4), [y2] "=&s"(y2), [y4] "=&s"(y4)
            : [x] "v"(x), [y] "v"(y), [t2] "s"(t2), [t4] "s"(t4));
}

// Metropolis acceptance mask of one 32-site word whose uniforms are the LCG
// outputs after `seed`: a site flips if k <= 0, else if its uniform x is below
// T_2 (one anti-aligned neighbour) or T_4 (none), i.e. x <= T - 1 (T >= 1).
// PAIRS: by shift_in_pair.
template <bool PAIRS>
__device__ __forceinline__ uint32_t lcg_accept_mask(uint32_t w, const Nb& n, uint32_t seed, const SweepArgs& a)
{
    const uint32_t d1 = w ^ n.up, d2 = w ^ n.dn, d3 = w ^ n.same, d4 = w ^ n.side;
    const uint32_t o12 = d1 | d2, a12 = d1 & d2, o34 = d3 | d4, a34 = d3 & d4;
    const uint32_t ge2 = a12 | a34 | (o12 & o34);
    const uint32_t any = o12 | o34;
    // T - 1 in 32 bits (T = 2^32 gives 2^32 - 1)
    const uint32_t t2m1 = (a.t2h << 16) + a.t2l - 1u;
    const uint32_t t4m1 = (a.t4h << 16) + a.t4l - 1u;
    uint32_t m2 = 0u, m4 = 0u;
    const auto output = [seed](int i) { return (uint32_t)((uint64_t)lcg_mul(i) * seed + (uint64_t)lcg_add(i)); };
    if constexpr (PAIRS) {
#pragma unroll
        for (int b = 32; b > 0; b -= 2) shift_in_pair(m2, m4, output(b), output(b - 1), t2m1, t4m1);
    } else {
#pragma unroll
        for (int b = 32; b > 0; --b) {
            const uint32_t x = output(b);
            m2 = shift_in_le(m2, x, t2m1);
            m4 = shift_in_le(m4, x, t4m1);
        }
    }
    return ge2 | (any & ~ge2 & m2) | (~any & m4);
}

// One colour of the LCG sweep for the lane's one word (register path).
template <int L, int C, bool PAIRS>
__device__ __forceinline__ void half_sweep_lcg(uint32_t (&own)[1], const uint32_t (&oth)[1], int lane, int gl,
                                               uint32_t seed, const SweepArgs& a)
{
    const Neighbours<L, C> nb(oth, lane, gl);
    own[0] ^= lcg_accept_mask<PAIRS>(own[0], nb.get(oth, 0), seed, a);
}

template <int L, int C, bool HB>
__device__ __forceinline__ void half_sweep(uint32_t (&own)[Geo<L>::K], const uint32_t (&oth)[Geo<L>::K], int lane,
                                           int gl, uint32_t g, uint32_t j, const SweepArgs& a, const PhiloxKeys& K)
{
    using Gm = Geo<L>;
    const Neighbours<L, C> nb(oth, lane, gl);
    const uint32_t ctr1 = 2u * g + (uint32_t)C;
    const HalfBlocks blocks{philox_half(ctr1, j, a.key0), a.key0, a.key1, K};
#pragma unroll
    for (int k = 0; k < Gm::K; ++k) {
        const uint32_t v = (uint32_t)(gl * Gm::K + k);
        if constexpr (HB)
            own[k] ^= heatbath_mask(own[k], nb.get(oth, k), v, blocks, a);
        else
            own[k] ^= accept_mask(own[k], nb.get(oth, k), v, blocks, a);
    }
}


// Decisions of the first 8 bit planes (Philox blocks 0 and 1) for NG words of
// one lane together.  A site flips if at least two of its four neighbours are
// anti-aligned (k = s h <= 0); a site with one anti-aligned neighbour (k = 2,
// `cls1`) or none (k = 4) flips if its uniform x is below T_2 or T_4.  The
// planes are compared high bit first with one uniform branch per plane over the
// two threshold bits, shared by the NG words.  The words are updated with
// their decided flips; `tie` receives the sites whose 8 high bits equal the
// threshold's (probability 2^-8 each), decided later by decide_word_tail.  With
// HB (heat-bath, the update of heatbath_mask) every site draws, the k = 0 sites
// are decided by plane 0, the k < 0 sites compare the complemented planes
// (`ng`) and are flipped provisionally, so that the tail's result xored on top
// gives their decision.  blk(g, kk) is Philox block kk of word g.
template <int NG, bool HB, class BLK>
__device__ __forceinline__ void decide8_group(uint32_t (&w)[NG], const Nb (&n)[NG], const BLK& blk,
                                              const SweepArgs& a, uint32_t (&tie)[NG], uint32_t (&cls1)[NG],
                                              uint32_t (&ng)[NG])
{
    uint32_t acc[NG], open[NG], zero[NG];  // zero: heat-bath k = 0 sites; Metropolis: any anti-aligned neighbour
    uint32_t need = 0u;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if constexpr (HB) {
            const HbClass c = hb_classes(w[g], n[g]);
            cls1[g] = c.cls1;
            ng[g] = c.neg;
            zero[g] = c.zero;
        } else {
            const uint32_t d1 = w[g] ^ n[g].up, d2 = w[g] ^ n[g].dn, d3 = w[g] ^ n[g].same, d4 = w[g] ^ n[g].side;
            const uint32_t o12 = d1 | d2, a12 = d1 & d2, o34 = d3 | d4, a34 = d3 & d4;
            const uint32_t ge2 = a12 | a34 | (o12 & o34);
            const uint32_t any = o12 | o34;
            cls1[g] = any & ~ge2;
            ng[g] = 0u;
            zero[g] = any;
            acc[g] = ge2;
            open[g] = 0xFFFFFFFFu;
        }
    }
    if constexpr (!HB) {
        if (__builtin_expect((a.t2h | a.t4h) > 0xFFFFu, 0)) {  // a threshold is 2^32 (beta ~ 0): always accepted
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (a.t2h > 0xFFFFu) acc[g] |= cls1[g];
                if (a.t4h > 0xFFFFu) acc[g] |= ~zero[g];
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) need |= ~acc[g];
    }
    // heat-bath draws for every site: its k = 0 sites are decided by plane 0
    // even when no site of the wave is left for the later planes
    if (HB || __any(need != 0u)) {
        uint32_t pl[8][NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const U4 P0 = blk(g, 0u), P1 = blk(g, 1u);
            pl[0][g] = P0.x, pl[1][g] = P0.y, pl[2][g] = P0.z, pl[3][g] = P0.w;
            pl[4][g] = P1.x, pl[5][g] = P1.y, pl[6][g] = P1.z, pl[7][g] = P1.w;
            if constexpr (HB) {
                acc[g] = zero[g] & ~pl[0][g];  // U_0 = 2^31: x < U_0 iff its top bit is 0
                open[g] = acc[g] | ~zero[g];
#pragma unroll
                for (int q = 0; q < 8; ++q) pl[q][g] ^= ng[g];
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) open_plane<NG>(pl[q], plane_bits(a, q), cls1, acc, open);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        w[g] ^= HB ? acc[g] ^ ng[g] : acc[g];
        tie[g] = open[g] & ~acc[g];
    }
}

// Orders the LDS accesses of one wave: everything before is complete and
// visible to every lane of the wave after.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Remaining comparison of the tied sites `mask` of word v (all tied after 8
// planes): Philox block 2 (planes 8-11) once for the word, block 3 (planes
// 12-15) once if a site of the wave is still tied, then the SWEEP-LOW half of
// each site still tied.  cls1 marks the sites of class k = 2, ngm (heat-bath)
// those that compare the complement of their uniform, k < 0.  Returns the
// sites whose (complemented) uniform is below their threshold, each decided
// exactly as a comparison of its whole 32-bit uniform would decide it.  The
// planes are compared for the whole word at once: the sites that are not
// tied have open = acc = 0 and stay so (deciding each tied site by itself, bit
// by bit, took 161 vector instructions per word and half sweep at L = 128
// against 144, and 2.10 ms per launch of 20 sweeps at R = 50000 against 1.68).
template <bool HB>
__device__ __forceinline__ uint32_t decide_word_tail(uint32_t v, uint32_t mask, uint32_t cls1, uint32_t ngm,
                                                     const PhiloxHalf& h, const SweepArgs& a, const PhiloxKeys& K)
{
    uint32_t acc[1] = {0u}, open[1] = {mask};
    const uint32_t c1[1] = {cls1};
#pragma unroll
    for (int kk = 2; kk < 4; ++kk) {
        if (!__any(open[0] != acc[0])) return acc[0];
        const U4 P = philox10_h(4u * v + (uint32_t)kk, a.tag | kStreamSweepHigh, h, a.key0, a.key1, K);
        uint32_t x[4][1] = {{P.x}, {P.y}, {P.z}, {P.w}};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (HB) x[q][0] ^= ngm;
            open_plane<1>(x[q], plane_bits(a, 4 * kk + q), c1, acc, open);
        }
    }
    uint32_t below = acc[0];
    mask = open[0] & ~acc[0];
    while (mask) {
        const uint32_t b = (uint32_t)__builtin_ctz(mask);
        mask &= mask - 1u;
        const uint32_t q = 32u * v + b;
        const U4 P = philox10_h(q >> 3, a.tag | kStreamSweepLow, h, a.key0, a.key1, K);
        const uint32_t word = pick(P, (q >> 1) & 3u);
        uint32_t lo = (q & 1u) ? (word & 0xFFFFu) : (word >> 16);
        if (HB && ((ngm >> b) & 1u)) lo ^= 0xFFFFu;
        if (lo < (((cls1 >> b) & 1u) ? a.t2l : a.t4l)) below |= 1u << b;
    }
    return below;
}

// Tie queue of one wave.  The sites still tied after decide8_group are rare
// (2^-8 each), so instead of evaluating the later Philox blocks for every
// word, every word that holds a tied site is queued in LDS and decided by one
// lane, which evaluates the later blocks once for all of the word's tied
// sites.  Entry i of the queue is the four words
//   q[4 i]      the word's number in the wave (the caller's encoding)
//   q[4 i + 1]  the word's tied sites
//   q[4 i + 2]  its sites of class k = 2
//   q[4 i + 3]  its sites that compare the complement of their uniform
// Each word's entries are placed by a wave vote: the lanes with a tie take
// consecutive entries in lane order.
// Queues the tied words of one group of NG words, id[g] their numbers, after
// the nq entries already queued.  If the queue would then hold more than
// min(a.qcap, kTieQueue) entries, every lane decides the group's words itself:
// own(g, tie, cls1, ng) does so for word g.
template <int NG, class OWN>
__device__ __forceinline__ void queue_ties(const uint32_t (&tie)[NG], const uint32_t (&cls1)[NG],
                                           const uint32_t (&ng)[NG], const uint32_t (&id)[NG], const SweepArgs& a,
                                           uint32_t* queue, uint32_t& nq, const OWN& own)
{
    uint64_t vote[NG];
    uint32_t total = 0u;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        vote[g] = __ballot(tie[g] != 0u);
        total += (uint32_t)__popcll(vote[g]);
    }
    if (__builtin_expect(nq + total > min(a.qcap, (uint32_t)kTieQueue), 0)) {
#pragma unroll 1
        for (int g = 0; g < NG; ++g) {
            uint32_t t = 0u, c = 0u, n = 0u;
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                t = (i == g) ? tie[i] : t;
                c = (i == g) ? cls1[i] : c;
                n = (i == g) ? ng[i] : n;
            }
            own(g, t, c, n);
        }
        return;
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (tie[g] != 0u) {
            const uint32_t lo = (uint32_t)vote[g], hi = (uint32_t)(vote[g] >> 32);
            const uint32_t i = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, nq));
            reinterpret_cast<uint4*>(queue)[i] = make_uint4(id[g], tie[g], cls1[g], ng[g]);
        }
        nq += (uint32_t)__popcll(vote[g]);
    }
}

// Decides the nq queued words, one per lane: half(id, &v) gives a word's index
// in its replica and the shared part of its Philox blocks, and apply(id, f)
// takes the additional flips of a word (each word is in one entry, so no two
// lanes touch the same word).
template <bool HB, class HALF, class APPLY>
__device__ __forceinline__ void resolve_ties(uint32_t nq, const SweepArgs& a, const PhiloxKeys& K,
                                             const uint32_t* queue, int lane, const HALF& half, const APPLY& apply)
{
    wave_lds_sync();
    for (uint32_t i = (uint32_t)lane; i < nq; i += 64u) {
        const uint4 e = reinterpret_cast<const uint4*>(queue)[i];
        uint32_t v;
        const PhiloxHalf h = half(e.x, &v);
        apply(e.x, decide_word_tail<HB>(v, e.y, e.z, e.w, h, a, K));
    }
    wave_lds_sync();
}

// Sign bits of 16 consecutive int8 spins: the even-x ones in byte 0, the odd-x
// ones in byte 1 (the bytes above are not meant).  Dword k puts its four sign
// bits at bit 2k of the bytes of x; the even sites are then in bytes 0 and 2 and
// the odd ones in 1 and 3, and the upper pair moves in between the lower one's
// bits.
__device__ __forceinline__ uint32_t pack16(const uint4& q)
{
    const uint32_t x = ((q.x >> 7) & 0x01010101u) | ((q.y >> 5) & 0x04040404u) | ((q.z >> 3) & 0x10101010u) |
                       ((q.w >> 1) & 0x40404040u);
    return x | (x >> 15);
}

// The reverse (bytes 2 and 3 of z are zero): each dword's four bits picked out
// of x, one per byte, select the bytes +1 (0x01) or -1 (0xFF).
__device__ __forceinline__ uint4 unpack16(uint32_t z)
{
    const uint32_t x = z | (z << 15);
    uint32_t w[4];
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) w[k] = __builtin_amdgcn_perm(0u, 0xFF01u, (x >> (2u * k)) & 0x01010101u);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Byte s of ev and od as unpack16 takes them (v_perm_b32: selector bytes 0-3
// take from the second operand, 4-7 from the first, 12 is zero).
__device__ __forceinline__ uint32_t byte_pair(uint32_t ev, uint32_t od, uint32_t s)
{
    return __builtin_amdgcn_perm(od, ev, 0x0C0C0400u + 0x0101u * s);
}

// Sign bits of 64 consecutive int8 spins -> (even-x bits, odd-x bits), and back.
// One running value per 16 bytes: as 64 single bits joined by an or-tree it held
// up to 30 temporaries, which put other values of the register-path kernels
// into scratch memory.
__device__ __forceinline__ void pack64(const uint4* src, uint32_t& ev, uint32_t& od)
{
    uint32_t z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = pack16(src[i]);
    const uint32_t lo = __builtin_amdgcn_perm(z[1], z[0], 0x05010400u);  // even 0, even 1, odd 0, odd 1
    const uint32_t hi = __builtin_amdgcn_perm(z[3], z[2], 0x05010400u);
    ev = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    od = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

__device__ __forceinline__ void unpack64(uint32_t ev, uint32_t od, uint4* dst)
{
#pragma unroll
    for (uint32_t i = 0; i < 4u; ++i) dst[i] = unpack16(byte_pair(ev, od, i));
}

// Row-parity blend between the even-x / odd-x bits of a 64-site chunk and the
// two colour words: colour 0 holds the even-x sites of even rows.
template <int L>
__device__ __forceinline__ uint32_t even_row_mask(uint32_t v)
{
    using Gm = Geo<L>;
    if constexpr (Gm::WIDE) {
        return (((v / Gm::WPR) & 1u) == 0u) ? 0xFFFFFFFFu : 0u;
    } else {
        return Seg<Gm::HW>::even();
    }
}

// Replica identity of a lane: group of G lanes per replica inside the wave.
struct LaneInfo {
    int lane, gl;
    uint32_t j;
    bool valid;
};

// Lane of thread `thread` in the wave `wave` of a run (register path).
template <int L>
__device__ __forceinline__ LaneInfo lane_info(const SweepArgs& a, int wave, uint32_t thread)
{
    using Gm = Geo<L>;
    LaneInfo li;
    li.lane = (int)(thread & 63u);
    li.gl = li.lane % Gm::G;
    int j = wave * Gm::REPW + li.lane / Gm::G;
    if constexpr (Gm::REPW == 1) j = __builtin_amdgcn_readfirstlane(j);
    li.j = (uint32_t)j;
    li.valid = j < a.n_rep;
    return li;
}

// Initial-state word (stream INIT): the INIT output word p >> 5 with
// p = c N/2 + q is exactly the 32-site word (c, v) of the bit store.
template <int L>
__device__ __forceinline__ uint32_t init_word(int c, uint32_t v, uint32_t j, const SweepArgs& a)
{
    const uint32_t idx = (uint32_t)(c * Geo<L>::NW) + v;
    return pick(philox10(idx >> 2, 0u, j, a.tag | kStreamInit, a.key0, a.key1), idx & 3u);
}

// Bytes of one replica in the spin store.
template <int L, bool INT8>
constexpr size_t replica_bytes()
{
    return INT8 ? (size_t)Geo<L>::N : Geo<L>::BITS_BYTES;
}

// The stored replica a sweep starts from for slot j: slot j of the store, or,
// when the sweep follows a resampling (a.parent set), replica parent[j] of the
// parent store, so that the copy of the resampling and the load of the sweep
// are one pass.
template <int L, bool INT8>
__device__ __forceinline__ const uint8_t* replica_in(const SweepArgs& a, uint32_t j)
{
    if (a.parent) return a.src + (size_t)a.parent[j] * replica_bytes<L, INT8>();
    return a.spin + (size_t)j * replica_bytes<L, INT8>();
}

// Load the colour-0 / colour-1 words of word index v of the replica at rep.
template <int L, bool INT8>
__device__ __forceinline__ void load_word(const uint8_t* rep, uint32_t v, uint32_t& w0, uint32_t& w1)
{
    using Gm = Geo<L>;
    if constexpr (INT8) {
        const uint4* base = reinterpret_cast<const uint4*>(rep);
        uint32_t ev, od;
        pack64(base + 4 * v, ev, od);
        const uint32_t em = even_row_mask<L>(v);
        w0 = (ev & em) | (od & ~em);
        w1 = (od & em) | (ev & ~em);
    } else {
        const uint32_t* base = reinterpret_cast<const uint32_t*>(rep);
        w0 = base[v];
        w1 = base[Gm::NW + v];
    }
}

template <int L, bool INT8>
__device__ __forceinline__ void store_word(const SweepArgs& a, uint32_t j, uint32_t v, uint32_t w0, uint32_t w1)
{
    using Gm = Geo<L>;
    if constexpr (INT8) {
        uint4* base = reinterpret_cast<uint4*>(a.spin + (size_t)j * Gm::N);
        const uint32_t em = even_row_mask<L>(v);
        unpack64((w0 & em) | (w1 & ~em), (w1 & em) | (w0 & ~em), base + 4 * v);
    } else {
        uint32_t* base = reinterpret_cast<uint32_t*>(a.spin + (size_t)j * Gm::BITS_BYTES);
        base[v] = w0;
        base[Gm::NW + v] = w1;
    }
}

// Stores the words of a wave's replicas in the int8 store (register path, G = NW
// lanes to a replica), 16 bytes per lane and access: access i of lane l covers
// the l-th 16 sites of the i-th quarter of the wave's 64 words, so that 64 lanes
// write 1024 consecutive bytes of a replica (of four, for L = 16).  One exchange
// brings word 16 i + l / 4 to the lane of its quad with l mod 4 = i, and the quad
// shares it from there.  Bound by memory in launches of few sweeps, where the
// partial lines of a lane writing the 64 bytes of its own word cost most.  In us,
// every lane its own word and so: one sweep of L = 32, R = 100000 48.3, 36.3;
// L = 64, R = 50000 83.3, 64.3; L = 16, R = 400000 47.8, 37.0; 20 sweeps of
// L = 32, R = 12000 48.1, 48.1.  The load keeps a word per lane: in this order
// it took 41 us where that took 36 (L = 32, R = 100000), as the words of a launch
// then arrive all at once, and its waves store all at once.
template <int L>
__device__ __forceinline__ void store_wave_int8(const SweepArgs& a, int wave, int lane, uint32_t v, uint32_t w0,
                                                uint32_t w1)
{
    const uint32_t em = even_row_mask<L>(v);
    const int from = 16 * (lane & 3) + (lane >> 2);  // the word this lane keeps
    const uint32_t ev = (uint32_t)__shfl((int)((w0 & em) | (w1 & ~em)), from);
    const uint32_t od = (uint32_t)__shfl((int)((w1 & em) | (w0 & ~em)), from);
    const uint32_t e[4] = {quad_lane<0>(ev), quad_lane<1>(ev), quad_lane<2>(ev), quad_lane<3>(ev)};
    const uint32_t o[4] = {quad_lane<0>(od), quad_lane<1>(od), quad_lane<2>(od), quad_lane<3>(od)};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        constexpr int CH = Geo<L>::N / 16;  // 16-byte chunks of a replica
        const int c = 64 * i + lane, j = wave * Geo<L>::REPW + c / CH;
        const uint4 q = unpack16(byte_pair(e[i], o[i], (uint32_t)lane & 3u));
        if (j < a.n_rep) reinterpret_cast<uint4*>(a.spin + (size_t)j * Geo<L>::N)[c % CH] = q;
    }
}

// Epilogue of a sweep launched with a.acc: the wave's replicas (E, M on the
// first lane of each valid group) are added to the population statistics,
// slot and histogram copy chosen by the wave's index.  The moment sums are
// summed over the wave first, so one lane issues one atomic per quantity; the
// energies go to the histogram copy with one atomic per distinct bin of the
// wave.  Integer sums, so the result does not depend on the order in which
// waves finish.  Called by every lane of the wave.
template <int L>
__device__ __forceinline__ void accumulate_stats(const SweepArgs& a, const LaneInfo& li, int32_t e, int32_t m)
{
    using Gm = Geo<L>;
    const bool lead = li.valid && li.gl == 0;
    uint64_t sE = 0, sE2 = 0, sA = 0, sM2 = 0, q_lo = 0, q_hi = 0;
    int32_t emin = 0x7FFFFFFF, emax = (int32_t)0x80000000;
    int b = 0;
    if (lead) {
        const int64_t e64 = e;
        const uint64_t am = (uint64_t)(m < 0 ? -(int64_t)m : (int64_t)m);
        const uint64_t m2 = am * am;                 // <= 2^32
        const uint64_t p_lo = m2 * m2, p_hi = __umul64hi(m2, m2);  // M^4 <= 2^64
        sE = (uint64_t)e64;
        sE2 = (uint64_t)(e64 * e64);
        sA = am;
        sM2 = m2;
        q_lo = p_lo & 0xFFFFFFFFull;
        q_hi = (p_lo >> 32) | (p_hi << 32);
        emin = emax = e;
        b = (e + 2 * Gm::N) >> 2;  // in [0, N] for |E| <= 2N
    }
    if constexpr (Gm::REPW > 1) {
#pragma unroll
        for (int off = 32; off >= Gm::G; off >>= 1) {
            sE += __shfl_xor(sE, off);
            sE2 += __shfl_xor(sE2, off);
            sA += __shfl_xor(sA, off);
            sM2 += __shfl_xor(sM2, off);
            q_lo += __shfl_xor(q_lo, off);
            q_hi += __shfl_xor(q_hi, off);
            emin = min(emin, __shfl_xor(emin, off));
            emax = max(emax, __shfl_xor(emax, off));
        }
    }
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(li.j / (uint32_t)Gm::REPW));
    if (li.lane == 0 && __builtin_amdgcn_readfirstlane((int)(emin <= emax))) {
        AccSlot* s = a.acc + (w % (uint32_t)kAccSlots);
        atomicAdd((unsigned long long*)&s->sumE, (unsigned long long)sE);
        atomicAdd((unsigned long long*)&s->sumE2, (unsigned long long)sE2);
        atomicAdd((unsigned long long*)&s->sumAbsM, (unsigned long long)sA);
        atomicAdd((unsigned long long*)&s->sumM2, (unsigned long long)sM2);
        atomicAdd((unsigned long long*)&s->m4lo, (unsigned long long)q_lo);
        atomicAdd((unsigned long long*)&s->m4hi, (unsigned long long)q_hi);
        atomicMin(&s->emin, emin);
        atomicMax(&s->emax, emax);
    }
    uint32_t* h = a.acc_hist + (size_t)(w % (uint32_t)kAccHists) * (size_t)a.nbins;
    if constexpr (Gm::REPW == 1) {
        if (li.lane == 0 && lead) atomicAdd(&h[b], 1u);
    } else {
        uint64_t pending = __ballot(lead);
        while (pending) {
            const int leader = __builtin_ctzll(pending);
            const int bv = __builtin_amdgcn_readlane(b, leader);
            const uint64_t same = __ballot(lead && b == bv);
            if (li.lane == leader) atomicAdd(&h[bv], (uint32_t)__popcll(same));
            pending &= ~same;
        }
    }
}

// E = 2 (anti-aligned bonds) - 2N and M = N - 2 (down spins), written by the
// first lane of the replica's group; with a.acc the epilogue above follows.
template <int L>
__device__ __forceinline__ void write_EM(const SweepArgs& a, const LaneInfo& li, uint32_t anti, uint32_t downs)
{
    using Gm = Geo<L>;
#pragma unroll
    for (int off = Gm::G / 2; off >= 1; off >>= 1) {
        anti += (uint32_t)__shfl_xor((int)anti, off);
        downs += (uint32_t)__shfl_xor((int)downs, off);
    }
    const int32_t e = 2 * (int32_t)anti - 2 * Gm::N, m = Gm::N - 2 * (int32_t)downs;
    if (li.valid && li.gl == 0) {
        a.E[li.j] = e;
        a.M[li.j] = m;
    }
    if (a.acc) accumulate_stats<L>(a, li, e, m);
}

// Priority of a wave among those of its SIMD: lower the further its sweeps have
// come.  Left to itself the SIMD issues from its oldest waves first, so these
// finish early and the last ones run with too few others to hide their
// latency: with every wave resident from the start, 7.8 of them per SIMD, L = 64
// ran at 0.7 of the rate that a long queue of waves reaches.  Three steps keep the
// waves of a SIMD together.  Where all waves fit the GPU at once (one_round)
// the steps lie late, so that what remains after the last is short; where
// waves queue for a place they lie early, as waves that end together leave
// their SIMD to a last round that starts together and may be thin.  Launches
// in ms without the priorities, with steps at 1/2, 1/4 and 1/8 of the sweeps
// left, and at 3/4, 1/2 and 1/4: L = 16, R = 80000, theta = 100: 0.329, 0.271,
// 0.283; L = 256, R = 3800, theta = 50: 1.57, 1.34, 1.39; L = 64, theta = 100,
// R = 8000: 0.475, 0.413, 0.422; queueing: L = 128, R = 50000, theta = 20:
// 1.61, 1.60, 1.57; R = 10000, theta = 50: 0.897, 0.856, 0.845; L = 64,
// R = 100000, theta = 40: 1.753, 1.789, 1.749.  (Waves that each took several
// replicas in turn, as many as fit, lost 22 % there: the oldest wave of each
// SIMD ran through all of its own first.)
template <bool ON>
struct Progress {
    int l2, l1, l0;  // sweeps left at which it steps down
    __device__ __forceinline__ Progress(int n, bool one_round)
        : l2(one_round ? n / 2 : 3 * n / 4), l1(one_round ? n / 4 : n / 2), l0(one_round ? n / 8 : n / 4)
    {
        if constexpr (ON) __builtin_amdgcn_s_setprio(3);
    }
    __device__ __forceinline__ void left(int n) const
    {
        if constexpr (!ON) return;
        if (n == l2) __builtin_amdgcn_s_setprio(2);
        if (n == l1) __builtin_amdgcn_s_setprio(1);
        if (n == l0) __builtin_amdgcn_s_setprio(0);
    }
};

// Energies, magnetisations and spins of a wave after its sweeps (register path).
template <int L, bool INT8>
__device__ __forceinline__ void write_regs(const SweepArgs& a, int wave, const LaneInfo& li, const uint32_t (&s0)[1],
                                           const uint32_t (&s1)[1])
{
    const uint32_t v = (uint32_t)li.gl;
    const Neighbours<L, 0> nb(s1, li.lane, li.gl);
    const Nb n = nb.get(s1, 0);
    const uint32_t anti = __popc(s0[0] ^ n.up) + __popc(s0[0] ^ n.dn) + __popc(s0[0] ^ n.same) + __popc(s0[0] ^ n.side);
    const uint32_t downs = __popc(s0[0]) + __popc(s1[0]);
    write_EM<L>(a, li, anti, downs);
    if constexpr (INT8)
        store_wave_int8<L>(a, wave, li.lane, v, s0[0], s1[0]);
    else if (li.valid)
        store_word<L, INT8>(a, li.j, v, s0[0], s1[0]);
}

// Register-resident sweep: each lane owns one word per colour (L <= 64).
// LCG: the in-line LCG variant; the word's seeds for both colours of a sweep
// come from one Philox block (outputs x and y).
template <int L, bool INT8, bool HB, bool LCG, bool PRIO>
__device__ __forceinline__ void sweep_regs(const SweepArgs& a, int wave, const LaneInfo& li,
                                           const Progress<PRIO>& progress)
{
    using Gm = Geo<L>;
    static_assert(Gm::K == 1, "one word per lane");
    const uint32_t v = (uint32_t)li.gl;
    uint32_t s0[1], s1[1];
    if (a.init) {
        s0[0] = init_word<L>(0, v, li.j, a);
        s1[0] = init_word<L>(1, v, li.j, a);
    } else if (li.valid) {
        load_word<L, INT8>(replica_in<L, INT8>(a, li.j), v, s0[0], s1[0]);
    } else {
        s0[0] = s1[0] = 0u;
    }
    const PhiloxKeys K = philox_keys(a.key0, a.key1);
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint32_t g = a.g0 + (uint32_t)t;
        progress.left(a.nsweeps - t);
        if constexpr (LCG) {
            const U4 P = philox10(v, g, li.j, a.tag | kStreamLcgSeed, a.key0, a.key1);
            half_sweep_lcg<L, 0, !PRIO>(s0, s1, li.lane, li.gl, P.x, a);
            half_sweep_lcg<L, 1, !PRIO>(s1, s0, li.lane, li.gl, P.y, a);
        } else {
            half_sweep<L, 0, HB>(s0, s1, li.lane, li.gl, g, li.j, a, K);
            half_sweep<L, 1, HB>(s1, s0, li.lane, li.gl, g, li.j, a, K);
        }
    }
    // the replica's number and its addresses are taken from the thread's number
    // again where a wave holds several replicas or the store is int8: kept through
    // the sweeps they need more registers than eight waves leave, and went to
    // scratch memory.  The bit store of L = 64 keeps them: taken again there they
    // fit as well, but the loop came out slower (100 sweeps, R = 20000: heat bath
    // 1003 us against 987, LCG 1438 against 1424)
    if constexpr (Gm::REPW > 1 || INT8) {
        uint32_t thread = threadIdx.x;
        __asm__("" : "+v"(thread));
        write_regs<L, INT8>(a, wave, lane_info<L>(a, wave, thread), s0, s1);
    } else {
        write_regs<L, INT8>(a, wave, li, s0, s1);
    }
}

// Sweep of a launch of few waves (L = 16 and 32): four lanes share a word, each
// with one of its four Philox blocks, so with four of the 16 planes.  A wave that
// has its SIMD to itself issues about one instruction in ten cycles whatever
// they are, so its time is its number of instructions: a quarter of the
// Philox rounds and of the planes per lane, the planes compared with the lane's
// own threshold bits (masks) instead of a branch per plane.  The lane's four
// planes give the sites below (lt) and equal to (eq) the threshold there, which
// are then joined over the quad, high planes first.  The results are those of
// sweep_regs.  L = 16, R = 1000, ten sweeps: 19.8 -> 7.9 us.
struct QuadPlanes {
    uint32_t m2[4], m4[4];  // the lane's four bits of T_2 and T_4 as masks
    __device__ __forceinline__ QuadPlanes(const SweepArgs& a, int kk)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int bit = 15 - (4 * kk + q);
            m2[q] = 0u - ((a.t2h >> bit) & 1u);
            m4[q] = 0u - ((a.t4h >> bit) & 1u);
        }
    }
};

// Word w of colour C after its half sweep.
template <int C, bool HB>
__device__ __forceinline__ uint32_t quad_word(uint32_t w, const Nb& n, int lane, uint32_t v, uint32_t g, uint32_t j,
                                              const SweepArgs& a, const PhiloxKeys& K, const QuadPlanes& T)
{
    const HalfBlocks blk{philox_half(2u * g + (uint32_t)C, j, a.key0), a.key0, a.key1, K};
    const U4 P = blk(4u * v + (uint32_t)(lane & 3), a.tag | kStreamSweepHigh);
    uint32_t x[4] = {P.x, P.y, P.z, P.w};
    uint32_t cls1, neg = 0u, zero = 0u, sure = 0u;
    if constexpr (HB) {
        const HbClass c = hb_classes(w, n);
        cls1 = c.cls1;
        neg = c.neg;
        zero = c.zero;
        sure = zero & ~quad_lane<0>(x[0]);  // U_0 = 2^31: x < U_0 iff its top bit is 0
    } else {
        const uint32_t d1 = w ^ n.up, d2 = w ^ n.dn, d3 = w ^ n.same, d4 = w ^ n.side;
        const uint32_t o12 = d1 | d2, a12 = d1 & d2, o34 = d3 | d4, a34 = d3 & d4;
        const uint32_t any = o12 | o34;
        sure = a12 | a34 | (o12 & o34);
        cls1 = any & ~sure;
        if (a.t2h > 0xFFFFu) sure |= cls1;  // a threshold of 2^32 (beta ~ 0): always accepted
        if (a.t4h > 0xFFFFu) sure |= ~any;
    }
    uint32_t lt = 0u, eq = 0xFFFFFFFFu;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t t = (cls1 & T.m2[q]) | (~cls1 & T.m4[q]);
        const uint32_t y = HB ? x[q] ^ neg : x[q];
        lt |= eq & t & ~y;
        eq &= ~(t ^ y);
    }
    const uint32_t e0 = quad_lane<0>(eq), e1 = quad_lane<1>(eq), e2 = quad_lane<2>(eq), e3 = quad_lane<3>(eq);
    const uint32_t l0 = quad_lane<0>(lt), l1 = quad_lane<1>(lt), l2 = quad_lane<2>(lt), l3 = quad_lane<3>(lt);
    const uint32_t below = l0 | (e0 & (l1 | (e1 & (l2 | (e2 & l3)))));
    uint32_t acc = sure | (below & ~zero);
    uint32_t tie = e0 & e1 & e2 & e3 & ~(sure | zero);
    while (tie) {  // as in accept_mask and heatbath_mask, the same on the four lanes
        const int b = __builtin_ctz(tie);
        tie &= tie - 1u;
        const uint32_t q = 32u * v + (uint32_t)b;
        const U4 Q = blk(q >> 3, a.tag | kStreamSweepLow);
        const uint32_t word = pick(Q, (q >> 1) & 3u);
        uint32_t lo = (q & 1u) ? (word & 0xFFFFu) : (word >> 16);
        if ((neg >> b) & 1u) lo ^= 0xFFFFu;
        const uint32_t tl = ((cls1 >> b) & 1u) ? a.t2l : a.t4l;
        if (lo < tl) acc |= 1u << b;
    }
    return w ^ acc ^ neg;
}

template <int L, int C, bool HB>
__device__ __forceinline__ void half_sweep_quads(uint32_t (&own)[1], const uint32_t (&oth)[1], int lane, uint32_t v,
                                                 uint32_t g, uint32_t j, const SweepArgs& a, const PhiloxKeys& K,
                                                 const QuadPlanes& T)
{
    const Neighbours<L, C, 4> nb(oth, lane, 0);
    own[0] = quad_word<C, HB>(own[0], nb.get(oth, 0), lane, v, g, j, a, K, T);
}

// Replicas of a wave of sweep_quads.
template <int L>
constexpr int quad_replicas()
{
    return 16 / Geo<L>::NW;
}

template <int L, bool INT8, bool HB>
__device__ __forceinline__ void sweep_quads(const SweepArgs& a, int wave)
{
    using Gm = Geo<L>;
    static_assert(Gm::K == 1 && Gm::NW <= 16 && !Gm::WIDE, "a replica's words fit a quarter of a wave");
    constexpr int QG = 4 * Gm::NW;  // lanes of a replica
    const int lane = (int)(threadIdx.x & 63u), kk = lane & 3;
    const uint32_t v = (uint32_t)((lane % QG) >> 2);
    const uint32_t j = (uint32_t)(wave * quad_replicas<L>() + lane / QG);
    const bool valid = (int)j < a.n_rep;
    uint32_t s0[1] = {0u}, s1[1] = {0u};
    if (valid) load_word<L, INT8>(replica_in<L, INT8>(a, j), v, s0[0], s1[0]);
    const PhiloxKeys K = philox_keys(a.key0, a.key1);
    const QuadPlanes T(a, kk);
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint32_t g = a.g0 + (uint32_t)t;
        half_sweep_quads<L, 0, HB>(s0, s1, lane, v, g, j, a, K, T);
        half_sweep_quads<L, 1, HB>(s1, s0, lane, v, g, j, a, K, T);
    }
    const Neighbours<L, 0, 4> nb(s1, lane, 0);
    const Nb n = nb.get(s1, 0);
    uint32_t anti = __popc(s0[0] ^ n.up) + __popc(s0[0] ^ n.dn) + __popc(s0[0] ^ n.same) + __popc(s0[0] ^ n.side);
    uint32_t downs = __popc(s0[0]) + __popc(s1[0]);
#pragma unroll
    for (int off = QG / 2; off >= 4; off >>= 1) {  // over the words; the lanes of a quad hold the same
        anti += (uint32_t)__shfl_xor((int)anti, off);
        downs += (uint32_t)__shfl_xor((int)downs, off);
    }
    if (!valid || kk != 0) return;
    store_word<L, INT8>(a, j, v, s0[0], s1[0]);
    if (v == 0u) {
        a.E[j] = 2 * (int32_t)anti - 2 * Gm::N;
        a.M[j] = Gm::N - 2 * (int32_t)downs;
    }
}

// Adds the per-lane counts of the W waves of a replica in lanes of the first
// wave, whose lane i < W returns with the sum of wave i; false in the others.
// red: W pairs of LDS words that nothing else uses any more.
template <int W>
__device__ __forceinline__ bool first_wave_sums(uint32_t* red, int lane, int wv, uint32_t& anti, uint32_t& downs)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        anti += (uint32_t)__shfl_xor((int)anti, off);
        downs += (uint32_t)__shfl_xor((int)downs, off);
    }
    if (lane == 0) {
        red[2 * wv] = anti;
        red[2 * wv + 1] = downs;
    }
    __syncthreads();
    anti = (lane < W) ? red[2 * lane] : 0u;
    downs = (lane < W) ? red[2 * lane + 1] : 0u;
    return wv == 0;
}

// The same for L = 64, whose 64 words take the four waves of a block: the words
// stand in LDS too (lds: [2][64]), where their vertical neighbours are read; the
// waves meet once per half sweep.
template <int C>
__device__ __forceinline__ Nb row_neighbours64(const uint32_t* oth, uint32_t v)
{
    Nb n;
    n.same = oth[v];
    n.up = oth[(v + 63u) & 63u];
    n.dn = oth[(v + 1u) & 63u];
    // (y + C) even: horizontal neighbour at h-1, else at h+1
    n.side = __builtin_amdgcn_alignbit(n.same, n.same, (((v + (uint32_t)C) & 1u) == 0u) ? 31u : 1u);
    return n;
}

template <bool INT8, bool HB>
__device__ __forceinline__ void sweep_quads64(const SweepArgs& a, uint32_t j, uint32_t* lds)
{
    const int lane = (int)(threadIdx.x & 63u), kk = lane & 3;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t v = threadIdx.x >> 2;
    uint32_t* c0 = lds;
    uint32_t* c1 = lds + 64;
    uint32_t w0, w1;
    load_word<64, INT8>(replica_in<64, INT8>(a, j), v, w0, w1);
    if (kk == 0) {
        c0[v] = w0;
        c1[v] = w1;
    }
    const PhiloxKeys K = philox_keys(a.key0, a.key1);
    const QuadPlanes T(a, kk);
    __syncthreads();
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint32_t g = a.g0 + (uint32_t)t;
        w0 = quad_word<0, HB>(w0, row_neighbours64<0>(c1, v), lane, v, g, j, a, K, T);
        if (kk == 0) c0[v] = w0;
        __syncthreads();
        w1 = quad_word<1, HB>(w1, row_neighbours64<1>(c0, v), lane, v, g, j, a, K, T);
        if (kk == 0) c1[v] = w1;
        __syncthreads();
    }
    const Nb n = row_neighbours64<0>(c1, v);
    uint32_t anti = __popc(w0 ^ n.up) + __popc(w0 ^ n.dn) + __popc(w0 ^ n.same) + __popc(w0 ^ n.side);
    uint32_t downs = __popc(w0) + __popc(w1);
    if (kk == 0) {
        store_word<64, INT8>(a, j, v, w0, w1);
    } else {
        anti = downs = 0u;
    }
    if (!first_wave_sums<4>(lds + 128, lane, wv, anti, downs)) return;
    LaneInfo li;
    li.lane = li.gl = lane;
    li.j = j;
    li.valid = true;
    write_EM<64>(a, li, anti, downs);
}

// LDS-resident sweep for rows of whole words (L >= 128): one wave owns one
// replica; word (k, lane) of a colour sits at k * 64 + lane, so the 64 lanes
// touch 64 consecutive words for every k.
template <int L>
struct LdsRep {
    using Gm = Geo<L>;
    static constexpr int K = Gm::K, WPR = Gm::WPR, RL = Gm::RL;
    uint32_t* w;  // [2][NW]
    __device__ __forceinline__ uint32_t& at(int c, int k, int gl) const { return w[c * Gm::NW + k * 64 + gl]; }
    // neighbour words (other colour 1 - C) of own word k of lane gl
    template <int C>
    __device__ __forceinline__ Nb nb(int k, int gl) const
    {
        constexpr int O = 1 - C;
        const int r = k / WPR, t = k - (k / WPR) * WPR;
        Nb n;
        n.same = at(O, k, gl);
        n.up = (r > 0) ? at(O, k - WPR, gl) : at(O, (RL - 1) * WPR + t, (gl + 63) & 63);
        n.dn = (r < RL - 1) ? at(O, k + WPR, gl) : at(O, t, (gl + 1) & 63);
        if (((r + C) & 1) == 0) {  // RL is even: row parity is the parity of r
            const int tp = (t == 0) ? WPR - 1 : t - 1;
            n.side = __builtin_amdgcn_alignbit(n.same, at(O, r * WPR + tp, gl), 31);
        } else {
            const int tn = (t == WPR - 1) ? 0 : t + 1;
            n.side = __builtin_amdgcn_alignbit(at(O, r * WPR + tn, gl), n.same, 1);
        }
        return n;
    }
};

// Orders the LDS accesses of the W waves that share a replica.
template <int W>
__device__ __forceinline__ void replica_lds_sync()
{
    if constexpr (W == 1)
        wave_lds_sync();
    else
        __syncthreads();
}

// One colour of a sweep on the LDS path: the lane's K words in chunks of
// SLOTS, each chunk followed by the wave's tie resolution.  With W waves to the
// replica, wave wv takes words [wv K / W, (wv + 1) K / W) of every lane.
template <int L, int C, bool HB, int W>
__device__ __forceinline__ void half_sweep_lds(const LdsRep<L>& rep, int gl, int wv, uint32_t g, uint32_t j,
                                               const SweepArgs& a, const PhiloxKeys& K, uint32_t* queue)
{
    using Gm = Geo<L>;
    constexpr int KW = Gm::K / W;
    constexpr int S = KW < Gm::SLOTS ? KW : Gm::SLOTS;
    constexpr int NG = S < 4 ? S : 4;  // groups of four words share the branches of decide8_group
    static_assert(Gm::K % W == 0 && KW % S == 0 && S % NG == 0, "slots divide the words of a lane");
    const PhiloxHalf h = philox_half(2u * g + (uint32_t)C, j, a.key0);
    const int kbase = W == 1 ? 0 : wv * KW;
#pragma unroll 1
    for (int k0 = kbase; k0 < kbase + KW; k0 += S) {
        uint32_t nq = 0u;
#pragma unroll
        for (int s0 = 0; s0 < S; s0 += NG) {
            uint32_t w[NG], tie[NG], cls1[NG], ng[NG], id[NG];
            Nb n[NG];
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                n[i] = rep.template nb<C>(k0 + s0 + i, gl);
                w[i] = rep.at(C, k0 + s0 + i, gl);
                id[i] = (uint32_t)((k0 + s0 + i) * 64 + gl);  // the word's place in the LDS replica
            }
            const auto blk = [&](int i, uint32_t kk) {
                return philox10_h(4u * (uint32_t)(gl * Gm::K + k0 + s0 + i) + kk, a.tag | kStreamSweepHigh, h,
                                  a.key0, a.key1, K);
            };
            decide8_group<NG, HB>(w, n, blk, a, tie, cls1, ng);
#pragma unroll
            for (int i = 0; i < NG; ++i) rep.at(C, k0 + s0 + i, gl) = w[i];
            const auto own = [&](int i, uint32_t t, uint32_t c, uint32_t m) {
                rep.at(C, k0 + s0 + i, gl) ^=
                    decide_word_tail<HB>((uint32_t)(gl * Gm::K + k0 + s0 + i), t, c, m, h, a, K);
            };
            if constexpr (KW == 1) {
                if (tie[0]) own(0, tie[0], cls1[0], ng[0]);
            } else {
                queue_ties<NG>(tie, cls1, ng, id, a, queue, nq, own);
            }
        }
        if (nq == 0u) continue;
        const auto half = [&](uint32_t w, uint32_t* v) {
            *v = (w & 63u) * (uint32_t)Gm::K + (w >> 6);
            return h;
        };
        const auto apply = [&](uint32_t w, uint32_t f) {
            if (f) atomicXor(&rep.w[C * Gm::NW + w], f);
        };
        resolve_ties<HB>(nq, a, K, queue, gl, half, apply);
    }
    replica_lds_sync<W>();
}

// One colour of an LCG sweep on the LDS path: every word of the lane in turn,
// its seed from the word's Philox block of this sweep (x: colour 0, y:
// colour 1).  The uniforms are whole 32-bit numbers, so there are no ties.
template <int L, int C, bool PAIRS>
__device__ __forceinline__ void half_sweep_lds_lcg(const LdsRep<L>& rep, int gl, uint32_t g, uint32_t j,
                                                   const SweepArgs& a)
{
    using Gm = Geo<L>;
#pragma unroll 1
    for (int k = 0; k < Gm::K; ++k) {
        const Nb n = rep.template nb<C>(k, gl);
        const uint32_t w = rep.at(C, k, gl);
        const U4 P = philox10u((uint32_t)(gl * Gm::K + k), g, j, a.tag | kStreamLcgSeed, a.key0, a.key1);
        rep.at(C, k, gl) = w ^ lcg_accept_mask<PAIRS>(w, n, C == 0 ? P.x : P.y, a);
    }
    wave_lds_sync();
}

// The LDS of the W waves of a replica: the replica [2][NW], then W tie queues.
template <int L, bool INT8, bool HB, bool LCG, bool PRIO, int W = 1>
__device__ __forceinline__ void sweep_lds(const SweepArgs& a, uint32_t j, uint32_t* lds, int wv = 0)
{
    static_assert(W == 1 || !LCG, "the LCG variant has one wave per replica");
    using Gm = Geo<L>;
    static_assert(Gm::WIDE && Gm::RL % 2 == 0 && Gm::G == 64, "LDS path layout");
    const Progress<PRIO> progress(a.nsweeps, a.one_round != 0);
    const LdsRep<L> rep{lds};
    uint32_t* queue = lds + 2 * Gm::NW + wv * kTieQueueWords;
    const int gl = (int)(threadIdx.x & 63u);
    const uint8_t* in = a.init ? nullptr : replica_in<L, INT8>(a, j);
    constexpr int KW = Gm::K / W;
    const int kbase = W == 1 ? 0 : wv * KW;
#pragma unroll 1
    for (int k = kbase; k < kbase + KW; ++k) {
        const uint32_t v = (uint32_t)(gl * Gm::K + k);
        uint32_t w0, w1;
        if (a.init) {
            w0 = init_word<L>(0, v, j, a);
            w1 = init_word<L>(1, v, j, a);
        } else {
            load_word<L, INT8>(in, v, w0, w1);
        }
        rep.at(0, k, gl) = w0;
        rep.at(1, k, gl) = w1;
    }
    replica_lds_sync<W>();
    const PhiloxKeys K = philox_keys(a.key0, a.key1);
    for (int t = 0; t < a.nsweeps; ++t) {
        const uint32_t g = a.g0 + (uint32_t)t;
        progress.left(a.nsweeps - t);
        if constexpr (LCG) {
            half_sweep_lds_lcg<L, 0, !PRIO>(rep, gl, g, j, a);
            half_sweep_lds_lcg<L, 1, !PRIO>(rep, gl, g, j, a);
        } else {
            half_sweep_lds<L, 0, HB, W>(rep, gl, wv, g, j, a, K, queue);
            half_sweep_lds<L, 1, HB, W>(rep, gl, wv, g, j, a, K, queue);
        }
    }
    uint32_t anti = 0, downs = 0;
#pragma unroll 1
    for (int k = kbase; k < kbase + KW; ++k) {
        const Nb n = rep.template nb<0>(k, gl);
        const uint32_t w0 = rep.at(0, k, gl), w1 = rep.at(1, k, gl);
        anti += __popc(w0 ^ n.up) + __popc(w0 ^ n.dn) + __popc(w0 ^ n.same) + __popc(w0 ^ n.side);
        downs += __popc(w0) + __popc(w1);
        store_word<L, INT8>(a, j, (uint32_t)(gl * Gm::K + k), w0, w1);
    }
    if constexpr (W > 1) {
        if (!first_wave_sums<W>(lds + 2 * Gm::NW, gl, wv, anti, downs)) return;
    }
    LaneInfo li;
    li.lane = gl;
    li.gl = gl;
    li.j = j;
    li.valid = true;
    write_EM<L>(a, li, anti, downs);
}

// Minimum waves per SIMD the sweep kernels are compiled for.  At L = 128 the
// grouped decision with the round keys in vector registers needs two registers
// more than fit four waves per SIMD; holding the kernel to four (two values go
// to scratch outside the inner loops) takes 1.59 ms per launch at R = 50000,
// theta = 20, against 1.78 with three waves (2.10 before the keys, the tail by
// planes and the plane block).  The register path fits eight without
// scratch memory; at 65 to 68 registers it held seven, so that 7500 waves no
// longer fitted at once (seven and eight waves, and now: L = 32, R = 30000, theta =
// 50: 0.258, 0.221, 0.217 ms in the int8 store, 0.269, 0.236, 0.215 with the
// heat bath; L = 64, R = 7777, theta = 20, heat bath: 0.124, 0.106, 0.092).
// The batch's kernel over several lattice sizes fits eight without being held to
// them (64 registers; seven for the LCG update, by its scalar registers): held,
// steps of 4 and 16 runs of one or three sizes took within 5 % of the same time.
template <int L>
constexpr int sweep_min_waves()
{
    return L == 128 ? 4 : (L >= 16 && L <= 64) ? 8 : 1;
}

// Waves of a sweep that the GPU holds at once: 256 CUs of 4 SIMDs, each with 8
// waves of the register path or 4 of the LDS path.
template <int L>
constexpr int sweep_resident_waves()
{
    return 1024 * (Geo<L>::K == 1 ? 8 : 4);
}

// Threads per block of the single-run sweep kernel.
template <int L>
constexpr int sweep_block()
{
    return Geo<L>::K == 1 ? kBlock : 64;
}

// Sweep entry shared by the single-run and batched kernels, for the block
// holding waves [wave0, wave0 + wpb) of a run (wpb = blockDim.x / 64); lds is
// the block's Geo<L>::lds_words(wpb) words (none on the register path).
// Waves share no barrier: each returns as soon as it holds no replica.  HB
// selects the heat-bath update instead of Metropolis; LCG the in-line LCG
// variant of the Metropolis sweep; PRIO the wave priorities (Progress).
template <int L, bool INT8, bool HB, bool LCG = false, bool PRIO = true>
__device__ __forceinline__ void sweep_waves(const SweepArgs& a, int wave0, uint32_t* lds)
{
    using Gm = Geo<L>;
    const int lane = (int)(threadIdx.x & 63u), wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wave = wave0 + wib;
    if (wave * Gm::RPWV >= a.n_rep) return;  // uniform per wave
    if constexpr (Gm::K == 1) {
        const Progress<PRIO> progress(a.nsweeps, a.one_round != 0);
        const LaneInfo li = lane_info<L>(a, wave, (uint32_t)lane);
        sweep_regs<L, INT8, HB, LCG, PRIO>(a, wave, li, progress);
    } else {
        sweep_lds<L, INT8, HB, LCG, PRIO>(a, (uint32_t)__builtin_amdgcn_readfirstlane(wave),
                                          lds + wib * Gm::WAVE_LDS_WORDS);
    }
}

}  // namespace dev
}  // namespace pa
