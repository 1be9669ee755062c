// device_common.hpp -- shared device helpers of libodust: the counter-based
// generator, uniform and normal draws, fixed-point accumulation and wave
// reductions.  Units inside the kernels are dimensionless: lengths in the
// electron Debye length r_De, times in 1/omega_pi, velocities in
// c_s = r_De omega_pi, charges in e.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace odk {

constexpr int kMaxDust = 32;
constexpr double kPi = 3.14159265358979323846;

// Random-stream purposes (third counter word).
enum : uint64_t { kInitPos = 0, kInitVel = 1, kColl = 2, kReinj = 3 };

// Per-ion event byte.
enum : uint8_t { kEvNone = 0, kEvExit = 1, kEvAbsBase = 2, kEvCollBit = 0x80 };

// Device status bits.
enum : int { kStNaN = 1, kStPlace = 2, kStOverflow = 4 };

// Fixed-point scales of the integer accumulators (two's-complement int64
// sums are associative, so the totals do not depend on the order in which
// blocks add them).
constexpr double kForceScale = 4294967296.0;    // 2^32: Eq. (1) sums, dimensionless
constexpr double kMomScale = 4294967296.0;      // 2^32: absorbed velocity sums, c_s

// Counters that every block adds to are spread over kSlots addresses (slot =
// block index mod kSlots): device-scope atomics on one address serialise, and
// thousands of blocks adding to one word would take tens of microseconds.
// Each slot of a counter has a 128-byte cache line of its own (the memory
// side performs atomics on a line one at a time), so a counter's slots are
// kPad64 (8-byte) or kPad32 (4-byte) words apart.
constexpr int kSlots = 64;
constexpr int kPad64 = 16, kPad32 = 32;

// Layout of one system's control block (device memory, int64/double words).
struct alignas(128) Ctl {
    unsigned long long acc[kMaxDust][8];   // [3] absorbed count, [4..6] sum v ([0..2], [7] unused)
    unsigned long long part[kSlots][kMaxDust][3];  // Eq.(1) sums, per slot (block index mod kSlots)
    unsigned long long n_exit[kSlots][kPad64];     // exits, per slot ([s][0])
    unsigned long long n_coll[kSlots][kPad64];     // collisions, per slot ([s][0])
    unsigned int ticket_slot[kSlots][kPad32];      // tail blocks of the slot that have finished ([s][0])
    unsigned int lost_seg[kSlots * kPad32];        // lost-list segment lengths (single system), [s * kPad32]
    double Q[kMaxDust];                    // charge, e
    double last[kMaxDust][16];             // [0] Q^n, [1..12] F parts (SI), [13] absorbed count
    double sums[kMaxDust][16];             // running sums over recorded steps
    long long step;                        // step counter n
    long long nrec;                        // recorded steps
    long long last_exit, last_coll;
    int status;
    unsigned int ticket;                   // slots of the tail whose blocks have all finished
    unsigned int lost_ticket;              // reinjection blocks that have finished
    int pad[3];
    long long pair_bad;                    // FP64: step + 1 of a pair sum that its words cannot hold
};
static_assert(offsetof(Ctl, n_exit) % 128 == 0 && offsetof(Ctl, n_coll) % 128 == 0 &&
                  offsetof(Ctl, ticket_slot) % 128 == 0 && offsetof(Ctl, lost_seg) % 128 == 0,
              "slot counters start on cache lines");

// ---------------------------------------------------------------------------
// Philox4x64 with 10 rounds (Salmon et al., SC'11): per round two 64x64->128
// products; the words are permuted and the high halves mixed with the key;
// the key advances by two Weyl increments between rounds.
struct U64x4 {
    uint64_t w[4];
};

__host__ __device__ inline void mul128(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo)
{
#if defined(__HIP_DEVICE_COMPILE__)
    lo = a * b;
    hi = __umul64hi(a, b);
#else
    unsigned __int128 p = (unsigned __int128)a * b;
    lo = (uint64_t)p;
    hi = (uint64_t)(p >> 64);
#endif
}

__host__ __device__ inline U64x4 philox(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                        uint64_t k0, uint64_t k1)
{
    const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t h0, l0, h1, l1;
        mul128(M0, c0, h0, l0);
        mul128(M1, c2, h1, l1);
        const uint64_t t0 = h1 ^ c1 ^ k0;
        const uint64_t t2 = h0 ^ c3 ^ k1;
        c0 = t0;
        c1 = l1;
        c2 = t2;
        c3 = l0;
        k0 += W0;
        k1 += W1;
    }
    U64x4 o;
    o.w[0] = c0; o.w[1] = c1; o.w[2] = c2; o.w[3] = c3;
    return o;
}

// Uniform strictly inside (0,1): 52 high bits plus one half, over 2^52.
__host__ __device__ inline double unit(uint64_t w)
{
    return ((double)(w >> 12) + 0.5) * 2.220446049250313080847e-16;
}

// Box-Muller: two standard normals from two uniforms.
__device__ inline void gauss2(double ua, double ub, double& g1, double& g2)
{
    const double m = sqrt(-2.0 * log(ua));
    double s, c;
    sincos(2.0 * kPi * ub, &s, &c);
    g1 = m * c;
    g2 = m * s;
}

// ---------------------------------------------------------------------------
// FP64 pieces of the screened pair term without a division.
//
// 1/sqrt(x), x > 0: the hardware estimate (about 24 correct bits) and one
// third-order Newton-Raphson correction, y (1 + e/2 + 3e^2/8) with
// e = 1 - x y^2 (the series of (1 - e)^(-1/2)), which triples the correct
// bits (measured on gfx950 within 1.3 ulp).
__device__ inline double rsq_f64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// 2^(j / 64), correctly rounded.
__constant__ const double kExp2Tab[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0,
    0x1.0874518759bc8p+0, 0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0,
    0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0, 0x1.172b83c7d517bp+0,
    0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0,
    0x1.2d285a6e4030bp+0, 0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0,
    0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0, 0x1.3dea64c123422p+0,
    0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0,
    0x1.56f4736b527dap+0, 0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0,
    0x1.6247eb03a5585p+0, 0x1.6623882552225p+0, 0x1.6a09e667f3bcdp+0,
    0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0,
    0x1.868d99b4492edp+0, 0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0,
    0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0, 0x1.9c49182a3f090p+0,
    0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0,
    0x1.bcc1e904bc1d2p+0, 0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0,
    0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0, 0x1.d5818dcfba487p+0,
    0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0,
    0x1.fa7c1819e90d8p+0,
};

// e^-r for 0 <= r, clamped at 700 (below 1e-304): r = -(n ln 2) / 64 + f with n
// rounded by adding 1.5 * 2^52, ln 2 / 64 split into a 32-bit head (n * head
// exact) and its remainder, |f| <= ln 2 / 128, 2^(n / 64) from the table (in
// LDS) and its exponent, e^f - 1 to degree 5 (remainder below 4e-17).  The
// method is Tang's (ACM Trans. Math. Software 15, 144, 1989).
__device__ __forceinline__ double exp_neg_tab(double r, const double* __restrict__ tab)
{
    const double magic = 6755399441055744.0;
    const double x = -fmin(r, 700.0);
    const double t = fma(x, 92.33248261689366, magic);
    const double n = t - magic;
    const int k = (int)(unsigned int)__builtin_bit_cast(unsigned long long, t);
    const double f = fma(n, -0x1.62e42fee00000p-7, fma(n, -0x1.a39ef35793c76p-39, x));
    double p = fma(f, 1.0 / 120.0, 1.0 / 24.0);
    p = fma(p, f, 1.0 / 6.0);
    p = fma(p, f, 0.5);
    p = fma(p, f, 1.0);
    const unsigned long long b = __builtin_bit_cast(unsigned long long, tab[k & 63]);
    const int hi = (int)(b >> 32) + ((k & ~63) << 14);
    const double s = __builtin_bit_cast(double, (unsigned long long)(unsigned int)hi << 32 | (unsigned int)b);
    return fma(s * f, p, s);
}

// Arrival number of each active lane's key: count[key]++ for every one of them,
// with one atomic for the lanes of a wave that share a key, as far as shared
// keys are found in the first lanes.  Where most ions fall into few bins, an
// atomic per ion on one address, 12 ns each, is what a sort would take.
__device__ __forceinline__ int arrive(int* __restrict__ count, int key, bool active)
{
    const int lane = threadIdx.x & 63;
    int lead = lane, add = active ? 1 : 0, rank = 0;
    unsigned long long todo = __ballot(active);
    while (todo) {
        const int first = __ffsll(todo) - 1;
        const unsigned long long same = __ballot(active && key == __shfl(key, first, 64)) & todo;
        if (__popcll(same) == 1) break;
        if (same >> lane & 1) {
            lead = first;
            rank = __popcll(same & ((1ull << lane) - 1ull));
            add = lane == first ? __popcll(same) : 0;
        }
        todo &= ~same;
    }
    int at = 0;
    if (add) at = atomicAdd(&count[key], add);
    return __shfl(at, lead, 64) + rank;
}

// How many of v[0 .. n) are below x, with loads in flight.
__device__ __forceinline__ int count_below(const int* __restrict__ v, int n, int x)
{
    int below = 0, k = 0;
    for (; k + 16 <= n; k += 16)
#pragma unroll
        for (int u = 0; u < 16; ++u) below += v[k + u] < x;
    for (; k < n; ++k) below += v[k] < x;
    return below;
}

// ---------------------------------------------------------------------------
// Wave64 sum of a 64-bit value: butterfly over the xor masks 32 and 16, then
// rotations by 8, 4, 2 and 1 within rows of 16 lanes, which after the steps
// before them bring the same values as the masks 8 to 1, without LDS.
template <int ROT>
__device__ inline unsigned long long row_rotate(unsigned long long b)
{
    const unsigned int lo = __builtin_amdgcn_mov_dpp((int)(unsigned int)b, 0x120 + ROT, 0xf, 0xf, true);
    const unsigned int hi = __builtin_amdgcn_mov_dpp((int)(unsigned int)(b >> 32), 0x120 + ROT, 0xf, 0xf, true);
    return (unsigned long long)hi << 32 | lo;
}

template <typename V>
__device__ inline V wave_sum(V v)
{
    static_assert(sizeof(V) == 8, "64-bit values");
    auto rot = [](auto r, V x) {
        return __builtin_bit_cast(V, row_rotate<decltype(r)::value>(__builtin_bit_cast(unsigned long long, x)));
    };
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
    v += rot(std::integral_constant<int, 8>{}, v);
    v += rot(std::integral_constant<int, 4>{}, v);
    v += rot(std::integral_constant<int, 2>{}, v);
    v += rot(std::integral_constant<int, 1>{}, v);
    return v;
}

__device__ inline unsigned long long to_fixed(double v, double scale, int* status)
{
    double s = v * scale;
    const double lim = 4.0e18;
    if (!(s < lim && s > -lim)) {   // also catches NaN
        atomicOr(status, (s != s) ? kStNaN : kStOverflow);
        s = 0.0;
    }
    return (unsigned long long)__double2ll_rn(s);
}

__host__ __device__ inline double from_fixed(unsigned long long v, double scale)
{
    return (double)(long long)v / scale;
}

}  // namespace odk
