// pairsym64.hpp -- the all-pairs ion-ion sum of FP64 systems, each pair once.
//
// The work items and the lane rotation are those of pairsym.hpp, in 64 bits.
// The totals of an ion are two int64 words, the second in units of 2^-38 of
// the first's: exact, so independent of the order of the items, and fine
// enough (2^-60 of a typical sum) that what a flush rounds stays below the
// rounding of the terms.  A flush too large for the words (a pair closer than
// about 1e-4 of the mean spacing) or not finite marks the step, and the step's
// second kernel then sums every pair one-sided instead.
// Bound by FP64 issue: 41 instructions per pair and 3 per direction.  The
// one-sided sum took 48 per ordered pair: 18.0 ms at 100,003 ions against
// 6.4, 1.22 against 0.15 at 12,345 and, in 8 blocks, 0.21 against 0.025 at 2,000.
#pragma once

#include "kernels.hpp"
#include "symitems.hpp"

namespace odk {

// (1 + r) e^-r / r^3 for the difference d.
__device__ __forceinline__ double sym64_f(double dx, double dy, double dz, const double* __restrict__ tab)
{
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const double ri = rsq_f64(r2);
    const double ri2 = ri * ri;
    return fma(ri2, ri, ri2) * exp_neg_tab(r2 * ri, tab);
}

// Lane l receives the value of lane l + 1 (mod 64).
__device__ __forceinline__ double rotate_down64(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned int lo = __builtin_amdgcn_mov_dpp((int)(unsigned int)b, 0x134, 0xf, 0xf, true);
    const unsigned int hi = __builtin_amdgcn_mov_dpp((int)(unsigned int)(b >> 32), 0x134, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

constexpr double kSym64Lo = 274877906944.0;     // 2^38

// Totals of one system: planes [6][stride] (x, y, z high words, then low),
// scale of the high word, the largest flush, and the step after which a flush
// did not fit (0: none did not).
struct Sym64 {
    unsigned long long* fix;
    long long stride;
    double scale, lim;
    long long* bad;         // Ctl::pair_bad
};

__device__ __forceinline__ void sym64_words(double v, const Sym64& s, long long step, unsigned long long* w0,
                                            unsigned long long* w1)
{
    const double a = v * s.scale, h = rint(a);
    if (!(fabs(h) < s.lim)) {                   // NaN too
        *s.bad = step + 1;
        return;
    }
    const long long lo = __double2ll_rn((a - h) * kSym64Lo);
    __hip_atomic_fetch_add(w0, (unsigned long long)(long long)h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(w1, (unsigned long long)lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Sym64Lds {
    double tab[64];
    double src[3][4][128];              // sub-tiles of 64 sources, each stored twice
    unsigned long long j[6][256];       // reactions on the tile's sources
};

// R target tile rows I .. I + R - 1 against the 64-ion sub-tiles [st0, st1) of
// the source tiles [J0, J1); for R == 1 the diagonal tile (J == I) is summed
// one-sided.
template <int R>
__device__ __forceinline__ void sym64_rows(const double* __restrict__ X, const double* __restrict__ Y,
                                           const double* __restrict__ Z, int N, int I, int J0, int J1, int st0,
                                           int st1, const Sym64& s, long long step, Sym64Lds& m)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double xt[R], yt[R], zt[R], ax[R], ay[R], az[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = (I + r) * 256 + threadIdx.x;
        xt[r] = X[i];
        yt[r] = Y[i];
        zt[r] = Z[i];
        ax[r] = ay[r] = az[r] = 0.0;
    }
    for (int J = J0; J < J1; ++J) {
        const int j = J * 256 + threadIdx.x;
        __syncthreads();
        {
            const double q[3] = {X[j], Y[j], Z[j]};
#pragma unroll
            for (int c = 0; c < 3; ++c) m.src[c][wv][lane] = m.src[c][wv][lane + 64] = q[c];
#pragma unroll
            for (int c = 0; c < 6; ++c) m.j[c][threadIdx.x] = 0ull;
        }
        __syncthreads();
        if (R == 1 && J == I) {
            for (int k = 64 * st0; k < 64 * st1; ++k) {
                const double dx = xt[0] - m.src[0][k >> 6][k & 63], dy = yt[0] - m.src[1][k >> 6][k & 63],
                             dz = zt[0] - m.src[2][k >> 6][k & 63];
                double f = sym64_f(dx, dy, dz, m.tab);
                f = k == (int)threadIdx.x ? 0.0 : f;
                ax[0] = fma(f, dx, ax[0]);
                ay[0] = fma(f, dy, ay[0]);
                az[0] = fma(f, dz, az[0]);
            }
            continue;
        }
        for (int st = st0; st < st1; ++st) {
            double jx = 0.0, jy = 0.0, jz = 0.0;
            const double *px = &m.src[0][st][lane], *py = &m.src[1][st][lane], *pz = &m.src[2][st][lane];
#pragma unroll 4
            for (int k = 0; k < 64; ++k) {
                const double qx = px[k], qy = py[k], qz = pz[k];        // source (lane + k) mod 64
                jx = rotate_down64(jx);
                jy = rotate_down64(jy);
                jz = rotate_down64(jz);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double dx = xt[r] - qx, dy = yt[r] - qy, dz = zt[r] - qz;
                    const double f = sym64_f(dx, dy, dz, m.tab);
                    ax[r] = fma(f, dx, ax[r]);
                    ay[r] = fma(f, dy, ay[r]);
                    az[r] = fma(f, dz, az[r]);
                    jx = fma(-f, dx, jx);
                    jy = fma(-f, dy, jy);
                    jz = fma(-f, dz, jz);
                }
            }
            // after 64 rotations lane l holds source (l + 63) mod 64
            const int sid = st * 64 + ((lane + 63) & 63);
            sym64_words(jx, s, step, &m.j[0][sid], &m.j[3][sid]);
            sym64_words(jy, s, step, &m.j[1][sid], &m.j[4][sid]);
            sym64_words(jz, s, step, &m.j[2][sid], &m.j[5][sid]);
        }
        __syncthreads();
        if (j < N && wv >= st0 && wv < st1)
#pragma unroll
            for (int c = 0; c < 6; ++c) atomicAdd(&s.fix[c * s.stride + j], m.j[c][threadIdx.x]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = (I + r) * 256 + threadIdx.x;
        if (i >= N) continue;
        sym64_words(ax[r], s, step, &s.fix[i], &s.fix[3 * s.stride + i]);
        sym64_words(ay[r], s, step, &s.fix[s.stride + i], &s.fix[4 * s.stride + i]);
        sym64_words(az[r], s, step, &s.fix[2 * s.stride + i], &s.fix[5 * s.stride + i]);
    }
}

__global__ __launch_bounds__(256) void pair_sym64_kernel(const double* __restrict__ xs, int Npad, int N,
                                                         const SymItem* __restrict__ items, Sym64 s,
                                                         const Ctl* __restrict__ ctl)
{
    __shared__ Sym64Lds m;
    if (threadIdx.x < 64) m.tab[threadIdx.x] = kExp2Tab[threadIdx.x];
    const SymItem it = items[blockIdx.x];
    const double *X = xs, *Y = xs + Npad, *Z = xs + 2 * (long long)Npad;
    const long long step = ctl->step;
    if (it.rows == 1) {
        sym64_rows<1>(X, Y, Z, N, it.I, it.J0, it.J1, it.st0, it.st1, s, step, m);
        return;
    }
    int J0 = it.J0;
    if (J0 == it.I) {                   // the rows' own tiles
        for (int r = 0; r < kSymRows; ++r)
            sym64_rows<1>(X, Y, Z, N, it.I + r, it.I + r, it.I + kSymRows, 0, 4, s, step, m);
        J0 = it.I + kSymRows;
    }
    if (J0 < it.J1) sym64_rows<kSymRows>(X, Y, Z, N, it.I, J0, it.J1, 0, 4, s, step, m);
}

// FP64 pair terms of one target against a staged tile of TJ sources;
// Self: the tile holds the target itself (source index `self`), whose term
// is dropped.
template <int TJ, bool Self>
__device__ __forceinline__ void f64_tile(const double4* __restrict__ tile, double xi, double yi, double zi,
                                         int self, const double* __restrict__ tab, double& sx, double& sy, double& sz)
{
    for (int k = 0; k < TJ; ++k) {
        const double4 q = tile[k];
        const double dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
        double f = sym64_f(dx, dy, dz, tab);
        if (Self) f = (k == self) ? 0.0 : f;
        sx += f * dx;
        sy += f * dy;
        sz += f * dz;
    }
}

// Per ion: the pair sum from its totals, which are cleared (or summed here
// one-sided, see above, or where the totals' memory was refused: s.fix null),
// the grain terms in FP64, drive and confinement field; the block's share of
// the Eq. (1) sums.
template <int BLOCK, int TJ>
__global__ __launch_bounds__(BLOCK) void pair_forces_f64(const double* __restrict__ xs,
                                                         double* __restrict__ acc,
                                                         PairArgs p, DustSet ds, Sym64 s,
                                                         Ctl* __restrict__ ctl)
{
    static_assert(BLOCK == TJ, "the block's own tile is the one source tile holding its targets");
    __shared__ double tab[64];
    __shared__ double4 tile[TJ];
    __shared__ double red[BLOCK / 64][kMaxDust][3];
    const int Npad = p.Npad;
    const double* X = xs;
    const double* Y = xs + Npad;
    const double* Z = xs + 2 * Npad;
    const int i0 = blockIdx.x * BLOCK;
    const int i = i0 + threadIdx.x;
    const double xi = X[i], yi = Y[i], zi = Z[i];
    double sx = 0.0, sy = 0.0, sz = 0.0;
    const bool one_sided = !s.fix || ctl->pair_bad == ctl->step + 1;
    if (p.ion_ion && !one_sided) {
        double t[3];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            t[c] = from_fixed(s.fix[c * s.stride + i], s.scale) +
                   from_fixed(s.fix[(c + 3) * s.stride + i], s.scale * kSym64Lo);
        sx = t[0];
        sy = t[1];
        sz = t[2];
    } else if (p.ion_ion) {
        if (threadIdx.x < 64) tab[threadIdx.x] = kExp2Tab[threadIdx.x];
        for (int j0 = 0; j0 < Npad; j0 += TJ) {
            __syncthreads();
            for (int t = threadIdx.x; t < TJ; t += BLOCK) {
                double4 q;
                q.x = X[j0 + t]; q.y = Y[j0 + t]; q.z = Z[j0 + t]; q.w = 0.0;
                tile[t] = q;
            }
            __syncthreads();
            if (j0 == i0)      // the block's own tile holds the self-pair
                f64_tile<TJ, true>(tile, xi, yi, zi, threadIdx.x, tab, sx, sy, sz);
            else
                f64_tile<TJ, false>(tile, xi, yi, zi, threadIdx.x, tab, sx, sy, sz);
        }
    }
    if (s.fix)
        for (int c = 0; c < 6; ++c) s.fix[c * s.stride + i] = 0ull;
    const bool live = i < p.N;
    double gx = p.Cd * sx, gy = p.Cd * sy, gz = p.Cd * sz + p.Ez;
    if (p.cf.on) {
        double ex, ey, ez;
        conf_field(p.cf, xi, yi, zi, ex, ey, ez);
        gx += ex; gy += ey; gz += ez;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int d = 0; d < ds.nd; ++d) {
        const double rx = xi - ds.pos[d][0], ry = yi - ds.pos[d][1], rz = zi - ds.pos[d][2];
        const double r2 = rx * rx + ry * ry + rz * rz;
        const double r = sqrt(r2);
        const double ir3 = 1.0 / (r2 * r);
        const double kq = p.Kq * ctl->Q[d] * ir3;
        gx += kq * rx; gy += kq * ry; gz += kq * rz;
        double f = live ? -(1.0 + r) * exp(-r) * ir3 : 0.0;
        double fx = wave_sum(f * rx), fy = wave_sum(f * ry), fz = wave_sum(f * rz);
        if (lane == 0) {
            red[wv][d][0] = fx;
            red[wv][d][1] = fy;
            red[wv][d][2] = fz;
        }
    }
    if (live) {
        acc[i] = gx;
        acc[Npad + i] = gy;
        acc[2 * Npad + i] = gz;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < ds.nd * 3; t += BLOCK) {
        const int d = t / 3, c = t % 3;
        double s = 0.0;
        for (int w = 0; w < BLOCK / 64; ++w) s += red[w][d][c];
        atomicAdd(&ctl->part[blockIdx.x % kSlots][d][c], to_fixed(s, kForceScale, &ctl->status));
    }
}

}  // namespace odk
