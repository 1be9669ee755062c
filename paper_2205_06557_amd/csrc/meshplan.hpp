// meshplan.hpp -- host side: how the ion-ion sum of a large system is split
// into a near part and a smooth far part (kernels: mesh.hpp).  Plain C++.
//
// The screened Coulomb energy e^-r / r is written L(r) + [e^-r / r - L(r)]
// with L a sum of Gaussians,
//   L(r) = sum_m w_m e^(-t_m^2 r^2),   t_m geometric from t_min to 2.8 / r_c,
// whose weights are fitted (least squares on the force) so that L equals the
// screened energy beyond r_c.  The bracket then vanishes beyond r_c and is
// summed over near pairs; L is smooth and is summed over all ions on a
// regular grid: charges spread with a Kaiser-Bessel window of ten nodes per
// axis, each Gaussian applied as three one-dimensional convolutions (a
// Gaussian is a product over the axes) with the window's transform divided
// out, and the potential's gradient taken with the window's derivative.
// With r_c / h = 7.5 cells and window shape 22 the grid adds less than 1e-7 of
// the rms acceleration (2^14 .. 2^20 ions, measured against 64-bit direct
// sums); the fit adds 5e-8 to 2.3e-7, growing with diag / r_c at a given number
// of Gaussians (mesh_plan).
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

namespace odk {

constexpr int kMeshP = 10;          // window nodes per axis
constexpr int kMeshM = 20;          // Gaussians at most ...
constexpr int kMeshMinM = 14;       // ... and at least
constexpr double kMeshFit = 3.2e-6; // |F - F_L| r r_c that a fit may leave beyond r_c
constexpr int kMeshWDeg = 18;       // degree of the window polynomial in 1 - 2 z^2
constexpr int kMeshNearDeg = 12;    // degree of the near part's polynomial in 1 - 2 r^2 / r_c^2
constexpr double kMeshBeta = 22.0;  // Kaiser-Bessel shape
constexpr double kMeshRatio = 7.5;  // r_c / h
constexpr double kMeshTop = 2.8;    // t_max r_c
constexpr int kMeshSub = 8;         // ions per box of the near search
constexpr double kMeshCol = 27.0;   // ions in the unit of volume that r_c is given in
constexpr int kMeshTile = 16;       // ions per group of targets
constexpr int kMeshKx = 4;          // column width in cells
constexpr int kMeshZsub = 2;        // sort bins per cell along z
constexpr int kMeshG = 4;           // a brick is kMeshG x kMeshG columns ...
constexpr int kMeshBz = 7;          // ... and kMeshBz cells along z
constexpr int kMeshSlab = kMeshBz * kMeshZsub;  // a brick's sort bins along z, about r_c thick
// nodes that the ions of a brick reach, per axis and in all
constexpr int kMeshLx = kMeshG * kMeshKx + kMeshP - 1, kMeshLz = kMeshBz + kMeshP - 1;
constexpr int kMeshNodes = kMeshLx * kMeshLx * kMeshLz;

// Constants of one system's split, passed to the kernels by value.
struct MeshArgs {
    int N, cap;                     // ions; sorted slots (columns padded to whole groups)
    int nc[3], n[3];                // grid cells and nodes (nc + 9) per axis
    int ncx, ncy, nzb;              // columns along x and y; sort bins per column
    int nbx, nby, nbz;              // bricks per axis
    int parts, gparts;              // blocks per brick that spread its charges, that gather its forces
    int ng;                         // entries of one Green's table (zero padded)
    long long cost_max;             // estimated cost (mesh_cost) above which a step is summed directly
    double R, Hh, h, inv_h;         // domain radius and half height; grid spacing
    float rc, rc2, irc2, cw;        // near radius, its square, -2 / rc^2; column width
    float near[kMeshNearDeg + 1];   // f_L(r) = -L'/r in powers of 1 - 2 r^2 / r_c^2
    double win[kMeshWDeg + 1];      // window in powers of s = 1 - 2 z^2
    int M;                          // Gaussians in use
    double w[kMeshM], th[kMeshM];   // weights; t_m h (zero beyond M)
};

// Least squares of an m x n system (column major A, overwritten) by
// Householder QR; columns scaled by the caller.
inline void mesh_lstsq(std::vector<double>& A, std::vector<double>& b, int m, int n, double* x)
{
    std::vector<double> d(n);
    for (int j = 0; j < n; ++j) {
        double* a = &A[(size_t)j * m];
        double s = 0.0;
        for (int i = j; i < m; ++i) s += a[i] * a[i];
        s = std::sqrt(s);
        const double alpha = a[j] > 0 ? -s : s;
        a[j] -= alpha;
        double vv = 0.0;
        for (int i = j; i < m; ++i) vv += a[i] * a[i];
        auto reflect = [&](double* c) {
            double dot = 0.0;
            for (int i = j; i < m; ++i) dot += a[i] * c[i];
            const double f = vv > 0 ? 2.0 * dot / vv : 0.0;
            for (int i = j; i < m; ++i) c[i] -= f * a[i];
        };
        for (int k = j + 1; k < n; ++k) reflect(&A[(size_t)k * m]);
        reflect(b.data());
        d[j] = alpha;
    }
    for (int j = n - 1; j >= 0; --j) {
        double t = b[j];
        for (int k = j + 1; k < n; ++k) t -= A[(size_t)k * m + j] * x[k];
        x[j] = t / d[j];
    }
}

// Interpolation of f at the deg + 1 extrema of the Chebyshev polynomial on
// [-1, 1] (end points among them), as powers of s.
template <typename F>
void mesh_cheb(const F& f, int deg, std::vector<double>& mono)
{
    const int n = deg + 1;
    std::vector<double> c(n, 0.0), fv(n);
    const double pi = 3.14159265358979323846;
    for (int k = 0; k < n; ++k) fv[k] = f(std::cos(pi * k / deg)) * (k == 0 || k == deg ? 0.5 : 1.0);
    for (int j = 0; j < n; ++j) {
        for (int k = 0; k < n; ++k) c[j] += fv[k] * std::cos(pi * j * k / deg);
        c[j] *= (j == 0 || j == deg ? 1.0 : 2.0) / deg;
    }
    // Chebyshev to monomial
    std::vector<double> t0(n, 0.0), t1(n, 0.0), t2(n);
    mono.assign(n, 0.0);
    t0[0] = 1.0;
    if (n > 1) t1[1] = 1.0;
    for (int j = 0; j < n; ++j) {
        for (int k = 0; k < n; ++k) mono[k] += c[j] * t0[k];
        t2.assign(n, 0.0);
        for (int k = 0; k + 1 < n; ++k) t2[k + 1] = 2.0 * t1[k];
        for (int k = 0; k < n; ++k) t2[k] -= t0[k];
        t0 = t1;
        t1 = t2;
    }
}

inline double mesh_i0(double x)
{
    double t = 1.0, s = 1.0;
    const double q = 0.25 * x * x;
    for (int k = 1; k < 200; ++k) {
        t *= q / ((double)k * k);
        s += t;
        if (t < 1e-18 * s) break;
    }
    return s;
}

// M Gaussians w e^(-t^2 r^2) whose force is fitted to that of e^-r / r on
// [r_c, diag].  Returns the largest |F - F_L| r r_c there (1 at
// r_c = r << 1 for F itself), infinity if the fit failed.
inline double mesh_fit(double rc, double diag, int M, double* t, double* w)
{
    constexpr int m = 160;
    double t2[kMeshM];
    const double t0 = std::max(0.2, 0.6 / diag), t1 = kMeshTop / rc;
    for (int j = 0; j < M; ++j) {
        t[j] = t0 * std::pow(t1 / t0, (double)j / (M - 1));
        t2[j] = t[j] * t[j];
    }
    std::vector<double> A((size_t)m * M), rhs(m), sc(M, 0.0);
    for (int i = 0; i < m; ++i) {
        const double r = rc * std::pow(diag * 1.01 / rc, (double)i / (m - 1));
        // weighted by r; r_c itself heavily, because pairs a little beyond it
        // are evaluated at r_c, where the near part has to vanish
        const double wt = i == 0 ? 1.0e4 : 1.0;
        rhs[i] = wt * (1.0 + r) * std::exp(-r) / r;
        for (int j = 0; j < M; ++j) A[(size_t)j * m + i] = wt * 2.0 * t2[j] * r * r * std::exp(-t2[j] * r * r);
    }
    for (int j = 0; j < M; ++j) {
        for (int i = 0; i < m; ++i) sc[j] = std::max(sc[j], std::fabs(A[(size_t)j * m + i]));
        for (int i = 0; i < m; ++i) A[(size_t)j * m + i] /= sc[j];
    }
    mesh_lstsq(A, rhs, m, M, w);
    double worst = 0.0;
    for (int j = 0; j < M; ++j) w[j] /= sc[j];
    for (int i = 0; i < m; ++i) {
        const double r = rc * std::pow(diag / rc, (double)i / (m - 1));
        double f = -(1.0 + r) * std::exp(-r) / (r * r * r);
        for (int j = 0; j < M; ++j) f += w[j] * 2.0 * t2[j] * std::exp(-t2[j] * r * r);
        const double e = std::fabs(f) * r * r * rc;
        if (!std::isfinite(e)) return HUGE_VAL;
        worst = std::max(worst, e);
    }
    return worst;
}

// Grid and columns for a near radius; false if the domain is outside what the
// split is made for.
inline bool mesh_dims(double R, double H, double rc, MeshArgs& a)
{
    const double h = rc / kMeshRatio;
    a.h = h;
    a.inv_h = 1.0 / h;
    a.R = R;
    a.Hh = 0.5 * H;
    a.nc[0] = a.nc[1] = (int)std::ceil(2.0 * R / h);
    a.nc[2] = (int)std::ceil(H / h);
    for (int c = 0; c < 3; ++c) {
        if (a.nc[c] < 8 || a.nc[c] > 500) return false;
        a.n[c] = a.nc[c] + kMeshP - 1;
    }
    a.ncx = a.ncy = (a.nc[0] + kMeshKx - 1) / kMeshKx;
    a.nzb = a.nc[2] * kMeshZsub;
    a.cw = (float)(kMeshKx * h);
    a.rc = (float)rc;
    a.rc2 = a.rc * a.rc;
    a.irc2 = -2.0f / a.rc2;
    return true;
}

// Blocks per brick, at most `most`, on `cus` compute units: each holds one block, a last
// round that is nearly empty costs as much as a full one, a block has 0.08 of
// a brick's work to do whatever its part (the brick's nodes in and out of
// LDS), and a tenth of the bricks lie in the corners outside the cylinder.
// More than one only where that should gain a tenth.  One against the blocks
// chosen, us per pair sum on 256: 336 / 281 at 40,960 ions (128 bricks), 405 / 382 at
// 2^16 (144), 638 / 597 at 2^17 (300; 612 with four to gather); 489 / 507 with four at
// 98,304 (275).
inline int mesh_parts(const MeshArgs& a, int most, int cus)
{
    const double bricks = 0.9 * a.nbx * a.nby * a.nbz;
    int best = 1;
    double cost = 0.9 * std::ceil(bricks / cus) * 1.08;
    for (int p = 2; p <= most; ++p) {
        const double c = std::ceil(bricks * p / cus) * (1.0 / p + 0.08);
        if (c < cost) {
            cost = c;
            best = p;
        }
    }
    return best;
}

// What a step may cost as a split, in near pairs of 1.1 ps: the direct sum's
// N^2 / 4,200 ns less 2.4 ns per ion for the kernels that do not depend on where
// the ions are (each has 0.1 ms besides).  Near pairs and the fullest column of a
// brick (340 ns per ion: one wave spreads it) count against it.  Uniform ions
// reach 0.38 of it at 40,960, 0.21 at 2^16 and 0.05 at 2^18; with 30 % of the ions in a
// ball of 0.1 r_De a pair sum took 4.5 ms at 40,960 ions, 7.4 at 2^16 and 31 at
// 2^18, with all of them 14, 24 and 101, against 0.53, 1.2 and 16 directly (0.64,
// 1.35 and 17.7 with the choice).
constexpr double kMeshPairNs = 1.1e-3, kMeshColumnNs = 340.0;

inline long long mesh_cost_max(long long N)
{
    return (long long)(((double)N * N / 4200.0 - 2.4 * N) / kMeshPairNs);
}

// The split of a system of N ions (dimensionless R, H) on a device of `cus`
// compute units.  False: use the direct sum.
//
// r_c trades near pairs (r_c^3) against the grid (its nodes go as r_c^-3, the
// convolutions as r_c^-4) and scales with the ion spacing: in units of
// (27 / n)^(1/3), a step took 0.61 ms at 1.6, 0.65 at 1.68, 0.65 at 1.75 and
// 0.66 at 1.82 for 2^17 ions; 1.11, 1.12, 1.14 and 1.10 for 2^18; 4.55, 4.44,
// 4.28 and 4.39 for 2^20.
inline bool mesh_plan(long long N, double R, double H, MeshArgs& a, int cus = 256)
{
    const double diag = std::sqrt(4.0 * R * R + H * H);
    if (diag > 24.0 || N < 1024 || N > (1ll << 26)) return false;
    const double pi = 3.14159265358979323846;
    const double n = (double)N / (pi * R * R * H), b = std::cbrt(kMeshCol / n);
    double rc = 0.0;
    for (double q = 1.75; q <= 6.0 && rc == 0.0; q *= 1.04) {
        const double r = q * b;
        if (r < 0.1) continue;
        if (r > 2.5 || r > 0.45 * diag) return false;
        // a larger r_c where the grid would have too many nodes
        if (mesh_dims(R, H, r, a) && (double)a.n[0] * a.n[1] * a.n[2] <= 3.0e7) rc = r;
    }
    if (rc == 0.0) return false;
    a.N = (int)N;
    const long long cap = (N + (kMeshTile - 1ll) * a.ncx * a.ncy + 63) / 64 * 64;
    if (cap > (1ll << 28)) return false;
    a.cap = (int)cap;
    a.nbx = (a.ncx + kMeshG - 1) / kMeshG;
    a.nby = (a.ncy + kMeshG - 1) / kMeshG;
    a.nbz = (a.nc[2] + kMeshBz - 1) / kMeshBz;
    a.cost_max = mesh_cost_max(N);
    a.parts = mesh_parts(a, 2, cus);
    a.gparts = mesh_parts(a, 3, cus);
    a.ng = std::max(a.n[0], a.n[2]) + 80;

    // As few Gaussians as fit to kMeshFit.  The fit's error of the acceleration,
    // relative to the rms over uniform ions, is then 4e-8 to 2.3e-7, below the
    // 3e-7 of the direct FP32 sum; 14 throughout left 1.3e-7 at 2^20 ions,
    // 3.4e-7 at 2^21, 9.8e-7 at 2^22 and 2.3e-6 at 2^23 (R = 3, H = 6 to 8),
    // against 1.3e-7, 1.1e-7 (15), 1.2e-7 (16) and 9.8e-8 (17).  A domain that
    // the most do not fit to it keeps the direct sum.
    double t[kMeshM];
    bool fits = false;
    for (a.M = kMeshMinM; a.M <= kMeshM && !fits; ++a.M) fits = mesh_fit(rc, diag, a.M, t, a.w) < kMeshFit;
    --a.M;
    if (!fits) return false;
    for (int j = 0; j < kMeshM; ++j) {
        a.th[j] = j < a.M ? t[j] * a.h : 0.0;
        if (j >= a.M) a.w[j] = 0.0;
    }
    // near part: f_L in powers of s = 1 - 2 r^2 / r_c^2
    std::vector<double> mono;
    mesh_cheb([&](double s) {
        const double y = 0.5 * (1.0 - s) * rc * rc;
        double f = 0.0;
        for (int j = 0; j < a.M; ++j) f += a.w[j] * 2.0 * (t[j] * t[j]) * std::exp(-(t[j] * t[j]) * y);
        return f;
    }, kMeshNearDeg, mono);
    for (int k = 0; k <= kMeshNearDeg; ++k) a.near[k] = (float)mono[k];
    // window I0(beta sqrt(1 - z^2)) / I0(beta) in powers of s = 1 - 2 z^2
    const double top = mesh_i0(kMeshBeta);
    mesh_cheb([&](double s) { return mesh_i0(kMeshBeta * std::sqrt(std::max(0.0, 0.5 * (1.0 + s)))) / top; },
              kMeshWDeg, mono);
    for (int k = 0; k <= kMeshWDeg; ++k) a.win[k] = mono[k];
    return true;
}

}  // namespace odk
