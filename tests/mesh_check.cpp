// Checks of the near / far split's plan (meshplan.hpp) over sizes and domains:
// the Gaussians against the screened force, the near polynomial, the window
// polynomial, and the sizes the kernels rely on.  Prints the number of plans.
#include <cstdio>
#include <cstdlib>

#include "../paper_2205_06557_amd/csrc/meshplan.hpp"

using namespace odk;

#define NEED(c)                                                              \
    do {                                                                     \
        if (!(c)) {                                                          \
            std::printf("failed: %s (N %lld R %g H %g)\n", #c, N, R, H);     \
            return 1;                                                        \
        }                                                                    \
    } while (0)

int main()
{
    int plans = 0;
    const double shapes[][2] = {{3, 6}, {3, 8}, {1.5, 14}, {8, 2.5}, {5, 5}, {3, 20}, {0.5, 0.5}, {60, 60}};
    for (const auto& s : shapes)
        for (long long N = 16384; N <= 1ll << 24; N = N * 3 / 2 + 7) {
            const double R = s[0], H = s[1];
            MeshArgs a{};
            if (!mesh_plan(N, R, H, a)) {
                NEED(R > 10 || R < 1 || N > 1 << 22);      // these domains and sizes are what it is for
                continue;
            }
            ++plans;
            const double rc = a.rc, diag = std::sqrt(4 * R * R + H * H);
            NEED(a.N == N && a.cap % kMeshTile == 0 && a.cap >= N);
            NEED(a.nc[0] * a.h >= 2 * R && a.nc[2] * a.h >= H && a.ncx * kMeshKx >= a.nc[0] && a.ncy * kMeshKx >= a.nc[1]);
            NEED(a.nbx * kMeshG >= a.ncx && a.nby * kMeshG >= a.ncy && a.nbz * kMeshBz >= a.nc[2]);
            // the nodes that any cell reaches lie in its brick's, and the grid holds them
            NEED(a.n[0] == a.nc[0] + kMeshP - 1 && a.n[2] == a.nc[2] + kMeshP - 1);
            NEED(a.ng >= a.n[0] + 79 && a.ng >= a.n[2] + 79 && (a.ng + 63) / 64 <= 65535);
            auto fl = [&](double r) {
                double f = 0;
                for (int j = 0; j < kMeshM; ++j) {
                    const double t = a.th[j] / a.h;
                    f += a.w[j] * 2 * t * t * std::exp(-t * t * r * r);
                }
                return f;
            };
            for (int i = 0; i <= 400; ++i) {
                // beyond r_c the Gaussians are the screened force
                const double r = rc * std::pow(diag / rc, i / 400.0), F = (1 + r) * std::exp(-r) / (r * r);
                NEED(std::fabs(fl(r) * r - F) * r * rc < 3e-5);
                // inside, the near polynomial is the Gaussians' force
                const double z = i / 400.0, y = z * rc;
                double p = 0, q = 0;
                for (int k = kMeshNearDeg; k >= 0; --k) p = p * (1 - 2 * z * z) + a.near[k];
                NEED(std::fabs(p - fl(y)) * y * rc * rc < 5e-6);
                for (int k = kMeshWDeg; k >= 0; --k) q = q * (1 - 2 * z * z) + a.win[k];
                NEED(std::fabs(q - mesh_i0(kMeshBeta * std::sqrt(1 - z * z)) / mesh_i0(kMeshBeta)) < 1e-11);
            }
            NEED(std::fabs(fl(rc) * rc * rc * rc - (1 + rc) * std::exp(-rc)) < 1e-8);
        }
    std::printf("%d plans\n", plans);
    return plans > 50 ? 0 : 1;
}
