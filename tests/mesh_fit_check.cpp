// The Gaussians of every plan of the near / far split reproduce the screened
// force beyond r_c to the level of the sizes that were measured against 64-bit
// sums (meshplan.hpp, kMeshFit), whatever the number of ions: the error per
// pair, |F - F_L| r r_c with F(r) = (1 + r) e^-r / r^2, at points between the
// fit's own.  Prints the largest and the number of plans.
#include <cstdio>

#include "../paper_2205_06557_amd/csrc/meshplan.hpp"

using namespace odk;

int main()
{
    const double shapes[][2] = {{3, 6}, {3, 8}, {1.5, 14}, {8, 2.5}, {5, 5}, {3, 20}, {0.6, 20}};
    int plans = 0, bad = 0;
    double top = 0.0;
    for (const auto& s : shapes)
        for (long long N = 40960; N <= 1ll << 26; N = N * 3 / 2 + 7) {
            MeshArgs a{};
            if (!mesh_plan(N, s[0], s[1], a)) continue;
            ++plans;
            const double rc = a.rc, diag = std::sqrt(4 * s[0] * s[0] + s[1] * s[1]);
            double worst = 0.0;
            for (int i = 0; i <= 3000; ++i) {
                const double r = rc * std::pow(diag / rc, i / 3000.0);
                double f = (1 + r) * std::exp(-r) / (r * r * r);
                for (int j = 0; j < kMeshM; ++j) {
                    const double t = a.th[j] / a.h;
                    f -= a.w[j] * 2 * t * t * std::exp(-t * t * r * r);
                }
                worst = std::max(worst, std::fabs(f) * r * r * rc);
            }
            // a tenth above the fit's limit: the error's peaks lie between the points it is tested at
            if (!(worst < 3.5e-6)) {
                std::printf("N %lld R %g H %g: %.2e\n", N, s[0], s[1], worst);
                ++bad;
            }
            top = std::max(top, worst);
        }
    std::printf("%d plans, largest error %.2e\n", plans, top);
    return plans > 70 && !bad ? 0 : 1;
}
