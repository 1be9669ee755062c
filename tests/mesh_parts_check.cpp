// Blocks per brick of the near / far split's plans: in the range that the
// kernels and the brick workspace are made for, every value among them, and
// none beyond one where the bricks alone fill the device many times over.
#include <cstdio>

#include "../paper_2205_06557_amd/csrc/meshplan.hpp"

using namespace odk;

int main()
{
    int seen[2][4] = {};
    for (int cus : {32, 80, 128, 256, 304})
        for (long long N = 40960; N <= 1 << 21; N = N * 5 / 4 + 7) {
            MeshArgs a{};
            if (!mesh_plan(N, 3.0, 6.0, a, cus)) return 1;
            if (a.parts < 1 || a.parts > 2 || a.gparts < 1 || a.gparts > 3) {
                std::printf("N %lld on %d: %d, %d\n", N, cus, a.parts, a.gparts);
                return 1;
            }
            ++seen[0][a.parts];
            ++seen[1][a.gparts];
            const double rounds = 0.9 * a.nbx * a.nby * a.nbz / cus;
            if (rounds > 8.0 && (a.parts > 1 || a.gparts > 1)) return 1;
            // without the device's size a plan is that of 256 compute units
            MeshArgs b{};
            if (cus == 256 && (!mesh_plan(N, 3.0, 6.0, b) || b.parts != a.parts || b.gparts != a.gparts)) return 1;
        }
    std::printf("%d %d, %d %d %d\n", seen[0][1], seen[0][2], seen[1][1], seen[1][2], seen[1][3]);
    return seen[0][1] && seen[0][2] && seen[1][1] && seen[1][2] && seen[1][3] ? 0 : 1;
}
