// Tiles that one cone's eight steps of a reverse launch can touch on grids so wide that the FP32
// rounding of a tip is cells, against the room that reverse_list_capacity leaves it: tips straight
// along the longer axis, moved and turned into cells by the expressions of the step.  Tiles of TX x
// TY cells with a halo of H cells.  A cone's box is listed unless its eight footprints of four cells
// need fewer entries, which then are.  Prints the most tiles, or the first grid whose tips need more
// than their room.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "internal.hpp"

int main(int argc, char** argv) {
    using namespace cuesim;
    const int TX = std::atoi(argv[1]), TY = std::atoi(argv[2]), H = std::atoi(argv[3]);
    int most = 0, checked = 0;
    for (const int axis : {0, 1})
        for (const int n : {1000, 1 << 20, 3000000, 20000000, 100000000, 200000000, 500000000,
                            1 << 30}) {
            const int core = axis == 0 ? TX : TY, tiles = (n + core - 1) / core;
            for (double step = 0.1; step < 40.0; step += 0.3) {
                const int nx = axis == 0 ? n : 2, ny = axis == 0 ? 2 : n;
                const int64_t room = (int64_t)reverse_list_capacity(nx, ny, 1, step);
                if (room >= 8 * std::min<int64_t>((3 + 2 * H) / core + 2, tiles)) continue;
                for (int k = 0; k < 400; ++k) {
                    float at = (float)n * (0.5f + 0.4f * (float)((k * 7919) % 400) / 400.0f) + (float)k;
                    int i0, i1;
                    float f;
                    corner(at, 1.0f, n, i0, f);
                    for (int s = 0; s < 7; ++s) at = std::fmaf((float)step, 1.0f, at);
                    corner(at, 1.0f, n, i1, f);
                    if (i1 > n - 3) continue;
                    const int first = std::max(std::max(i0 - 1, 0) - H, 0) / core;
                    const int last = std::min((std::min(i1 + 2, n - 1) + H) / core, tiles - 1);
                    ++checked;
                    if (last - first + 1 > room) {
                        std::printf("%d cells along axis %d, steps of %g: %d tiles, room for %lld\n",
                                    n, axis, step, last - first + 1, (long long)room);
                        return 1;
                    }
                    most = std::max(most, last - first + 1);
                }
            }
        }
    std::printf("%d %d\n", most, checked);
    return 0;
}
