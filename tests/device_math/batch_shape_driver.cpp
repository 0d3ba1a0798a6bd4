// The launch shape that the library plans for a batch, and the one that each member then gets.
// Arguments: depth and row width / 64 asked for, then for every member nx ny species step_len/dx cones tile_height.
// Prints the planned depth and, per member, depth and height of its plan; then, of the whole plan,
// the member that does not fit (-1: all do), row width / 64, depth and every member's row width / 64
// and depth with them.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tiled.hpp"

int main(int argc, char** argv) {
    using namespace cuesim;
    const int asked = std::atoi(argv[1]), cols = std::atoi(argv[2]), n = (argc - 3) / 6;
    const int cpl = cols ? cols : 2;
    std::vector<sim_params> p(n);
    std::vector<const sim_params*> at(n);
    for (int i = 0; i < n; ++i) {
        char** a = argv + 3 + 6 * i;
        p[i] = sim_params{};
        p[i].nx = std::atoi(a[0]);
        p[i].ny = std::atoi(a[1]);
        p[i].n_species = std::atoi(a[2]);
        p[i].dx = 1.0;
        p[i].step_len = std::atof(a[3]);
        p[i].n_cones = std::atoi(a[4]);
        p[i].tile_height = std::atoi(a[5]);
        p[i].dim = 2;
        p[i].block_steps = asked;
        p[i].tile_cols_per_lane = cols;
        at[i] = &p[i];
    }
    std::vector<int> height;
    const int depth = tiled_batch_shape(at.data(), n, cpl, height);
    std::printf("%d", depth);
    for (int i = 0; i < n; ++i) {
        const int b = asked ? asked : depth ? depth : kDefaultBlockSteps;
        const TiledPlan t = tiled_plan(2, p[i].nx, p[i].ny, 1, p[i].n_species, p[i].step_len, b,
                                       p[i].n_cones, cpl, depth ? height[i] : p[i].tile_height,
                                       false);
        std::printf(" %d %d", t.block_steps, t.height);
    }
    std::printf("\n");
    BatchPlan plan;
    const int misfit = tiled_batch_plan(at.data(), n, plan);
    std::printf("%d %d %d", misfit, plan.cpl, plan.block_steps);
    for (int i = 0; i < n && misfit < 0; ++i) {
        const TiledPlan& t = plan.members[i];
        std::printf(" %d %d", t.cpl, t.block_steps);
    }
    std::printf("\n");
    return 0;
}
