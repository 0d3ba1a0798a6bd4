// Launches over the widest and thinnest grids that are accepted (host code): every reverse tile has
// one workgroup, and no launch has 2^32 threads along an axis.  Prints "ok" or what is wrong.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "internal.hpp"
#include "tiled.hpp"

using namespace cuesim;

static int wrong(const char* what, int64_t a, int64_t b, int64_t c) {
    std::printf("%s: %lld %lld %lld\n", what, (long long)a, (long long)b, (long long)c);
    return 1;
}

int main() {
    const int64_t limit = (int64_t)1 << 32;
    for (int n : {1, 7, 8, 9, 470, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 3 << 20,
                  reverse_tiles(1 << 30, 2), reverse_tiles(2, 1 << 30)}) {
        const ReverseGrid g = reverse_grid(n);
        if ((int64_t)g.per_slice * 512 + ((int64_t)1 << 22) * 512 >= limit || g.slices > 65535)
            return wrong("reverse grid", n, g.slices, g.per_slice);
        std::vector<bool> seen(n, false);
        int64_t count = 0;
        for (int z = 0; z < g.slices; ++z)
            for (int x = 0; x < g.per_slice; ++x) {
                const int t = g.tile(x, z);
                if (t < 0) return wrong("reverse tile", n, x, z);
                if (t >= n) continue;
                if (seen[t]) return wrong("reverse tile twice", n, x, z);
                seen[t] = true;
                ++count;
            }
        if (count != n) return wrong("reverse tiles", n, count, g.slices);
    }
    // volumes a few cells thin, and the largest cube
    for (int ns : {1, 2})
        for (auto v : {std::vector<int>{2, 2, 536870911}, {2, 2, 100000000}, {2, 500000000, 2},
                       {1000000000, 2, 1}, {3, 9, 70000000}, {1290, 1290, 1290}, {97, 64, 51}}) {
            if (v[2] < 2) v[2] = 2, v[0] /= 2;
            Field3D f;
            f.nx = v[0];
            f.ny = v[1];
            f.nz = v[2];
            f.n_species = ns;
            const float* in[2] = {};
            float* out[2] = {};
            const StencilCoef coef[2] = {};
            const Field3DArgs a = field3d_args(f, in, out, coef);
            const int64_t boxes = (int64_t)ns * a.tx * a.ty * a.tz;
            if (a.tx * a.ty <= 1 << 22 && boxes * 512 >= limit)
                return wrong("boxes", v[0], v[1], v[2]);
            if ((int64_t)a.tz * a.planes < v[2] || a.planes % 4 != 0)
                return wrong("planes", v[2], a.tz, a.planes);
        }
    // tiled launches
    for (int ns : {1, 2})
        for (int block : {0, 8, 16})
            for (auto v : {std::vector<int>{1 << 30, 2}, {1000000000, 2}, {700000000, 2},
                           {640000000, 3}, {100000000, 20}, {46340, 46340}, {2, 1 << 30}}) {
                const TiledPlan p = tiled_plan(2, v[0], v[1], 1, ns, 0.5, block, 100000);
                const int waves = p.shape == kWide ? 16 : p.shape == kTwo ? 12 : 8;
                if (p.block_steps > 1 && ((int64_t)p.n_tiles + 8 + 1024) * 64 * waves >= limit)
                    return wrong("tiles", v[0], p.n_tiles, p.block_steps);
            }
    std::printf("ok\n");
    return 0;
}
