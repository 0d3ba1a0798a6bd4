// Host build of tile_place (internal.hpp): for every number of tiles to a row that a grid of at
// most 2^31 - 1 cells can have (tiles of TX x TY cells, at least two rows of cells), the first and
// the last tile of every row of tiles.  Prints the number of rows checked, or the first tile that
// is misplaced.
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "internal.hpp"

int main(int argc, char** argv) {
    const int64_t TX = std::atoi(argv[1]), TY = std::atoi(argv[2]), cells = 2147483647;
    int64_t rows = 0;
    for (int64_t tiles_x = 1; (tiles_x - 1) * TX + 1 <= cells / 2; ++tiles_x) {
        const int64_t least = tiles_x == 1 ? 2 : (tiles_x - 1) * TX + 1;
        const int64_t tiles_y = (cells / least + TY - 1) / TY;
        for (int64_t row = 0; row < tiles_y; ++row, ++rows)
            for (int64_t col : {(int64_t)0, tiles_x - 1}) {
                const int2 at = cuesim::tile_place((int)(row * tiles_x + col), (int)tiles_x);
                if (at.x == col && at.y == row) continue;
                std::printf("tile %lld of %lld to a row: column %d row %d\n",
                            (long long)(row * tiles_x + col), (long long)tiles_x, at.x, at.y);
                return 1;
            }
    }
    std::printf("%lld rows\n", (long long)rows);
    return 0;
}
