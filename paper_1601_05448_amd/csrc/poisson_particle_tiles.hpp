// The tiles of the deposit's last kernel, k_part_cells (poisson_particles.hip): their
// rows, their order over the blocks, and where their rows begin in the list of runs.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/poisson.h"
#include "poisson_internal.hpp"

namespace pois {

// Divisions by the lengths, 2^a or 3 2^a, are shifts and one product, by the rows of
// a tile one product: with the compiler's own, k_part_runs took 13.5 us for 10^6
// particles on 512^3 instead of 11.8.
struct LineDivide {
    unsigned shift, third;  // third: the length has a factor 3
    __host__ __device__ unsigned operator()(unsigned x) const {
        x >>= shift;
        return third ? (unsigned)(((unsigned long long)x * 0xAAAAAAABull) >> 33) : x;
    }
};

inline LineDivide line_divide(int n) {
    LineDivide d{0u, n % 3 == 0 ? 1u : 0u};
    for (int m = d.third ? n / 3 : n; m > 1; m /= 2) ++d.shift;
    return d;
}

// The tiles of k_part_cells: `rows` rows of one plane, tiles_y of them per plane.
// Where their rows begin in the list of runs is kept in 2 tiles_y edges per plane, in
// the order of their rows: row 0; rows j0 - 1 and j0 of every later tile; row ny - 1
// (the row below row 0).  After the last plane's comes the end of the list.
struct TileGeom {
    int nx, ny, rows, tiles_y;
    unsigned tiles, group;  // all tiles, neighbouring tiles of a block
    LineDivide by_nx, by_ny;
    unsigned inv_rows;  // 65536 / rows, rounded up: exact quotients up to 1024 for rows <= 8
    // edges up to and with the row of the cell
    __host__ __device__ unsigned edges_to(unsigned cell) const {
        const unsigned row = by_nx(cell), k = by_ny(row), j = row - k * (unsigned)ny, last = (unsigned)tiles_y - 1;
        const unsigned above = ((j + 1) * inv_rows) >> 16;
        return k * 2u * (unsigned)tiles_y + 1u + (above < last ? above : last) + ((j * inv_rows) >> 16) +
               (j + 1 == (unsigned)ny ? 1u : 0u);
    }
    __host__ __device__ unsigned edges() const { return 2u * tiles; }
};

constexpr unsigned kSpanMax = 32;  // tiles of a block at most: one thread per bound (of eight)

// Tile m of block b of nb, whose groups are `group` tiles.
__host__ __device__ __forceinline__ unsigned block_tile(unsigned m, unsigned group, unsigned b, unsigned nb) {
    const unsigned g = m / group;
    return (g * nb + b) * group + (m - g * group);
}

// Rows of a tile of k_part_cells: eight, or what fits 32 KB of LDS (four blocks per
// CU), fewer where that leaves the chip without four blocks per CU.  More rows share
// the row below the tile (10^6 particles on 512^3: 510, 432 and 436 us with 2, 4 and 8
// rows; on 64 x 512 x 512, x first: 350, 270 and 220; 3 10^5 on 768 x 192 x 384: 221 with
// 2 and 205 with 5).  Then as many tiles per block as leave eight blocks per CU.
inline int tile_rows(const GridArgs& g) {
    int rows = std::max(1, std::min({g.ny, 8, 4096 / g.nx}));
    while (rows > 1 && (long long)g.nz * ((g.ny + rows - 1) / rows) < 1024) rows = (rows + 1) / 2;
    return rows;
}

// Neighbouring tiles of a block, up to kTileGroup of them: neighbours are written a
// little faster, tiles far apart share out a crowd (10^6 particles on 512^3, uniform /
// in one plane: 1 of 16 tiles 444 / 443 us, 2 432 / 469, 4 431 / 525, 8 437 / 686).
constexpr unsigned kTileGroup = 2;

inline TileGeom tile_geom(const GridArgs& g) {
    const int rows = tile_rows(g), tiles_y = (g.ny + rows - 1) / rows;
    const unsigned tiles = (unsigned)g.nz * (unsigned)tiles_y;
    return TileGeom{g.nx, g.ny, rows, tiles_y, tiles, std::clamp(tiles / 2048u, 1u, kTileGroup),
                    line_divide(g.nx), line_divide(g.ny), (65536u + (unsigned)rows - 1) / (unsigned)rows};
}

inline unsigned tile_blocks(const TileGeom& tg) {
    const unsigned groups = (tg.tiles + tg.group - 1) / tg.group;
    const unsigned span = std::clamp(groups / 2048u, 1u, kSpanMax / kTileGroup);
    return (groups + span - 1) / span;
}

}  // namespace pois
