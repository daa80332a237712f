"""The tiles of the deposit's last kernel, on the CPU over every grid of supported
lengths: each tile belongs to one block, the divisions are exact, and the edges that
the list of runs gets at its cells are those that the tiles read (against plain
searches)."""
import os
import subprocess

from paper_1601_05448_amd import build as B

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "poisson_particle_tiles.hpp"
using namespace pois;
static const int L[] = {4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024};
#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); return 1; } } while (0)
int main() {
    for (int n : L) {
        const LineDivide d = line_divide(n);
        for (unsigned x = 0; x <= (1u << 30); x += x < 5000000u || x > (1u << 30) - 5000000u ? 1u : 977u)
            CHECK(d(x) == x / (unsigned)n, "%u / %d\n", x, n);
    }
    for (int nx : L) for (int ny : L) for (int nz : L) {
        GridArgs g{};
        g.nx = nx; g.ny = ny; g.nz = nz;
        const TileGeom tg = tile_geom(g);
        CHECK((tg.rows * nx + 0) * 8 <= 32768 || tg.rows == 1, "lds %d %d\n", nx, tg.rows);
        const unsigned nb = tile_blocks(tg);
        std::vector<char> seen(tg.tiles, 0);
        for (unsigned b = 0; b < nb; ++b) {
            bool ended = false;
            for (unsigned m = 0; m < kSpanMax; ++m) {
                const unsigned t = block_tile(m, tg.group, b, nb);
                if (t >= tg.tiles) { ended = true; continue; }
                CHECK(!ended && !seen[t], "tile %u of %d %d %d\n", t, nx, ny, nz);
                seen[t] = 1;
            }
        }
        for (char c : seen) CHECK(c, "a tile of %d %d %d has no block\n", nx, ny, nz);
        // edges_to counts the edges up to a row; edge e of a plane lies at this row:
        auto row_of = [&](int e) {
            return e == 0 ? 0 : e == 2 * tg.tiles_y - 1 ? ny - 1 : e % 2 ? (e + 1) / 2 * tg.rows - 1 : e / 2 * tg.rows;
        };
        for (int k : {0, 1, nz - 1}) for (int j = 0; j < ny; ++j) for (int i : {0, nx - 1}) {
            unsigned want = (unsigned)k * 2u * (unsigned)tg.tiles_y;
            for (int e = 0; e < 2 * tg.tiles_y; ++e) want += row_of(e) <= j ? 1u : 0u;
            CHECK(tg.edges_to(((unsigned)k * ny + j) * (unsigned)nx + i) == want, "edges %d %d %d\n", nx, ny, j);
        }
        // the edges a tile reads: max(j0 - 1, 0), j1, ny - 1 and the plane's end
        for (int jt = 0; jt < tg.tiles_y; ++jt) {
            const int j0 = jt * tg.rows, j1 = j0 + tg.rows < ny ? j0 + tg.rows : ny;
            CHECK(row_of(jt == 0 ? 0 : 2 * jt - 1) == (j0 > 0 ? j0 - 1 : 0), "first row %d\n", jt);
            CHECK(2 * jt + 2 == 2 * tg.tiles_y ? j1 == ny : row_of(2 * jt + 2) == j1, "end row %d\n", jt);
        }
    }
    std::printf("ok\n");
    return 0;
}
"""


def test_tiles_and_edges(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-O2", "-std=c++20", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", B.CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=240)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
