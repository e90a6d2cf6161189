// Host-side checks of paper_1901_02211_amd/csrc/wilson_site.h, built by tests/test_tiles_host.py: the blocks of the
// stencils cover every site of a lattice once.  Exit status 0 = all pass.
#include <cstdio>
#include <vector>

#include "../../paper_1901_02211_amd/csrc/wilson_site.h"

static int failures = 0;

static smpq::Geom geometry(int nx, int ny, int nz, int nt, int band) {
    smpq::Geom g{};
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.nt = nt;
    g.V = nx * ny * nz * nt;
    g.band = band;
    return g;
}

// Any-lattice tiles, whatever band the other variants' fields hold (kind 0 takes any value there).
static void any_tiles(int nx, int ny, int nz, int nt, int band) {
    const smpq::Geom g = geometry(nx, ny, nz, nt, band);
    int ty, m;
    smpq::any_tile(g, ty, m);
    if (ty == 0) return;   // consecutive sites
    const int threads = (m * nx * ty + 63) / 64 * 64;
    std::vector<int> seen(g.V, 0);
    bool inside = threads <= smpq::kBlock && (ty == ny || 2 * nx <= threads);   // the halo rows' threads
    for (int tile = 0; tile < smpq::any_blocks(g); ++tile)
        for (int t = 0; t < threads; ++t) {
            const smpq::AnySite a = smpq::any_site(g, ty, m, tile, t);
            const int s = (a.pl * ny + a.y0) * nx + a.i;
            if (a.pl < 0 || a.pl >= nz * nt || s < 0 || s >= g.V || a.mi >= m || a.here < 1 || a.y0 + a.here > ny)
                inside = false;
            else if (a.ok)
                ++seen[s];
        }
    bool once = true;
    for (int n : seen) once = once && n == 1;
    if (!inside || !once) {
        std::printf("FAIL %d x %d x %d x %d, band %d: %s\n", nx, ny, nz, nt, band,
                    inside ? "a site missing or twice" : "outside the lattice");
        ++failures;
    }
}

// The plane order of the tiles that have a band.
static void bands(int nz, int nt) {
    for (int band = 1; band <= nz; ++band) {
        if (nz % band) continue;
        const smpq::Geom g = geometry(16, 16, nz, nt, band);
        std::vector<int> seen(nz * nt, 0);
        for (int p = 0; p < nz * nt; ++p) {
            const int pl = smpq::plane_order(p, g);
            if (pl >= 0 && pl < nz * nt) ++seen[pl];
        }
        for (int n : seen)
            if (n != 1) {
                std::printf("FAIL planes %d x %d, band %d\n", nz, nt, band);
                ++failures;
                break;
            }
    }
}

int main() {
    const int planes[][2] = {{1, 1}, {4, 1}, {1, 3}, {2, 5}, {4, 6}};
    for (int nx : {1, 2, 3, 5, 6, 8, 12, 16, 17, 24, 63, 64, 65, 100, 127, 128, 129, 256, 300})
        for (int ny : {1, 2, 3, 4, 7, 10, 12, 16, 17, 24, 33, 128, 256})
            for (const auto &pl : planes)
                for (int band : {1, 2, 3, 7, 0, -1}) any_tiles(nx, ny, pl[0], pl[1], band);
    for (const auto &pl : planes) bands(pl[0], pl[1]);
    bands(12, 5);
    std::printf("%d failures\n", failures);
    return failures == 0 ? 0 : 1;
}
