// Which sites the blocks of the stencils cover, for the kernels and for host checks.
#pragma once
#include "kernels.h"

namespace smpq {

// Plane p of the block order -> (z, t) plane index z + nz t.  The planes are taken in bands of
// g.band consecutive z: t runs over the whole extent inside a band, so that the +-t
// neighbours of a plane were staged g.band blocks earlier (still in L2) rather than nz.  Needs a band
// that divides nz.
__host__ __device__ __forceinline__ int plane_order(int p, const Geom &g) {
    if (g.band == 1) return p;
    const int per = g.band * g.nt, b = p / per, i = p % per;
    return b * g.band + i % g.band + g.nz * (i / g.band);
}

// Rows ty of one plane and planes m of a kTileAny block (ty = ny where m > 1); ty = 0: kTileNone.
__host__ __device__ __forceinline__ void any_tile(const Geom &g, int &ty, int &m) {
    const int nxy = g.nx * g.ny, planes = g.nz * g.nt;
    m = 1;
    if (nxy <= kBlock) {
        ty = g.ny;
        m = kBlock / nxy < planes ? kBlock / nxy : planes;
    } else if (g.nx <= kBlock / 2) {
        int tiles = (nxy + kBlock - 1) / kBlock;
        while ((g.ny + tiles - 1) / tiles * g.nx > kBlock) ++tiles;
        ty = (g.ny + tiles - 1) / tiles;
        if (ty < 2) ty = 0;
    } else {
        ty = 0;
    }
}

// Blocks per right-hand side of a kTileAny launch, or of a kTileNone one where no tile fits.
inline int any_blocks(const Geom &g) {
    int ty, m;
    any_tile(g, ty, m);
    if (ty == 0) return (g.V + kBlock - 1) / kBlock;
    const int planes = g.nz * g.nt;
    return m > 1 ? (planes + m - 1) / m : planes * ((g.ny + ty - 1) / ty);
}

// Thread t of tile `tile` of a kTileAny launch: site i of the tile's rows, which start at row y0 of plane
// pl = z + nz t (the planes in their own order: no variant for any lattice has a band) and of which
// `here` lie in the plane; mi numbers the planes of a block with several.  ok is false for an idle
// thread, which gets the tile's first site.
struct AnySite {
    int pl, mi, y0, here, i;
    bool ok;
};
__host__ __device__ __forceinline__ AnySite any_site(const Geom &g, int ty, int m, int tile, int t) {
    const int nxy = g.nx * g.ny;
    AnySite a{0, 0, 0, ty, t, true};
    if (m > 1) {
        a.mi = t / nxy;
        a.pl = tile * m + a.mi;
        a.i = t - a.mi * nxy;
        a.ok = a.mi < m && a.pl < g.nz * g.nt;
    } else {
        const int tiles_per_plane = (g.ny + ty - 1) / ty;
        a.pl = tile / tiles_per_plane;
        a.y0 = tile % tiles_per_plane * ty;
        a.here = g.ny - a.y0 < ty ? g.ny - a.y0 : ty;
        a.ok = t < g.nx * a.here;
    }
    if (!a.ok) {
        a.i = a.mi = 0;
        if (m > 1) a.pl = tile * m;
    }
    return a;
}

}  // namespace smpq
