// Per-site Wilson hopping term and the sites of the stencils' blocks, written once for the GPU kernels and for
// host checks.
//
// hop(x) = sum_mu [ P(-s)_mu U_mu(x) psi(x + mu) + P(+s)_mu U_mu(x - mu)^dag psi(x - mu) ],
// with P(s)_mu = 1 - s gamma_mu, s = +1 for D_W and s = -1 for D_W^dag (the adjoint swaps
// the two projectors), so that D_W psi = psi - kappa hop (section 1, Eq. 3).
//
// Chiral basis: gamma_mu = [[0, A_mu], [A_mu^dag, 0]] with A_x = -i sigma_1,
// A_y = -i sigma_2, A_z = -i sigma_3, A_t = 1.  (1 - s gamma_mu) psi has upper half
// h = psi_up - s A_mu psi_dn and lower half -s A_mu^dag h, so each hop projects to a
// two-spinor, multiplies it by the link and rebuilds the lower half.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace smpq {

template <class T>
struct cpx {
    T re, im;
};

template <class T>
__host__ __device__ __forceinline__ cpx<T> operator+(cpx<T> a, cpx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <class T>
__host__ __device__ __forceinline__ cpx<T> operator-(cpx<T> a, cpx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <class T>
__host__ __device__ __forceinline__ cpx<T> operator*(T s, cpx<T> a) { return {s * a.re, s * a.im}; }
// i * a
template <class T>
__host__ __device__ __forceinline__ cpx<T> mul_i(cpx<T> a) { return {-a.im, a.re}; }
// a * b
template <class T>
__host__ __device__ __forceinline__ cpx<T> cmul(cpx<T> a, cpx<T> b) {
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// conj(a) * b
template <class T>
__host__ __device__ __forceinline__ cpx<T> cjmul(cpx<T> a, cpx<T> b) {
    return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
// a * b + c with a single rounding
__host__ __device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
// the products in FP64 with their rounding written out, so that every kernel rounds them alike (left to the
// compiler, which of the two products is fused differed between two forms of one kernel)
__host__ __device__ __forceinline__ cpx<double> cmul(cpx<double> a, cpx<double> b) {
    return {fmadd(a.re, b.re, -(a.im * b.im)), fmadd(a.re, b.im, a.im * b.re)};
}
__host__ __device__ __forceinline__ cpx<double> cjmul(cpx<double> a, cpx<double> b) {
    return {fmadd(a.re, b.re, a.im * b.im), fmadd(a.re, b.im, -(a.im * b.re))};
}
// c + a * b and c + conj(a) * b as chains of fused multiply-adds: sums of complex products
// written this way take 4 instructions per term instead of 6 (the compiler does not
// reassociate a sum of products into such a chain by itself)
template <class T>
__host__ __device__ __forceinline__ cpx<T> cfma(cpx<T> a, cpx<T> b, cpx<T> c) {
    return {fmadd(a.re, b.re, fmadd(-a.im, b.im, c.re)), fmadd(a.re, b.im, fmadd(a.im, b.re, c.im))};
}
template <class T>
__host__ __device__ __forceinline__ cpx<T> cjfma(cpx<T> a, cpx<T> b, cpx<T> c) {
    return {fmadd(a.re, b.re, fmadd(a.im, b.im, c.re)), fmadd(a.re, b.im, fmadd(-a.im, b.re, c.im))};
}

// Upper two spin rows of (1 - S gamma_MU) psi; psi[spin*3 + colour], h[spin*3 + colour].
template <int MU, int S, class T>
__host__ __device__ __forceinline__ void project(const cpx<T> p[12], cpx<T> h[6]) {
    constexpr T s = static_cast<T>(S);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cpx<T> p0 = p[a], p1 = p[3 + a], p2 = p[6 + a], p3 = p[9 + a];
        if constexpr (MU == 0) {        // A = -i sigma_1:  A psi_dn = (-i p3, -i p2)
            h[a] = p0 + s * mul_i(p3);
            h[3 + a] = p1 + s * mul_i(p2);
        } else if constexpr (MU == 1) { // A = -i sigma_2 = [[0,-1],[1,0]]: A psi_dn = (-p3, p2)
            h[a] = p0 + s * p3;
            h[3 + a] = p1 - s * p2;
        } else if constexpr (MU == 2) { // A = -i sigma_3 = diag(-i, i): A psi_dn = (-i p2, i p3)
            h[a] = p0 + s * mul_i(p2);
            h[3 + a] = p1 - s * mul_i(p3);
        } else {                        // A = 1
            h[a] = p0 - s * p2;
            h[3 + a] = p1 - s * p3;
        }
    }
}

// acc += (1 - S gamma_MU) spinor whose upper half is g (lower half = -S A^dag g); FIRST: acc = it
// (adding to zeros costs an instruction per real).
template <int MU, int S, bool FIRST = false, class T>
__host__ __device__ __forceinline__ void accumulate(cpx<T> acc[12], const cpx<T> g[6]) {
    constexpr T s = static_cast<T>(S);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cpx<T> g0 = g[a], g1 = g[3 + a];
        cpx<T> l0, l1;                  // A^dag g
        if constexpr (MU == 0) {        // A^dag = i sigma_1: A^dag g = (i g1, i g0)
            l0 = mul_i(g1);
            l1 = mul_i(g0);
        } else if constexpr (MU == 1) { // A^dag = [[0,1],[-1,0]]: A^dag g = (g1, -g0)
            l0 = g1;
            l1 = T(-1) * g0;
        } else if constexpr (MU == 2) { // A^dag = diag(i, -i): A^dag g = (i g0, -i g1)
            l0 = mul_i(g0);
            l1 = T(-1) * mul_i(g1);
        } else {
            l0 = g0;
            l1 = g1;
        }
        if constexpr (FIRST) {
            acc[a] = g0;
            acc[3 + a] = g1;
            acc[6 + a] = T(-1) * (s * l0);
            acc[9 + a] = T(-1) * (s * l1);
        } else {
            acc[a] = acc[a] + g0;
            acc[3 + a] = acc[3 + a] + g1;
            acc[6 + a] = acc[6 + a] - s * l0;
            acc[9 + a] = acc[9 + a] - s * l1;
        }
    }
}

// g = U h for both spin rows (U row-major u[row*3 + col]).
template <class T>
__host__ __device__ __forceinline__ void su3_mul(const cpx<T> u[9], const cpx<T> h[6], cpx<T> g[6]) {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            g[3 * sp + a] = cfma(u[3 * a + 2], h[3 * sp + 2], cfma(u[3 * a + 1], h[3 * sp + 1], cmul(u[3 * a], h[3 * sp])));
}

// g = U^dag h.
template <class T>
__host__ __device__ __forceinline__ void su3_dag_mul(const cpx<T> u[9], const cpx<T> h[6], cpx<T> g[6]) {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            g[3 * sp + a] = cjfma(u[6 + a], h[3 * sp + 2], cjfma(u[3 + a], h[3 * sp + 1], cjmul(u[a], h[3 * sp])));
}

// Neighbour indices of site s on the periodic lattice (x fastest).
struct Nbr {
    int fwd[4], bwd[4];
};

__host__ __device__ __forceinline__ Nbr neighbours(int s, int nx, int ny, int nz, int nt) {
    Nbr n;
    const int sxy = nx * ny, sxyz = sxy * nz;
    const int x = s % nx, y = (s / nx) % ny, z = (s / sxy) % nz, t = s / sxyz;
    n.fwd[0] = (x == nx - 1) ? s - (nx - 1) : s + 1;
    n.bwd[0] = (x == 0) ? s + (nx - 1) : s - 1;
    n.fwd[1] = (y == ny - 1) ? s - (ny - 1) * nx : s + nx;
    n.bwd[1] = (y == 0) ? s + (ny - 1) * nx : s - nx;
    n.fwd[2] = (z == nz - 1) ? s - (nz - 1) * sxy : s + sxy;
    n.bwd[2] = (z == 0) ? s + (nz - 1) * sxy : s - sxy;
    n.fwd[3] = (t == nt - 1) ? s - (nt - 1) * sxyz : s + sxyz;
    n.bwd[3] = (t == 0) ? s + (nt - 1) * sxyz : s - sxyz;
    return n;
}

// ------------------------------------------------------------------ sites of a block
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
