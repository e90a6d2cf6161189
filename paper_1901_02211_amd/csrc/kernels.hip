// Device kernels of the overlap charge-density path on gfx950 (CDNA4, wave64).
//
//  k_dslash_rl     Wilson stencil D_W / D_W^dag (section 1, Eq. 3) in FP64 and FP32, one site per
//                  thread: on xy-tiles staged in LDS, or on consecutive sites of any lattice
//  k_dslash_f32_*  FP32 stencils that hold a site's eight links in registers for several
//                  right-hand sides: one 16x16 xy-plane per block in LDS (_plane; _plane_xyl with
//                  its x and y links there too), xy-tiles of any width <= 64 with halo rows (_tile).
//                  All take an optional epilogue "+ sigma aux" with a fused <aux, out> partial for
//                  H^2 + sigma (Eq. 4).
//  k_cg_init ...   multi-shift CG for (D_W^dag D_W + q_i) x_i = b (Eqs. 6-8): the stencil
//                  epilogues sum <p, A p> = |D_W p|^2 + s0 |p|^2 in the first stencil and
//                  update the residual in the second; scalar recurrences on the device (one wave
//                  per right-hand side); every K iterations one update of all active shifts'
//                  directions and of y = c_0 b + sum_i c_i x_i from the residuals kept since the
//                  last one; FP64 residual replacement.
//  k_contract      q(x) += 1/2 [gamma5 D_ov phi](x, alpha, a) on the probed sites (Eq. 16), or
//                  the probing estimate of tr D_W^-1 (x, x) from the unshifted solve.
//  k_multi_dot ... low-mode deflation: many dot products and linear combinations at once
//                  (Lanczos reorthogonalisation, Ritz vectors), deflated sources and terms.
//  k_block_mean_abs  locality of D_ov (Eq. 12): mean |D_ov(x, . ; y, .)| per site.
//
// Vectors that a kernel touches once (search directions, residuals, running sums, stencil
// outputs) use non-temporal loads and stores; stencil inputs and links stay cached, since
// neighbouring sites and right-hand-side groups reuse them through L2.
// Reductions are two-pass and fixed-order (per-block partials, then one wave per
// right-hand side), so every FP64 result is bitwise reproducible from run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <type_traits>

#include "kernels.h"
#include "wilson_site.h"

namespace smpq {

// ------------------------------------------------------------------ storage units
// A storage unit (16 bytes) of site s of a plane that starts at a block-uniform address: the
// address stays in scalar registers and the site's byte offset in 32 bits (V < 2^27), one vector
// register for every plane instead of a 64-bit sum for each.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <class W, class V>
__device__ __forceinline__ W *at_site(V *plane, int s) {
    using bytes = typename std::conditional<std::is_const<W>::value, const char, char>::type;
    return reinterpret_cast<W *>(reinterpret_cast<bytes *>(plane) + (unsigned)s * 16u);
}
__device__ __forceinline__ double2 unit_get(const double2 *plane, int s) { return *at_site<const double2>(plane, s); }
__device__ __forceinline__ float4 unit_get(const float4 *plane, int s) { return *at_site<const float4>(plane, s); }
__device__ __forceinline__ f64x2 unit_get_nt(const double2 *plane, int s) {
    return __builtin_nontemporal_load(at_site<const f64x2>(plane, s));
}
__device__ __forceinline__ f32x4 unit_get_nt(const float4 *plane, int s) {
    return __builtin_nontemporal_load(at_site<const f32x4>(plane, s));
}

// One storage unit of a spinor: FP64 one complex (double2), FP32 two complexes (float4).  _stream:
// non-temporal, for vectors a kernel touches once.
__device__ __forceinline__ void unit_load(const double2 *p, size_t vs, int k, int s, cpx<double> v[1]) {
    const double2 t = unit_get(p + k * vs, s);
    v[0] = {t.x, t.y};
}
__device__ __forceinline__ void unit_load(const float4 *p, size_t vs, int k, int s, cpx<float> v[2]) {
    const float4 t = unit_get(p + k * vs, s);
    v[0] = {t.x, t.y};
    v[1] = {t.z, t.w};
}
__device__ __forceinline__ void unit_load_stream(const double2 *p, size_t vs, int k, int s, cpx<double> v[1]) {
    const f64x2 t = unit_get_nt(p + k * vs, s);
    v[0] = {t.x, t.y};
}
__device__ __forceinline__ void unit_load_stream(const float4 *p, size_t vs, int k, int s, cpx<float> v[2]) {
    const f32x4 t = unit_get_nt(p + k * vs, s);
    v[0] = {t.x, t.y};
    v[1] = {t.z, t.w};
}
__device__ __forceinline__ void unit_store_stream(double2 *p, size_t vs, int k, int s, const cpx<double> v[1]) {
    const f64x2 t = {v[0].re, v[0].im};
    __builtin_nontemporal_store(t, at_site<f64x2>(p + k * vs, s));
}
__device__ __forceinline__ void unit_store_stream(float4 *p, size_t vs, int k, int s, const cpx<float> v[2]) {
    const f32x4 t = {v[0].re, v[0].im, v[1].re, v[1].im};
    __builtin_nontemporal_store(t, at_site<f32x4>(p + k * vs, s));
}

template <class T>
struct Store;

template <>
struct Store<double> {
    using vec = double2;
    using link = double2;
    static constexpr int units = 12;
    __device__ static __forceinline__ void load(const double2 *p, size_t vs, int s, cpx<double> v[12]) {
#pragma unroll
        for (int c = 0; c < 12; ++c) unit_load(p, vs, c, s, v + c);
    }
};

template <>
struct Store<float> {
    using vec = float4;
    using link = float4;   // two rows of the SU(3) link: (u00,u01), (u02,u10), (u11,u12)
    static constexpr int units = 6;
    __device__ static __forceinline__ void load(const float4 *p, size_t vs, int s, cpx<float> v[12]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) unit_load(p, vs, k, s, v + 2 * k);
    }
};

// FP64 links: all nine entries, [mu][row*3 + col][site] double2.
// FP32 links: the first two rows, [mu][3][site] float4; the third row is rebuilt as
// conj(row0 x row1), exact for a special unitary matrix.
__device__ __forceinline__ void unpack_rows(float4 a, float4 b, float4 c, cpx<float> u[9]) {
    u[0] = {a.x, a.y};
    u[1] = {a.z, a.w};
    u[2] = {b.x, b.y};
    u[3] = {b.z, b.w};
    u[4] = {c.x, c.y};
    u[5] = {c.z, c.w};
    const cpx<float> r0 = cfma(u[1], u[5], -1.0f * cmul(u[2], u[4]));
    const cpx<float> r1 = cfma(u[2], u[3], -1.0f * cmul(u[0], u[5]));
    const cpx<float> r2 = cfma(u[0], u[4], -1.0f * cmul(u[1], u[3]));
    u[6] = {r0.re, -r0.im};
    u[7] = {r1.re, -r1.im};
    u[8] = {r2.re, -r2.im};
}

template <class T>
__device__ __forceinline__ void load_link(const typename Store<T>::link *U, int V, int mu, int s, cpx<T> u[9]);

template <>
__device__ __forceinline__ void load_link<double>(const double2 *U, int V, int mu, int s, cpx<double> u[9]) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 t = unit_get(U + (size_t)(mu * 9 + k) * V, s);
        u[k] = {t.x, t.y};
    }
}

template <>
__device__ __forceinline__ void load_link<float>(const float4 *U, int V, int mu, int s, cpx<float> u[9]) {
    unpack_rows(unit_get(U + (size_t)(mu * 3) * V, s), unit_get(U + (size_t)(mu * 3 + 1) * V, s),
                unit_get(U + (size_t)(mu * 3 + 2) * V, s), u);
}

// Hardware dispatches consecutive workgroups round-robin over the 8 XCDs; give each XCD
// a contiguous range of sites so that stencil neighbours share that XCD's L2.
__device__ __forceinline__ int xcd_swizzle(int b, int nb) {
    const int q = nb >> 3, r = nb & 7, xcd = b & 7, k = b >> 3;
    return xcd * q + (xcd < r ? xcd : r) + k;
}

// Neighbours of site s = (x, y) of the (z, t) plane pl = z + nz t without per-thread integer
// divisions (the plane is uniform over a block, so the z and t offsets are too).  The tile
// kernels read the +x and +y neighbours from LDS: fwd[0] and fwd[1] are left at s.
__device__ __forceinline__ Nbr plane_neighbours(int s, int x, int y, int pl, int nx, int ny, int nz, int nt) {
    const int zc = pl % nz, tc = pl / nz;
    const int sxy = nx * ny, sxyz = sxy * nz;
    Nbr nb;
    nb.fwd[0] = nb.fwd[1] = s;
    nb.bwd[0] = x == 0 ? s + (nx - 1) : s - 1;
    nb.bwd[1] = y == 0 ? s + (ny - 1) * nx : s - nx;
    nb.fwd[2] = s + (zc == nz - 1 ? -(nz - 1) * sxy : sxy);
    nb.bwd[2] = s + (zc == 0 ? (nz - 1) * sxy : -sxy);
    nb.fwd[3] = s + (tc == nt - 1 ? -(nt - 1) * sxyz : sxyz);
    nb.bwd[3] = s + (tc == 0 ? (nt - 1) * sxyz : -sxyz);
    return nb;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Sum of n partials in a fixed order by one wave (lane l takes l, l+64, ...).
__device__ __forceinline__ double wave_sum_partials(const double *p, int n) {
    double v = 0.0;
    for (int i = threadIdx.x & 63; i < n; i += 64) v += p[i];
    return wave_sum(v);
}

// alpha = |r|^2 / <p, A p> from the first stencil's partials; not ok (breakdown) unless the
// product is positive and finite.  Every wave that sums them gets the same value.
__device__ __forceinline__ double step_length(const double *pap_partials, int npart, double rr, bool &ok) {
    const double pap = wave_sum_partials(pap_partials, npart);
    ok = pap > 0.0 && isfinite(pap);
    return rr / pap;
}

__device__ __forceinline__ int slot_of(const Slots &sl, int k) { return sl.list ? sl.list[k] : k; }
__device__ __forceinline__ int slot_count(const Slots &sl) { return sl.count ? *sl.count : sl.n; }

// ------------------------------------------------------------------ stencil epilogues
// At one site, d = [D in](s) (D_W, or D_W^dag) and self = in(s):
//   EPI 0  out = d
//   EPI 1  out = d + sigma aux;                         returns Re <aux, out>(s)
//   EPI 3  out = d;                                     returns |d|^2 + sigma |self|^2
//   EPI 2  a = d + sigma aux, not stored; out = r - alpha a with the residual r at out + r_ofs;
//          returns |r - alpha a|^2 (a slot whose status is not OK keeps r: alpha is taken as 0)
// In a CG iteration on H^2 + sigma (D_W^dag D_W + sigma) the first stencil D_W p with EPI 3
// yields <p, (H^2 + sigma) p> = |D_W p|^2 + sigma |p|^2, so alpha is known before the second
// stencil, which with EPI 2 updates r directly and never writes (H^2 + sigma) p.  The vectors
// are read and written one storage unit at a time, so that few extra registers are live.
template <class T>
__device__ __forceinline__ double norm2(cpx<T> v) {
    return (double)v.re * (double)v.re + (double)v.im * (double)v.im;
}
// one entry's share of |d|^2 + sigma |e|^2
template <class T>
__device__ __forceinline__ double norm_term(cpx<T> d, cpx<T> e, T sigma) {
    return (double)d.re * (double)d.re + (double)d.im * (double)d.im +
           (double)sigma * ((double)e.re * (double)e.re + (double)e.im * (double)e.im);
}
// epilogues 3 and 2 on a spinor in registers (k_cg_small), the same sums in the same order
template <class T>
__device__ __forceinline__ double norm_step(const cpx<T> d[12], const cpx<T> self[12], T sigma) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 12; ++c) acc += norm_term(d[c], self[c], sigma);
    return acc;
}
template <class T>
__device__ __forceinline__ double residual_step(cpx<T> d[12], const cpx<T> a[12], cpx<T> r[12], T sigma, T alpha) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        d[c] = d[c] + sigma * a[c];
        r[c] = r[c] - alpha * d[c];
        acc += norm2(r[c]);
    }
    return acc;
}

template <class T, int EPI>
__device__ __forceinline__ double stencil_epilogue(cpx<T> d[12], const cpx<T> self[12],
                                                   const typename Store<T>::vec *aux,
                                                   typename Store<T>::vec *out, size_t vs, int s, T sigma,
                                                   T alpha, bool ok, ptrdiff_t r_ofs) {
    constexpr int UN = Store<T>::units, CU = 12 / UN;   // units per spinor, complexes per unit
    double acc = 0.0;
    if constexpr (EPI == 2) {
        if (!ok) alpha = T(0);   // a broken-down slot keeps its residual
    }
#pragma unroll
    for (int k = 0; k < UN; ++k) {
        cpx<T> *dk = d + k * CU;
        if constexpr (EPI == 1 || EPI == 2) {
            cpx<T> a[CU];
            unit_load(aux, vs, k, s, a);
#pragma unroll
            for (int j = 0; j < CU; ++j) {
                dk[j] = dk[j] + sigma * a[j];
                if constexpr (EPI == 1)
                    acc += (double)a[j].re * (double)dk[j].re + (double)a[j].im * (double)dk[j].im;
            }
        }
        if constexpr (EPI == 2) {
            cpx<T> r[CU];
            unit_load_stream(out + r_ofs, vs, k, s, r);
#pragma unroll
            for (int j = 0; j < CU; ++j) {
                r[j] = r[j] - alpha * dk[j];
                acc += norm2(r[j]);
            }
            unit_store_stream(out, vs, k, s, r);
        } else {
            if constexpr (EPI == 3) {
#pragma unroll
                for (int j = 0; j < CU; ++j) {
                    const cpx<T> e = self[k * CU + j];
                    acc += norm_term(dk[j], e, sigma);
                }
            }
            unit_store_stream(out, vs, k, s, dk);
        }
    }
    return acc;
}

// ------------------------------------------------------------------ Wilson stencil
// The hopping term at one site from global memory (the contraction's stencil).
template <int MU, int SF, class T>
__device__ __forceinline__ void hop_dir(const typename Store<T>::link *U, int V, size_t vs,
                                        const typename Store<T>::vec *in, int s, const Nbr &nb, cpx<T> acc[12]) {
    cpx<T> u[9], p[12], h[6], g[6];
    load_link<T>(U, V, MU, s, u);
    Store<T>::load(in, vs, nb.fwd[MU], p);
    project<MU, SF>(p, h);
    su3_mul(u, h, g);
    accumulate<MU, SF>(acc, g);
    load_link<T>(U, V, MU, nb.bwd[MU], u);
    Store<T>::load(in, vs, nb.bwd[MU], p);
    project<MU, -SF>(p, h);
    su3_dag_mul(u, h, g);
    accumulate<MU, -SF>(acc, g);
}

template <class T, int SF>
__device__ __forceinline__ void hop_site(const typename Store<T>::link *U, const Geom &g,
                                         const typename Store<T>::vec *in, int s, cpx<T> acc[12]) {
    const Nbr nb = neighbours(s, g.nx, g.ny, g.nz, g.nt);
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = {T(0), T(0)};
    hop_dir<0, SF, T>(U, g.V, g.vs, in, s, nb, acc);
    hop_dir<1, SF, T>(U, g.V, g.vs, in, s, nb, acc);
    hop_dir<2, SF, T>(U, g.V, g.vs, in, s, nb, acc);
    hop_dir<3, SF, T>(U, g.V, g.vs, in, s, nb, acc);
}

// FP32 stencil on xy-tiles: a block of nx * ty threads (ty = g.tile_y rows, a divisor of ny)
// covers rows y0 .. y0 + ty - 1 of one (z, t) plane, one site per thread.  For each
// right-hand side the block stages those rows plus one halo row on each side (periodic in y)
// in LDS, so the +-x and +-y neighbours come from LDS and only +-z and +-t from global memory
// (their rows are the tiles of the neighbouring planes).  The eight two-row links a site needs
// (U_mu(x) and U_mu(x - mu)) are held in registers and applied to NR right-hand sides in turn.
template <int NR, bool DAG, int EPI>
__global__ __launch_bounds__(kBlock) void k_dslash_f32_tile(const float4 *__restrict__ U, const float4 *__restrict__ in,
                                                            size_t in_stride, size_t in_extra,
                                                            float4 *__restrict__ out, size_t out_stride,
                                                            const float4 *__restrict__ aux, size_t aux_stride,
                                                            size_t aux_extra, Geom g, float kappa, float sigma,
                                                            Slots sl, int nsb, double *__restrict__ partial,
                                                            size_t pstride, const double *__restrict__ alpha,
                                                            const int *__restrict__ status, ptrdiff_t r_ofs,
    const int *__restrict__ done) {
    constexpr int SF = DAG ? -1 : 1;
    constexpr int kTileSites = kBlock + 2 * 64;
    __shared__ float4 tile[6][kTileSites];
    const int L = xcd_swizzle(blockIdx.x, gridDim.x);
    const int sb = L % nsb, rg = L / nsb;
    const int cnt = slot_count(sl);
    const int k0 = rg * NR;
    if (k0 >= cnt) return;  // uniform over the block
    const int nx = g.nx, ny = g.ny, ty = g.tile_y;
    const int tiles_per_plane = ny / ty;
    const int pl = plane_order(sb / tiles_per_plane, g), y0 = (sb % tiles_per_plane) * ty;
    const int x = threadIdx.x % nx, yl = threadIdx.x / nx;
    const int plane0 = pl * nx * ny;
    const int s = plane0 + (y0 + yl) * nx + x;   // every site is valid: V is a multiple of the tile
    const Nbr nb = plane_neighbours(s, x, y0 + yl, pl, nx, ny, g.nz, g.nt);
    // halo loads: threads 0 .. 2nx-1 also fetch row y0 - 1 (first nx) or y0 + ty (next nx)
    const bool halo = (int)threadIdx.x < 2 * nx;
    const int hrow = threadIdx.x < (unsigned)nx ? 0 : ty + 1;
    const int hy = threadIdx.x < (unsigned)nx ? (y0 + ny - 1) % ny : (y0 + ty) % ny;
    const int hsite = plane0 + hy * nx + x;
    const int hl = hrow * nx + x;
    float4 lf[4][3], lb[4][3];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            lf[mu][j] = unit_get(U + (size_t)(mu * 3 + j) * g.V, s);
            lb[mu][j] = unit_get(U + (size_t)(mu * 3 + j) * g.V, nb.bwd[mu]);
        }
    const int me = (yl + 1) * nx + x;
    const int xf = (yl + 1) * nx + (x == nx - 1 ? 0 : x + 1);
    const int xb = (yl + 1) * nx + (x == 0 ? nx - 1 : x - 1);
    const int yf = me + nx, yb = me - nx;
    double dot[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) dot[r] = 0.0;
#pragma unroll 1
    for (int r = 0; r < NR; ++r) {
        const int k = k0 + r;
        if (k >= cnt) break;  // uniform over the block
        const int slot = slot_of(sl, k);
        if (done && done[slot]) continue;  // uniform over the block
        const float4 *src = in + slot * in_stride + in_extra;
        __syncthreads();  // the previous right-hand side is done with the tile
#pragma unroll
        for (int j = 0; j < 6; ++j) tile[j][me] = unit_get(src + j * g.vs, s);
        if (halo) {
#pragma unroll
            for (int j = 0; j < 6; ++j) tile[j][hl] = unit_get(src + j * g.vs, hsite);
        }
        cpx<float> acc[12], u[9], p[12], h[6], w[6];
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = {0.f, 0.f};
#define SMPQ_GLOBAL_HOP(MU)                                                          \
        unpack_rows(lf[MU][0], lf[MU][1], lf[MU][2], u);                             \
        Store<float>::load(src, g.vs, nb.fwd[MU], p);                                \
        project<MU, SF>(p, h);                                                       \
        su3_mul(u, h, w);                                                            \
        accumulate<MU, SF>(acc, w);                                                  \
        unpack_rows(lb[MU][0], lb[MU][1], lb[MU][2], u);                             \
        Store<float>::load(src, g.vs, nb.bwd[MU], p);                                \
        project<MU, -SF>(p, h);                                                      \
        su3_dag_mul(u, h, w);                                                        \
        accumulate<MU, -SF>(acc, w);
        SMPQ_GLOBAL_HOP(2)
        SMPQ_GLOBAL_HOP(3)
#undef SMPQ_GLOBAL_HOP
        __syncthreads();  // the tile is complete
#define SMPQ_TILE_LOAD(L, P)                                                         \
        _Pragma("unroll") for (int j = 0; j < 6; ++j) {                              \
            const float4 t_ = tile[j][L];                                            \
            P[2 * j] = {t_.x, t_.y};                                                 \
            P[2 * j + 1] = {t_.z, t_.w};                                             \
        }
#define SMPQ_TILE_HOP(MU, LF, LB)                                                    \
        unpack_rows(lf[MU][0], lf[MU][1], lf[MU][2], u);                             \
        SMPQ_TILE_LOAD(LF, p)                                                        \
        project<MU, SF>(p, h);                                                       \
        su3_mul(u, h, w);                                                            \
        accumulate<MU, SF>(acc, w);                                                  \
        unpack_rows(lb[MU][0], lb[MU][1], lb[MU][2], u);                             \
        SMPQ_TILE_LOAD(LB, p)                                                        \
        project<MU, -SF>(p, h);                                                      \
        su3_dag_mul(u, h, w);                                                        \
        accumulate<MU, -SF>(acc, w);
        SMPQ_TILE_HOP(0, xf, xb)
        SMPQ_TILE_HOP(1, yf, yb)
#undef SMPQ_TILE_HOP
        cpx<float> v[12];
        SMPQ_TILE_LOAD(me, p)
#undef SMPQ_TILE_LOAD
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = p[c] - kappa * acc[c];
        dot[r] = stencil_epilogue<float, EPI>(v, p, aux + slot * aux_stride + aux_extra, out + slot * out_stride, g.vs,
                                              s, sigma, EPI == 2 ? (float)alpha[slot] : 0.f,
                                              EPI == 2 ? status[slot] == kStatusOK : true, r_ofs);
    }
    if constexpr (EPI != 0) {
        __shared__ double lds[NR][kBlock / 64];
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        const int nw = blockDim.x >> 6;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const double t = wave_sum(dot[r]);
            if (lane == 0) lds[r][wv] = t;
        }
        __syncthreads();
        if ((int)threadIdx.x < NR && k0 + (int)threadIdx.x < cnt) {
            double t = 0.0;
            for (int i = 0; i < nw; ++i) t += lds[threadIdx.x][i];
            partial[(size_t)slot_of(sl, k0 + threadIdx.x) * pstride + sb] = t;
        }
    }
}

template <int NR, bool DAG, int EPI, bool XYL>
__device__ __forceinline__ void dslash_f32_plane_body(const float4 *__restrict__ U, const float4 *__restrict__ in,
                                                             size_t in_stride, size_t in_extra,
                                                             float4 *__restrict__ out, size_t out_stride,
                                                             const float4 *__restrict__ aux, size_t aux_stride,
                                                             size_t aux_extra, Geom g, float kappa, float sigma,
                                                             Slots sl, int nsb, double *__restrict__ partial,
                                                             size_t pstride, const double *__restrict__ alpha,
                                                             const int *__restrict__ status, ptrdiff_t r_ofs,
    const int *__restrict__ done) {
    constexpr int SF = DAG ? -1 : 1;
    __shared__ float4 tile[6][kBlock];
    // XYL: the plane's x and y links in LDS (the backward ones are the neighbours' forward
    // links within the plane), so that fewer registers per thread hold links
    __shared__ float4 lxy[XYL ? 2 : 1][3][XYL ? kBlock : 1];
    const int L = xcd_swizzle(blockIdx.x, gridDim.x);
    const int sb = L % nsb, rg = L / nsb;
    const int cnt = slot_count(sl);
    const int k0 = rg * NR;
    if (k0 >= cnt) return;  // uniform over the block
    const int base = plane_order(sb, g) * kBlock;
    const int s = base + threadIdx.x;  // every site is valid: V is a multiple of the plane
    const Nbr nb = neighbours(s, g.nx, g.ny, g.nz, g.nt);
    float4 lf[4][3], lb[4][3];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (XYL && mu < 2) {
                if constexpr (XYL) lxy[mu][j][threadIdx.x] = unit_get(U + (size_t)(mu * 3 + j) * g.V, s);
                continue;   // visible after the first barrier of the loop below
            }
            lf[mu][j] = unit_get(U + (size_t)(mu * 3 + j) * g.V, s);
            lb[mu][j] = unit_get(U + (size_t)(mu * 3 + j) * g.V, nb.bwd[mu]);
        }
    const int xf = nb.fwd[0] - base, xb = nb.bwd[0] - base, yf = nb.fwd[1] - base, yb = nb.bwd[1] - base;
    // EPI 1: per right-hand side, the block's <aux, out> is summed per wave at once and the
    // wave sums kept in LDS (no accumulators held across the loop)
    __shared__ double ldsdot[EPI != 0 ? NR : 1][kBlock / 64];
    [[maybe_unused]] const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll 1
    for (int r = 0; r < NR; ++r) {
        const int k = k0 + r;
        if (k >= cnt) break;  // uniform over the block
        const int slot = slot_of(sl, k);
        if (done && done[slot]) continue;  // uniform over the block
        const float4 *src = in + slot * in_stride + in_extra;
        __syncthreads();  // the previous right-hand side is done with the tile
#pragma unroll
        for (int j = 0; j < 6; ++j) tile[j][threadIdx.x] = unit_get(src + j * g.vs, s);
        cpx<float> acc[12], u[9], p[12], h[6], w[6];
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = {0.f, 0.f};
#define SMPQ_GLOBAL_HOP(MU)                                                          \
        unpack_rows(lf[MU][0], lf[MU][1], lf[MU][2], u);                             \
        Store<float>::load(src, g.vs, nb.fwd[MU], p);                                \
        project<MU, SF>(p, h);                                                       \
        su3_mul(u, h, w);                                                            \
        accumulate<MU, SF>(acc, w);                                                  \
        unpack_rows(lb[MU][0], lb[MU][1], lb[MU][2], u);                             \
        Store<float>::load(src, g.vs, nb.bwd[MU], p);                                \
        project<MU, -SF>(p, h);                                                      \
        su3_dag_mul(u, h, w);                                                        \
        accumulate<MU, -SF>(acc, w);
        SMPQ_GLOBAL_HOP(2)
        SMPQ_GLOBAL_HOP(3)
#undef SMPQ_GLOBAL_HOP
        __syncthreads();  // the tile is complete
#define SMPQ_TILE_LOAD(L, P)                                                         \
        _Pragma("unroll") for (int j = 0; j < 6; ++j) {                              \
            const float4 t_ = tile[j][L];                                            \
            P[2 * j] = {t_.x, t_.y};                                                 \
            P[2 * j + 1] = {t_.z, t_.w};                                             \
        }
#define SMPQ_TILE_HOP(MU, LF, LB)                                                    \
        if constexpr (XYL) unpack_rows(lxy[MU][0][threadIdx.x], lxy[MU][1][threadIdx.x],  \
                                       lxy[MU][2][threadIdx.x], u);                  \
        else unpack_rows(lf[MU][0], lf[MU][1], lf[MU][2], u);                        \
        SMPQ_TILE_LOAD(LF, p)                                                        \
        project<MU, SF>(p, h);                                                       \
        su3_mul(u, h, w);                                                            \
        accumulate<MU, SF>(acc, w);                                                  \
        if constexpr (XYL) unpack_rows(lxy[MU][0][LB], lxy[MU][1][LB], lxy[MU][2][LB], u); \
        else unpack_rows(lb[MU][0], lb[MU][1], lb[MU][2], u);                        \
        SMPQ_TILE_LOAD(LB, p)                                                        \
        project<MU, -SF>(p, h);                                                      \
        su3_dag_mul(u, h, w);                                                        \
        accumulate<MU, -SF>(acc, w);
        SMPQ_TILE_HOP(0, xf, xb)
        SMPQ_TILE_HOP(1, yf, yb)
#undef SMPQ_TILE_HOP
        cpx<float> v[12];
        SMPQ_TILE_LOAD(threadIdx.x, p)
#undef SMPQ_TILE_LOAD
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = p[c] - kappa * acc[c];
        double d = stencil_epilogue<float, EPI>(v, p, aux + slot * aux_stride + aux_extra, out + slot * out_stride,
                                                g.vs, s, sigma, EPI == 2 ? (float)alpha[slot] : 0.f,
                                                EPI == 2 ? status[slot] == kStatusOK : true, r_ofs);
        if constexpr (EPI != 0) {
            d = wave_sum(d);
            if (lane == 0) ldsdot[r][wv] = d;
        }
    }
    if constexpr (EPI != 0) {
        __syncthreads();
        if ((int)threadIdx.x < NR && k0 + (int)threadIdx.x < cnt) {
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < kBlock / 64; ++i) t += ldsdot[threadIdx.x][i];
            partial[(size_t)slot_of(sl, k0 + threadIdx.x) * pstride + sb] = t;
        }
    }
}


template <int NR, bool DAG, int EPI>
__global__ __launch_bounds__(kBlock) void k_dslash_f32_plane(const float4 *__restrict__ U, const float4 *__restrict__ in,
                                                             size_t in_stride, size_t in_extra,
                                                             float4 *__restrict__ out, size_t out_stride,
                                                             const float4 *__restrict__ aux, size_t aux_stride,
                                                             size_t aux_extra, Geom g, float kappa, float sigma,
                                                             Slots sl, int nsb, double *__restrict__ partial,
                                                             size_t pstride, const double *__restrict__ alpha,
                                                             const int *__restrict__ status, ptrdiff_t r_ofs,
    const int *__restrict__ done) {
    dslash_f32_plane_body<NR, DAG, EPI, false>(U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra,
                                               g, kappa, sigma, sl, nsb, partial, pstride, alpha, status, r_ofs, done);
}

// The same with the x and y links in LDS, at 3 waves per SIMD.
template <int NR, bool DAG, int EPI>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_dslash_f32_plane_xyl(
    const float4 *__restrict__ U, const float4 *__restrict__ in, size_t in_stride, size_t in_extra,
    float4 *__restrict__ out, size_t out_stride, const float4 *__restrict__ aux, size_t aux_stride, size_t aux_extra,
    Geom g, float kappa, float sigma, Slots sl, int nsb, double *__restrict__ partial, size_t pstride,
    const double *__restrict__ alpha, const int *__restrict__ status, ptrdiff_t r_ofs,
    const int *__restrict__ done) {
    dslash_f32_plane_body<NR, DAG, EPI, true>(U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra,
                                              g, kappa, sigma, sl, nsb, partial, pstride, alpha, status, r_ofs, done);
}

// Stencil with the links read for every right-hand side (or pair of them) instead of held in
// registers, one site per thread, the block's sites staged in LDS so that the +-x and +-y
// neighbours come from there and only +-z and +-t from global memory.  TILE: the blocks' sites,
//   kTileExact  nx * ty sites, a multiple of 64, of one (z, t) plane (FP64 kind 1, FP32 kind 4)
//   kTileAny    the same for any plane, with idle threads: several whole planes where they are small,
//               else ty rows of one plane, the last tile of a plane maybe shorter (kind 0)
//   kTileNone   256 consecutive sites, all neighbours through the caches (kind 0, nx > 128)
// A tile that is not whole planes has one halo row on each side.  Links: in FP32 their first two rows (48
// bytes), the third rebuilt as conj(row0 x row1) (exact for SU(3) up to rounding); in FP64 all nine
// entries (FULL), or two rows (96 of 144 bytes) in the solver's iterations where the caller chose that.
enum { kTileExact, kTileAny, kTileNone };

// u's third row from its first two
__device__ __forceinline__ void third_row(cpx<double> u[9]) {
    const cpx<double> r0 = cfma(u[1], u[5], -1.0 * cmul(u[2], u[4]));
    const cpx<double> r1 = cfma(u[2], u[3], -1.0 * cmul(u[0], u[5]));
    const cpx<double> r2 = cfma(u[0], u[4], -1.0 * cmul(u[1], u[3]));
    u[6] = {r0.re, -r0.im};
    u[7] = {r1.re, -r1.im};
    u[8] = {r2.re, -r2.im};
}
__device__ __forceinline__ void load_link64_rows(const double2 *U, int V, int mu, int s, cpx<double> u[9]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double2 t = unit_get(U + (size_t)(mu * 9 + k) * V, s);
        u[k] = {t.x, t.y};
    }
    third_row(u);
}
template <bool FULL>
__device__ __forceinline__ void load_link_rows(const double2 *U, int V, int mu, int s, cpx<double> u[9]) {
    if constexpr (FULL) load_link<double>(U, V, mu, s, u);
    else load_link64_rows(U, V, mu, s, u);
}
template <bool FULL>
__device__ __forceinline__ void load_link_rows(const float4 *U, int V, int mu, int s, cpx<float> u[9]) {
    load_link<float>(U, V, mu, s, u);
}
// A tile in LDS is held as [site][unit], so that a spinor's units are immediate offsets from one
// address.  Its sites are 96 bytes apart in FP32 and 208 (one unit of padding) in FP64: eight
// lanes' 16-byte accesses then fall on different banks.
template <class T>
constexpr int tile_units = Store<T>::units + (std::is_same<T, double>::value ? 1 : 0);

__device__ __forceinline__ void tile_read(const double2 *tile, int l, cpx<double> p[12]) {
    const double2 *q = tile + l * tile_units<double>;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const double2 t = q[j];
        p[j] = {t.x, t.y};
    }
}
__device__ __forceinline__ void tile_read(const float4 *tile, int l, cpx<float> p[12]) {
    const float4 *q = tile + l * tile_units<float>;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const float4 t = q[j];
        p[2 * j] = {t.x, t.y};
        p[2 * j + 1] = {t.z, t.w};
    }
}

// P right-hand sides are carried at once: two in FP32 where a block has more than one.  Every link
// read, its third row (27 instructions) and the address arithmetic then serve two, and the loads
// of one overlap the products of the other; two accumulators, two spinors and one link fit the 168
// VGPRs of three waves per SIMD, and two tiles of the largest plane (49 KB) three blocks per CU.
// In FP64 the second accumulator would leave one wave per SIMD.
//
// Waves per SIMD the kernel is compiled for: three for a pair in FP32; three for the FP64 solver's
// two epilogues (3 and 2) on tiles with one right-hand side per block, which fit the 168 VGPRs of three
// waves (with rebuilt rows four are spilled) and are 9 % faster so than at two.
template <class T, int P, int EPI, int TILE, bool ONE>
struct RlWaves {
    static constexpr int min = std::is_same<T, double>::value ? ((TILE == kTileExact ? ONE : TILE == kTileAny) && (EPI == 2 || EPI == 3) ? 3 : 1)
                                                              : (P == 2 ? 3 : 1);
};
constexpr int kMaxNR = 8;   // right-hand sides per block

template <class T, int P, bool DAG, int EPI, int TILE, bool FULL, bool ONE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(RlWaves<T, P, EPI, TILE, ONE>::min, 8))) void k_dslash_rl(
    const typename Store<T>::link *__restrict__ U, const typename Store<T>::vec *__restrict__ in, size_t in_stride,
    size_t in_extra, typename Store<T>::vec *__restrict__ out, size_t out_stride,
    const typename Store<T>::vec *__restrict__ aux, size_t aux_stride, size_t aux_extra, Geom g, int nr, int IL, T kappa,
    T sigma, Slots sl, int nsb, double *__restrict__ partial, size_t pstride, ResidualStep rstep,
    const int *__restrict__ done) {
    using vec = typename Store<T>::vec;
    using link = typename Store<T>::link;
    constexpr int SF = DAG ? -1 : 1;
    constexpr int UN = Store<T>::units;
    constexpr bool LDS = TILE != kTileNone;
    const int NR = ONE ? 1 : nr;   // right-hand sides of the block (ONE: no loop, fewer registers live)
    extern __shared__ __align__(16) unsigned char tile_raw[];
    vec *tile = reinterpret_cast<vec *>(tile_raw);   // [P][tsites][tile_units]
    constexpr int TU = tile_units<T>;
    const int L = xcd_swizzle(blockIdx.x, gridDim.x);
    // block order: groups of IL right-hand-side groups, tiles, then the IL groups of one tile
    // fastest (IL = 1: the tiles of one right-hand-side group in a row)
    const int grp = L / (nsb * IL), rem = L - grp * nsb * IL;
    const int sb = rem / IL, rg = grp * IL + (rem - sb * IL);
    const int cnt = slot_count(sl);
    const int k0 = rg * NR;
    if (k0 >= cnt) return;  // uniform over the block
    int s, tsites = 0;
    Nbr nb;
    [[maybe_unused]] int me = 0, xf = 0, xb = 0, yf = 0, yb = 0, hsite = 0, hl = 0;
    [[maybe_unused]] bool halo = false, site_ok = true;
    if constexpr (LDS) {
        const int nx = g.nx, ny = g.ny;
        int ty = g.tile_y, m = 1;
        if constexpr (TILE == kTileAny) any_tile(g, ty, m);
        const bool whole = ty == ny;             // whole planes: y wraps inside the tile
        const int rows = whole ? ty : ty + 2;    // rows of a plane held in LDS
        tsites = m * rows * nx;
        int pl, y0, here = ty, i = threadIdx.x, mi = 0;
        if constexpr (TILE == kTileAny) {
            const AnySite a = any_site(g, ty, m, sb, threadIdx.x);
            pl = a.pl;
            y0 = a.y0;
            here = a.here;
            i = a.i;
            mi = a.mi;
            site_ok = a.ok;              // idle: the tile's first site, nothing stored
        } else {
            const int tiles_per_plane = ny / ty;
            pl = plane_order(sb / tiles_per_plane, g);
            y0 = (sb % tiles_per_plane) * ty;
        }
        const bool halo_thread = !whole && (int)threadIdx.x < 2 * nx;
        const int x = i % nx, yl = i / nx;
        const int plane0 = pl * nx * ny;
        s = plane0 + (y0 + yl) * nx + x;
        nb = plane_neighbours(s, x, y0 + yl, pl, nx, ny, g.nz, g.nt);
        // LDS row of tile row yl: shifted by the lower halo row when there is one
        const int off = mi * rows + (whole ? 0 : 1);
        me = (yl + off) * nx + x;
        xf = (yl + off) * nx + (x == nx - 1 ? 0 : x + 1);
        xb = (yl + off) * nx + (x == 0 ? nx - 1 : x - 1);
        yf = whole ? (off + (yl + 1) % ty) * nx + x : me + nx;
        yb = whole ? (off + (yl + ty - 1) % ty) * nx + x : me - nx;
        halo = halo_thread;
        const int hx = threadIdx.x % nx;
        const int hrow = threadIdx.x < (unsigned)nx ? 0 : here + 1;
        const int hy = threadIdx.x < (unsigned)nx ? (y0 + ny - 1) % ny : (y0 + here) % ny;
        hsite = plane0 + hy * nx + hx;
        hl = hrow * nx + hx;
    } else {
        s = sb * kBlock + threadIdx.x;
        site_ok = s < g.V;
        s = site_ok ? s : 0;   // threads past the last site compute site 0 and store nothing
        nb = neighbours(s, g.nx, g.ny, g.nz, g.nt);
    }
    __shared__ double ldsdot[EPI != 0 ? kMaxNR : 1][kBlock / 64];
    [[maybe_unused]] const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    [[maybe_unused]] const int nw = blockDim.x >> 6;
#pragma unroll 1
    for (int r = 0; r < NR; r += P) {
        const int k = k0 + r;
        if (k >= cnt) break;  // uniform over the block
        // the P right-hand sides of this turn; one that is missing or done takes the other's
        // vectors and stores nothing
        int slot[P];
        bool live[P];
        bool any = false;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            live[q] = k + q < cnt && r + q < NR;
            slot[q] = live[q] ? slot_of(sl, k + q) : 0;
            live[q] = live[q] && !(done && done[slot[q]]);
            any = any || live[q];
        }
        if (!any) continue;  // uniform over the block
        const vec *src[P];
#pragma unroll
        for (int q = 0; q < P; ++q) {
            if (P == 2 && !live[q]) slot[q] = slot[P - 1 - q];
            src[q] = in + slot[q] * in_stride + in_extra;
        }
        // the links are re-read for every turn: an empty asm makes the base pointer opaque in
        // each iteration, so that the compiler does not hoist all eight links out of the loop
        // into registers
        const link *Ur = U;
        asm volatile("" : "+s"(Ur));
        if constexpr (LDS) {
            __syncthreads();  // the previous turn is done with the tile
#pragma unroll
            for (int q = 0; q < P; ++q) {
#pragma unroll
                for (int j = 0; j < UN; ++j) tile[(q * tsites + me) * TU + j] = unit_get(src[q] + j * g.vs, s);
                if (halo) {
#pragma unroll
                    for (int j = 0; j < UN; ++j) tile[(q * tsites + hl) * TU + j] = unit_get(src[q] + j * g.vs, hsite);
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // the staging loads are not held across the hops
        }
        cpx<T> acc[P][12], u[9], p[P][12], h[6], w[6];
#define SMPQ_HOPQ(MU, Q)                                                             \
        project<MU, SF>(p[Q], h);                                                    \
        su3_mul(u, h, w);                                                            \
        accumulate<MU, SF, MU == 2>(acc[Q], w);
#define SMPQ_HOPQ_B(MU, Q)                                                           \
        project<MU, -SF>(p[Q], h);                                                   \
        su3_dag_mul(u, h, w);                                                        \
        accumulate<MU, -SF>(acc[Q], w);
#define SMPQ_HOPT(MU, LOADF, LOADB)                                                  \
        load_link_rows<FULL>(Ur, g.V, MU, s, u);                                           \
        LOADF(0)                                                                     \
        if constexpr (P == 2) { LOADF(P - 1) }                                       \
        SMPQ_HOPQ(MU, 0)                                                             \
        if constexpr (P == 2) { SMPQ_HOPQ(MU, P - 1) }                               \
        load_link_rows<FULL>(Ur, g.V, MU, nb.bwd[MU], u);                                  \
        LOADB(0)                                                                     \
        if constexpr (P == 2) { LOADB(P - 1) }                                       \
        SMPQ_HOPQ_B(MU, 0)                                                           \
        if constexpr (P == 2) { SMPQ_HOPQ_B(MU, P - 1) }
#define SMPQ_G2F(Q) Store<T>::load(src[Q], g.vs, nb.fwd[2], p[Q]);
#define SMPQ_G2B(Q) Store<T>::load(src[Q], g.vs, nb.bwd[2], p[Q]);
#define SMPQ_G3F(Q) Store<T>::load(src[Q], g.vs, nb.fwd[3], p[Q]);
#define SMPQ_G3B(Q) Store<T>::load(src[Q], g.vs, nb.bwd[3], p[Q]);
#define SMPQ_T(Q, L_, G_)                                                            \
        if constexpr (LDS) { tile_read(tile + (Q) * tsites * TU, L_, p[Q]); }                \
        else { Store<T>::load(src[Q], g.vs, G_, p[Q]); }
#define SMPQ_T0F(Q) SMPQ_T(Q, xf, nb.fwd[0])
#define SMPQ_T0B(Q) SMPQ_T(Q, xb, nb.bwd[0])
#define SMPQ_T1F(Q) SMPQ_T(Q, yf, nb.fwd[1])
#define SMPQ_T1B(Q) SMPQ_T(Q, yb, nb.bwd[1])
        // one direction at a time: loads of later directions hoisted above earlier ones would hold
        // more links and spinors in registers than the occupancy target allows
        SMPQ_HOPT(2, SMPQ_G2F, SMPQ_G2B)
        __builtin_amdgcn_sched_barrier(0);
        SMPQ_HOPT(3, SMPQ_G3F, SMPQ_G3B)
        if constexpr (LDS) __syncthreads();  // the tile is complete
        else __builtin_amdgcn_sched_barrier(0);
        SMPQ_HOPT(0, SMPQ_T0F, SMPQ_T0B)
        __builtin_amdgcn_sched_barrier(0);
        SMPQ_HOPT(1, SMPQ_T1F, SMPQ_T1B)
        {
            // the sums are complete here: without this the compiler sinks their arithmetic into
            // the conditional stores below, past every scheduling barrier, and spills
#pragma unroll
            for (int q = 0; q < P; ++q)
#pragma unroll
                for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(acc[q][c].re), "+v"(acc[q][c].im));
        }
#pragma unroll
        for (int q = 0; q < P; ++q) {
            if (P > 1 && !live[q]) continue;  // uniform over the block
            cpx<T> v[12];
            SMPQ_T(q, me, s)
#pragma unroll
            for (int c = 0; c < 12; ++c) v[c] = p[q][c] - kappa * acc[q][c];
            T al = T(0);   // epilogue 2: the step along p, 0 after a breakdown
            if constexpr (EPI == 2) {
                if (rstep.npart > 0) {
                    bool ok;
                    const double a = step_length(rstep.pap + (size_t)slot[q] * pstride, rstep.npart,
                                                 rstep.rr[slot[q]], ok);
                    al = ok ? (T)a : T(0);
                } else {
                    al = rstep.status[slot[q]] == kStatusOK ? (T)rstep.alpha[slot[q]] : T(0);
                }
            }
            double d = 0.0;
            if (TILE == kTileExact || site_ok)
                d = stencil_epilogue<T, EPI>(v, p[q], aux + slot[q] * aux_stride + aux_extra,
                                             out + slot[q] * out_stride, g.vs, s, sigma, al,
                                             true, rstep.r_ofs);
            if constexpr (EPI != 0) {
                d = wave_sum(d);
                if (lane == 0) ldsdot[r + q][wv] = d;
            }
        }
#undef SMPQ_T1B
#undef SMPQ_T1F
#undef SMPQ_T0B
#undef SMPQ_T0F
#undef SMPQ_T
#undef SMPQ_G3B
#undef SMPQ_G3F
#undef SMPQ_G2B
#undef SMPQ_G2F
#undef SMPQ_HOPT
#undef SMPQ_HOPQ_B
#undef SMPQ_HOPQ
    }
    if constexpr (EPI != 0) {
        __syncthreads();
        if ((int)threadIdx.x < NR && k0 + (int)threadIdx.x < cnt) {
            double t = 0.0;
            for (int i = 0; i < nw; ++i) t += ldsdot[threadIdx.x][i];
            partial[(size_t)slot_of(sl, k0 + threadIdx.x) * pstride + sb] = t;
        }
    }
}

__host__ __device__ int site_blocks(const Geom &g) { return (g.V + kBlock - 1) / kBlock; }
size_t partial_stride(const Geom &g) { return (size_t)12 * site_blocks(g); }
bool plane_tileable(const Geom &g) { return g.nx * g.ny == kBlock; }

int tile_rows(int nx, int ny) {
    if (nx > 64) return 0;
    for (int ty = kBlock / nx; ty >= 2; --ty)
        if (ny % ty == 0 && (nx * ty) % 64 == 0) return ty;
    return 0;
}

static int tile_blocks(const Geom &g) { return g.V / (g.nx * g.tile_y); }

// g with the FP32 variant of one direction in f32_kind, f32_nr and f32_il
static Geom for_direction(const Geom &g, int prec, bool dag) {
    Geom d = g;
    if (prec != 0 && dag) {
        d.f32_kind = g.f32_dag_kind;
        d.f32_nr = g.f32_dag_nr;
        d.f32_il = g.f32_dag_il;
    }
    return d;
}

// The variant of a launch on n right-hand sides where none was chosen (g.adapt).  Measured on
// 16^3 x 32 (120 right-hand sides), 24^4 (24), 8^4 (192) and 12^4 (48), per launch:
//  - D_W in FP32: kind 1 with its links in registers for 8 on 16 x 16 planes (0.77 ms against 0.88 with
//    links read per pair), unless that leaves fewer than two blocks per CU; elsewhere the links
//    are read for every right-hand side (8^4: 0.037 ms against 0.062 with kind 2; 24^4: 0.55
//    against 0.60)
//  - D_W^dag in FP32: links read per pair on 256-site tiles where that leaves eight blocks per CU
//    (1.33 ms against 1.75 with kind 1), else for every right-hand side (8^4: 0.070 against 0.149,
//    24^4: 0.75 against 1.20)
//  - FP64: links read for every right-hand side, two in turn where a tile is one wave and there are
//    many (a whole 8^4 map 74.4 ms against 76.9; 24^4, larger tiles: 901 against 822)
//  - any-lattice tiles in FP32: one right-hand side per block; two per link read leave half as many blocks
//    and are 0 to 20 % slower in whole solves of 12 to 96 right-hand sides (10^4 x 12 12.6 ms against
//    10.9, 6 x 10 x 6 x 14 x 96 30.5 against 28.2) and within 2 % with more (12^4 x 192 202 against 205)
//  - tiles: exact ones where they fit, else kTileAny (12^4 in FP64, two-row links: 0.416 ms a pair of
//    stencils against 0.449 without LDS and with right-hand sides interleaved over the lanes)
//  - two right-hand sides of a tile in a row (interleave 2) wherever links are read for one or two, in FP64
//    four on 16 x 16 planes: whole FP64 links then come from L2 more often (four 12^4 classes 115 -> 105 ms
//    and 48 right-hand sides on 130 x 4^3 69 -> 61 with 2 against 1, 16^4 classes 324 -> 315 with 4
//    against 2; four on 24^4, tiles with halo rows, 822 -> 873); FP32 kind 0 takes 1
// Results do not depend on the choice.
static Geom adapted(Geom d, int prec, bool dag, int n) {
    const bool exact = d.tile_y > 0;
    const int il = n > 1 ? 2 : 1;
    if (prec == 0) {
        d.f64_kind = exact ? 1 : 0;
        d.f64_lgr = 0;
        d.f64_nr = exact && d.nx * d.tile_y == 64 && (long long)tile_blocks(d) * n >= 16 * 256 ? 2 : 1;
        d.f64_il = exact && plane_tileable(d) && n >= 4 ? 4 : il;
        return d;
    }
    const long long work = exact ? (long long)tile_blocks(d) * n : 0;   // tiles x right-hand sides
    if (!dag && plane_tileable(d) && work >= 8 * 512) {
        d.f32_kind = 1;
        d.f32_nr = 8;
        d.f32_il = 1;
    } else {
        d.f32_kind = exact ? 4 : 0;
        d.f32_nr = exact && dag && d.nx * d.tile_y == kBlock && d.tile_y == d.ny && work >= 2 * 2048 ? 2 : 1;
        d.f32_il = exact ? il : 1;
    }
    return d;
}

int dslash_partials(int prec, const Geom &g, bool dag) {
    if (prec == 0) return g.f64_kind == 1 ? tile_blocks(g) : any_blocks(g);
    const Geom d = for_direction(g, prec, dag);
    if (d.f32_kind == 0) return any_blocks(d);
    return d.f32_kind == 2 || d.f32_kind == 4 ? tile_blocks(d) : site_blocks(d);
}

// Whether the variant in g's f32_kind or f64_kind can compute alpha itself.
static bool links_per_turn(int prec, const Geom &d) { return prec == 0 || d.f32_kind == 4 || d.f32_kind == 0; }

bool dslash_takes_partials(int prec, const Geom &g, bool dag) {
    return g.adapt ? prec == 0 || dag : links_per_turn(prec, for_direction(g, prec, dag));
}

static bool il_ok(int il) { return il == 1 || il == 2 || il == 4 || il == 8 || il == 16; }

static bool valid_f32(const Geom &g);

bool valid_tuning(int prec, const Geom &g) {
    if (prec != 0) return valid_f32(g) && valid_f32(for_direction(g, prec, true));
    if (g.f64_kind == 1)
        return g.tile_y > 0 && g.tile_y == tile_rows(g.nx, g.ny) && g.band >= 1 && g.nz % g.band == 0 &&
               (g.f64_nr == 1 || g.f64_nr == 2 || g.f64_nr == 4 || g.f64_nr == 8) && il_ok(g.f64_il);
    return g.f64_kind == 0 && g.f64_lgr >= 0 && g.f64_lgr <= 2 && g.f64_il == 1;
}

static bool valid_f32(const Geom &g) {
    if (g.f32_kind != 4 && g.f32_il != 1) return false;   // the interleave applies to kind 4 only
    const bool nr_tile = g.f32_nr == 4 || g.f32_nr == 8 || g.f32_nr == 16;
    if (g.f32_kind == 1 || g.f32_kind == 3) return plane_tileable(g) && nr_tile && g.band >= 1 && g.nz % g.band == 0;
    const bool tiled = g.tile_y > 0 && g.tile_y == tile_rows(g.nx, g.ny);
    const bool band_ok = g.band >= 1 && g.nz % g.band == 0;
    if (g.f32_kind == 2) return tiled && nr_tile && band_ok;
    if (g.f32_kind == 4)
        return tiled && band_ok && (g.f32_nr == 1 || g.f32_nr == 2 || g.f32_nr == 4 || g.f32_nr == 8) && il_ok(g.f32_il);
    return g.f32_kind == 0 && (g.f32_nr == 1 || g.f32_nr == 2 || g.f32_nr == 4 || g.f32_nr == 8);
}

// The kernels that read the links for every turn, nr right-hand sides per block.
template <class T, int P, bool DAG, int EPI, int TILE, bool FULL, bool ONE>
static void launch_rl_t(const void *U, const void *in, size_t in_stride, size_t in_extra, void *out, size_t out_stride,
                        const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g, int nr, int il,
                        double kappa, double sigma, Slots sl, int max_slots, double *partial, const ResidualStep &rstep,
                        const int *done, hipStream_t st) {
    using vec = typename Store<T>::vec;
    using link = typename Store<T>::link;
    int ty = g.tile_y, m = 1;
    if (TILE != kTileExact) any_tile(g, ty, m);
    const int nsb = TILE == kTileExact ? tile_blocks(g) : any_blocks(g);
    // right-hand-side groups, rounded up to whole interleave groups (the extra blocks exit)
    const int ngr = ((max_slots + nr - 1) / nr + il - 1) / il * il;
    const int threads = TILE == kTileNone ? kBlock : (m * g.nx * ty + 63) / 64 * 64;
    const int rows = ty == g.ny ? ty : ty + 2;
    const size_t lds = TILE == kTileNone ? 0 : (size_t)P * m * rows * g.nx * tile_units<T> * sizeof(vec);
    hipLaunchKernelGGL((k_dslash_rl<T, P, DAG, EPI, TILE, FULL, ONE>), dim3(nsb * ngr), dim3(threads), lds, st,
                       (const link *)U, (const vec *)in, in_stride, in_extra, (vec *)out, out_stride, (const vec *)aux,
                       aux_stride, aux_extra, g, nr, il, (T)kappa, (T)sigma, sl, nsb, partial, partial_stride(g), rstep, done);
}

template <class T, bool DAG, int EPI>
static void launch_rl(bool exact, const void *U, const void *in, size_t in_stride, size_t in_extra, void *out,
                      size_t out_stride, const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g, int nr,
                      int il, double kappa, double sigma, Slots sl, int max_slots, double *partial,
                      const ResidualStep &rstep, const int *done, hipStream_t st) {
    const auto go = [&](auto fn) {
        fn(U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra, g, nr, il, kappa, sigma, sl,
           max_slots, partial, rstep, done, st);
    };
    int ty, m;
    any_tile(g, ty, m);
    if constexpr (std::is_same<T, double>::value) {
        // Links are read in full unless the caller chose the tile variant (f64_kind 1), whose iterations
        // (epilogues 2 and 3) rebuild third rows where those of the loaded links are within rounding of it;
        // D_W itself and H^2 + sigma keep the links as loaded.  A rebuilt row takes the error of D_W from
        // 1.7e-16 to 4.8e-16 of its largest entry, and that of D_ov at the finest tolerance from
        // 4.31e-15 to 4.38e-15, for up to 4 % of an FP64 solve (four 16^4 classes, r = 4: 303 ms in full, 290
        // with two rows; four points on 12^4 99.8 and 99.0).
        const bool rows = (EPI == 2 || EPI == 3) && exact && !g.adapt && !g.f64_full;
        if constexpr (EPI == 2 || EPI == 3) {
            if (rows && nr == 1) return go(launch_rl_t<double, 1, DAG, EPI, kTileExact, false, true>);
            if (rows) return go(launch_rl_t<double, 1, DAG, EPI, kTileExact, false, false>);
        }
        if (exact && nr == 1) go(launch_rl_t<double, 1, DAG, EPI, kTileExact, true, true>);
        else if (exact) go(launch_rl_t<double, 1, DAG, EPI, kTileExact, true, false>);
        else if (ty > 0 && nr == 1) go(launch_rl_t<double, 1, DAG, EPI, kTileAny, true, true>);
        else if (ty > 0) go(launch_rl_t<double, 1, DAG, EPI, kTileAny, true, false>);
        else go(launch_rl_t<double, 1, DAG, EPI, kTileNone, true, false>);
    } else {
        if (exact && nr > 1) go(launch_rl_t<float, 2, DAG, EPI, kTileExact, false, false>);
        else if (exact) go(launch_rl_t<float, 1, DAG, EPI, kTileExact, false, true>);
        else if (ty > 0 && nr > 1) go(launch_rl_t<float, 2, DAG, EPI, kTileAny, false, false>);
        else if (ty > 0) go(launch_rl_t<float, 1, DAG, EPI, kTileAny, false, true>);
        else if (nr > 1) go(launch_rl_t<float, 2, DAG, EPI, kTileNone, false, false>);
        else go(launch_rl_t<float, 1, DAG, EPI, kTileNone, false, true>);
    }
}

template <class T, bool DAG, int EPI>
static void launch_dslash_t(const void *U, const void *in, size_t in_stride, size_t in_extra, void *out,
                            size_t out_stride, const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g,
                            double kappa, double sigma, Slots sl, int max_slots, double *partial,
                            const ResidualStep &rstep, const int *done, hipStream_t st) {
    const bool lds = g.f64_kind == 1;
    launch_rl<T, DAG, EPI>(lds, U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra, g,
                           lds ? g.f64_nr : 1 << g.f64_lgr, g.f64_il, kappa, sigma, sl, max_slots, partial,
                           rstep, done, st);
}

template <int NR, bool DAG, int EPI, int KIND>
static void launch_f32(const void *U, const void *in, size_t in_stride, size_t in_extra, void *out, size_t out_stride,
                       const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g, double kappa, double sigma,
                       Slots sl, int max_slots, double *partial, const ResidualStep &rstep, const int *done,
                       hipStream_t st) {
    const int nsb = KIND == 2 ? tile_blocks(g) : site_blocks(g);
    const int ngr = (max_slots + NR - 1) / NR;
    if constexpr (KIND == 2)
        hipLaunchKernelGGL((k_dslash_f32_tile<NR, DAG, EPI>), dim3(nsb * ngr), dim3(g.nx * g.tile_y), 0, st,
                           (const float4 *)U, (const float4 *)in, in_stride, in_extra, (float4 *)out, out_stride,
                           (const float4 *)aux, aux_stride, aux_extra, g, (float)kappa, (float)sigma, sl, nsb, partial,
                           partial_stride(g), rstep.alpha, rstep.status, rstep.r_ofs, done);
    else if constexpr (KIND == 3)
        hipLaunchKernelGGL((k_dslash_f32_plane_xyl<NR, DAG, EPI>), dim3(nsb * ngr), dim3(kBlock), 0, st,
                           (const float4 *)U, (const float4 *)in, in_stride, in_extra, (float4 *)out, out_stride,
                           (const float4 *)aux, aux_stride, aux_extra, g, (float)kappa, (float)sigma, sl, nsb, partial,
                           partial_stride(g), rstep.alpha, rstep.status, rstep.r_ofs, done);
    else if constexpr (KIND == 1)
        hipLaunchKernelGGL((k_dslash_f32_plane<NR, DAG, EPI>), dim3(nsb * ngr), dim3(kBlock), 0, st,
                           (const float4 *)U, (const float4 *)in, in_stride, in_extra, (float4 *)out, out_stride,
                           (const float4 *)aux, aux_stride, aux_extra, g, (float)kappa, (float)sigma, sl, nsb, partial,
                           partial_stride(g), rstep.alpha, rstep.status, rstep.r_ofs, done);
}

template <bool DAG, int EPI>
static void launch_f32_tuned(const void *U, const void *in, size_t in_stride, size_t in_extra, void *out,
                             size_t out_stride, const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g,
                             double kappa, double sigma, Slots sl, int max_slots, double *partial,
                             const ResidualStep &rstep, const int *done, hipStream_t st) {
#define SMPQ_F32(NR, PL)                                                                                       \
    launch_f32<NR, DAG, EPI, PL>(U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra, g, kappa, \
                                 sigma, sl, max_slots, partial, rstep, done, st)
    if (g.f32_kind == 4 || g.f32_kind == 0) {
        launch_rl<float, DAG, EPI>(g.f32_kind == 4, U, in, in_stride, in_extra, out, out_stride, aux, aux_stride,
                                   aux_extra, g, g.f32_nr, g.f32_il, kappa, sigma, sl, max_slots, partial, rstep, done, st);
    } else if (g.f32_kind == 2) {
        if (g.f32_nr == 4) SMPQ_F32(4, 2);
        else if (g.f32_nr == 16) SMPQ_F32(16, 2);
        else SMPQ_F32(8, 2);
    } else if (g.f32_kind == 1) {
        if (g.f32_nr == 4) SMPQ_F32(4, 1);
        else if (g.f32_nr == 16) SMPQ_F32(16, 1);
        else SMPQ_F32(8, 1);
    } else {
        if (g.f32_nr == 4) SMPQ_F32(4, 3);
        else if (g.f32_nr == 16) SMPQ_F32(16, 3);
        else SMPQ_F32(8, 3);
    }
#undef SMPQ_F32
}

void launch_dslash(int prec, bool dag, int epi, const void *U, const void *in, size_t in_stride, size_t in_extra,
                   void *out, size_t out_stride, const void *aux, size_t aux_stride, size_t aux_extra, const Geom &g,
                   double kappa, double sigma, Slots sl, int max_slots, double *partial, hipStream_t st,
                   const ResidualStep &rstep, const int *done) {
    using Fn = void (*)(const void *, const void *, size_t, size_t, void *, size_t, const void *, size_t, size_t,
                        const Geom &, double, double, Slots, int, double *, const ResidualStep &, const int *, hipStream_t);
    if (!g.adapt && !valid_tuning(prec, g)) throw std::invalid_argument("stencil variant does not fit this lattice");
    if (epi < 0 || epi > 3) throw std::invalid_argument("unknown stencil epilogue");
    if (epi == 2 && (rstep.npart > 0 ? !rstep.pap || !rstep.rr : !rstep.alpha || !rstep.status))
        throw std::invalid_argument("the residual epilogue needs alpha and status, or what they follow from");
    // [precision][dagger][epilogue]; the FP32 stencil is built for the combinations the solver,
    // the autotuner and smpq_apply_dw use
    static const Fn table[2][2][4] = {
        {{launch_dslash_t<double, false, 0>, launch_dslash_t<double, false, 1>, launch_dslash_t<double, false, 2>,
          launch_dslash_t<double, false, 3>},
         {launch_dslash_t<double, true, 0>, launch_dslash_t<double, true, 1>, launch_dslash_t<double, true, 2>,
          launch_dslash_t<double, true, 3>}},
        {{launch_f32_tuned<false, 0>, nullptr, nullptr, launch_f32_tuned<false, 3>},
         {launch_f32_tuned<true, 0>, launch_f32_tuned<true, 1>, launch_f32_tuned<true, 2>, nullptr}}};
    const Fn f = table[prec == 0 ? 0 : 1][dag ? 1 : 0][epi];
    if (!f) throw std::invalid_argument("stencil epilogue not built for this precision and direction");
    const Geom d = g.adapt ? adapted(g, prec, dag, max_slots) : for_direction(g, prec, dag);
    if (rstep.npart > 0 && !links_per_turn(prec, d))
        throw std::invalid_argument("this stencil variant needs alpha computed before it");
    f(U, in, in_stride, in_extra, out, out_stride, aux, aux_stride, aux_extra, d, kappa, sigma, sl, max_slots, partial, rstep, done, st);
}

// ------------------------------------------------------------------ element-wise kernels
// Element-wise kernels work on one storage unit per thread: a float4 (two complex
// entries) in FP32 or a double2 (one complex entry) in FP64.  Block b of a slot covers
// unit u = b / nsb and sites (b % nsb)*256 + [0, 256), so a wave reads 64 consecutive
// units of one component plane.
template <class T>
struct Unit {
    using vec = typename Store<T>::vec;
    static constexpr int C = 12 / Store<T>::units;
    __device__ static __forceinline__ void load(const vec *p, size_t vs, int u, int s, cpx<T> *v) {
        unit_load(p, vs, u, s, v);
    }
    __device__ static __forceinline__ void store(vec *p, size_t vs, int u, int s, const cpx<T> *v) {
        if constexpr (C == 1) *at_site<vec>(p + u * vs, s) = make_double2(v[0].re, v[0].im);
        else *at_site<vec>(p + u * vs, s) = make_float4(v[0].re, v[0].im, v[1].re, v[1].im);
    }
    // streamed (non-temporal) vector load/store: data touched once per kernel
    __device__ static __forceinline__ void load_stream(const vec *p, size_t vs, int u, int s, cpx<T> *v) {
        unit_load_stream(p, vs, u, s, v);
    }
    __device__ static __forceinline__ void store_stream(vec *p, size_t vs, int u, int s, const cpx<T> *v) {
        unit_store_stream(p, vs, u, s, v);
    }
};

// FP64 complex entry c of an FP64 spinor (double2 planes), streamed (non-temporal)
__device__ __forceinline__ cpx<double> ld64_stream(const double2 *p, size_t vs, int c, int s) {
    const f64x2 t = unit_get_nt(p + c * vs, s);
    return {t.x, t.y};
}
__device__ __forceinline__ void st64_stream(double2 *p, size_t vs, int c, int s, cpx<double> v) {
    const f64x2 t = {v.re, v.im};
    __builtin_nontemporal_store(t, at_site<f64x2>(p + c * vs, s));
}

// A shifted search direction in 16 bits: one FP32 unit (4 reals) in 8 bytes, holding p / scale.
// Conversions round to nearest even (v_cvt_pk_f16_f32 / v_cvt_pk_bf16_f32 on gfx950).
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
template <int D>
struct Dir16;
template <>
struct Dir16<kDirF16> {
    using v = f16x4;
};
template <>
struct Dir16<kDirBF16> {
    using v = bf16x4;
};

template <int D>
__device__ __forceinline__ void load_dir16(const void *p, size_t vs, int u, int s, float scale, cpx<float> v[2]) {
    using h = typename Dir16<D>::v;
    const h t = __builtin_nontemporal_load(reinterpret_cast<const h *>(p) + u * vs + s);
    const f32x4 f = __builtin_convertvector(t, f32x4);
    v[0] = {f.x * scale, f.y * scale};
    v[1] = {f.z * scale, f.w * scale};
}
template <int D>
__device__ __forceinline__ void store_dir16(void *p, size_t vs, int u, int s, float inv_scale, const cpx<float> v[2]) {
    using h = typename Dir16<D>::v;
    const f32x4 f = {v[0].re * inv_scale, v[0].im * inv_scale, v[1].re * inv_scale, v[1].im * inv_scale};
    __builtin_nontemporal_store(__builtin_convertvector(f, h), reinterpret_cast<h *>(p) + u * vs + s);
}

// FP64 complex entry c of an FP64 spinor (double2 planes)
__device__ __forceinline__ cpx<double> ld64(const double2 *p, size_t vs, int c, int s) {
    const double2 t = unit_get(p + c * vs, s);
    return {t.x, t.y};
}
__device__ __forceinline__ void st64(double2 *p, size_t vs, int c, int s, cpx<double> v) {
    *at_site<double2>(p + c * vs, s) = make_double2(v.re, v.im);
}

__device__ __forceinline__ void block_partial(double v, double *partial, size_t idx) {
    __shared__ double lds[kBlock / 64];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) t += lds[i];
        partial[idx] = t;
    }
}

// Entry c of the source of a slot at site s.
__device__ __forceinline__ cpx<double> source_entry(const Source &src, int slot, int c, int s, size_t vs) {
    cpx<double> v;
    if (src.b) {
        v = ld64(src.b + (size_t)slot * 12 * vs, vs, c, s);
    } else {
        const bool on = (src.colour[s] == src.slot_class[slot]) && (c == src.slot_comp[slot]);
        v = {on ? 1.0 : 0.0, 0.0};
    }
    // deflated modes projected out: b - sum_i <u_i, b> u_i
    for (int i = 0; i < src.dk; ++i) {
        const double2 a = src.dcoef[(size_t)slot * src.dk + i];
        const cpx<double> u = ld64(src.du + (size_t)i * 12 * vs, vs, c, s);
        v.re -= a.x * u.re - a.y * u.im;
        v.im -= a.x * u.im + a.y * u.re;
    }
    return v;
}

int unit_parts(int prec, const Geom &g) { return (prec == 0 ? 12 : 6) * site_blocks(g); }

// r = b, p_i = b for every shift, y = c0 b (FP64), x0 = 0 (FP32 path only; the FP64 path has no
// x0); partial = |b|^2 per block.
template <class T, int D>
__global__ __launch_bounds__(kBlock) void k_cg_init(Geom g, Source src, int NS, double c0,
                                                    typename Store<T>::vec *r, size_t rst,
                                                    typename Store<T>::vec *p, size_t pst, double2 *y, double2 *x0,
                                                    double *partial, size_t pstride) {
    constexpr int C = Unit<T>::C;
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    const size_t rs = Store<T>::units * g.vs;
    double nrm = 0.0;
    if (s < g.V) {
        cpx<T> bt[C];
        double2 *ys = y + (size_t)slot * 12 * g.vs;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int c = u * C + i;
            const cpx<double> b = source_entry(src, slot, c, s, g.vs);
            bt[i] = {(T)b.re, (T)b.im};
            nrm += (double)bt[i].re * bt[i].re + (double)bt[i].im * bt[i].im;
            st64(ys, g.vs, c, s, c0 * b);
            if (x0) st64(x0 + (size_t)slot * 12 * g.vs, g.vs, c, s, {0.0, 0.0});
        }
        Unit<T>::store(r + slot * rst, g.vs, u, s, bt);
        if constexpr (D == kDirF32) {
            for (int i = 0; i < NS; ++i) Unit<T>::store(p + slot * pst + i * rs, g.vs, u, s, bt);
        } else {
            // the base direction; the 16-bit ones follow from r once |b| is known (k_dir16_init)
            Unit<T>::store(p + slot * pst, g.vs, u, s, bt);
        }
    }
    block_partial(nrm, partial, (size_t)slot * pstride + blockIdx.x);
}

void launch_cg_init(int prec, const Geom &g, const Source &src, int nslots, int NS, double c0, void *r, size_t rst,
                    void *p, size_t pst, double2 *y, double2 *x0, double *partial, int dir, hipStream_t st) {
    dim3 grid(unit_parts(prec, g), nslots);
    if (prec == 0) {
        if (dir != kDirF32) throw std::invalid_argument("16-bit directions need the FP32 path");
        hipLaunchKernelGGL((k_cg_init<double, kDirF32>), grid, dim3(kBlock), 0, st, g, src, NS, c0, (double2 *)r, rst,
                           (double2 *)p, pst, y, x0, partial, partial_stride(g));
        return;
    }
    if (dir == kDirF32)
        hipLaunchKernelGGL((k_cg_init<float, kDirF32>), grid, dim3(kBlock), 0, st, g, src, NS, c0, (float4 *)r, rst,
                           (float4 *)p, pst, y, x0, partial, partial_stride(g));
    else   // only the base direction's layout depends on the 16-bit format
        hipLaunchKernelGGL((k_cg_init<float, kDirF16>), grid, dim3(kBlock), 0, st, g, src, NS, c0, (float4 *)r, rst,
                           (float4 *)p, pst, y, x0, partial, partial_stride(g));
}

// 16-bit directions: p_i = b = r for every shift but the base, stored with the scale that
// k_scalars_init set from |b| (so that the entries of any source are near 1).
template <int D>
__global__ __launch_bounds__(kBlock) void k_dir16_init(Geom g, MSState S, const float4 *r, size_t rst, void *ph) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const size_t rs = Store<float>::units * g.vs;
    cpx<float> v[2];
    Unit<float>::load(r + slot * rst, g.vs, u, s, v);
    for (int i = 0; i < S.NS; ++i)
        if (i != S.i0)
            store_dir16<D>(static_cast<typename Dir16<D>::v *>(ph) + ((size_t)slot * S.NS + i) * rs, g.vs, u, s,
                           (float)(1.0 / S.sh_scale[slot * S.NS + i]), v);
}

void launch_dir16_init(const Geom &g, const MSState &s, int nslots, const void *r, size_t rst, int dir, void *ph,
                       hipStream_t st) {
    dim3 grid(unit_parts(1, g), nslots);
    if (dir == kDirF16)
        hipLaunchKernelGGL(k_dir16_init<kDirF16>, grid, dim3(kBlock), 0, st, g, s, (const float4 *)r, rst, ph);
    else if (dir == kDirBF16)
        hipLaunchKernelGGL(k_dir16_init<kDirBF16>, grid, dim3(kBlock), 0, st, g, s, (const float4 *)r, rst, ph);
    else
        throw std::invalid_argument("launch_dir16_init: not a 16-bit format");
}

// ------------------------------------------------------------------ CG scalars (one wave per slot)
// Lane i holds shift i (NS <= 32).  Slots >= nslots are not part of this batch and start finished.
__global__ void k_scalars_init(MSState S, int npart, int nslots) {
    const int slot = blockIdx.x;
    const double rr = slot < nslots ? wave_sum_partials(S.partial + (size_t)slot * S.pstride, npart) : 0.0;
    const int i = threadIdx.x;
    if (i < S.NS) {
        const int k = slot * S.NS + i;
        S.zeta[k] = 1.0;
        S.zeta_prev[k] = 1.0;
        S.sh_active[k] = rr > 0.0;
        S.sh_iters[k] = 0;
        S.sh_scale[k] = rr > 0.0 ? sqrt(rr) * S.dir_norm : 1.0;
    }
    if (i != 0) return;
    S.rr[slot] = rr;
    S.bnorm[slot] = sqrt(rr);
    S.alpha_prev[slot] = 1.0;
    S.beta_prev[slot] = 0.0;
    S.alpha[slot] = 0.0;
    S.beta[slot] = 0.0;
    S.done[slot] = !(rr > 0.0);
    S.iters[slot] = 0;
    S.status[slot] = kStatusOK;
    S.blk_n[slot] = 0;
    S.fl_m[slot] = 0;
    S.fl_act[slot] = rr > 0.0 ? (unsigned)((1ull << S.NS) - 1) : 0u;
    S.cnt_entries[slot] = 0;
    S.cnt_active[slot] = 0;
    S.cnt_fl[slot] = 0;
    S.cnt_fl_r[slot] = 0;
    S.cnt_fl_p[slot] = 0;
}

void launch_scalars_init(const MSState &s, int npart, int nslots, hipStream_t st) {
    hipLaunchKernelGGL(k_scalars_init, dim3(s.B), dim3(64), 0, st, s, npart, nslots);
}

// alpha_k = |r_k|^2 / <p_k, A p_k>.
__global__ void k_scalars_alpha(MSState S, int npart) {
    if ((int)blockIdx.x >= *S.count) return;
    const int slot = S.list[blockIdx.x];
    if (S.done[slot]) return;
    bool ok;
    const double a = step_length(S.partial + (size_t)slot * S.pstride, npart, S.rr[slot], ok);
    if (threadIdx.x != 0) return;
    S.alpha[slot] = ok ? a : 0.0;
    if (!ok) S.status[slot] = kStatusBreakdown;
}

void launch_scalars_alpha(const MSState &s, int npart, hipStream_t st) {
    hipLaunchKernelGGL(k_scalars_alpha, dim3(s.B), dim3(64), 0, st, s, npart);
}

// The shifts' recurrences of one slot, one wave, lane i = shift i (NS <= 32): the state of a lane's
// shift and of the slot, advanced after each residual update.
struct ShiftLane {
    double z, zp;                  // zeta^i and the one before
    double alpha_prev, beta_prev;
    double lim, delta, c;          // tol |b|, q_i - q_base, c_i
    int act, it, j;                // shift active; iterations of the solve and of the block
    long long entries, steps;      // listed shifts and iterations since load()

    __device__ __forceinline__ void load(const MSState &S, int slot) {
        const int i = threadIdx.x & 63, k = slot * S.NS + (i < S.NS ? i : 0);
        z = S.zeta[k];
        zp = S.zeta_prev[k];
        act = i < S.NS && S.sh_active[k];
        alpha_prev = S.alpha_prev[slot];
        beta_prev = S.beta_prev[slot];
        lim = S.tol * S.bnorm[slot];
        delta = S.delta[i < S.NS ? i : 0];
        c = S.c[i < S.NS ? i : 0];
        it = S.iters[slot];
        j = S.blk_n[slot];
        entries = steps = 0;
    }
    // After the step a: beta_k = |r_{k+1}|^2/|r_k|^2; per active shift the new zeta, the block's
    // coefficients alpha^i, beta^i and zeta^i, and convergence (zeta^i_{k+1} |r_{k+1}| <= tol |b|).
    // The base shift's direction keeps being updated while any shift of the slot is active (its
    // alpha^i is 0 once it has converged).  Returns whether one still is.
    template <class T>
    __device__ __forceinline__ bool advance(const MSState &S, int slot, double a, double rr, double rrn) {
        const int i = threadIdx.x & 63;
        const double b = rrn / rr;
        bool conv = false;
        const bool listed = act || i == S.i0;
        if (i < S.NS) {
            double ha = 0.0, hb = i == S.i0 ? b : 0.0, hz = i == S.i0 ? 1.0 : 0.0;
            if (act) {
                const double zn = z * zp * alpha_prev /
                                  (a * beta_prev * (zp - z) + zp * alpha_prev * (1.0 + delta * a));
                const double ratio = zn / z;
                conv = zn * sqrt(rrn) <= lim;
                ha = a * ratio;
                hb = b * ratio * ratio;
                hz = zn;
                if (conv) S.sh_iters[slot * S.NS + i] = it + 1;
                zp = z;
                z = zn;
            }
            const size_t h = ((size_t)slot * S.K + j) * S.NS + i;
            S.h_a[h] = ha;
            S.h_cy[h] = c * ha;
            static_cast<T *>(S.h_b)[h] = (T)hb;
            static_cast<T *>(S.h_z)[h] = (T)hz;
        }
        if (S.vec16 && i == 0) S.h_rr[(size_t)slot * S.K + j] = rrn;
        entries += __popcll(__ballot(listed));
        act = act && !conv;
        alpha_prev = a;
        beta_prev = b;
        ++it;
        ++j;
        ++steps;
        return __ballot(act) != 0;
    }
    __device__ __forceinline__ void store(const MSState &S, int slot, bool still, double rr, double *rr_out) const {
        const int i = threadIdx.x & 63;
        if (i < S.NS) {
            const int k = slot * S.NS + i;
            S.zeta[k] = z;
            S.zeta_prev[k] = zp;
            S.sh_active[k] = act;
        }
        if (i != 0) return;
        if (!still) S.done[slot] = 1;   // slot finished: no direction needs updating any more
        S.cnt_entries[slot] += entries;
        S.cnt_active[slot] += steps;
        S.alpha_prev[slot] = alpha_prev;
        S.beta_prev[slot] = beta_prev;
        S.beta[slot] = beta_prev;
        rr_out[slot] = rr;
        S.iters[slot] = it;
        S.blk_n[slot] = j;
    }
};

template <class T>
__device__ __forceinline__ void advance_shifts(const MSState &S, int slot, double a, double rr, double rrn,
                                               double *rr_out) {
    ShiftLane lane;
    lane.load(S, slot);
    const bool still = lane.advance<T>(S, slot, a, rr, rrn);
    lane.store(S, slot, still, rrn, rr_out);
}

template <class T>
__global__ void k_scalars_beta(MSState S, int npart) {
    if ((int)blockIdx.x >= *S.count) return;
    const int slot = S.list[blockIdx.x];
    if (S.done[slot]) return;
    const double rrn = wave_sum_partials(S.partial2 + (size_t)slot * S.pstride, npart);
    if (S.status[slot] != kStatusOK) {
        if (threadIdx.x == 0) S.done[slot] = 1;
        return;
    }
    advance_shifts<T>(S, slot, S.alpha[slot], S.rr[slot], rrn, S.rr);
}

void launch_scalars_beta(int prec, const MSState &s, int npart, hipStream_t st) {
    if (prec == 0)
        hipLaunchKernelGGL(k_scalars_beta<double>, dim3(s.B), dim3(64), 0, st, s, npart);
    else
        hipLaunchKernelGGL(k_scalars_beta<float>, dim3(s.B), dim3(64), 0, st, s, npart);
}

// ------------------------------------------------------------------ base direction
// z r + b p, rounded as b p + (z r) with one fused step: the same in every kernel that advances a
// direction.
template <class T>
__device__ __forceinline__ cpx<T> next_direction(T z, cpx<T> r, T b, cpx<T> p) {
    return {fmadd(b, p.re, z * r.re), fmadd(b, p.im, z * r.im)};
}

// p_out = r + beta p_in: three streamed vectors, bound by HBM.  With partials (np_pap > 0) every
// wave sums |r|^2 itself and the slot's first one advances the scalars: on lattices with at most
// kFusedPartials partials this and the stencil's own alpha save two launches of 4.5 us in an
// iteration (D_ov of one 8^4 spinor spent 9 of 34 us in them).  |r|^2 goes to the other of two
// buffers, since other blocks still read the old one; that they may see the slot done already
// does no harm, its direction is not needed any more.
template <class T>
__global__ __launch_bounds__(kBlock) void k_base_direction(Geom g, MSState S, const typename Store<T>::vec *r,
                                                           size_t rst, const typename Store<T>::vec *p_in,
                                                           typename Store<T>::vec *p_out, size_t pst, int np_pap,
                                                           int np_rr, const double *rr_in, double *rr_out) {
    constexpr int C = Unit<T>::C;
    if ((int)blockIdx.y >= *S.count) return;
    const int slot = S.list[blockIdx.y];
    if (S.done[slot]) return;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    double beta;
    if (np_pap > 0) {
        const double rr = rr_in[slot];
        const double rrn = wave_sum_partials(S.partial2 + (size_t)slot * S.pstride, np_rr);
        beta = rrn / rr;
        if (blockIdx.x == 0 && threadIdx.x < 64) {
            bool ok;
            const double a = step_length(S.partial + (size_t)slot * S.pstride, np_pap, rr, ok);
            if (ok) {
                advance_shifts<T>(S, slot, a, rr, rrn, rr_out);
            } else if (threadIdx.x == 0) {
                S.status[slot] = kStatusBreakdown;
                S.done[slot] = 1;
            }
        }
    } else {
        beta = S.beta[slot];
    }
    if (s >= g.V) return;
    const T b = (T)beta;
    cpx<T> rv[C], pv[C];
    Unit<T>::load_stream(r + slot * rst, g.vs, u, s, rv);
    Unit<T>::load_stream(p_in + slot * pst, g.vs, u, s, pv);
#pragma unroll
    for (int j = 0; j < C; ++j) pv[j] = next_direction(T(1), rv[j], b, pv[j]);
    Unit<T>::store_stream(p_out + slot * pst, g.vs, u, s, pv);
}

void launch_base_direction(int prec, const Geom &g, const MSState &s, const void *r, size_t rst, const void *p_in,
                           void *p_out, size_t pst, int np_pap, int np_rr, const double *rr_in, double *rr_out,
                           hipStream_t st) {
    dim3 grid(unit_parts(prec, g), s.B);
    if (prec == 0)
        hipLaunchKernelGGL(k_base_direction<double>, grid, dim3(kBlock), 0, st, g, s, (const double2 *)r, rst,
                           (const double2 *)p_in, (double2 *)p_out, pst, np_pap, np_rr, rr_in, rr_out);
    else
        hipLaunchKernelGGL(k_base_direction<float>, grid, dim3(kBlock), 0, st, g, s, (const float4 *)r, rst,
                           (const float4 *)p_in, (float4 *)p_out, pst, np_pap, np_rr, rr_in, rr_out);
}

// ------------------------------------------------------------------ small lattices
// Iterations of a solve with one workgroup per right-hand side: on a lattice of at most
// kSmallThreads sites the whole of one vector fits a CU's LDS, and a right-hand side needs no other
// workgroup, so that an iteration is five barriers instead of three launches of 9 to 17 us that
// each leave most of the chip idle.  The vector that the stencil reads is in LDS, the residuals and
// links come from L2, and the first wave advances the shifts' recurrences.  Bound by the latency of
// one or two waves per SIMD (LDS, links, reductions).  A whole 4^4 map of 192 right-hand sides:
// FP64 11.1 -> 4.2 ms; 96 point sources on 420 sites (two tiles) in FP64 6.5 ms, mixed 3.9 ms
// against about 10 in separate launches.
// The sums have the order of the separate kernels (tiles of the stencil's blocks, their waves, one
// wave over the tiles), so that results are equal bit for bit.
template <class T>
struct RawLink {
    static constexpr int n = std::is_same<T, float>::value ? 3 : 9;
    typename Store<T>::link v[n];
    __device__ __forceinline__ void load(const typename Store<T>::link *U, int V, int mu, int s) {
#pragma unroll
        for (int k = 0; k < n; ++k) v[k] = unit_get(U + (size_t)(mu * n + k) * V, s);
    }
    __device__ __forceinline__ void unpack(cpx<T> u[9]) const {
        if constexpr (std::is_same<T, float>::value) {
            unpack_rows(v[0], v[1], v[2], u);
        } else {
#pragma unroll
            for (int k = 0; k < n; ++k) u[k] = {v[k].x, v[k].y};
        }
    }
};

template <class T, bool EXACT, int MAXT>
__global__ __launch_bounds__(MAXT) void k_cg_small(const typename Store<T>::link *__restrict__ U, Geom g,
                                                            MSState S, int tpt, int np, T kappa, T sigma,
                                                            const typename Store<T>::vec *p_in,
                                                            typename Store<T>::vec *p_out, size_t pst,
                                                            typename Store<T>::vec *ring, int n0, int iters) {
    using vec = typename Store<T>::vec;
    using link = typename Store<T>::link;
    constexpr int TU = tile_units<T>, UN = Store<T>::units, CU = 12 / UN;
    extern __shared__ __align__(16) unsigned char tile_raw[];
    vec *field = reinterpret_cast<vec *>(tile_raw);   // [site][tile_units]
    __shared__ double red[2][kSmallThreads / 64];
    __shared__ int finished;
    // (p, tmp and an accumulator in registers at once would not fit the 256 of two waves per SIMD)
    if ((int)blockIdx.x >= *S.count) return;
    const int slot = S.list[blockIdx.x];
    if (S.done[slot]) return;
    // the thread's site, as the stencil's tiles order them
    const int sb = threadIdx.x / tpt, i = threadIdx.x - sb * tpt;
    int s;
    bool ok_site = true;
    if constexpr (EXACT) {
        const int tiles_per_plane = g.ny / g.tile_y;
        s = plane_order(sb / tiles_per_plane, g) * g.nx * g.ny + (sb % tiles_per_plane) * g.tile_y * g.nx + i;
    } else {
        int ty, m;
        any_tile(g, ty, m);
        const AnySite a = any_site(g, ty, m, sb, i);   // idle: computes a site, stores and adds nothing
        s = (a.pl * g.ny + a.y0) * g.nx + a.i;
        ok_site = a.ok;
    }
    const Nbr nb = neighbours(s, g.nx, g.ny, g.nz, g.nt);
    const size_t rs = UN * g.vs;
    vec *rp = ring + (size_t)slot * S.K * rs;
    double rr = S.rr[slot];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wpt = tpt >> 6;
    if (threadIdx.x == 0) finished = 0;
    const auto put = [&](const cpx<T> *v) {
        if (!ok_site) return;
#pragma unroll
        for (int k = 0; k < UN; ++k) {
            if constexpr (CU == 1) field[s * TU + k] = make_double2(v[k].re, v[k].im);
            else field[s * TU + k] = make_float4(v[2 * k].re, v[2 * k].im, v[2 * k + 1].re, v[2 * k + 1].im);
        }
    };
    // the sum over the block in the order of the separate kernels; its barrier also ends the reads of
    // the field before it
    const auto total = [&](double d, int which) {
        d = wave_sum(d);
        if (lane == 0) red[which][wv] = d;
        __syncthreads();
        double v = 0.0;
        if (lane < np)
            for (int k = 0; k < wpt; ++k) v += red[which][lane * wpt + k];
        return wave_sum(v);
    };
    cpx<T> acc[12], u[9], q[12], h[6], w[6];
    // D_W or D_W^dag of the field at the own site, q = the field there
    // Each link is loaded one hop ahead (its rows as stored), since one or two waves per SIMD hide little
    // of the latency of L2; in FP64 only up to 256 threads, whose registers hold two links of 36 (on 512
    // threads 139-192 were spilled, a map of four classes on 4^3 x 8 8.7 ms against 6.8 so).
    constexpr bool kAhead = std::is_same<T, float>::value || MAXT <= 256;
    [[maybe_unused]] RawLink<T> l0, l1;
#define SMPQ_SMALL_HOP(MU, SF, CUR, LSITE, NEXT, NMU, NSITE, SITE, MUL, FIRST)       \
        if constexpr (kAhead) {                                                      \
            NEXT.load(Ur, g.V, NMU, NSITE);                                          \
            __builtin_amdgcn_sched_barrier(0);                                       \
            CUR.unpack(u);                                                           \
        }                                                                            \
        tile_read(field, SITE, q);                                                   \
        project<MU, SF>(q, h);                                                       \
        if constexpr (!kAhead) {                                                     \
            __builtin_amdgcn_sched_barrier(0);                                       \
            load_link<T>(Ur, g.V, MU, LSITE, u);                                     \
        }                                                                            \
        MUL(u, h, w);                                                                \
        accumulate<MU, SF, FIRST>(acc, w);                                           \
        __builtin_amdgcn_sched_barrier(0);
    // l0 holds U_z(x) before and after
#define SMPQ_SMALL_HOPS(SF)                                                                     \
        SMPQ_SMALL_HOP(2, SF, l0, s, l1, 2, nb.bwd[2], nb.fwd[2], su3_mul, true)                \
        SMPQ_SMALL_HOP(2, -SF, l1, nb.bwd[2], l0, 3, s, nb.bwd[2], su3_dag_mul, false)          \
        SMPQ_SMALL_HOP(3, SF, l0, s, l1, 3, nb.bwd[3], nb.fwd[3], su3_mul, false)               \
        SMPQ_SMALL_HOP(3, -SF, l1, nb.bwd[3], l0, 0, s, nb.bwd[3], su3_dag_mul, false)          \
        SMPQ_SMALL_HOP(0, SF, l0, s, l1, 0, nb.bwd[0], nb.fwd[0], su3_mul, false)               \
        SMPQ_SMALL_HOP(0, -SF, l1, nb.bwd[0], l0, 1, s, nb.bwd[0], su3_dag_mul, false)          \
        SMPQ_SMALL_HOP(1, SF, l0, s, l1, 1, nb.bwd[1], nb.fwd[1], su3_mul, false)               \
        SMPQ_SMALL_HOP(1, -SF, l1, nb.bwd[1], l0, 2, s, nb.bwd[1], su3_dag_mul, false)          \
        _Pragma("unroll") for (int c = 0; c < 12; ++c)                                          \
            asm volatile("" : "+v"(acc[c].re), "+v"(acc[c].im));
    if constexpr (kAhead) l0.load(U, g.V, 2, s);
    __shared__ ShiftLane shifts[64];
    if (wv == 0) shifts[lane].load(S, slot);
    Store<T>::load(p_in + slot * pst, g.vs, s, q);
    put(q);
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < iters; ++it) {
        // opaque in each iteration, so that the links are not hoisted into registers (as in k_dslash_rl)
        const link *Ur = U;
        asm volatile("" : "+s"(Ur));
        // tmp = D_W p, <p, (H^2 + sigma) p>
        SMPQ_SMALL_HOPS(1)
        cpx<T> p[12];
        tile_read(field, s, p);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = p[c] - kappa * acc[c];
        const double pap = total(ok_site ? norm_step<T>(acc, p, sigma) : 0.0, 0);
        if (!(pap > 0.0) || !isfinite(pap)) {   // uniform over the block
            if (wv == 0) shifts[lane].store(S, slot, false, rr, S.rr);
            if (threadIdx.x == 0) S.status[slot] = kStatusBreakdown;
            return;
        }
        const double a = rr / pap;
        put(acc);
        __syncthreads();
        // r -= alpha (D_W^dag tmp + sigma p)
        SMPQ_SMALL_HOPS(-1)
        tile_read(field, s, q);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = q[c] - kappa * acc[c];
        const int n = n0 + it;
        Store<T>::load(rp + (size_t)(n == 0 ? S.K - 1 : n - 1) * rs, g.vs, s, q);
        double d = residual_step<T>(acc, p, q, sigma, (T)a);
        if (ok_site) {
#pragma unroll
            for (int k = 0; k < UN; ++k) unit_store_stream(rp + (size_t)n * rs, g.vs, k, s, q + k * CU);
        } else {
            d = 0.0;
        }
        const double rrn = total(d, 1);
        // the next direction goes to the field first, so that no spinor is held beside the recurrences
        const T b = (T)(rrn / rr);
#pragma unroll
        for (int c = 0; c < 12; ++c) q[c] = next_direction(T(1), q[c], b, p[c]);
        put(q);
        if (wv == 0) {
            ShiftLane sh = shifts[lane];
            const bool still = sh.template advance<T>(S, slot, a, rr, rrn);
            if (!still || it == iters - 1) sh.store(S, slot, still, rrn, S.rr);
            else shifts[lane] = sh;
            if (lane == 0 && !still) finished = 1;
        }
        rr = rrn;
        __syncthreads();
        if (finished) return;   // uniform over the block; its direction is not needed any more
    }
#undef SMPQ_SMALL_HOPS
#undef SMPQ_SMALL_HOP
    if (ok_site) {
        tile_read(field, s, q);
#pragma unroll
        for (int k = 0; k < UN; ++k) unit_store_stream(p_out + slot * pst, g.vs, k, s, q + k * CU);
    }
}

// Threads of a k_cg_small block where one fits the lattice and the default variants are in use, else 0.
static int small_block(int prec, const Geom &g, int &tpt, int &np) {
    if (!g.adapt) return 0;
    if (g.tile_y > 0) {
        tpt = g.nx * g.tile_y;
        np = tile_blocks(g);
    } else {
        int ty, m;
        any_tile(g, ty, m);
        if (ty == 0) return 0;
        tpt = (m * g.nx * ty + 63) / 64 * 64;
        np = any_blocks(g);
    }
    return (long long)tpt * np <= kSmallThreads && g.V <= kSmallThreads ? tpt * np : 0;
}

bool small_lattice(int prec, const Geom &g) {
    int tpt, np;
    return small_block(prec, g, tpt, np) > 0;
}

template <class T>
static void launch_cg_small_t(const Geom &g, const MSState &s, const void *U, double kappa, double sigma,
                              const void *p_in, void *p_out, size_t pst, void *ring, int n0, int iters,
                              hipStream_t st) {
    using vec = typename Store<T>::vec;
    using link = typename Store<T>::link;
    constexpr bool dbl = std::is_same<T, double>::value;
    int tpt, np;
    const int threads = small_block(dbl ? 0 : 1, g, tpt, np);
    if (threads == 0 || n0 + iters > s.K) throw std::invalid_argument("not a small lattice, or too many iterations");
    const size_t lds = (size_t)g.V * tile_units<T> * sizeof(vec);
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(s.B), dim3(threads), lds, st, (const link *)U, g, s, tpt, np, (T)kappa, (T)sigma,
                           (const vec *)p_in, (vec *)p_out, pst, (vec *)ring, n0, iters);
    };
    // up to 256 threads the block has a SIMD's registers per wave
    const bool exact = g.tile_y > 0;
    if constexpr (dbl) {
        if (threads <= 256) return exact ? go(k_cg_small<T, true, 256>) : go(k_cg_small<T, false, 256>);
    }
    if (exact) go(k_cg_small<T, true, kSmallThreads>);
    else go(k_cg_small<T, false, kSmallThreads>);
}

void launch_cg_small(int prec, const Geom &g, const MSState &s, const void *U, double kappa, double sigma,
                     const void *p_in, void *p_out, size_t pst, void *ring, int n0, int iters, hipStream_t st) {
    if (prec == 0)
        launch_cg_small_t<double>(g, s, U, kappa, sigma, p_in, p_out, pst, ring, n0, iters, st);
    else
        launch_cg_small_t<float>(g, s, U, kappa, sigma, p_in, p_out, pst, ring, n0, iters, st);
}

// ------------------------------------------------------------------ block update of the shifts
// One wave per slot, lane i = shift i.
__global__ void k_block_end(MSState S, int base_inline, int dir) {
    const int slot = blockIdx.x, i = threadIdx.x;
    const int m = S.blk_n[slot];
    const bool on = i < S.NS;
    const int k = slot * S.NS + (on ? i : 0);
    const bool active = on && S.sh_active[k];
    const bool was = on && (S.fl_act[slot] >> i & 1);
    const bool write = on && !S.done[slot] && (i == S.i0 ? base_inline != 0 : active);
    const unsigned rd = (unsigned)__ballot(was || write), wr = (unsigned)__ballot(write),
                   now = (unsigned)__ballot(active);
    if (i == 0) S.fl_m[slot] = m;
    if (m == 0) return;
    if (on && dir != kDirF32) {
        // 16-bit directions: the stored p_i is decoded with its current scale and the new one is
        // stored divided by zeta^i |r| dir_norm, which keeps its entries near 1
        S.s_sold[k] = S.sh_scale[k];
        double sc = S.zeta[k] * sqrt(S.rr[slot]) * S.dir_norm;
        if (!(sc > 0.0) || !isfinite(sc)) sc = S.sh_scale[k];
        if (write) S.sh_scale[k] = sc;
        S.s_snew[k] = 1.0 / sc;
    }
    if (i != 0) return;
    S.blk_n[slot] = 0;
    S.fl_rd[slot] = rd;
    S.fl_wr[slot] = wr;
    S.fl_act[slot] = now;
    S.cnt_fl[slot] += 1;
    S.cnt_fl_r[slot] += m;
    S.cnt_fl_p[slot] += __popc(rd) + __popc(wr);
}

void launch_block_end(const MSState &s, bool base_inline, int dir, hipStream_t st) {
    hipLaunchKernelGGL(k_block_end, dim3(s.B), dim3(64), 0, st, s, base_inline ? 1 : 0, dir);
}

// The rounding of vectors that the stencil reads, mode 1: FP16 after division by sqrt(|r|^2 / (24 V)), where
// the entries of a vector of norm |r| lie near 1; mode 2: BF16 (FP32's exponent range); to nearest even.
struct Round16 {
    int mode;
    float sc, inv;
    __device__ __forceinline__ Round16(int m, double rr, int V) : mode(m) {
        const float scale = mode == 1 ? (float)sqrt(rr / (24.0 * (double)V)) : 1.f;
        sc = scale > 0.f ? scale : 1.f;
        inv = 1.f / sc;
    }
    __device__ __forceinline__ float operator()(float x) const {
        return mode == 1 ? (float)(_Float16)(x * inv) * sc : (float)(__bf16)x;
    }
};

// acc += w v in FP64
template <class T>
__device__ __forceinline__ void add_scaled(double w, cpx<T> v, cpx<double> &acc) {
    acc.re = fmadd(w, (double)v.re, acc.re);
    acc.im = fmadd(w, (double)v.im, acc.im);
}

// The iterations l = 0 .. m-1 of a block for every listed shift: y += c_i a p_i and, for the base
// shift, x0 += a p_i (FP64 sums of products that are exact in FP64 for FP32 vectors), then
// p_i = z r_l + b p_i.  The NS <= CH directions are held in registers while the block's residuals stream
// by, so that a direction is read and written once per block instead of once per iteration and
// y and x0 are read and written once: per site and iteration, in FP32 with n listed shifts,
// 96 (1 + 2 n / K) + 768 / K bytes against 96 (1 + 2 n) + 192 .. 768.  Bound by HBM (the FP64
// sums, four instructions a direction and real, take half of that time).  Against an update in
// every iteration: four 16^4 classes (r = 4) in FP64 559 -> 366 ms, a whole 8^4 map (r = 2) in mixed
// precision 99.5 -> 61.0 ms, eight unshifted 16^4 classes 376 -> 291 ms.  All shifts take part in one
// pass, so that the order of the sums is that of an update in every iteration.
template <class T, int CH, int D, bool XS>
__global__ __launch_bounds__(kBlock) void k_block_update(
    Geom g, int NS, int K, int i0, const int *__restrict__ fl_m, const unsigned *__restrict__ fl_rd,
    const unsigned *__restrict__ fl_wr, const double *__restrict__ h_cy, const double *__restrict__ h_a,
    const T *__restrict__ h_z, const T *__restrict__ h_b, const double *__restrict__ s_sold,
    const double *__restrict__ s_snew, const typename Store<T>::vec *__restrict__ ring, typename Store<T>::vec *p,
    size_t pst, int base_sel, double2 *y, double2 *x0, void *ph, double2 *xs, int vec16,
    const double *__restrict__ h_rr) {
    using vec = typename Store<T>::vec;
    constexpr bool DIR16 = D == kDirF16 || D == kDirBF16;
    constexpr int C = Unit<T>::C;
    const int slot = blockIdx.y;
    const int m = fl_m[slot];
    if (m == 0) return;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const unsigned rd = fl_rd[slot], wr = fl_wr[slot];
    const size_t rs = Store<T>::units * g.vs, r64 = 12 * g.vs;
    const vec *rp = ring + (size_t)slot * K * rs;
    vec *pp = p + slot * pst;
    const bool with_x = x0 && (rd >> i0 & 1);
    cpx<double> ya[C], xa[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        ya[c] = ld64_stream(y + slot * r64, g.vs, u * C + c, s);
        xa[c] = {0.0, 0.0};
        if (with_x) xa[c] = ld64_stream(x0 + slot * r64, g.vs, u * C + c, s);
    }
    cpx<T> pv[CH][C];
    cpx<double> xv[XS ? CH : 1][C];
#pragma unroll
    for (int i = 0; i < CH; ++i) {   // rd holds no bit of a shift >= NS
#pragma unroll
        for (int c = 0; c < C; ++c) pv[i][c] = {T(0), T(0)};
        if (rd >> i & 1) {
            if (!DIR16 || i == i0)
                Unit<T>::load_stream(pp + (i == i0 ? base_sel : i) * rs, g.vs, u, s, pv[i]);
            else if constexpr (DIR16)
                load_dir16<D>(static_cast<typename Dir16<D>::v *>(ph) + ((size_t)slot * NS + i) * rs, g.vs, u, s,
                              (float)s_sold[slot * NS + i], pv[i]);
            if constexpr (XS) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    xv[i][c] = ld64_stream(xs + ((size_t)slot * NS + i) * r64, g.vs, u * C + c, s);
            }
        }
    }
    cpx<T> next[C];
    Unit<T>::load_stream(rp, g.vs, u, s, next);
#pragma unroll 1
    for (int l = 0; l < m; ++l) {
        cpx<T> rv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) rv[c] = next[c];
        if (l + 1 < m) Unit<T>::load_stream(rp + (l + 1) * rs, g.vs, u, s, next);
        const size_t h = ((size_t)slot * K + l) * NS;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (rd >> i & 1) {
                const double cy = h_cy[h + i];
                const T z = h_z[h + i], b = h_b[h + i];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    add_scaled(cy, pv[i][c], ya[c]);
                    if constexpr (XS) add_scaled(h_a[h + i], pv[i][c], xv[i][c]);
                }
                if (with_x && i == i0) {
                    const double a = h_a[h + i];
#pragma unroll
                    for (int c = 0; c < C; ++c) add_scaled(a, pv[i][c], xa[c]);
                }
#pragma unroll
                for (int c = 0; c < C; ++c) pv[i][c] = next_direction(z, rv[c], b, pv[i][c]);
                if constexpr (D == kDirVec16) {
                    if (i == i0) {   // as k_round16 stored it for the next iteration's stencil
                        const Round16 round(vec16, h_rr[(size_t)slot * K + l], g.V);
#pragma unroll
                        for (int c = 0; c < C; ++c) pv[i][c] = {round(pv[i][c].re), round(pv[i][c].im)};
                    }
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        if (rd >> i & 1) {
            if (wr >> i & 1) {
                if (!DIR16 || i == i0)
                    Unit<T>::store_stream(pp + (i == i0 ? base_sel : i) * rs, g.vs, u, s, pv[i]);
                else if constexpr (DIR16)
                    store_dir16<D>(static_cast<typename Dir16<D>::v *>(ph) + ((size_t)slot * NS + i) * rs, g.vs, u, s,
                                   (float)s_snew[slot * NS + i], pv[i]);
            }
            if constexpr (XS) {
#pragma unroll
                for (int c = 0; c < C; ++c)
                    st64_stream(xs + ((size_t)slot * NS + i) * r64, g.vs, u * C + c, s, xv[i][c]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        st64_stream(y + slot * r64, g.vs, u * C + c, s, ya[c]);
        if (with_x) st64_stream(x0 + slot * r64, g.vs, u * C + c, s, xa[c]);
    }
}

template <class T, int CH, int D, bool XS>
static void launch_block_update_t(const Geom &g, const MSState &s, const void *ring, void *p, size_t pst, int base_sel,
                                  double2 *y, double2 *x0, void *ph, double2 *xs, hipStream_t st) {
    using vec = typename Store<T>::vec;
    dim3 grid(unit_parts(std::is_same<T, double>::value ? 0 : 1, g), s.B);
    hipLaunchKernelGGL((k_block_update<T, CH, D, XS>), grid, dim3(kBlock), 0, st, g, s.NS, s.K, s.i0, s.fl_m, s.fl_rd,
                       s.fl_wr, s.h_cy, s.h_a, (const T *)s.h_z, (const T *)s.h_b, s.s_sold, s.s_snew, (const vec *)ring, (vec *)p, pst, base_sel, y, x0, ph, xs, s.vec16, s.h_rr);
}

// Registers for as many directions as the solve has: one (the trace of D_W^-1, refinement and inner
// solves), up to 8, up to 14 (the usual order of the sign function), up to 32.
template <class T, int D, bool XS>
static void launch_block_update_d(const Geom &g, const MSState &s, const void *ring, void *p, size_t pst, int base_sel,
                                  double2 *y, double2 *x0, void *ph, double2 *xs, hipStream_t st) {
    if (s.NS == 1)
        launch_block_update_t<T, 1, D, XS>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (s.NS <= 8)
        launch_block_update_t<T, 8, D, XS>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (s.NS <= 14)
        launch_block_update_t<T, 14, D, XS>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else
        launch_block_update_t<T, 32, D, XS>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
}

void launch_block_update(int prec, const Geom &g, const MSState &s, const void *ring, void *p, size_t pst,
                         int base_sel, double2 *y, double2 *x0, int dir, void *ph, double2 *xs, hipStream_t st) {
    if (xs && dir != kDirF32) throw std::invalid_argument("the per-shift check needs FP32 or FP64 directions");
    if (prec == 0 && dir != kDirF32) throw std::invalid_argument("16-bit directions need the FP32 path");
    if (prec == 0 && xs)
        launch_block_update_d<double, kDirF32, true>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (prec == 0)
        launch_block_update_d<double, kDirF32, false>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (dir == kDirF16)
        launch_block_update_d<float, kDirF16, false>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (dir == kDirBF16)
        launch_block_update_d<float, kDirBF16, false>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (s.vec16 && s.K > 1 && xs)
        launch_block_update_d<float, kDirVec16, true>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (s.vec16 && s.K > 1)   // with K = 1 the base direction is rounded once it is stored
        launch_block_update_d<float, kDirVec16, false>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else if (xs)
        launch_block_update_d<float, kDirF32, true>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
    else
        launch_block_update_d<float, kDirF32, false>(g, s, ring, p, pst, base_sel, y, x0, ph, xs, st);
}

// Evaluated precision: an FP32 vector of every listed slot rounded in place to what 16-bit storage would
// hold.  Applied to the vectors the stencil reads (the base direction and D_W p) after the
// kernels that write them, so that those compute in FP32 and only storage is emulated.
__global__ __launch_bounds__(kBlock) void k_round16(Geom g, MSState S, float4 *v, size_t slot_stride, size_t extra,
                                                    int mode) {
    if ((int)blockIdx.y >= *S.count) return;
    const int slot = S.list[blockIdx.y];
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    float4 *p = v + slot * slot_stride + extra + (size_t)u * g.vs + s;
    const Round16 round(mode, S.rr[slot], g.V);
    const float4 t = *p;
    *p = make_float4(round(t.x), round(t.y), round(t.z), round(t.w));
}

void launch_round16(const Geom &g, const MSState &s, void *v, size_t slot_stride, size_t extra, int mode,
                    hipStream_t st) {
    dim3 grid(unit_parts(1, g), s.B);
    hipLaunchKernelGGL(k_round16, grid, dim3(kBlock), 0, st, g, s, (float4 *)v, slot_stride, extra, mode);
}

// Ordered list of the slots still iterating: one block, each thread counting a contiguous range
// of slots (one thread walking all of them waits for a load per slot: 24 us for 192 slots).
__global__ __launch_bounds__(kBlock) void k_compact(MSState S) {
    __shared__ int wave_n[kBlock / 64];
    const int per = (S.B + kBlock - 1) / kBlock;
    const int beg = min(S.B, (int)threadIdx.x * per), end = min(S.B, beg + per);
    int n = 0;
    for (int slot = beg; slot < end; ++slot) n += !S.done[slot];
    int before = n;   // inclusive prefix sum over the wave
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(before, off);
        if (lane >= off) before += t;
    }
    if (lane == 63) wave_n[wv] = before;
    __syncthreads();
    int at = before - n, total = 0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) {
        if (i < wv) at += wave_n[i];
        total += wave_n[i];
    }
    for (int slot = beg; slot < end; ++slot)
        if (!S.done[slot]) S.list[at++] = slot;
    if (threadIdx.x == 0) *S.count = total;
}

void launch_compact(const MSState &s, hipStream_t st) {
    hipLaunchKernelGGL(k_compact, dim3(1), dim3(kBlock), 0, st, s);
}

// Residual replacement: r = b - (H^2 + s) x0 evaluated in FP64 (ap64 holds (H^2 + s) x0),
// stored in the iteration precision; partial |r|^2 of the stored values.
template <class T>
__global__ __launch_bounds__(kBlock) void k_reliable(Geom g, MSState S, Source src, const double2 *ap64,
                                                     size_t ast, typename Store<T>::vec *r, size_t rst) {
    constexpr int C = Unit<T>::C;
    if ((int)blockIdx.y >= *S.count) return;
    const int slot = S.list[blockIdx.y];
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    double nrm = 0.0;
    if (s < g.V) {
        cpx<T> rv[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int c = u * C + i;
            const cpx<double> d = source_entry(src, slot, c, s, g.vs) - ld64(ap64 + slot * ast, g.vs, c, s);
            rv[i] = {(T)d.re, (T)d.im};
            nrm += (double)rv[i].re * rv[i].re + (double)rv[i].im * rv[i].im;
        }
        Unit<T>::store(r + slot * rst, g.vs, u, s, rv);
    }
    block_partial(nrm, S.partial, (size_t)slot * S.pstride + blockIdx.x);
}

void launch_reliable(int prec, const Geom &g, const MSState &s, const Source &src, const double2 *ap64, size_t ast,
                     void *r, size_t rst, hipStream_t st) {
    dim3 grid(unit_parts(prec, g), s.B);
    if (prec == 0)
        hipLaunchKernelGGL(k_reliable<double>, grid, dim3(kBlock), 0, st, g, s, src, ap64, ast, (double2 *)r, rst);
    else
        hipLaunchKernelGGL(k_reliable<float>, grid, dim3(kBlock), 0, st, g, s, src, ap64, ast, (float4 *)r, rst);
}

__global__ void k_scalars_rr(MSState S, int npart) {
    if ((int)blockIdx.x >= *S.count) return;
    const int slot = S.list[blockIdx.x];
    const double rr = wave_sum_partials(S.partial + (size_t)slot * S.pstride, npart);
    if (threadIdx.x == 0) S.rr[slot] = rr;
}

void launch_scalars_rr(const MSState &s, int npart, hipStream_t st) {
    hipLaunchKernelGGL(k_scalars_rr, dim3(s.B), dim3(64), 0, st, s, npart);
}

// ------------------------------------------------------------------ per-shift check
// out = b - ap64 in FP64 for the first nslots slots; partial |out|^2 per block.
__global__ __launch_bounds__(kBlock) void k_resid64(Geom g, Source src, const double2 *ap64, double2 *out,
                                                    double *partial, size_t pstride) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    double nrm = 0.0;
    if (s < g.V) {
        const size_t o = (size_t)slot * 12 * g.vs;
        const cpx<double> d = source_entry(src, slot, u, s, g.vs) - ld64(ap64 + o, g.vs, u, s);
        st64(out + o, g.vs, u, s, d);
        nrm = d.re * d.re + d.im * d.im;
    }
    block_partial(nrm, partial, (size_t)slot * pstride + blockIdx.x);
}

void launch_resid64(const Geom &g, int nslots, const Source &src, const double2 *ap64, double2 *out,
                    double *partial, size_t pstride, hipStream_t st) {
    hipLaunchKernelGGL(k_resid64, dim3(unit_parts(0, g), nslots), dim3(kBlock), 0, st, g, src, ap64, out, partial,
                       pstride);
}

__global__ void k_slot_sums(const double *partial, size_t pstride, int npart, double *sums) {
    const double v = wave_sum_partials(partial + (size_t)blockIdx.x * pstride, npart);
    if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

void launch_slot_sums(int nslots, const double *partial, size_t pstride, int npart, double *sums, hipStream_t st) {
    hipLaunchKernelGGL(k_slot_sums, dim3(nslots), dim3(64), 0, st, partial, pstride, npart, sums);
}

__global__ __launch_bounds__(kBlock) void k_zero_unflagged(Geom g, const int *flag, double2 *v) {
    const int slot = blockIdx.y;
    if (flag[slot]) return;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s < g.V) st64(v + (size_t)slot * 12 * g.vs, g.vs, u, s, {0.0, 0.0});
}

void launch_zero_unflagged(const Geom &g, int nslots, const int *flag, double2 *v, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_unflagged, dim3(unit_parts(0, g), nslots), dim3(kBlock), 0, st, g, flag, v);
}

__global__ __launch_bounds__(kBlock) void k_refine_acc(Geom g, const double2 *e, double c, double2 *ysave,
                                                       double2 *xsi, size_t xs_stride) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const size_t o = (size_t)slot * 12 * g.vs;
    const cpx<double> ev = ld64(e + o, g.vs, u, s);
    st64(ysave + o, g.vs, u, s, ld64(ysave + o, g.vs, u, s) + c * ev);
    double2 *xp = xsi + (size_t)slot * xs_stride;
    st64(xp, g.vs, u, s, ld64(xp, g.vs, u, s) + ev);
}

void launch_refine_acc(const Geom &g, int nslots, const double2 *e, double c, double2 *ysave, double2 *xsi,
                       size_t xs_stride, hipStream_t st) {
    hipLaunchKernelGGL(k_refine_acc, dim3(unit_parts(0, g), nslots), dim3(kBlock), 0, st, g, e, c, ysave, xsi,
                       xs_stride);
}

// ------------------------------------------------------------------ contraction (Eq. 16)
// For each probed site x of class position ci and each component j (slot 12 ci + j):
//   q(x)  += 1/2 gamma5_jj (1 + Re[D_W y_slot](x, j)),   qi(x) += 1/2 gamma5_jj Im[D_W y_slot](x, j),
// since gamma5 D_ov phi = gamma5 (phi + D_W y) with eps phi = gamma5 D_W y.
// INV (trace of D_W^-1): y_slot = (D_W^dag D_W)^-1 phi and D_W^-1 phi = g_j gamma5 D_W y_slot
// (from D_W^-1 = D_W^dag (D_W D_W^dag)^-1, D_W D_W^dag = gamma5 D_W^dag D_W gamma5 and
// gamma5 phi = g_j phi), so component j of D_W^-1 phi at x is [D_W y_slot](x, j):
//   t(x) += [D_W y_slot](x, j)  (real part into qx, imaginary part into qxi).
// With deflated modes (dk > 0), eps phi gains sum_i c_i w_i (w_i = H u_i / sqrt(theta_i),
// c_i = <u_i, phi>), which adds 1/2 sum_i c_i w_i(x, j) to [gamma5 D_ov phi](x, j) / 2.
template <bool INV>
__global__ __launch_bounds__(kBlock) void k_contract(Geom g, const double2 *U64, const double2 *y, double kappa,
                                                     const int *batch_classes, const int *class_ptr,
                                                     const int *class_sites, double *qx, double *qxi,
                                                     const double2 *dw, const double2 *dcoef, int dk) {
    const int ci = blockIdx.y;
    const int cls = batch_classes[ci];
    const int beg = class_ptr[cls], end = class_ptr[cls + 1];
    const int k = beg + blockIdx.x * kBlock + threadIdx.x;
    if (k >= end) return;
    const int x = class_sites[k];
    double q = 0.0, qi = 0.0;
#pragma unroll 1
    for (int j = 0; j < 12; ++j) {
        const double2 *yv = y + (size_t)(12 * ci + j) * 12 * g.vs;
        cpx<double> acc[12];
        hop_site<double, 1>(U64, g, yv, x, acc);
        const cpx<double> self = ld64(yv, g.vs, j, x);
        const double dre = self.re - kappa * acc[j].re;
        const double dim = self.im - kappa * acc[j].im;
        if constexpr (INV) {
            q += dre;
            qi += dim;
        } else {
            const double g5 = (j < 6) ? 0.5 : -0.5;
            q += g5 * (1.0 + dre);
            qi += g5 * dim;
            const int slot = 12 * ci + j;
            for (int i = 0; i < dk; ++i) {
                const double2 a = dcoef[(size_t)slot * dk + i];
                const cpx<double> w = ld64(dw + (size_t)i * 12 * g.vs, g.vs, j, x);
                q += 0.5 * (a.x * w.re - a.y * w.im);
                qi += 0.5 * (a.x * w.im + a.y * w.re);
            }
        }
    }
    qx[x] = q;
    qxi[x] = qi;
}

void launch_contract(const Geom &g, const double2 *U64, const double2 *y, double kappa, const int *batch_classes,
                     int n_classes, int max_class_size, const int *class_ptr, const int *class_sites, double *qx,
                     double *qxi, bool inverse, const double2 *dw, const double2 *dcoef, int dk, hipStream_t st) {
    dim3 grid((max_class_size + kBlock - 1) / kBlock, n_classes);
    if (inverse)
        hipLaunchKernelGGL(k_contract<true>, grid, dim3(kBlock), 0, st, g, U64, y, kappa, batch_classes, class_ptr,
                           class_sites, qx, qxi, nullptr, nullptr, 0);
    else
        hipLaunchKernelGGL(k_contract<false>, grid, dim3(kBlock), 0, st, g, U64, y, kappa, batch_classes, class_ptr,
                           class_sites, qx, qxi, dw, dcoef, dk);
}

// ------------------------------------------------------------------ locality of D_ov (Eq. 12)
// d holds D_W y_j for the twelve point-source columns j of site `site` (slot stride 12 vs);
// column j of D_ov is e_{site,j} + d_j.  m(x) = (1/144) sum_{i,j} |D_ov(x i; site j)|.
__global__ __launch_bounds__(kBlock) void k_block_mean_abs(Geom g, const double2 *d, int site, double *m) {
    const int x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= g.V) return;
    double acc = 0.0;
#pragma unroll 1
    for (int j = 0; j < 12; ++j) {
        const double2 *col = d + (size_t)j * 12 * g.vs;
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            cpx<double> v = ld64(col, g.vs, i, x);
            if (x == site && i == j) v.re += 1.0;
            acc += sqrt(v.re * v.re + v.im * v.im);
        }
    }
    m[x] = acc / 144.0;
}

void launch_block_mean_abs(const Geom &g, const double2 *d, int site, double *m, hipStream_t st) {
    hipLaunchKernelGGL(k_block_mean_abs, dim3((g.V + kBlock - 1) / kBlock), dim3(kBlock), 0, st, g, d, site, m);
}

// ------------------------------------------------------------------ Lanczos helpers (FP64, one vector)
__global__ __launch_bounds__(kBlock) void k_lanczos_update(Geom g, double2 *w, const double2 *v, const double2 *vprev,
                                                           double alpha, double beta, double *partial) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    double nrm = 0.0;
    if (s < g.V) {
        const size_t i = c * g.vs + s;
        double2 t = w[i];
        const double2 a = v[i], b = vprev[i];
        t.x -= alpha * a.x + beta * b.x;
        t.y -= alpha * a.y + beta * b.y;
        w[i] = t;
        nrm = t.x * t.x + t.y * t.y;
    }
    block_partial(nrm, partial, blockIdx.x);
}

void launch_lanczos_update(const Geom &g, double2 *w, const double2 *v, const double2 *vprev, double alpha,
                           double beta, double *partial, hipStream_t st) {
    hipLaunchKernelGGL(k_lanczos_update, dim3(unit_parts(0, g)), dim3(kBlock), 0, st, g, w, v, vprev, alpha, beta,
                       partial);
}

// Entry i (real and imaginary parts in order of site, spin, colour) of the start vector: 2 u - 1, u
// the i-th SplitMix64 uniform of stream seed, as splitmix64_uniform gives it on the host.
__device__ __forceinline__ double start_entry(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    z ^= z >> 31;
    return 2.0 * ((double)(z >> 11) * 0x1.0p-53) - 1.0;
}

// The Lanczos helpers below run one thread per site through its twelve components, so that a
// vector's sum leaves site_blocks partials, few enough for every wave of the next kernel to add up.
__global__ __launch_bounds__(kBlock) void k_random_start(Geom g, uint64_t seed, double2 *w, double *partial) {
    const int s = blockIdx.x * kBlock + threadIdx.x;
    double nrm = 0.0;
    if (s < g.V) {
        for (int c = 0; c < 12; ++c) {
            const uint64_t i = 24 * (uint64_t)s + 2 * c;
            const cpx<double> v = {start_entry(seed, i), start_entry(seed, i + 1)};
            st64(w, g.vs, c, s, v);
            nrm += v.re * v.re + v.im * v.im;
        }
    }
    block_partial(nrm, partial, blockIdx.x);
}

void launch_random_start(const Geom &g, uint64_t seed, double2 *w, double *partial, hipStream_t st) {
    hipLaunchKernelGGL(k_random_start, dim3(site_blocks(g)), dim3(kBlock), 0, st, g, seed, w, partial);
}

// One Lanczos step on vectors kept unnormalised: n = |u| from its partials (the last step's beta),
// alpha = <u, w> / n^2 from the stencil's, w = (w - alpha u) / n - (n / n_prev) u_prev, and w's
// partial |w|^2.  Dividing here instead of in a kernel of its own leaves three launches a step; on
// one right-hand side each is bound by its latency, 8 us on 8^3 x 16 (bounds there 9.4 -> 7.9 ms).
__global__ __launch_bounds__(kBlock) void k_lanczos_step(Geom g, double2 *w, const double2 *u, const double2 *uprev,
                                                         const double *dot_partials, int np,
                                                         const double *norm_partials, int np_u, double *alpha_out,
                                                         double *norm, double *partial) {
    const int s = blockIdx.x * kBlock + threadIdx.x;
    const double n2 = wave_sum_partials(norm_partials, np_u);
    const double n = sqrt(n2), inv = 1.0 / n;
    const double a = wave_sum_partials(dot_partials, np) / n2;
    const double b = uprev ? n / norm[-1] : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *alpha_out = a;
        *norm = n;
    }
    double nrm = 0.0;
    if (s < g.V) {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            cpx<double> t = ld64(w, g.vs, c, s);
            const cpx<double> x = ld64(u, g.vs, c, s);
            t = inv * (t - a * x);
            if (uprev) t = t - b * ld64(uprev, g.vs, c, s);
            st64(w, g.vs, c, s, t);
            nrm += t.re * t.re + t.im * t.im;
        }
    }
    block_partial(nrm, partial, blockIdx.x);
}

void launch_lanczos_step(const Geom &g, double2 *w, const double2 *u, const double2 *uprev, const double *dot_partials,
                         int np, const double *norm_partials, int np_u, double *alpha_out, double *norm,
                         double *partial, hipStream_t st) {
    hipLaunchKernelGGL(k_lanczos_step, dim3(site_blocks(g)), dim3(kBlock), 0, st, g, w, u, uprev, dot_partials, np,
                       norm_partials, np_u, alpha_out, norm, partial);
}

// v = w / |w|, |w| from its np partials.
__global__ __launch_bounds__(kBlock) void k_lanczos_scale(Geom g, double2 *v, const double2 *w,
                                                          const double *partials, int np) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    const double beta = sqrt(wave_sum_partials(partials, np));
    if (s >= g.V) return;
    const cpx<double> t = ld64(w, g.vs, c, s);
    st64(v, g.vs, c, s, (1.0 / beta) * t);
}

void launch_lanczos_scale(const Geom &g, double2 *v, const double2 *w, const double *partials, int np,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_lanczos_scale, dim3(unit_parts(0, g)), dim3(kBlock), 0, st, g, v, w, partials, np);
}

__global__ __launch_bounds__(kBlock) void k_scale(Geom g, double2 *dst, const double2 *src, double f) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const double2 t = src[c * g.vs + s];
    dst[c * g.vs + s] = make_double2(f * t.x, f * t.y);
}

void launch_scale(const Geom &g, double2 *dst, const double2 *src, double f, hipStream_t st) {
    hipLaunchKernelGGL(k_scale, dim3(unit_parts(0, g)), dim3(kBlock), 0, st, g, dst, src, f);
}

// ------------------------------------------------------------------ low-mode deflation (FP64)
// Complex block sum of (re, im) written to partial[idx] and partial[idx + stride].
__device__ __forceinline__ void block_partial_c(double re, double im, double *partial, size_t idx, size_t stride) {
    __shared__ double lds[2][kBlock / 64];
    re = wave_sum(re);
    im = wave_sum(im);
    if ((threadIdx.x & 63) == 0) {
        lds[0][threadIdx.x >> 6] = re;
        lds[1][threadIdx.x >> 6] = im;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) {
            a += lds[0][i];
            b += lds[1][i];
        }
        partial[idx] = a;
        partial[idx + stride] = b;
    }
}

// partial[(2 i + {0,1}) np + block] = Re, Im of the block's share of <q_i, w>, i < nq,
// q_i = Q + i qstride; grid (np = unit_parts(0, g), nq).
__global__ __launch_bounds__(kBlock) void k_multi_dot(Geom g, const double2 *Q, size_t qstride, const double2 *w,
                                                      double *partial) {
    const int nsb = site_blocks(g);
    const int np = gridDim.x;
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    const int i = blockIdx.y;
    double re = 0.0, im = 0.0;
    if (s < g.V) {
        const double2 q = Q[(size_t)i * qstride + c * g.vs + s], x = w[c * g.vs + s];
        re = q.x * x.x + q.y * x.y;
        im = q.x * x.y - q.y * x.x;
    }
    block_partial_c(re, im, partial, (size_t)(2 * i) * np + blockIdx.x, np);
}

// out[i] = sum of the np partials of pair i, in a fixed order (one wave per i).
__global__ void k_reduce_pairs(const double *partial, int np, double2 *out) {
    const int i = blockIdx.x;
    const double re = wave_sum_partials(partial + (size_t)(2 * i) * np, np);
    const double im = wave_sum_partials(partial + (size_t)(2 * i + 1) * np, np);
    if (threadIdx.x == 0) out[i] = make_double2(re, im);
}

// w -= sum_{i < nq} h_i q_i, or w = sum_{i < nq} h_i q_i when overwrite is set.
__global__ __launch_bounds__(kBlock) void k_multi_axpy(Geom g, const double2 *Q, size_t qstride, int nq,
                                                       const double2 *h, double2 *w, int overwrite) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const size_t o = c * g.vs + s;
    double ar = 0.0, ai = 0.0;
#pragma unroll 4
    for (int i = 0; i < nq; ++i) {
        const double2 q = Q[(size_t)i * qstride + o], hh = h[i];
        ar += hh.x * q.x - hh.y * q.y;
        ai += hh.x * q.y + hh.y * q.x;
    }
    if (overwrite) {
        w[o] = make_double2(ar, ai);
    } else {
        const double2 t = w[o];
        w[o] = make_double2(t.x - ar, t.y - ai);
    }
}

// v = f gamma5 v (gamma5 = +1 on spins 0, 1 and -1 on spins 2, 3; component c = 3 spin + colour).
__global__ __launch_bounds__(kBlock) void k_g5_scale(Geom g, double2 *v, double f) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const double ff = c < 6 ? f : -f;
    const double2 t = v[c * g.vs + s];
    v[c * g.vs + s] = make_double2(ff * t.x, ff * t.y);
}

// Deflation coefficients of probing sources: coef[slot k + i] = <u_i, phi_slot> = sum over the
// sites x of the slot's class of conj(u_i(x, comp)); grid (k, nslots).
__global__ __launch_bounds__(kBlock) void k_defl_coef_probe(Geom g, const double2 *u, int k, const int *slot_class,
                                                            const int *slot_comp, const int *class_ptr,
                                                            const int *class_sites, double2 *coef) {
    const int i = blockIdx.x, slot = blockIdx.y;
    const int cls = slot_class[slot], comp = slot_comp[slot];
    const double2 *ui = u + (size_t)i * 12 * g.vs + comp * g.vs;
    double re = 0.0, im = 0.0;
    for (int t = class_ptr[cls] + threadIdx.x; t < class_ptr[cls + 1]; t += kBlock) {
        const double2 v = ui[class_sites[t]];
        re += v.x;
        im -= v.y;
    }
    __shared__ double lds[2][kBlock / 64];
    re = wave_sum(re);
    im = wave_sum(im);
    if ((threadIdx.x & 63) == 0) {
        lds[0][threadIdx.x >> 6] = re;
        lds[1][threadIdx.x >> 6] = im;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int j = 0; j < kBlock / 64; ++j) {
            a += lds[0][j];
            b += lds[1][j];
        }
        coef[(size_t)slot * k + i] = make_double2(a, b);
    }
}

// out_slot += gamma5 sum_i coef[slot k + i] w_i  (D_ov b of deflated modes), grid (units, nslots).
__global__ __launch_bounds__(kBlock) void k_add_defl(Geom g, double2 *out, const double2 *w, int k,
                                                     const double2 *coef) {
    const int nsb = site_blocks(g);
    const int c = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    const int slot = blockIdx.y;
    if (s >= g.V) return;
    double ar = 0.0, ai = 0.0;
    for (int i = 0; i < k; ++i) {
        const double2 a = coef[(size_t)slot * k + i], v = w[(size_t)i * 12 * g.vs + c * g.vs + s];
        ar += a.x * v.x - a.y * v.y;
        ai += a.x * v.y + a.y * v.x;
    }
    const double f = c < 6 ? 1.0 : -1.0;
    double2 &o = out[(size_t)slot * 12 * g.vs + c * g.vs + s];
    o = make_double2(o.x + f * ar, o.y + f * ai);
}

void launch_multi_dot(const Geom &g, const double2 *Q, size_t qstride, int nq, const double2 *w, double *partial,
                      double2 *out, hipStream_t st) {
    const int np = unit_parts(0, g);
    hipLaunchKernelGGL(k_multi_dot, dim3(np, nq), dim3(kBlock), 0, st, g, Q, qstride, w, partial);
    hipLaunchKernelGGL(k_reduce_pairs, dim3(nq), dim3(64), 0, st, partial, np, out);
}

void launch_multi_axpy(const Geom &g, const double2 *Q, size_t qstride, int nq, const double2 *h, double2 *w,
                       bool overwrite, hipStream_t st) {
    hipLaunchKernelGGL(k_multi_axpy, dim3(unit_parts(0, g)), dim3(kBlock), 0, st, g, Q, qstride, nq, h, w,
                       overwrite ? 1 : 0);
}

void launch_g5_scale(const Geom &g, double2 *v, double f, hipStream_t st) {
    hipLaunchKernelGGL(k_g5_scale, dim3(unit_parts(0, g)), dim3(kBlock), 0, st, g, v, f);
}

void launch_defl_coef_probe(const Geom &g, const double2 *u, int k, const int *slot_class, const int *slot_comp,
                            const int *class_ptr, const int *class_sites, int nslots, double2 *coef, hipStream_t st) {
    hipLaunchKernelGGL(k_defl_coef_probe, dim3(k, nslots), dim3(kBlock), 0, st, g, u, k, slot_class, slot_comp,
                       class_ptr, class_sites, coef);
}

void launch_add_defl(const Geom &g, double2 *out, const double2 *w, int k, const double2 *coef, int nslots,
                     hipStream_t st) {
    hipLaunchKernelGGL(k_add_defl, dim3(unit_parts(0, g), nslots), dim3(kBlock), 0, st, g, out, w, k, coef);
}

// ------------------------------------------------------------------ precision conversion
__global__ __launch_bounds__(kBlock) void k_to_f32(Geom g, const double2 *src, float4 *dst) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const double2 *sp = src + (size_t)slot * 12 * g.vs;
    const double2 a = sp[(2 * u) * g.vs + s], b = sp[(2 * u + 1) * g.vs + s];
    dst[(size_t)slot * 6 * g.vs + u * g.vs + s] = make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
}

__global__ __launch_bounds__(kBlock) void k_to_f64(Geom g, const float4 *src, double2 *dst) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    const float4 t = src[(size_t)slot * 6 * g.vs + u * g.vs + s];
    double2 *dp = dst + (size_t)slot * 12 * g.vs;
    dp[(2 * u) * g.vs + s] = make_double2(t.x, t.y);
    dp[(2 * u + 1) * g.vs + s] = make_double2(t.z, t.w);
}

// Host spinor layout [rhs][site][spin*3 + colour] complex128 <-> device [rhs][unit][site] double2.
__global__ __launch_bounds__(kBlock) void k_aos_to_soa(Geom g, const double2 *aos, double2 *soa) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    soa[((size_t)slot * 12 + u) * g.vs + s] = aos[((size_t)slot * g.V + s) * 12 + u];
}

__global__ __launch_bounds__(kBlock) void k_soa_to_aos(Geom g, const double2 *soa, double2 *aos) {
    const int slot = blockIdx.y;
    const int nsb = site_blocks(g);
    const int u = blockIdx.x / nsb;
    const int s = (blockIdx.x % nsb) * kBlock + threadIdx.x;
    if (s >= g.V) return;
    aos[((size_t)slot * g.V + s) * 12 + u] = soa[((size_t)slot * 12 + u) * g.vs + s];
}

void launch_layout(bool to_soa, const Geom &g, const double2 *src, double2 *dst, int nslots, hipStream_t st) {
    dim3 grid(unit_parts(0, g), nslots);
    if (to_soa)
        hipLaunchKernelGGL(k_aos_to_soa, grid, dim3(kBlock), 0, st, g, src, dst);
    else
        hipLaunchKernelGGL(k_soa_to_aos, grid, dim3(kBlock), 0, st, g, src, dst);
}

void launch_convert(int to_prec, const Geom &g, const void *src, void *dst, int nslots, hipStream_t st) {
    dim3 grid(unit_parts(1, g), nslots);
    if (to_prec == 1)
        hipLaunchKernelGGL(k_to_f32, grid, dim3(kBlock), 0, st, g, (const double2 *)src, (float4 *)dst);
    else
        hipLaunchKernelGGL(k_to_f64, grid, dim3(kBlock), 0, st, g, (const float4 *)src, (double2 *)dst);
}

// ------------------------------------------------------------------ calibration
// dst = src over n float4 (grid-stride), with cached or non-temporal loads and stores: kernels of
// known size (n * 16 bytes read and written) for scaling hardware byte counters.
template <bool NT>
__global__ __launch_bounds__(kBlock) void k_stream_copy(const float4 *__restrict__ src, float4 *__restrict__ dst,
                                                        size_t n) {
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        if constexpr (NT) {
            const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(src + i));
            __builtin_nontemporal_store(t, reinterpret_cast<f32x4 *>(dst + i));
        } else {
            dst[i] = src[i];
        }
    }
}

void launch_stream_copy(bool nontemporal, const void *src, void *dst, size_t n_float4, hipStream_t st) {
    const size_t blocks = std::min<size_t>((n_float4 + kBlock - 1) / kBlock, 8192);
    if (nontemporal)
        hipLaunchKernelGGL(k_stream_copy<true>, dim3((unsigned)blocks), dim3(kBlock), 0, st, (const float4 *)src,
                           (float4 *)dst, n_float4);
    else
        hipLaunchKernelGGL(k_stream_copy<false>, dim3((unsigned)blocks), dim3(kBlock), 0, st, (const float4 *)src,
                           (float4 *)dst, n_float4);
}

}  // namespace smpq
