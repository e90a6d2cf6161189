// Launch interface of the device kernels (kernels.hip) used by the C ABI (api.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace smpq {

constexpr int kBlock = 256;

// Geometry + storage strides.  A spinor of one right-hand side is stored as
// components [unit][site] with unit stride `vs` (the padded volume): FP64 uses 12
// double2 units (one complex each), FP32 uses 6 float4 units (two complexes each).
// FP64 links are [mu][row*3 + col][site] double2; FP32 links keep the first two rows,
// [mu][3][site] float4 holding (u00,u01), (u02,u10), (u11,u12).
struct Geom {
    int nx, ny, nz, nt, V;
    size_t vs;
    // stencil variants (smpq_tuning in smpq.h).  f32_kind: 0 any lattice, f32_nr right-hand sides per
    // block; 1 and 3 a 16x16 xy-plane per block in LDS, links in registers for f32_nr sides (3: x and y
    // links in LDS); 2 xy-tiles of tile_y rows with halo rows, links in registers; 4 the same tiles, links
    // read for every side or every two.  f64_kind: 0 any lattice, 2^f64_lgr sides per block; 1 xy-tiles,
    // f64_nr per block.  band: z-band of the plane order of kinds 1 to 4.  tile_y = tile_rows(nx, ny) (0
    // when no tile fits).  f32_il / f64_il: in FP32 kind 4 and FP64 kind 1 consecutive blocks take that
    // many groups of right-hand sides of one tile before the next tile, so that the tile's links are
    // still in L2
    int f32_kind, f32_nr, f64_lgr, band, tile_y;
    int f64_kind, f64_nr;
    int f32_il, f64_il;
    int adapt;      // no variant chosen: each launch takes the one that suits its size
    int f64_full;   // a chosen f64_kind 1 reads all nine link entries too (else two rows, the third rebuilt)
    // the FP32 variant of the D_W^dag launches (f32_kind, f32_nr and f32_il above apply to D_W):
    // the two stencils of a CG iteration have different epilogues and favour different variants
    int f32_dag_kind, f32_dag_nr, f32_dag_il;
};

// Right-hand-side addressing: slot k of a launch uses offset (slot * slot_stride + extra)
// units from the base pointer, where slot = list[k] (or k when list is null) and the
// number of slots is *count (or n when count is null).
struct Slots {
    const int *list;
    const int *count;
    int n;
};

// Per-batch multi-shift CG state (all device pointers; one entry per slot, slot*NS + shift, or
// (slot*K + j)*NS + shift for iteration j of a block).
//
// The shifted systems are updated once per block of up to K iterations: the residuals r_1 .. r_m of
// the block's m iterations stay in a ring of K vectors per right-hand side, with the coefficients
// of every shift, and the block update runs the recurrences y += c_i a p_i, p_i = z r + b p_i of
// all its iterations in registers.  The arithmetic is that of an update in every iteration, so
// results do not depend on K.
struct MSState {
    int B, NS, i0, K;
    double tol;
    double *rr, *rr1;    // |r|^2 (rr1: every other iteration where its readers and writer overlap)
    double *bnorm, *alpha, *alpha_prev, *beta, *beta_prev;
    double *zeta, *zeta_prev;
    int *sh_active, *sh_iters;
    int *done, *iters, *status;
    // the current block: iterations done and their coefficients, [slot][K][NS]: c_i a, a, and z and b
    // in the iteration precision
    int *blk_n;
    double *h_cy, *h_a;
    void *h_z, *h_b;
    // the block update: number of residuals, masks of the shifts active at the block's start (or to
    // be written) and of those to write
    int *fl_m;
    unsigned *fl_act, *fl_rd, *fl_wr;
    // 16-bit shifted directions: p_i is stored as p_i / sh_scale[slot NS + i]; the scale that
    // decodes the stored direction and the reciprocal of the one the block update stores with
    double *sh_scale, *s_sold, *s_snew;
    // the vectors the stencil reads rounded to 16 bits (0: not, 1: FP16, 2: BF16), and |r|^2 after each
    // iteration of the block, [slot][K], from which the block update scales the base direction alike
    int vec16;
    double *h_rr;
    double dir_norm;     // 1 / sqrt(24 V): a direction of norm n has entries of size ~ n dir_norm
    long long *cnt_entries, *cnt_active;               // listed shifts, iterations
    long long *cnt_fl, *cnt_fl_r, *cnt_fl_p;           // block updates, residuals and directions they moved
    const double *c, *delta;
    double *partial;     // per-block partial sums, slot stride pstride
    double *partial2;    // the same of the second stencil of an iteration
    size_t pstride;
    int *list, *count;
};

// Source of the right-hand sides: probing (class, spin-colour component) or explicit FP64 vectors.
struct Source {
    const int *colour;      // probing: colour of each site
    const int *slot_class;  // probing: class of each slot
    const int *slot_comp;   // probing: component (spin*3 + colour) of each slot
    const double2 *b;       // explicit: FP64 vectors, slot stride 12*vs (null for probing)
    // deflation: the source is b - sum_{i < dk} dcoef[slot dk + i] u_i, u_i = du + i 12 vs
    const double2 *du = nullptr;
    const double2 *dcoef = nullptr;
    int dk = 0;
};

enum { kStatusOK = 0, kStatusBreakdown = 1 };

// With d = in - kappa * hop(in) (D_W in, or D_W^dag in when dag):
//   epi 0: out = d
//   epi 1: out = d + sigma * aux, partial[slot][block] = Re <aux, out>
//   epi 3: out = d, partial = |d|^2 + sigma |in|^2   (= <in, (H^2 + sigma) in> when dag = 0)
//   epi 2: out = r - alpha[slot] (d + sigma * aux), r read at out + rstep.r_ofs units (out = r when
//          status[slot] is not OK); partial = |out|^2 (the product d + sigma aux is not stored)
// done (nullable): slots whose flag is set are skipped.
// prec: 0 = FP64, 1 = FP32 (FP32: epi 0 both ways, epi 3 with dag = 0, epi 1 and 2 with
// dag = 1).  The kernel variant comes from g's tuning fields; epilogues 1-3 write
// dslash_partials(prec, g) partials per slot.
// Epilogue 2's step: alpha and status per slot, or (npart > 0, dslash_takes_partials) |r|^2 and the
// npart partials of <p, A p> they follow from, slot stride partial_stride.
struct ResidualStep {
    const double *alpha = nullptr;
    const int *status = nullptr;
    ptrdiff_t r_ofs = 0;
    const double *pap = nullptr, *rr = nullptr;
    int npart = 0;
};
void launch_dslash(int prec, bool dag, int epi, const void *U, const void *in, size_t in_stride,
                   size_t in_extra, void *out, size_t out_stride, const void *aux, size_t aux_stride,
                   size_t aux_extra, const Geom &g, double kappa, double sigma, Slots sl, int max_slots,
                   double *partial, hipStream_t st, const ResidualStep &rstep = {}, const int *done = nullptr);
bool dslash_takes_partials(int prec, const Geom &g, bool dag);   // the variant can compute alpha itself
__host__ __device__ int site_blocks(const Geom &g);   // blocks of 256 sites
int dslash_partials(int prec, const Geom &g, bool dag);   // partials per slot of the stencil epilogue
bool plane_tileable(const Geom &g);   // the xy-plane has exactly 256 sites
// Rows per xy-tile: the largest divisor ty >= 2 of ny with nx * ty <= 256 and a multiple of 64
// (nx <= 64); 0 when there is none.
int tile_rows(int nx, int ny);
bool valid_tuning(int prec, const Geom &g);            // g's tuning names an instantiated variant
int unit_parts(int prec, const Geom &g);        // partials per slot written by element-wise kernels
size_t partial_stride(const Geom &g);           // slot stride of the partial buffer (>= both)

// Storage of the shifted search directions p_i (i != base) in the FP32 path: FP32, or FP16 /
// BF16 scaled by a per-direction FP64 factor (the base direction, which the stencil reads,
// stays FP32).  With 16-bit storage, p holds only the base direction of each slot and ph the NS
// directions in 16 bits (the base entry unused).
enum { kDirF32 = 0, kDirF16 = 1, kDirBF16 = 2, kDirVec16 = 3 };   // the last: see vec16

// r = p_i = b, y = c0 b; FP32 path: x0 = 0 (null otherwise).  r and p have slot strides rst and
// pst (units).  With 16-bit directions only r and the base direction are written;
// launch_dir16_init writes the others after launch_scalars_init has set their scales from |b|.
void launch_cg_init(int prec, const Geom &g, const Source &src, int nslots, int NS, double c0, void *r, size_t rst,
                    void *p, size_t pst, double2 *y, double2 *x0, double *partial, int dir, hipStream_t st);
void launch_dir16_init(const Geom &g, const MSState &s, int nslots, const void *r, size_t rst, int dir, void *ph,
                       hipStream_t st);
void launch_scalars_init(const MSState &s, int npart, int nslots, hipStream_t st);
void launch_scalars_alpha(const MSState &s, int npart, hipStream_t st);
void launch_scalars_beta(int prec, const MSState &s, int npart, hipStream_t st);
// p_out = r + beta p_in of the base system, slots of the list that are not done; r at
// slot * rst, p_in and p_out at slot * pst units.  np_pap > 0: instead of launch_scalars_alpha and
// _beta, from the np_pap and np_rr partials of the two stencils, |r|^2 read from rr_in and
// written to rr_out (another buffer); at most kFusedPartials of each.
constexpr int kFusedPartials = 64;
void launch_base_direction(int prec, const Geom &g, const MSState &s, const void *r, size_t rst, const void *p_in,
                           void *p_out, size_t pst, int np_pap, int np_rr, const double *rr_in, double *rr_out,
                           hipStream_t st);
// Small lattices: up to `iters` iterations of the base system and the shifts' recurrences for every
// listed slot in one launch (one workgroup per slot), from iteration n0 of the block: p_in and p_out
// as the base direction's buffers, the residuals written to the ring.  Needs K > 1 and
// n0 + iters <= K.
constexpr int kSmallThreads = 512;
bool small_lattice(int prec, const Geom &g);
void launch_cg_small(int prec, const Geom &g, const MSState &s, const void *U, double kappa, double sigma,
                     const void *p_in, void *p_out, size_t pst, void *ring, int n0, int iters, hipStream_t st);
// Ends the block: what the block update has to do, blk_n = 0, and the new scales of 16-bit
// directions.  base_inline: the block update writes the base direction too.
void launch_block_end(const MSState &s, bool base_inline, int dir, hipStream_t st);
// The block update: y, x0 (null in the FP64 path) and every direction that is still needed,
// from the ring (slot stride K vectors) and the directions at the block's start (the base one at
// entry base_sel of the slot's directions; slot stride pst units).  xs (null, or FP64 vectors
// [slot][NS][12][vs]) receives every shift's own solution.
void launch_block_update(int prec, const Geom &g, const MSState &s, const void *ring, void *p, size_t pst,
                         int base_sel, double2 *y, double2 *x0, int dir, void *ph, double2 *xs, hipStream_t st);
void launch_compact(const MSState &s, hipStream_t st);
// Evaluated precision: FP32 vectors of the listed slots (v + slot * slot_stride + extra, in
// float4 units) rounded in place to FP16 (mode 1, scaled by sqrt(|r|^2 / (24 V)) of the slot)
// or BF16 (mode 2).
void launch_round16(const Geom &g, const MSState &s, void *v, size_t slot_stride, size_t extra, int mode,
                    hipStream_t st);
void launch_reliable(int prec, const Geom &g, const MSState &s, const Source &src, const double2 *ap64, size_t ast,
                     void *r, size_t rst, hipStream_t st);
void launch_scalars_rr(const MSState &s, int npart, hipStream_t st);

// Per-shift check (FP64 vectors, slot stride 12 vs, the first nslots slots):
// resid64: out = b - ap64 (b from src), partial[slot][block] = |out|^2 (unit_parts(0, g) blocks);
// slot_sums: sums[slot] = sum of the slot's npart partials (fixed order);
// zero_unflagged: v[slot] = 0 where flag[slot] == 0;
// refine_acc: ysave[slot] += c e[slot], xsi[slot] += e[slot] (xsi slot stride xs_stride units).
void launch_resid64(const Geom &g, int nslots, const Source &src, const double2 *ap64, double2 *out,
                    double *partial, size_t pstride, hipStream_t st);
void launch_slot_sums(int nslots, const double *partial, size_t pstride, int npart, double *sums, hipStream_t st);
void launch_zero_unflagged(const Geom &g, int nslots, const int *flag, double2 *v, hipStream_t st);
void launch_refine_acc(const Geom &g, int nslots, const double2 *e, double c, double2 *ysave, double2 *xsi,
                       size_t xs_stride, hipStream_t st);

// Low-mode deflation helpers (FP64 vectors [12][vs]).  multi_dot: out[i] = <q_i, w> for
// q_i = Q + i qstride, i < nq (partial: 2 nq unit_parts doubles); multi_axpy: w -= sum h_i q_i,
// or w = sum h_i q_i with overwrite; g5_scale: v = f gamma5 v; defl_coef_probe: coef[slot k +
// i] = <u_i, phi_slot> for probing sources; add_defl: out_slot += gamma5 sum_i coef w_i.
void launch_multi_dot(const Geom &g, const double2 *Q, size_t qstride, int nq, const double2 *w, double *partial,
                      double2 *out, hipStream_t st);
void launch_multi_axpy(const Geom &g, const double2 *Q, size_t qstride, int nq, const double2 *h, double2 *w,
                       bool overwrite, hipStream_t st);
void launch_g5_scale(const Geom &g, double2 *v, double f, hipStream_t st);
void launch_defl_coef_probe(const Geom &g, const double2 *u, int k, const int *slot_class, const int *slot_comp,
                            const int *class_ptr, const int *class_sites, int nslots, double2 *coef, hipStream_t st);
void launch_add_defl(const Geom &g, double2 *out, const double2 *w, int k, const double2 *coef, int nslots,
                     hipStream_t st);

// m(x) = mean |D_ov(x i; site j)| over the 144 entries, from d_j = D_W y_j of the twelve
// point-source columns of `site` (Eq. 12).
void launch_block_mean_abs(const Geom &g, const double2 *d, int site, double *m, hipStream_t st);

// q(x) contraction (Eq. 16) for the classes of one batch; slot = 12*class_pos + comp.
// inverse: the trace density of D_W^-1 from y = (D_W^dag D_W)^-1 phi instead.  dk deflated
// modes add their exact-sign part from dw (H u_i / sqrt(theta_i)) and dcoef ([slot][dk]).
void launch_contract(const Geom &g, const double2 *U64, const double2 *y, double kappa, const int *batch_classes,
                     int n_classes, int max_class_size, const int *class_ptr, const int *class_sites, double *qx,
                     double *qxi, bool inverse, const double2 *dw, const double2 *dcoef, int dk, hipStream_t st);

// Lanczos helpers (single FP64 vector); the update writes unit_parts(0, g) partials
void launch_lanczos_update(const Geom &g, double2 *w, const double2 *v, const double2 *vprev, double alpha,
                           double beta, double *partial, hipStream_t st);
// Lanczos on one vector with its scalars on the device: random_start: the SplitMix64 vector of
// `seed`, unnormalised, and site_blocks partials of its |.|^2; step: n = *norm = |u| from its np_u
// norm_partials, *alpha_out = (sum of the np dot_partials) / n^2, w = (w - alpha u) / n -
// (n / norm[-1]) uprev (uprev null in the first step), site_blocks partials of |w|^2;
// scale: v = w / |w|, |w| from its np partials.
void launch_random_start(const Geom &g, uint64_t seed, double2 *w, double *partial, hipStream_t st);
void launch_lanczos_step(const Geom &g, double2 *w, const double2 *u, const double2 *uprev, const double *dot_partials,
                         int np, const double *norm_partials, int np_u, double *alpha_out, double *norm,
                         double *partial, hipStream_t st);
void launch_lanczos_scale(const Geom &g, double2 *v, const double2 *w, const double *partials, int np,
                          hipStream_t st);
void launch_scale(const Geom &g, double2 *dst, const double2 *src, double f, hipStream_t st);
// dst = src over n float4 with cached (nontemporal = false) or non-temporal loads and stores:
// kernels of known size for scaling hardware byte counters
void launch_stream_copy(bool nontemporal, const void *src, void *dst, size_t n_float4, hipStream_t st);
// layout conversion between FP64 (double2 x 12) and FP32 (float4 x 6) spinors, n slots
void launch_convert(int to_prec, const Geom &g, const void *src, void *dst, int nslots, hipStream_t st);
// host spinor layout [slot][site][12] double2 (V sites per slot) <-> device [slot][12][vs]
void launch_layout(bool to_soa, const Geom &g, const double2 *src, double2 *dst, int nslots, hipStream_t st);

}  // namespace smpq
