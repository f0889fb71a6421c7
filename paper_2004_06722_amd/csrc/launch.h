// Host-callable launchers of the device kernels.
#pragma once

#include "bp_internal.h"

namespace bp {

// operator kernels (ops.hip)
bool kernels_cover(int p, int q, int quad);
int64_t plane_epb(int p1, int q, int which);
// work-groups (= energy partial rows) of one operator launch for `which`;
// apply_blocks is the largest over mass and stiffness (partial buffer size)
int64_t apply_rows(const bp_op_s *op, int which);
int64_t apply_blocks(const bp_op_s *op);
// threads of a work-group of the stiffness operator
int apply_threads(const bp_op_s *op);
// partial rows that any one operator application may write (buffer sizing)
int64_t max_partial_rows(const bp_op_s *op);
// The node order of the vectors a launch reads and writes. Internal: the
// solves' own, element-interior nodes stored by their element (own). Caller's:
// the vectors of bp_apply, bp_diag, bp_grad_kappa and bp_mass_misfit as they
// come, every node added, where the numbering allows it (by_internal_order in
// capi.cpp). An operator launch alone is about 10% slower so, but permuting u in
// and w out is two launches and 2 x 147 us more at p = 8, E = 47,520 in a
// lexicographic order (bp_apply 789 -> 562 us; 17.6 -> 12 us at E = 120, p = 5).
struct NodeMap {
  const int32_t *idx;
  int own;
};
inline NodeMap internal_map(const bp_op_s *op) { return {op->idx, op->n_owned > 0 ? 1 : 0}; }
inline NodeMap caller_map(const bp_op_s *op) { return {op->idx_c, 0}; }
// w, in the order of m, is clear before (the Gauss-Legendre mass overwrites it)
int launch_apply(const bp_op_s *op, int which, bool f32, const NodeMap &m, const void *u, void *w,
                 bool masked, double *part, const int *done, hipStream_t s);
// mass element kernel with element-local output: op->wl (op->wl32 if f32)
// [ncomp][nelem][p1^3] = B_L (Q u), zero at masked nodes; needs op->tr_pair
// (Gauss-Legendre operators). launch_apply(BP_MASS) runs it and then
// gather_local; the PCG iteration fuses the gather into the residual update.
int launch_mass_wl(const bp_op_s *op, bool f32, const NodeMap &m, const void *u, bool masked,
                   double *part, const int *done, hipStream_t s);
// w_L = A_L u_L (or B_L u_L) per element, no gather or scatter; uL and wL are
// [ncomp][nelem][p1^3] in the precision of f32
int launch_apply_local(const bp_op_s *op, int which, bool f32, const void *uL, void *wL,
                       hipStream_t s);
int launch_diag(const bp_op_s *op, int which, const NodeMap &m, double *d, bool masked,
                hipStream_t s);
// G [E][6][q^3] and Bt [E][q^3] from the node coordinates X [E][p1^3][3] (device);
// *bad (device, preset to INT_MAX) gets the smallest element with det J <= 0
int launch_geometry(const bp_op_s *op, const double *X, double *G, double *Bt, int *bad,
                    hipStream_t s);
int launch_grad_kappa(const bp_op_s *op, const NodeMap &m, const double *lam, const double *u,
                      double *g, hipStream_t s);

// vector kernels (vec.hip); sizes are global nodes n and components nc
// CG vector kernels give each work-group kVecThreads nodes (vec_blocks; FP32
// iteration kernels two per thread, FP64 one); fills and
// conversions use a capped grid-stride grid (grid_blocks). Up to
// kDirectRows pairs of block partial sums go straight to the final fixed-order
// single-work-group sum (one launch less per reduction on small meshes; eight
// columns of 16,290 rows took it 28 us; one column folded or direct, 40 iterations:
// 17,576 rows 7603 and 7600 us, 21,952 rows 9399 and 9450, 29,791 rows 12,396 and
// 12,370);
// more are first folded to at most kStage2Rows rows, stored right after
// the partials.
constexpr int kVecThreads = 256;
constexpr int64_t kVecMaxBlocks = 2048;
constexpr int64_t kStage2Rows = 256;
constexpr int64_t kDirectRows = 16384;
int64_t vec_blocks(int64_t n);
int64_t grid_blocks(int64_t n);
void fill_f64(double *x, int64_t n, double v, hipStream_t s);
void fill_f32(float *x, int64_t n, float v, hipStream_t s);
// Gk = kappa G per point (and its FP32 copy if Gk32); kappa is in the caller's
// [E][c][b][a] point order, G stored reversed when qrev = q (else qrev = 0)
void scale_geometry(const double *G, const double *kappa, double *Gk, float *Gk32, int qrev,
                    int64_t nelem, int nq, hipStream_t s);
// Bb = beta_q * Bt (beta_q NULL: the constant beta), and its FP32 copy if Bb32;
// point orders as for scale_geometry
void scale_mass(const double *Bt, const double *beta_q, double beta, double *Bb, float *Bb32,
                int nq, int qrev, int64_t count, hipStream_t s);
void to_f32(const double *src, float *dst, int64_t n, hipStream_t s);
void invert_diag(const double *d, double *dinv, float *dinv32, int64_t n, hipStream_t s);

// CG steps; part holds per-block partial sums, sc the device scalars.
// Where perm is given, b and x0 are in the caller's order, and x0 is copied
// into x if sc->x0_zero is set (otherwise x holds it).
template <typename T>
void cg_init(int nc, int64_t n, const T *b, const T *x0, T *x, const int32_t *perm, T *r, T *w,
             T *p, const T *dinv, double *part, DevScalars *sc, hipStream_t s);
// clears sc->x0_zero if any entry of x is not zero
void scan_nonzero(const double *x, int64_t count, DevScalars *sc, hipStream_t s);
// check = false (a fixed number of iterations): the kernels do not stop on
// the done flag, so their loads need not wait for it
void cg_fin_alpha(int nc, const double *part, int64_t nb, DevScalars *sc, hipStream_t s,
                  bool check = true);
// n_own: nodes [0, n_own) are written whole by the operator (internal
// order), so w is cleared from n_own on
template <typename T>
void cg_update_r(int nc, int64_t n, T *r, T *w, const T *dinv, double *part, DevScalars *sc,
                 hipStream_t s, bool check = true, int64_t n_own = 0);
void cg_fin_beta(int nc, int64_t nb, const double *part, DevScalars *sc, hipStream_t s,
                 bool check = true);
template <typename T>
void cg_update_xp(int nc, int64_t n, T *x, T *p, const T *z, DevScalars *sc, hipStream_t s,
                  bool check = true);

// The fused iteration of small and mid-size meshes. The residual update
// computes alpha itself from the operator's partials pa[nba][nc] and writes its
// own partials into pr ([rxp_rows(n)][2 nc]); the direction update computes beta
// and the convergence test from pr. Three launches per iteration instead of
// five; parity = iteration index & 1 (selects the r.z slot, DevScalars::rzs).
// One node per thread up to kFusedRows groups of 256, kRxpNodes beyond, so that
// the tables that every work-group reduces stay short.
constexpr int64_t kFusedRows = 1024;
constexpr int kRxpNodes = 4;
// the wider form: components, and the bounds of its tables. Five launches ->
// three, 40 iterations in us: at the bounds one component gains 7-8% (BP3 p = 7,
// E = 14^3, 948 rows, 2055 -> 1897; p = 3, 26^3, product 0.9M, 1914 -> 1770), three 11%
// (BP4 p = 7, 12^3, 1.04M, 3701 -> 3305), four 15% (BP6 p = 9, 8^3, 0.8M, 2537 ->
// 2163). Beyond them it still gains, less with the product: BP3 p = 7, 17^3 (2.8M)
// 3150 -> 2908, p = 3, 32^3 (2.9M) 2970 -> 2854, BP4 p = 7, 13^3 (1.7M) 3833 -> 3428,
// 15^3 (3.9M) 5478 -> 5199; BP5 p = 7, 20^3 (22M) 3883 -> 3911, FP32 2779 -> 2937, p =
// 3, 34^3 (10M) 3008 -> 3035. The bounds are the sizes that were tried first, not
// the last ones that gain.
constexpr int kFusedWide = 4;
constexpr int64_t kFused3ApplyRows = 4096, kFused3Product = int64_t(1) << 20;
int64_t rxp_rows(int64_t n);  // partial rows of the fused vector kernels
bool cg_fused_fits(int nc, int64_t n, int64_t nb_apply);
template <typename T>
void cg_update_r_fused(int nc, int64_t n, T *z, T *w, const T *dinv, const double *pa,
                       int64_t nba, double *pr, DevScalars *sc, int parity, hipStream_t s,
                       bool check, int64_t n_own);
template <typename T>
void cg_update_xp_fused(int nc, int64_t n, T *x, T *p, const T *z, const double *pr,
                        DevScalars *sc, int parity, hipStream_t s, bool check);

// The two-launch iteration of small and mid-size meshes (collocated
// stiffness, one component, p1 <= 9; PZIter; cg_fused2_fits): the operator
// launch forms p_k = z_k + beta p_{k-1} while gathering and takes the
// stopping test on r_k; cg_update_rxp_fused then
// stores p_k, updates x and z = dinv r and writes the partials of the next
// r.z and r.r into pr. cg_fin_rxp_fused, once after the last iteration,
// reduces pr into the scalars the host reads (r.z, r.r, and the stopping
// test of the last iterate).
// The bounds of the two partial tables: every work-group of each launch reads
// the other's. Four launches (FP32: five) -> two, 40 iterations in us, inside and
// outside each bound:
// - product of the two: FP64 p = 5, E = 26^3 (5.5M) 3856 -> 3638, p = 6, 22^3
//   (4.9M) 3879 -> 3626, p = 4, 28^3 (6.2M) 3106 -> 3117, 30^3 (9.3M) 3545 -> 3700;
//   FP32 p = 7, 16^3 (5.8M) 1806 -> 1775, 17^3 (8.3M) 2038 -> 2062, 18^3 (11.7M)
//   2299 -> 2422;
// - vector rows: p = 8, 16^3 (2097 rows) 3102 -> 3017; 17^3 (2512) 3635 -> 3454
//   would gain as well;
// - operator work-groups: p = 1, 50^3 (7813) 1410 -> 1328, 54^3 (9842) 1578 -> 1630;
// - vector rows per thread of the operator, FP64 (a work-group of one wave, p = 1, 2,
//   3, 7, sums them in that many dependent steps): p = 7, 14^3 (15) 1770 -> 1765,
//   15^3 (18) 2067 -> 2092 (60 iterations in another run 3164-3247 -> 3148-3162),
//   16^3 (22) 2280 -> 2396, 17^3 (26) 2716 -> 3131; p = 3, 32^3 (14) 2650 -> 2643.
//   The FP32 kernel gains to 22 a thread (above).
constexpr int64_t kFused2VecRows = 2400, kFused2ApplyRows = 8192, kFused2ThreadRows = 20;
constexpr int64_t kFused2Product = int64_t(9) << 20;
// threads: of the operator's work-groups, in FP64 (0: no bound of rows per thread)
bool cg_fused2_fits(int64_t n, int64_t nb_apply, int threads);
bool apply_pz_supported(const bp_op_s *op, int which);
template <typename T>
int launch_apply_pz(const bp_op_s *op, const T *p, T *w, bool masked, double *part,
                    const int *done, const PZIter<T> &pz, hipStream_t s);
template <typename T>
void cg_update_rxp_fused(int64_t n, T *x, T *p, T *z, T *w, const T *dinv, const double *pa,
                         int64_t nba, double *pr, DevScalars *sc, int parity, hipStream_t s,
                         bool check, bool first, int64_t n_own);
void cg_fin_rxp_fused(int64_t n, const double *pr, DevScalars *sc, hipStream_t s);
// The four-launch form (one component, above those bounds): the operator
// launch (PZIter with fused = 0: beta from k_fin_beta), cg_fin_alpha,
// cg_update_rxp (p, x and z in one pass; partials for cg_fin_beta),
// cg_fin_beta.
bool cg_streams(int64_t n);  // FP64 vectors of n entries take the streaming kernels
template <typename T>
void cg_update_rxp(int64_t n, T *x, T *p, T *z, T *w, const T *dinv, double *part,
                   DevScalars *sc, hipStream_t s, bool check, bool first, int64_t n_own);

// pair and list of bp_op_s from the sorted slots: those of node v are
// pos[off[v]], ..., pos[off[v + 1] - 1], the records of nodes 256 b, ... start at
// list[rec[b]]
void slot_records(int64_t n, const int32_t *off, const int32_t *rec, const int32_t *pos,
                  int2 *pair, int4 *list, hipStream_t s);
// transposed gather Q^T w_L: w[c][g] = sum of wl[c][.] over the slots of node
// v = iperm[g] or g (pair and list as in bp_op_s), ascending (wl is [nc][nl]);
// skipped while *done (done may be NULL)
template <typename T>
void gather_local(int nc, int64_t n, int64_t nl, const int2 *pair, const int4 *list,
                  const int32_t *iperm, const T *wl, T *w, const int *done, hipStream_t s);
// cg_update_r with w = Q^T w_L gathered per node (no w vector is read,
// written or cleared)
template <typename T>
void cg_update_r_gather(int nc, int64_t n, int64_t nl, T *r, const T *wl, const int2 *pair,
                        const int4 *list, const T *dinv, double *part, DevScalars *sc,
                        hipStream_t s, bool check = true);

// single-reduction PCG: init (r, u = dinv r, p = s = w = 0; partials r.u, r.r,
// b.b), the fused vector update (partials r.u, r.r), and the finisher that
// combines them with the operator's (u, A u) partials (alpha, beta, flags)
void sr_init(int nc, int64_t n, const double *b, const double *x0, double *x,
             const int32_t *perm, double *w, double *u, double *p, double *sv,
             const double *dinv, double *part, DevScalars *sc, hipStream_t s);
template <typename T>
void sr_update(int nc, int64_t n, T *x, T *u, T *w, T *p, T *sv, const T *dinv, double *part,
               DevScalars *sc, hipStream_t s, bool check = true, int64_t n_own = 0);

// vectors [nc][n] between the caller's node order and the internal one,
// both as gathers: in, dst[c][v] = src[c][perm[v]] (perm[v] = the caller's
// id of internal node v); out, dst[c][g] = src[c][iperm[g]] (iperm[g] = the
// internal id of the caller's node g; NULL: g itself); nothing is done if *skip
template <typename T>
void permute_in(int nc, int64_t n, const int32_t *perm, const T *src, T *dst, hipStream_t s,
                const int *skip = nullptr);
template <typename T>
void permute_out(int nc, int64_t n, const int32_t *iperm, const T *src, T *dst, hipStream_t s);
// a gather map in the other node order: out[k] = map[in[k]], Dirichlet signs kept
void map_ids(const int32_t *in, const int32_t *map, int32_t *out, int64_t count, hipStream_t s);
void sr_fin(bool first, int nc, double *pv, int64_t nbv, double *pa, int64_t nba,
            DevScalars *sc, hipStream_t s);

// residual replacement after an iteration that stopped before its direction
// update: r holds the new residual and becomes z = dinv r (the form the
// iteration keeps); r.z and r.r of it, then the pending p = z + beta p with
// beta = (r.z)_new / (r.z)_old (the search direction is kept); r.r becomes
// the reference norm; clears done/halted
template <typename T>
void cg_restart(int nc, int64_t n, T *r, T *p, const T *dinv, double *part,
                DevScalars *sc, hipStream_t s);

// sc->pap[c] = sum over the rows of column c of the operator's energy table
// part[rows][nc] (fixed order); part + rows nc holds the stage-1 rows
void operator_energies(int nc, double *part, int64_t rows, DevScalars *sc, hipStream_t s);
// collocated mass: w = M u with the assembled diagonal md (caller's order), its
// entries (0 on masked nodes), and the misfit's gradient and energy rows [vec_blocks(n)][nc]; assemble_mass sums
// that diagonal from Bt over the map's count slots (the same bits whatever the
// order of arrival; hi and lo: n words of scratch each) and makes it negative on
// the map's Dirichlet nodes
template <typename T>
void mass_diagonal(int nc, int64_t n, const double *md, const T *u, T *w, bool masked,
                   hipStream_t s);
void mass_entries(int64_t n, const double *md, double *d, bool masked, hipStream_t s);
void misfit_diagonal(int nc, int64_t n, const double *md, const double *u, const double *ut,
                     double *grad, double *part, hipStream_t s);
void assemble_mass(const int32_t *idx, const double *Bt, int64_t count, int64_t n, double *md,
                   double *hi, double *lo, hipStream_t s);
// d = a - b over count entries (d may be a)
void difference(const double *a, const double *b, double *d, int64_t count, hipStream_t s);

// defect correction helpers (FP64 outer loop)
void dc_residual(int nc, int64_t n, const double *b, double *r, double *w, const double *dinv,
                 double *part, DevScalars *sc, hipStream_t s);
void dc_accumulate(int64_t n, double *x, const float *d, hipStream_t s);

}  // namespace bp
