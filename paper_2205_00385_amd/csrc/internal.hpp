// Internal declarations of the AARMR HIP library (gfx950).
//
// Layout: DOF vectors are SoA [3][n_node] in FP64 (or FP32 inside the
// refinement form); elements and nodes are x-fastest.  The fixed-DOF mask is
// one byte per node with bit c set when component c is fixed.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "aarmr.h"
#include "inv_plan.hpp"
#include "walsh.hpp"

namespace aarmr {

constexpr int kRedBlocks = 512;    // partial-sum blocks of one reduction
constexpr int kFusedBlocks = 2048; // block limit of the CG updates with folded reductions
constexpr int kRedSlots = 24;      // dot products one reduction launch can hold
constexpr int kMaxIt = 4096;       // bound of cg_maxit (scalar history length)

// nz == 0 is the plane-stress grid: nx * ny unit squares, (nx+1)(ny+1)
// nodes with 2 DOFs each.
struct Grid {
  int nx, ny, nz;          // elements
  int64_t ne, nn;          // elements, nodes
};

inline Grid make_grid(int nx, int ny, int nz) {
  Grid g;
  g.nx = nx; g.ny = ny; g.nz = nz;
  g.ne = (int64_t)nx * ny * (nz > 0 ? nz : 1);
  g.nn = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
  return g;
}

// Reduction scratch: per-slot block partials.
struct RedScratch {
  double* partial;     // [kRedSlots][kRedBlocks]
};

// A small SPD system A x = b (n x n, row stride lda, entries averaged with
// their transpose) that is solved when its entries are finished (n = 0: none);
// not positive definite: bit 4 of *bad and x = 0.
struct SmallSolve {
  int n, lda;
  const double *A, *b;
  double* x;
  unsigned* bad;
};

// k dot products a_i . b_i (b_i == nullptr: plain sum of a_i) of vectors of
// element type T, accumulated and returned in FP64.
// Load cases solved in lock step by one set of launches: case l's vectors
// start at l * vs, its CG scalars at l * ss, its workgroup partials at l * ps
// and its host-visible partials at l * hs; active (device, n entries): 0 for
// a case that has finished, whose updates are then skipped.  n = 1 with zero
// strides is the single-case solve.
struct MultiRhs {
  int n = 1;
  int64_t vs = 0;
  int ss = 0, ps = 0, hs = 0;
  const int* active = nullptr;
};

template <typename T>
struct DotSetT {
  const T* a[kRedSlots];
  const T* b[kRedSlots];
  double* out[kRedSlots];
  int k;               // number of products
  int64_t n;           // length
};
using DotSet = DotSetT<double>;

// ---- fine-level operator (element-by-element, reflection-blocked) --------
// y = A v = Df K Df v + (I - Df) v for any v (any_input), or y = Df K v for a v
// that is zero on fixed DOFs (then equal to both A v and Df K Df v), the form
// every solver-internal product uses.
// tz: launch shape word, 0 the grid's default shape (kernels_ebe.hip).
void launch_ebe(const Grid& g, const WalshConsts& K, const double* E, const uint8_t* mask,
                const double* v, double* y, bool any_input, hipStream_t s, int tz = 0);
void launch_ebe_f32(const Grid& g, const WalshConsts& K, const float* E, const uint8_t* mask,
                    const float* v, float* y, hipStream_t s, int tz = 0, int nr = 1);
// The solver's product feeding a damped-Jacobi sweep: out = v + omega dinv
// (b - A v), out distinct from v.
void launch_ebe_jacobi(const Grid& g, const WalshConsts& K, const double* E, const uint8_t* mask,
                       const double* v, const double* b, const double* dinv, double omega,
                       double* out, hipStream_t s, int tz = 0);
// The same two products with CG's dot product folded in: each workgroup w
// writes part[w], the sum over the nodes it owns of v . y (launch_ebe_dot,
// p^T A p) or b . out (launch_ebe_jacobi_dot: r^T z); the return
// value is the number of partials.  part holds ebe_partials_max(g) entries.
int ebe_partials_max(const Grid& g);
int launch_ebe_dot(const Grid& g, const WalshConsts& K, const double* E, const uint8_t* mask,
                   const double* v, double* y, double* part, hipStream_t s, int tz = 0);
int launch_ebe_jacobi_dot(const Grid& g, const WalshConsts& K, const double* E,
                          const uint8_t* mask, const double* v, const double* b,
                          const double* dinv, double omega, double* out, double* part,
                          hipStream_t s, int tz = 0);
// FP32 forms of the two (vectors FP32, partials summed in FP64).
int launch_ebe_f32_dot(const Grid& g, const WalshConsts& K, const float* E, const uint8_t* mask,
                       const float* v, float* y, double* part, hipStream_t s, int tz = 0,
                       int nr = 1, int pst = 0);
int launch_ebe_jacobi_f32_dot(const Grid& g, const WalshConsts& K, const float* E,
                              const uint8_t* mask, const float* v, const float* b,
                              const float* dinv, float omega, float* out, double* part,
                              hipStream_t s, int tz = 0, int nr = 1, int pst = 0);
void launch_energy_walsh(const Grid& g, const WalshConsts& K, const uint8_t* mask,
                         const double* u, double* energy, hipStream_t s);
void launch_simp(int64_t ne, const double* rho, double E0, double Emin, double p, double* E,
                 float* E32, unsigned* bad, hipStream_t s);
void launch_diff(int64_t n, const double* a, const double* b, double* out, hipStream_t s);
// ncomp: DOFs per node (3, or 2 on the plane-stress grid)
void launch_build_mask(int64_t nn, const int64_t* fixed, int64_t nfixed, uint8_t* mask,
                       unsigned* bad, hipStream_t s, int ncomp = 3);
void launch_mask_diff(int64_t nn, const uint8_t* a, const uint8_t* b, unsigned* flags,
                      hipStream_t s);
void launch_diag_fine(const Grid& g, const double* KE, const double* E, const uint8_t* mask,
                      double* dinv, float* dinv32, hipStream_t s);
void launch_dc_accum(int64_t ne, const double* rho, const double* energy, double E0, double Emin,
                     double p, double* dc, int first, hipStream_t s);

// ---- multigrid ------------------------------------------------------------
// Stored element matrices are symmetric 24x24, packed (upper triangle,
// row-major: 300 entries) and entry-major, K[sym_index(r,c) * n_elem + w], w an
// element's place in its level's list of stored elements (kernels_level.hip).
constexpr int kSymEntries = 300;
__host__ __device__ constexpr int sym_index(int r, int c) {
  return r <= c ? r * 24 - (r * (r - 1)) / 2 + (c - r) : c * 24 - (c * (c - 1)) / 2 + (r - c);
}
// The coarse levels' buffers (index 0 unused, null).
constexpr int kCountSplit = 2 * AARMR_MAX_LEVELS, kCounts = 3 * AARMR_MAX_LEVELS;
struct LevelTable {
  int nlev = 0;
  int nx[AARMR_MAX_LEVELS] = {}, ny[AARMR_MAX_LEVELS] = {}, nz[AARMR_MAX_LEVELS] = {};
  int ne[AARMR_MAX_LEVELS] = {}, nn[AARMR_MAX_LEVELS] = {};
  uint8_t* eflag[AARMR_MAX_LEVELS] = {};    // [ne] 1: contains a fixed fine DOF
  uint8_t* special[AARMR_MAX_LEVELS] = {};  // [nn] 1: node of a flagged element
  int* eidx[AARMR_MAX_LEVELS] = {};         // [ne] place in the list of stored elements, or -1
  int* elist[AARMR_MAX_LEVELS] = {};        // [ne] stored elements: those with a special node, or flagged
  int* nlist[AARMR_MAX_LEVELS] = {};        // [nn] special nodes
  int* corner[AARMR_MAX_LEVELS] = {};       // [8][nn] stored elements around the special nodes
  double* mom[AARMR_MAX_LEVELS] = {};       // levels >= 2: [27][ne] moments of the moduli
  double* Esplit = nullptr;                 // split level 1: the fine moduli, 0 in flagged elements
  double* Kst[AARMR_MAX_LEVELS] = {};       // [300][ne] stored matrices
  int* part = nullptr;                      // level_list_blocks() counts
  int* counts = nullptr;                    // [2 level]: stored elements, [2 level + 1]: special nodes,
                                            // [kCountSplit + level]: 1 if the level is split
};
// What one level's product reads; nspecial and split as read back by the host,
// or, with count (the number on the device), the most nodes there can be and, if
// the level may be split, gate (on the device: 1 if it is).
struct LevelArgs {
  int level, nx, ny, nz, nspecial;
  const int *count, *gate;
  bool split;
  double gam;  // 2^-level
  const double* mom;
  const double* Esplit;
  const uint8_t* special;
  const int* nlist;
  const int* corner;
  const double* Kst;
};
bool level_may_split(int nx, int ny, int nz);
int64_t level_list_blocks(const Grid* lg, int nlev);
// Flags, lists and special nodes of every level >= 1 from the fine mask.
void launch_level_lists(const LevelTable& T, const uint8_t* mask, hipStream_t s);
// What a product marches on: moments of a level >= 2, from the fine moduli (2) or
// from the level above; the moduli of a split level 1.  After the lists.
void launch_level_moments(const LevelTable& T, int level, const double* E, hipStream_t s);
void launch_level_moduli(const LevelTable& T, const double* E, hipStream_t s);
// Matrices of the listed elements; level l - 1 done before level l.
void launch_level_store(const LevelTable& T, int level, const WalshConsts& K, const double* E,
                        const uint8_t* mask, hipStream_t s);
void launch_level_diag(const LevelTable& T, int level, const WalshConsts& K, const double* E,
                       double* dinv, float* dinv32, hipStream_t s);
// mode 0: y = A v; 1: y = v + omega jd (jb - A v); 2: y = jb - A v.  y distinct
// from v.  E: the fine moduli (level 1).
void launch_level_product(const LevelArgs& L, const WalshConsts& K, const double* E, int mode,
                          const double* v, double* y, const double* jb, const double* jd,
                          double omega, hipStream_t s);
// FP32 products of the refinement form (kernels_l32.hip), modes as above; nr
// load cases one after another.  Level 1: Bw = W M_0 W / 64 (24 x 24, M_0 child
// 0's Galerkin matrix, Walsh x component basis, index 3k + s), Y a [24][ne]
// element-product buffer per load case, nlist the stored elements as read back
// by the host.  Levels >= 2: element matrices Ke, made by launch_elemmat_f32
// from the moments (C: [300][28], the matrix per unit moment) and the stored
// matrices.
void launch_elemmat_f32(const Grid& g, const double* C, const double* mom, const double* Kst,
                        const int* list, const int* count, float* K, hipStream_t s);
void launch_apply_elemmat_f32(const Grid& g, const float* Ke, int mode, const float* v, float* y,
                              const float* jb, const float* jd, float omega, int nr,
                              hipStream_t s);
void launch_apply_l1_f32(const Grid& g, const double* Kst, const float* Bw, const float* Ef,
                         const uint8_t* eflag, const int* list, int nlist, int mode,
                         const float* v, float* Y, float* y, const float* jb, const float* jd,
                         float omega, int nr, hipStream_t s);
void launch_restrict_jacobi_f32(const Grid& coarse, const float* bf, const float* tf,
                                const uint8_t* mask, float* bc, const float* dinv_c, float omega,
                                float* xc, hipStream_t s, int nr = 1);
// Transfers act per component; ncomp = 2 on the plane-stress grid (nz = 0).
// o: the coarse vector's order (null: [component][node]), set where the coarse
// level is the coarsest.
void launch_restrict(const Grid& coarse, const double* bf, const double* tf, const uint8_t* mask,
                     double* bc, hipStream_t s, int ncomp = 3, const CoarseOrder* o = nullptr);
void launch_prolong_add(const Grid& fine, const double* xc, const uint8_t* mask, double* xf,
                        hipStream_t s, int ncomp = 3, const CoarseOrder* o = nullptr);
void launch_jacobi_first(int64_t n3, const double* b, const double* dinv, double omega, double* x,
                         hipStream_t s);
// The restriction that also forms the coarse level's first damped-Jacobi sweep
// xc = omega dinv_c bc.
void launch_restrict_jacobi(const Grid& coarse, const double* bf, const double* tf,
                            const uint8_t* mask, double* bc, const double* dinv_c, double omega,
                            double* xc, hipStream_t s, int ncomp);
void launch_jacobi_update(int64_t n3, const double* b, const double* t, const double* dinv,
                          double omega, double* x, hipStream_t s);
// The dense coarsest operator with its unknowns in the order o, and its
// inverse in place (A SPD) by the plan's steps.  tasks: the plan's, in device
// memory; scratch: inv_scratch_doubles(plan) doubles.
void launch_assemble_dense(const Grid& g, const CoarseOrder& o, const double* Ke, double* A,
                           hipStream_t s);
int64_t inv_scratch_doubles(const InvPlan& plan);
void launch_invert(const InvPlan& plan, const InvTask* tasks, double* A, double* scratch,
                   hipStream_t s);
void launch_gemv(int n, const double* A, const double* x, double* y, hipStream_t s);
// FP32 V-cycle pieces (FP32 vectors; the coarsest inverse alone is read in FP64).
void launch_restrict_f32(const Grid& coarse, const float* bf, const float* tf,
                         const uint8_t* mask, float* bc, hipStream_t s, int nr = 1,
                         const CoarseOrder* o = nullptr);
void launch_prolong_add_f32(const Grid& fine, const float* xc, const uint8_t* mask, float* xf,
                            hipStream_t s, int nr = 1, const CoarseOrder* o = nullptr);
void launch_jacobi_first_f32(int64_t n3, const float* b, const float* dinv, float omega, float* x,
                             hipStream_t s, int nr = 1);
void launch_jacobi_update_f32(int64_t n3, const float* b, const float* t, const float* dinv,
                              float omega, float* x, hipStream_t s, int nr = 1);
void launch_gemv_f32(int n, const double* A, const float* x, float* y, hipStream_t s, int nr = 1);

// ---- vector kernels and reductions ----------------------------------------
void launch_multidot(const DotSet& d, const RedScratch& rs, hipStream_t s,
                     const SmallSolve& S = SmallSolve{});
// The partials alone, product k's in slot k; and the finish of slot 0.
void launch_multidot_partials(const DotSet& d, double* partial, hipStream_t s);
void launch_dot_finish(int64_t n, const double* partial, double* out, hipStream_t s);
void launch_multidot_f32(const DotSetT<float>& d, const RedScratch& rs, hipStream_t s);
// FP32 direction update after a separate r^T z; the scalars stay FP64 in
// device memory and the update is formed in FP64 before rounding to FP32.
void launch_cg_p_f32(int64_t n, const double* rz_new, const double* rz_old, const float* z,
                     float* p, hipStream_t s);
// Refinement transfers: dst32 = src64 / sqrt(*nrm2);  x64 += sqrt(*nrm2) d32.
void launch_to_f32_scaled(int64_t n, const double* src, const double* nrm2, float* dst,
                          hipStream_t s);
void launch_add_scaled_f32(int64_t n, const float* d, const double* nrm2, double* x,
                           hipStream_t s);
void launch_copy_f32(int64_t n, const float* src, float* dst, hipStream_t s);
void launch_copy_masked(const Grid& g, const double* src, const uint8_t* mask, double* dst,
                        hipStream_t s, int ncomp = 3);
void launch_sub(int64_t n, const double* a, const double* b, double* out, hipStream_t s);
// CG with folded reductions.  dot_blocks(n): the block count of one dot's
// partials; fused_blocks(n): that of the fused updates (each finishes the
// dot partials it needs); launch_dot_partials writes a^T b's partials to
// part[0..dot_blocks(n)).
int dot_blocks(int64_t n);
int fused_blocks(int64_t n);
void launch_dot_partials(int64_t n, const double* a, const double* b, double* part,
                         hipStream_t s);
// pq finished from the n_part entries of pq_part (n_part <= 0: dot_blocks(n)),
// stored to *pq and rr_part[fused_blocks(n)]; x += alpha p, r -= alpha q with
// alpha = *rz / pq; rr_part[0..fused_blocks(n)) = partials of r^T r;
// z0 = omega dinv r unless z0 is null.
void launch_cg_xr_fused(int64_t n, const double* rz, const double* pq_part, int n_part,
                        double* pq, double* x, double* r, const double* p, const double* q,
                        double* rr_part, const double* dinv, double omega, double* z0,
                        hipStream_t s);
// rz_new finished from the n_part entries of rz_part (n_part <= 0:
// dot_blocks(n)), stored to *rz_new; p = z + (rz_new / *rz_old) p.
void launch_cg_p_fused(int64_t n, const double* rz_part, int n_part, double* rz_new,
                       const double* rz_old, const double* z, double* p, hipStream_t s);
// The FP32 forms (FP32 vectors, FP64 scalars and partials); the x/r update
// also stores *rz at rr_part[fused_blocks(n) + 1] and always writes z0.
void launch_cg_xr_fused_f32(int64_t n, const double* rz, const double* pq_part, int n_part,
                            double* pq, float* x, float* r, const float* p, const float* q,
                            double* rr_part, const float* dinv, float omega, float* z0,
                            hipStream_t s,
                            const MultiRhs& mr = MultiRhs());
void launch_cg_p_fused_f32(int64_t n, const double* rz_part, int n_part, double* rz_new,
                           const double* rz_old, const float* z, float* p, hipStream_t s,
                            const MultiRhs& mr = MultiRhs());
void launch_scale_by_inv_sqrt(int64_t n, const double* src, const double* nrm2, double* dst,
                              hipStream_t s);
// out = sum_j coef[j] * V_j (+ add) with coefficients read from device memory
void launch_lincomb(int64_t n, int k, const double* const* V, const double* coef, double sign,
                    const double* add, double* out, hipStream_t s);
// launch_lincomb whose coefficients are coef or, with coef null, the sums of
// slots 0..k - 1 of `from`; partials of out . W_j (null: out . out) to slot j
// of `partial`, j < nw.  out may be add.
void launch_lincomb_dots(int64_t n, int k, const double* const* V, const double* coef,
                         const double* from, double sign, const double* add, double* out, int nw,
                         const double* const* W, double* partial, hipStream_t s);
// Gram-Schmidt keep test on a projected column (n0, n1: squared norms before
// and after the projections, n1 null: the sum of the partials part): dst = src
// / sqrt(n1) and *keep = 1 when sqrt(n1) > tau sqrt(n0), else dst = 0 and
// *keep = 0.
void launch_gs_keep(int64_t n, const double* src, const double* n0, const double* n1,
                    const double* part, double tau, double* dst, double* keep, hipStream_t s);
// Thin SVD of the small n x n matrix T (row-major): left singular vectors of
// sigma > tau sigma_1, decreasing, column by column into coef[j * n + i];
// their count (as a double) into *kept.
void launch_small_svd(int n, const double* T, double tau, double* coef, double* kept,
                      hipStream_t s);

// ---- plane stress (bilinear quadrilaterals, grids with nz = 0) -------------
// Coarse element matrices are symmetric 8x8, packed (upper triangle,
// row-major: 36 entries) and entry-major like the 3D ones.  KE: the 8x8
// unit-modulus element stiffness, row-major, DOF 2a + c of corner a = dx + 2dy.
constexpr int kSymEntries2 = 36;
__host__ __device__ constexpr int sym_index2(int r, int c) {
  return r <= c ? r * 8 - (r * (r - 1)) / 2 + (c - r) : c * 8 - (c * (c - 1)) / 2 + (r - c);
}
// energy_e = u_e^T KE w_e (w = u: strain energy)
void launch_q4_energy(const Grid& g, const double* KE, const uint8_t* mask, const double* u,
                      const double* w, double* energy, hipStream_t s);
// Grounded springs on single DOFs (passed by value to the kernels).
struct SpringSet {
  int n;
  int64_t dof[AARMR_MAX_SPRINGS];
  double k[AARMR_MAX_SPRINGS];
};
// Product of the fine operator.  mode 0: y = A v; 1: y = v + omega dinv (b -
// A v), y distinct from v; 2: y = b - A v.  any_input: any v, identity rows on
// fixed DOFs; otherwise v is zero there.  part (or null): partials of v . y
// (mode 0) or b . y (mode 1), at most q4_partials_max(g); the return value is
// the number of workgroups.
int q4_partials_max(const Grid& g);
int launch_q4_fine(const Grid& g, const double* KE, const double* E, const uint8_t* mask,
                   const SpringSet& S, int mode, bool any_input, const double* v, double* y,
                   const double* b, const double* dinv, double omega, double* part,
                   hipStream_t s);
// The same modes for a coarse level's element matrices.
void launch_q4_coarse(const Grid& g, const double* Ke, int mode, const double* v, double* y,
                      const double* b, const double* dinv, double omega, hipStream_t s);
void launch_springs_diag(const SpringSet& S, const Grid& g, const uint8_t* mask, double* dinv,
                         hipStream_t s);
// level-1 contribution (Df P)^T S (Df P); coarse = the level-1 grid
void launch_springs_galerkin(const SpringSet& S, const Grid& coarse, const uint8_t* mask,
                             double* Kc, hipStream_t s);
void launch_q4_diag(const Grid& g, const double* KE, const double* E, const uint8_t* mask,
                    double* dinv, hipStream_t s);
// Level 1: (Df P)^T K (Df P) per parent from the fine moduli and mask.
void launch_q4_galerkin_from_fine(const Grid& coarse, const double* KE, const double* E,
                                  const uint8_t* mask, double* Kc, hipStream_t s);
void launch_q4_galerkin_from_coarse(const Grid& coarse, const double* Kf, double* Kc,
                                    hipStream_t s);
void launch_q4_diag_elemmat(const Grid& g, const double* Ke, double* dinv, hipStream_t s);
void launch_q4_assemble_dense(const Grid& g, const CoarseOrder& o, const double* Ke, double* A,
                              hipStream_t s);

// ---- filter, OC --------------------------------------------------------------
// Cone weights max(0, r - |d|) of the filter offsets, (2R+1)^3 with
// R = ceil(r) - 1, offset (dk, dj, di) at ((dk + R)(2R+1) + dj + R)(2R+1) + di + R.
void filter_weights(double r, double* W);
int filter_taps(double r);
void launch_filter_rowsum(const Grid& g, double r, double* Hs, hipStream_t s);
void launch_filter(const Grid& g, double r, const double* W, int mode, const double* Hs,
                   const double* in, double* out, hipStream_t s);
void launch_fill(int64_t n, double v, double* out, hipStream_t s);
void launch_fill_f32(int64_t n, float v, float* out, hipStream_t s);
// OC bisection, kOcLevels steps per launch.  Launch `round` (0, 1, ...) walks
// the steps that launch round - 1's volumes decide and leaves the partials of
// the volumes sum_j cw_j x_new_j for the kOcTrials multipliers of the next
// steps; launch_oc_final, after launches 0..round - 1, walks the last ones and,
// if the bisection is done, forms x_new at the last multiplier evaluated
// (else x_new is left alone).  scratch: kOcScratchDoubles,
// two states (l1, l2, lmid, done, steps; launch r writes state r & 1) and two
// sets of partials; nothing in it need be cleared.
constexpr int kOcLevels = 5, kOcTrials = (1 << kOcLevels) - 1;
constexpr int kOcParts = 256, kOcThreads = 512;  // workgroups and their threads
constexpr int kOcState = 8;
constexpr int kOcMaxRounds = 200 / kOcLevels;  // the bisection takes 200 steps at most
constexpr int kOcScratchDoubles = 2 * kOcState + 2 * kOcTrials * kOcParts;
void launch_oc_round(int64_t ne, const double* x, const double* dc, const double* dv,
                     const double* cw, double move, double eta, double target, int round,
                     double* scratch, hipStream_t s);
void launch_oc_final(int64_t ne, const double* x, const double* dc, const double* dv, double move,
                     double eta, double target, int round, double* scratch, double* xnew,
                     hipStream_t s);

}  // namespace aarmr
