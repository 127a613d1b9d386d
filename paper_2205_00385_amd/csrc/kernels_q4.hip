// Plane-stress path (the paper's 2D examples, Sections 4.1, 4.2.1, 4.3): the
// bilinear quadrilateral (Q4) operator, its element energies and Jacobi
// diagonal, and the 2D Galerkin hierarchy (Algorithm 2) with 8x8 coarse
// element matrices.  Grids are nx x ny unit squares, nodes x-fastest
// (i + (nx+1) j), local corner a = dx + 2 dy, DOF vectors SoA [2][n_node].
#include <algorithm>

#include "internal.hpp"

namespace aarmr {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

__host__ __device__ constexpr int s2(int r, int c) { return sym_index2(r, c); }

// Weight of parent corner A (0/1) at refined position pos (0, 1, 2) along an axis.
__host__ __device__ constexpr double phi1q(int pos, int A) {
  return pos == 1 ? 0.5 : ((pos >> 1) == A ? 1.0 : 0.0);
}

// Product of the fine operator (FINE: moduli E, masks, springs) or of a coarse
// level's packed element matrices Ke.  MODE 0: y = A v; 1: a damped-Jacobi
// sweep, y = v + omega dinv (b - A v), y distinct from v; 2: the residual
// y = b - A v.  any_input: any v, A v = v on fixed DOFs; otherwise v is zero
// there, and so is A v.
// With part non-null each workgroup also writes part[blockIdx.x], its sum of
// v . y (MODE 0) or b . y (MODE 1): the partials of CG's dot products.
//
// These launches are bound by their chain of loads, not by bytes: wavefront a
// of a workgroup takes the elements of which its 64 nodes are corner a, so a
// thread has one element's loads, all in flight, and row pairs of the fine KE
// are wave-uniform; the four sums meet in LDS, where wavefront c finishes
// component c with operands it loaded at the start.  At 320x160 a thread per
// node took 6.5 us for the fine product, 5.4 us for a coarse one and 2.8 us
// each for the sweep and the dot products; 4.0 to 4.8 us (fine) and 3.7 us
// (coarse) for all of it now.
//
// With part a workgroup takes several groups of 64 nodes above kQ4Blocks, since
// every workgroup of the CG updates reads all the partials (16384 of them: the
// 1024x1024 solve 5.7 -> 6.4 ms).  Without it there is one group a workgroup: at
// four workgroups a CU the loads were not hidden (1024x1024 25.6 -> 21.2 us,
// 2048x2048 91.0 -> 73.3 us, 4096x4096 450 -> 391 us; two groups a workgroup 21.8,
// 74.6 and 391 us).  A thread per node took 27.1, 83.5 and 372 us.
constexpr int kQ4Nodes = 64, kQ4Blocks = 1024;
template <bool FINE, int MODE>
__global__ void __launch_bounds__(4 * kQ4Nodes) k_q4_product(
    int nx, int ny, const double* __restrict__ Kmat, const double* __restrict__ E,
    const uint8_t* __restrict__ mask, bool any_input, const double* __restrict__ v,
    double* __restrict__ y, const double* __restrict__ b, const double* __restrict__ dinv,
    double omega, double* __restrict__ part, SpringSet S) {
  __shared__ double sums[4][2][kQ4Nodes], dots[2];
  const uint32_t nxp = nx + 1, nn = nxp * (ny + 1), ne = (uint32_t)nx * ny;
  const int lane = threadIdx.x & 63, a = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double dacc = 0.0;
  for (uint32_t base = blockIdx.x * kQ4Nodes; base < nn; base += gridDim.x * kQ4Nodes) {
    const uint32_t n = base + lane, nc = n < nn ? n : nn - 1;
    const int j = (int)(nc / nxp), i = (int)(nc - (uint32_t)j * nxp);
    const int ex = i - (a & 1), ey = j - (a >> 1);
    const bool eok = ex >= 0 && ex < nx && ey >= 0 && ey < ny;
    const uint32_t cx = min(max(ex, 0), nx - 1), cy = min(max(ey, 0), ny - 1);
    const uint32_t e = cx + (uint32_t)nx * cy;
    // what finishes component a of node nc
    double vn = 0.0, bn = 0.0, dn = 0.0;
    uint32_t mn = 0;
    if (a < 2) {
      const int64_t d = (int64_t)a * nn + nc;
      vn = v[d];
      if (MODE) bn = b[d];
      if (MODE == 1) dn = dinv[d];
      if (FINE) mn = mask[nc];
    }
    double ve[8], k0[8], k1[8];
    uint32_t me[4] = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t nb = cx + (c & 1) + nxp * (cy + (c >> 1));
      ve[2 * c] = v[nb];
      ve[2 * c + 1] = v[(int64_t)nn + nb];
      if (FINE && any_input) me[c] = mask[nb];
    }
    const double w = FINE ? E[e] : 1.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (FINE) {
        k0[q] = Kmat[16 * a + q];
        k1[q] = Kmat[16 * a + 8 + q];
      } else {
        k0[q] = Kmat[(int64_t)s2(2 * a, q) * ne + e];
        k1[q] = Kmat[(int64_t)s2(2 * a + 1, q) * ne + e];
      }
    }
    double t0 = 0.0, t1 = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double x = ((me[q >> 1] >> (q & 1)) & 1u) ? 0.0 : ve[q];
      t0 = fma(k0[q], x, t0);
      t1 = fma(k1[q], x, t1);
    }
    sums[a][0][lane] = eok ? w * t0 : 0.0;
    sums[a][1][lane] = eok ? w * t1 : 0.0;
    __syncthreads();
    if (a < 2 && n < nn) {
      const int64_t d = (int64_t)a * nn + n;
      double Av = (sums[0][a][lane] + sums[1][a][lane]) + (sums[2][a][lane] + sums[3][a][lane]);
      if (FINE) {
        for (int t = 0; t < S.n; ++t)
          if (S.dof[t] == d) Av = fma(S.k[t], vn, Av);
        if ((mn >> a) & 1u) Av = any_input ? vn : 0.0;
      }
      const double out = MODE == 0 ? Av : MODE == 1 ? fma(omega * dn, bn - Av, vn) : bn - Av;
      y[d] = out;
      dacc = fma(MODE ? bn : vn, out, dacc);
    }
    __syncthreads();  // the sums are read before the next nodes' are written
  }
  if (part) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dacc += __shfl_down(dacc, off, 64);
    if (a < 2 && lane == 0) dots[a] = dacc;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = dots[0] + dots[1];
  }
}

// energy_e = u_e^T KE w_e (unit modulus; w = u: the strain energy), fixed
// DOFs read as zero.
__global__ void k_q4_energy(int nx, int ny, const double* __restrict__ KE,
                            const uint8_t* __restrict__ mask, const double* __restrict__ u,
                            const double* __restrict__ w, double* __restrict__ energy) {
  const int64_t nn = (int64_t)(nx + 1) * (ny + 1);
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)nx * ny) return;
  const int ex = (int)(e % nx), ey = (int)(e / nx);
  double ue[8], we[8];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int64_t nb = (int64_t)(ex + (b & 1)) + (int64_t)(nx + 1) * (ey + (b >> 1));
    const uint8_t mb = mask[nb];
    ue[2 * b] = (mb & 1) ? 0.0 : u[nb];
    ue[2 * b + 1] = (mb & 2) ? 0.0 : u[nn + nb];
    we[2 * b] = (mb & 1) ? 0.0 : w[nb];
    we[2 * b + 1] = (mb & 2) ? 0.0 : w[nn + nb];
  }
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) t = fma(KE[r * 8 + q], we[q], t);
    s = fma(ue[r], t, s);
  }
  energy[e] = s;
}

// Inverse Jacobi diagonal of the fine operator (identity on fixed DOFs).
__global__ void k_q4_diag(int nx, int ny, const double* __restrict__ KE,
                          const double* __restrict__ E, const uint8_t* __restrict__ mask,
                          double* __restrict__ dinv) {
  const int64_t nn = (int64_t)(nx + 1) * (ny + 1);
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= nn) return;
  const int i = (int)(n % (nx + 1)), j = (int)(n / (nx + 1));
  double d[2] = {0.0, 0.0};
  for (int a = 0; a < 4; ++a) {
    const int ex = i - (a & 1), ey = j - (a >> 1);
    if (ex < 0 || ex >= nx || ey < 0 || ey >= ny) continue;
    const double w = E[(int64_t)ex + (int64_t)nx * ey];
    for (int c = 0; c < 2; ++c) d[c] += w * KE[(2 * a + c) * 9];
  }
  const uint8_t m = mask[n];
  for (int c = 0; c < 2; ++c) dinv[c * nn + n] = (((m >> c) & 1) || d[c] == 0.0) ? 1.0 : 1.0 / d[c];
}

// acc += P_c^T K P_c for child c of a parent (upper triangles, packed), P_c
// the child's bilinear interpolation from the parent's corners.
template <int C>
__device__ __forceinline__ void galerkin_child(const double (&K)[kSymEntries2],
                                               double (&acc)[kSymEntries2]) {
  constexpr int dx = C & 1, dy = C >> 1;
#pragma unroll
  for (int I = 0; I < 8; ++I)
#pragma unroll
    for (int J = I; J < 8; ++J)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const double pa = phi1q(dx + (a & 1), (I >> 1) & 1) * phi1q(dy + (a >> 1), I >> 2);
        if (pa == 0.0) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const double pb = phi1q(dx + (b & 1), (J >> 1) & 1) * phi1q(dy + (b >> 1), J >> 2);
          if (pb != 0.0)
            acc[s2(I, J)] = fma(pa * pb, K[s2(2 * a + (I & 1), 2 * b + (J & 1))], acc[s2(I, J)]);
        }
      }
}

// Galerkin matrix of every parent of the coarse grid (cnx x cny), one thread
// per parent: Kc = sum over the four children c of P_c^T K_c P_c.  FROM_FINE:
// K_c = E_c KE with the rows and columns of fixed fine DOFs removed (masked
// P); otherwise K_c is the previous level's packed matrix.  A child's 36
// entries are loaded at once and its share of all 36 sums formed in
// registers; small workgroups spread a level over the device (parents of
// 320x160, 160x80 and 80x40 children: 70, 122 and 122 us with a loop over
// entries that loaded operand by operand, 13.4, 6.2 and 6.2 us now).
template <bool FROM_FINE, int C>
__device__ __forceinline__ void galerkin_add(int cx, int cy, int cnx, int64_t fne,
                                             const double* __restrict__ KE,
                                             const double* __restrict__ E,
                                             const uint8_t* __restrict__ mask,
                                             const double* __restrict__ Kf,
                                             double (&acc)[kSymEntries2]) {
  const int fx = 2 * cx + (C & 1), fy = 2 * cy + (C >> 1);
  const int64_t fe = fx + (int64_t)(2 * cnx) * fy;
  double K[kSymEntries2];
  if (FROM_FINE) {
    const double w = E[fe];
    uint32_t fixed = 0;  // bit 2 a + c: DOF c of corner a
#pragma unroll
    for (int a = 0; a < 4; ++a)
      fixed |= (mask[fx + (a & 1) + (int64_t)(2 * cnx + 1) * (fy + (a >> 1))] & 3u) << (2 * a);
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int q = r; q < 8; ++q)
        K[s2(r, q)] = (((fixed >> r) | (fixed >> q)) & 1u) ? 0.0 : w * KE[r * 8 + q];
  } else {
#pragma unroll
    for (int t = 0; t < kSymEntries2; ++t) K[t] = Kf[(int64_t)t * fne + fe];
  }
  galerkin_child<C>(K, acc);
}
template <bool FROM_FINE>
__global__ void __launch_bounds__(64) k_q4_galerkin(int cnx, int cny, const double* __restrict__ KE,
                                                    const double* __restrict__ E,
                                                    const uint8_t* __restrict__ mask,
                                                    const double* __restrict__ Kf,
                                                    double* __restrict__ Kc) {
  const int64_t cne = (int64_t)cnx * cny;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= cne) return;
  const int cy = (int)(e / cnx), cx = (int)(e - (int64_t)cy * cnx);
  double acc[kSymEntries2];
#pragma unroll
  for (int t = 0; t < kSymEntries2; ++t) acc[t] = 0.0;
  galerkin_add<FROM_FINE, 0>(cx, cy, cnx, 4 * cne, KE, E, mask, Kf, acc);
  galerkin_add<FROM_FINE, 1>(cx, cy, cnx, 4 * cne, KE, E, mask, Kf, acc);
  galerkin_add<FROM_FINE, 2>(cx, cy, cnx, 4 * cne, KE, E, mask, Kf, acc);
  galerkin_add<FROM_FINE, 3>(cx, cy, cnx, 4 * cne, KE, E, mask, Kf, acc);
#pragma unroll
  for (int t = 0; t < kSymEntries2; ++t) Kc[(int64_t)t * cne + e] = acc[t];
}

__global__ void k_q4_diag_elemmat(int nx, int ny, const double* __restrict__ Ke,
                                  double* __restrict__ dinv) {
  const int64_t nn = (int64_t)(nx + 1) * (ny + 1);
  const int64_t ne = (int64_t)nx * ny;
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= nn) return;
  const int i = (int)(n % (nx + 1)), j = (int)(n / (nx + 1));
  double d[2] = {0.0, 0.0};
  for (int a = 0; a < 4; ++a) {
    const int ex = i - (a & 1), ey = j - (a >> 1);
    if (ex < 0 || ex >= nx || ey < 0 || ey >= ny) continue;
    const int64_t e = (int64_t)ex + (int64_t)nx * ey;
    for (int c = 0; c < 2; ++c) d[c] += Ke[(int64_t)s2(2 * a + c, 2 * a + c) * ne + e];
  }
  for (int c = 0; c < 2; ++c) dinv[c * nn + n] = d[c] == 0.0 ? 1.0 : 1.0 / d[c];
}

// Grounded springs (one thread each; the host merges repeated DOFs, so no
// two threads touch one DOF).
// The inverse Jacobi diagonal with the spring stiffness added.
__global__ void k_springs_diag(SpringSet S, int64_t nn, const uint8_t* __restrict__ mask,
                               double* __restrict__ dinv) {
  const int t = threadIdx.x;
  if (t >= S.n) return;
  const int64_t d = S.dof[t];
  const int64_t node = d % nn;
  if ((mask[node] >> (int)(d / nn)) & 1) return;
  dinv[d] = 1.0 / (1.0 / dinv[d] + S.k[t]);
}

// (Df P)^T S (Df P) for the springs S of the fine grid, added to the level-1
// matrices: the fine DOF of a spring interpolates from the corners of one
// parent (any parent containing it), so k w w^T lands in that parent's
// matrix.  One thread walks the springs in order (two may share a parent).
__global__ void k_springs_galerkin(SpringSet S, int cnx, int cny, const uint8_t* __restrict__ mask,
                                   double* __restrict__ Kc) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int fnx = 2 * cnx;
  const int64_t fnn = (int64_t)(fnx + 1) * (2 * cny + 1);
  const int64_t cne = (int64_t)cnx * cny;
  for (int t = 0; t < S.n; ++t) {
    const int64_t d = S.dof[t];
    const int64_t node = d % fnn;
    const int c = (int)(d / fnn);
    if ((mask[node] >> c) & 1) continue;
    const int fi = (int)(node % (fnx + 1)), fj = (int)(node / (fnx + 1));
    const int px = min(fi >> 1, cnx - 1), py = min(fj >> 1, cny - 1);
    const int lx = fi - 2 * px, ly = fj - 2 * py;
    const int64_t e = (int64_t)px + (int64_t)cnx * py;
    for (int A = 0; A < 4; ++A) {
      const double wa = phi1q(lx, A & 1) * phi1q(ly, A >> 1);
      if (wa == 0.0) continue;
      for (int B = A; B < 4; ++B) {
        const double wb = phi1q(lx, B & 1) * phi1q(ly, B >> 1);
        if (wb == 0.0) continue;
        double& k = Kc[(int64_t)s2(2 * A + c, 2 * B + c) * cne + e];
        k = fma(S.k[t] * wa, wb, k);
      }
    }
  }
}

// Dense coarsest operator with the unknowns in the order o; one wavefront per
// row, zeroed first (coalesced), then lanes take the 18 columns of the 9-node
// neighbourhood: an entry sums, over the elements around the row's node in
// corner order a = 0..3, the entries coupling the two nodes.
__global__ void __launch_bounds__(256) k_q4_assemble_dense(int nx, int ny, CoarseOrder o,
                                                           const double* __restrict__ Ke,
                                                           double* __restrict__ A) {
  const int nxp = nx + 1, nn = nxp * (ny + 1), ne = nx * ny, nd = 2 * nn;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool active = item < nd;  // wave-uniform; every wave reaches the barrier
  const int c = item / nn, n = item % nn;
  const int i = n % nxp, j = n / nxp;
  const int row = c * o.sc + i * o.si + j * o.sj;
  double* Ar = A + (int64_t)(active ? row : 0) * nd;
  if (active)
    for (int t = lane; t < nd; t += 64) Ar[t] = 0.0;
  __syncthreads();  // the zeros are stored before the same addresses are rewritten
  if (!active || lane >= 18) return;
  const int d = lane / 9, nb = lane % 9;
  const int bi = i + nb % 3 - 1, bj = j + nb / 3 - 1;
  if (bi < 0 || bi > nx || bj < 0 || bj > ny) return;
  double acc = 0.0;
  for (int a = 0; a < 4; ++a) {
    const int ex = i - (a & 1), ey = j - (a >> 1);
    if (ex < 0 || ex >= nx || ey < 0 || ey >= ny) continue;
    const int dx = bi - ex, dy = bj - ey;
    if (dx < 0 || dx > 1 || dy < 0 || dy > 1) continue;
    acc += Ke[(int64_t)s2(2 * a + c, 2 * (dx + 2 * dy) + d) * ne + ex + nx * ey];
  }
  const int col = d * o.sc + bi * o.si + bj * o.sj;
  Ar[col] = (col == row && acc == 0.0) ? 1.0 : acc;  // dead coarse DOF: identity row
}

}  // namespace

int q4_partials_max(const Grid& g) {
  return (int)std::min<int64_t>((g.nn + kQ4Nodes - 1) / kQ4Nodes, kQ4Blocks);
}

// Workgroups of a product without partials (a launch holds below 2^32 threads).
static int q4_blocks(const Grid& g) {
  return (int)std::min<int64_t>((g.nn + kQ4Nodes - 1) / kQ4Nodes, 1 << 22);
}

int launch_q4_fine(const Grid& g, const double* KE, const double* E, const uint8_t* mask,
                   const SpringSet& S, int mode, bool any_input, const double* v, double* y,
                   const double* b, const double* dinv, double omega, double* part,
                   hipStream_t s) {
  const int nb = part ? q4_partials_max(g) : q4_blocks(g);
  auto k = mode == 1   ? k_q4_product<true, 1>
           : mode == 2 ? k_q4_product<true, 2>
                       : k_q4_product<true, 0>;
  k<<<nb, 4 * kQ4Nodes, 0, s>>>(g.nx, g.ny, KE, E, mask, any_input, v, y, b, dinv, omega, part, S);
  return nb;
}

void launch_q4_coarse(const Grid& g, const double* Ke, int mode, const double* v, double* y,
                      const double* b, const double* dinv, double omega, hipStream_t s) {
  auto k = mode == 1   ? k_q4_product<false, 1>
           : mode == 2 ? k_q4_product<false, 2>
                       : k_q4_product<false, 0>;
  k<<<q4_blocks(g), 4 * kQ4Nodes, 0, s>>>(g.nx, g.ny, Ke, nullptr, nullptr, false, v, y, b, dinv, omega,
                                          nullptr, SpringSet{});
}

void launch_q4_energy(const Grid& g, const double* KE, const uint8_t* mask, const double* u,
                      const double* w, double* energy, hipStream_t s) {
  k_q4_energy<<<nblk(g.ne, 256), 256, 0, s>>>(g.nx, g.ny, KE, mask, u, w, energy);
}

void launch_springs_diag(const SpringSet& S, const Grid& g, const uint8_t* mask, double* dinv,
                         hipStream_t s) {
  if (S.n > 0) k_springs_diag<<<1, 64, 0, s>>>(S, g.nn, mask, dinv);
}

void launch_springs_galerkin(const SpringSet& S, const Grid& coarse, const uint8_t* mask,
                             double* Kc, hipStream_t s) {
  if (S.n > 0) k_springs_galerkin<<<1, 64, 0, s>>>(S, coarse.nx, coarse.ny, mask, Kc);
}

void launch_q4_diag(const Grid& g, const double* KE, const double* E, const uint8_t* mask,
                    double* dinv, hipStream_t s) {
  k_q4_diag<<<nblk(g.nn, 256), 256, 0, s>>>(g.nx, g.ny, KE, E, mask, dinv);
}

void launch_q4_galerkin_from_fine(const Grid& coarse, const double* KE, const double* E,
                                  const uint8_t* mask, double* Kc, hipStream_t s) {
  k_q4_galerkin<true><<<nblk(coarse.ne, 64), 64, 0, s>>>(coarse.nx, coarse.ny, KE, E, mask,
                                                           nullptr, Kc);
}

void launch_q4_galerkin_from_coarse(const Grid& coarse, const double* Kf, double* Kc,
                                    hipStream_t s) {
  k_q4_galerkin<false><<<nblk(coarse.ne, 64), 64, 0, s>>>(coarse.nx, coarse.ny, nullptr,
                                                            nullptr, nullptr, Kf, Kc);
}

void launch_q4_diag_elemmat(const Grid& g, const double* Ke, double* dinv, hipStream_t s) {
  k_q4_diag_elemmat<<<nblk(g.nn, 256), 256, 0, s>>>(g.nx, g.ny, Ke, dinv);
}

void launch_q4_assemble_dense(const Grid& g, const CoarseOrder& o, const double* Ke, double* A,
                              hipStream_t s) {
  k_q4_assemble_dense<<<(unsigned)((2 * g.nn + 3) / 4), 256, 0, s>>>(g.nx, g.ny, o, Ke, A);
}

}  // namespace aarmr
