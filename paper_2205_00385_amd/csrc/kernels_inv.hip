// The coarsest solve of the V-cycle (Algorithm 2): the dense operator of the
// coarsest level and its explicit inverse.
//
// Inverse by the symmetric sweep operator.  Sweeping a pivot block K maps
//   A_KK -> -P (P = A_KK^-1),  A_IK -> A_IK P,  A_IJ -> A_IJ - A_IK P A_KJ
// for every other I, J, swept or not, and keeps A symmetric; when every block
// is swept, A holds -A^-1.  Only tiles on or above the diagonal are kept: with
// c_i = A_iK and T_i = c_i P,
//   A_IJ -= T_I c_J^T,  A_IK = T_I,  A_KK = -P.
// The unknowns are ordered plane by plane and dissected (inv_plan.hpp), so a
// step sweeps the blocks of several independent planes side by side and
// touches only the rows coupled with them.
//
// A step is a chain: its first tile (about 10 us: the launch, two dependent
// loads, two 64^3 products), then that tile's 64x64 inverse for the next step
// (another 10), so the number of steps sets the time.  Dissected, the 1911
// unknowns of a 12x6x6 coarsest grid take 12 steps instead of the 30 of a
// plain block elimination, and a sixth of its arithmetic: 0.29 ms against
// 0.93 ms per inversion; 1722 unknowns of a 40x20 plane grid 0.13 against
// 0.84 ms (6 steps, 27); 4131 of a 16x8x8 grid 1.0 against 3.9 ms (20, 65).
#include "internal.hpp"

namespace aarmr {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Dense coarsest operator with the unknowns in the plan's order.  One
// wavefront per row: the row is zeroed (coalesced stores), then lanes take the
// 81 columns of the 27-node neighbourhood (3 components each); an entry is the
// sum, over the elements around the row's node in corner order a = 0..7, of
// the element matrices' entries coupling the two nodes.  A row with zero
// diagonal (a coarse DOF no free fine DOF interpolates from) becomes an
// identity row.  32-bit indices: the coarsest order is at most 8192.
__global__ void __launch_bounds__(256) k_assemble_dense(int nx, int ny, int nz, CoarseOrder o,
                                                        const double* __restrict__ Ke,
                                                        double* __restrict__ A) {
  const int nxp = nx + 1, nyp = ny + 1;
  const int nn = nxp * nyp * (nz + 1), ne = nx * ny * nz, nd = 3 * nn;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool active = item < nd;  // wave-uniform; every wave reaches the barrier
  const int c = item / nn, n = item % nn;
  const int i = n % nxp, j = (n / nxp) % nyp, k = n / (nxp * nyp);
  const int row = c * o.sc + i * o.si + j * o.sj + k * o.sk;
  double* Ar = A + (int64_t)(active ? row : 0) * nd;
  if (active)
    for (int t = lane; t < nd; t += 64) Ar[t] = 0.0;
  __syncthreads();  // the zeros are stored before the same addresses are rewritten
  if (!active) return;
  for (int l = lane; l < 81; l += 64) {
    const int cc = l / 27, d = l % 27;
    const int bi = i + d % 3 - 1, bj = j + (d / 3) % 3 - 1, bk = k + d / 9 - 1;
    if (bi < 0 || bi > nx || bj < 0 || bj > ny || bk < 0 || bk > nz) continue;
    double acc = 0.0;
    for (int a = 0; a < 8; ++a) {
      const int ex = i - (a & 1), ey = j - ((a >> 1) & 1), ez = k - (a >> 2);
      if (ex < 0 || ex >= nx || ey < 0 || ey >= ny || ez < 0 || ez >= nz) continue;
      const int dx = bi - ex, dy = bj - ey, dz = bk - ez;  // corner of the column node
      if (dx < 0 || dx > 1 || dy < 0 || dy > 1 || dz < 0 || dz > 1) continue;
      const int b = dx + 2 * dy + 4 * dz;
      const int e = ex + nx * (ey + ny * ez);
      acc += Ke[(int64_t)sym_index(3 * a + c, 3 * b + cc) * ne + e];
    }
    const int col = cc * o.sc + bi * o.si + bj * o.sj + bk * o.sk;
    Ar[col] = (col == row && acc == 0.0) ? 1.0 : acc;
  }
}

// 1/x from the hardware reciprocal estimate and two Newton steps.
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// Inverse of a symmetric positive definite 4x4 block by its 2x2 blocks (one
// reciprocal per 2x2 block): D = [[A, B], [B^T, C]], W = A^-1 B,
// S = C - B^T W, D^-1 = [[A^-1 + W S^-1 W^T, -W S^-1], [., S^-1]].
__device__ __forceinline__ void invert4(const double (&D)[4][4], double (&P)[4][4]) {
  const double ra = recip(fma(D[0][0], D[1][1], -D[0][1] * D[0][1]));
  const double a00 = D[1][1] * ra, a01 = -D[0][1] * ra, a11 = D[0][0] * ra;
  double W[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    W[0][j] = fma(a00, D[0][2 + j], a01 * D[1][2 + j]);
    W[1][j] = fma(a01, D[0][2 + j], a11 * D[1][2 + j]);
  }
  const double s00 = fma(-D[0][2], W[0][0], fma(-D[1][2], W[1][0], D[2][2]));
  const double s01 = fma(-D[0][2], W[0][1], fma(-D[1][2], W[1][1], D[2][3]));
  const double s11 = fma(-D[0][3], W[0][1], fma(-D[1][3], W[1][1], D[3][3]));
  const double rs = recip(fma(s00, s11, -s01 * s01));
  const double t00 = s11 * rs, t01 = -s01 * rs, t11 = s00 * rs;
  P[2][2] = t00;
  P[2][3] = P[3][2] = t01;
  P[3][3] = t11;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    P[i][2] = P[2][i] = -fma(W[i][0], t00, W[i][1] * t01);
    P[i][3] = P[3][i] = -fma(W[i][0], t01, W[i][1] * t11);
  }
  P[0][0] = fma(-P[0][2], W[0][0], fma(-P[0][3], W[0][1], a00));
  P[0][1] = P[1][0] = fma(-P[0][2], W[1][0], fma(-P[0][3], W[1][1], a01));
  P[1][1] = fma(-P[1][2], W[1][0], fma(-P[1][3], W[1][1], a11));
}

// 64x64 FP64 tile in LDS, row p, column i at p * 64 + (i ^ 8 (p & 3)).  An
// MFMA operand read (lanes l: row 4kk + l/16, 16 consecutive columns) then
// spreads its four 16-lane groups over both bank halves, two groups each:
// two passes, the minimum for 64 doubles, without padding (two tiles fill
// the 64 KB a workgroup may hold).
__device__ __forceinline__ int swz(int p, int i) { return p * 64 + (i ^ ((p & 3) << 3)); }

constexpr int kP = kInvBlock * kInvBlock;  // doubles of a tile

// Invert the ni x ni block x (each wavefront a strip of 16 rows in four 16x16
// MFMA tiles, tile element v of lane (lk, li) = row 16 w + lk + 4 v, column
// 16 jb + li; the identity beyond ni) and store the inverse at P (row stride
// 64).  The symmetric sweep again, four pivots K = [4k, 4k + 4) at a time: the
// wavefront that holds the pivot rows p publishes them in LDS, every lane
// inverts the 4x4 pivot block D itself (Q = D^-1), and one MFMA per tile does
// the rank-4 update x -= (c Q) p, c_i being column i of p by symmetry.  The
// new pivot rows Q p, pivot columns c Q and pivot block -Q come from the same
// MFMA: their accumulators are cleared, the A operand of pivot rows is +Q and
// the B operand of pivot columns is minus the identity.  One barrier per four
// pivots.  sm: 512 doubles, free to overwrite.
__device__ __forceinline__ void store_pivot(double* sm, int ni, f64x4 (&x)[4], double* P) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int nst = (ni + 3) / 4;
  for (int wk = 0; 4 * wk < nst; ++wk) {
#pragma unroll
    for (int vk = 0; vk < 4; ++vk) {
      const int k = 4 * wk + vk;
      if (k >= nst) break;  // uniform
      double* p = sm + (vk & 1) * 256;  // two buffers: one barrier a step
      if (w == wk) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) p[swz(lk, 16 * jb + li)] = x[jb][vk];
      }
      __syncthreads();
      double D[4][4], Q[4][4], c[4], r[4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = a; b < 4; ++b) D[a][b] = p[swz(a, 4 * k + b)];
#pragma unroll
      for (int q = 0; q < 4; ++q) c[q] = p[swz(q, 16 * w + li)];
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) r[jb] = p[swz(lk, 16 * jb + li)];
      invert4(D, Q);
      double ql[4];  // column lk of Q
#pragma unroll
      for (int q = 0; q < 4; ++q)
        ql[q] = lk < 2 ? (lk == 0 ? Q[q][0] : Q[q][1]) : (lk == 2 ? Q[q][2] : Q[q][3]);
      const int l4 = li & 3;
      const bool in_k = (li >> 2) == vk;  // row (A) or column (B) li of strip or tile wk is a pivot's
      double t = -c[0] * ql[0];
#pragma unroll
      for (int q = 1; q < 4; ++q) t = fma(-c[q], ql[q], t);
      if (w == wk) {
        if (in_k) t = l4 < 2 ? (l4 == 0 ? ql[0] : ql[1]) : (l4 == 2 ? ql[2] : ql[3]);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) x[jb][vk] = 0.0;
      }
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        if (jb == wk && in_k) {
          r[jb] = lk == l4 ? -1.0 : 0.0;
#pragma unroll
          for (int v = 0; v < 4; ++v) x[jb][v] = 0.0;
        }
        x[jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(t, r[jb], x[jb], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int jb = 0; jb < 4; ++jb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * w + lk + 4 * v;
      if (i < ni) P[i * kInvBlock + 16 * jb + li] = -x[jb][v];
    }
}

// Buffer resource over an array of `bytes` bytes (below 2^31): loads at or
// beyond it return 0 and stores are dropped, so a block's edge costs one
// select per lane (kOut) instead of a branch per element.
constexpr uint32_t kOut = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const double* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), (short)0, (int)bytes, 0x00020000);
}
// The row offset is added to the lane's (not carried in the scalar operand):
// the range check then sees the whole offset.
__device__ __forceinline__ double bld(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t row) {
  return __builtin_bit_cast(double,
                            __builtin_amdgcn_raw_buffer_load_b64(r, (int)(off + row), 0, 0));
}
__device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t row, double x) {
  __builtin_amdgcn_raw_buffer_store_b64(
      __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), x), r,
      (int)(off + row), 0, 0);
}

// acc[jb] += sgn sum_p X[p][16 w + i] Y[p][16 jb + j] over the first 4 nk rows.
__device__ __forceinline__ void product(const double* X, const double* Y, int nk, double sgn, int w,
                                        int li, int lk, f64x4 (&acc)[4]) {
  for (int kk = 0; kk < nk; ++kk) {
    const int p = 4 * kk + lk;
    const double a = sgn * X[swz(p, 16 * w + li)];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
      acc[jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Y[swz(p, 16 * jb + li)], acc[jb], 0, 0, 0);
  }
}

// One step of the plan, one workgroup per task.  It reads the step's pivot
// inverses Pc (slot q at q * 64 mr, mr the most rows of a block) and panels
// Cc[q & 1][p][i] = c_i[p] (mr rows of stride n) and writes the next step's into
// Pn and Cn, so no workgroup reads what another writes; every tile of A has one writer.  Entries of a tile that
// lie in a next pivot's row or column are also its panel's.  All products on
// FP64 MFMA.  The code is kept short (buffer accesses, rolled loops): it runs
// once per workgroup, and an early version of 77 KB spent its time fetching
// instructions.
__global__ void __launch_bounds__(256, 2) k_inv_step(int n, int mr, double* __restrict__ A,
                                                     const InvTask* __restrict__ tasks,
                                                     const double* __restrict__ Pc,
                                                     double* __restrict__ Pn,
                                                     const double* __restrict__ Cc,
                                                     double* __restrict__ Cn) {
  __shared__ double sm[2 * kP];
  double* sP = sm;       // pivot inverse [p][q], later c_J [p][j]
  double* sX = sm + kP;  // c_I [p][i], later T [q][i]
  const InvTask t = tasks[blockIdx.x];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t cs = (int64_t)mr * n, ps = (int64_t)mr * kInvBlock;  // strides of panels, pivots
  const uint32_t rs = (uint32_t)n * 8;        // row stride in bytes
  const int I0 = t.i0, J0 = t.j0, ni = t.ni, nj = t.nj;
  const bool inverts = t.nrow >= 0 && I0 == J0;
  // the next step waits for the workgroups that invert its pivots: their
  // waves go first where another workgroup shares the compute unit
  if (inverts) __builtin_amdgcn_s_setprio(3);
  if (t.kind == kInvPanel) {  // from the upper triangle
    double* C = Cn + (t.nrow & 1) * cs;
#pragma unroll 4
    for (int r = 0; r < 16; ++r) {
      const int p = w + 4 * r, j = lane;
      if (p < ni && j < nj)
        C[(int64_t)p * n + J0 + j] =
            J0 > I0 ? A[(int64_t)(I0 + p) * n + J0 + j] : A[(int64_t)(J0 + j) * n + I0 + p];
    }
    return;
  }
  if (t.kind == kInvDiag) {
    const double* P = Pc + t.p0 * ps;
#pragma unroll 4
    for (int r = 0; r < 16; ++r) {
      const int p = w + 4 * r;
      if (p < ni && lane < ni) A[(int64_t)(I0 + p) * n + I0 + lane] = -P[p * kInvBlock + lane];
    }
    return;
  }
  const bool cross = t.kind != kInvTile;
  // O: the block whose T is formed
  const int O0 = t.kind == kInvCrossJ ? J0 : I0, no = t.kind == kInvCrossJ ? nj : ni;
  // this lane's elements of the tile: row 16 w + lk + 4 v, column 16 jb + li
  const uint32_t row0 = (uint32_t)(16 * w + lk) * rs;
  uint32_t to[4];
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) to[jb] = 16 * jb + li < nj ? row0 + 8u * (16 * jb + li) : kOut;
  const auto rA = rsrc(A + (int64_t)I0 * n + J0, (int64_t)(ni - 1) * rs + 8 * nj);
  f64x4 acc[4];
  if (!cross) {
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[jb][v] = bld(rA, to[jb], 4 * v * rs);
  }
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int q = h == 0 ? t.p0 : t.p1;
    if (q < 0) break;
    const int kb = h == 0 ? t.kb0 : t.kb1, k0 = h == 0 ? t.k00 : t.k01;
    const int nk = (kb + 3) / 4;
    const double* C = Cc + (q & 1) * cs;
    const auto rP = rsrc(Pc + q * ps, kb * kInvBlock * 8);
    const auto rO = rsrc(C + O0, (int64_t)(kb - 1) * rs + 8 * no);
    const auto rJ = rsrc(C + J0, (int64_t)(kb - 1) * rs + 8 * nj);
    // every global load in flight before the first LDS store; zero beyond the blocks
    const uint32_t po = lane < kb ? 8u * (w * kInvBlock + lane) : kOut;
    const uint32_t oo = lane < no ? w * rs + 8u * lane : kOut;
    const uint32_t jo = (!cross && lane < nj) ? w * rs + 8u * lane : kOut;
    double pv[16], xv[16], cj[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      pv[r] = bld(rP, po, 4 * r * kInvBlock * 8);
      xv[r] = bld(rO, oo, 4 * r * rs);
      cj[r] = bld(rJ, jo, 4 * r * rs);
    }
    if (h > 0) __syncthreads();  // the previous pivot's operands are read
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sP[swz(w + 4 * r, lane)] = pv[r];
      sX[swz(w + 4 * r, lane)] = xv[r];
    }
    __syncthreads();
    f64x4 T[4];  // T[16w + i][16jb + j] = sum_p c[16w + i][p] P[p][16jb + j]
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) T[jb] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (16 * w < no) product(sX, sP, nk, 1.0, w, li, lk, T);
    __syncthreads();
    // stage T as [q][i]; c_J as [p][j] replaces P
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
      for (int v = 0; v < 4; ++v) sX[swz(16 * jb + li, 16 * w + lk + 4 * v)] = T[jb][v];
    if (cross) {
      const int nx = t.kind == kInvCrossI ? t.nrow : t.ncol;
      const auto rC = rsrc(Cn + (nx & 1) * cs + k0, nx >= 0 ? (int64_t)(no - 1) * rs + 8 * kb : 0);
      const auto rB = rsrc(A + (int64_t)O0 * n + k0,
                           t.kind == kInvCrossI ? (int64_t)(no - 1) * rs + 8 * kb : 0);
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        const uint32_t o = 16 * jb + li < kb ? row0 + 8u * (16 * jb + li) : kOut;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          bst(rB, o, 4 * v * rs, T[jb][v]);
          bst(rC, o, 4 * v * rs, T[jb][v]);  // next panel, rows of K
        }
      }
      if (t.kind == kInvCrossI) return;
      __syncthreads();
      const auto rK = rsrc(A + (int64_t)k0 * n + O0, (int64_t)(kb - 1) * rs + 8 * no);
#pragma unroll
      for (int r = 0; r < 16; ++r)  // A[k0 + c][O0 + i] = T[i][c], coalesced along i
        bst(rK, oo, 4 * r * rs, sX[swz(w + 4 * r, lane)]);
      return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) sP[swz(w + 4 * r, lane)] = cj[r];
    __syncthreads();
    if (16 * w < ni) product(sX, sP, nk, -1.0, w, li, lk, acc);
  }
  const bool row = t.nrow >= 0 && !inverts, col = t.ncol >= 0 && !inverts;
  const auto rR = rsrc(Cn + (t.nrow & 1) * cs + J0, row ? (int64_t)(ni - 1) * rs + 8 * nj : 0);
#pragma unroll
  for (int jb = 0; jb < 4; ++jb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      bst(rA, to[jb], 4 * v * rs, acc[jb][v]);
      bst(rR, to[jb], 4 * v * rs, acc[jb][v]);  // block I is a next pivot
    }
  if (col) {  // block J is a next pivot: staged to be coalesced along i
    __syncthreads();
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
      for (int v = 0; v < 4; ++v) sX[swz(16 * jb + li, 16 * w + lk + 4 * v)] = acc[jb][v];
    __syncthreads();
    const auto rC = rsrc(Cn + (t.ncol & 1) * cs + I0, (int64_t)(nj - 1) * rs + 8 * ni);
    const uint32_t o = lane < ni ? w * rs + 8u * lane : kOut;
#pragma unroll
    for (int r = 0; r < 16; ++r) bst(rC, o, 4 * r * rs, sX[swz(w + 4 * r, lane)]);
    return;
  }
  if (!inverts) return;
#pragma unroll
  for (int jb = 0; jb < 4; ++jb)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * w + lk + 4 * v >= ni || 16 * jb + li >= ni)
        acc[jb][v] = 16 * w + lk + 4 * v == 16 * jb + li ? 1.0 : 0.0;
  __syncthreads();  // sP and sX are read
  store_pivot(sm, ni, acc, Pn + t.nrow * ps);
}

// After the last step: A = -A on and above the diagonal, mirrored below it.
__global__ void __launch_bounds__(256) k_inv_finish(int n, double* __restrict__ A) {
  __shared__ double sX[kInvBlock][kInvBlock + 1];
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bi > bj) return;
  const int I0 = bi * kInvBlock, J0 = bj * kInvBlock, tid = threadIdx.x;
  for (int x = tid; x < kP; x += 256) {
    const int r = x / 64, c = x % 64;
    if (I0 + r < n && J0 + c < n) sX[r][c] = -A[(int64_t)(I0 + r) * n + J0 + c];
  }
  __syncthreads();
  for (int x = tid; x < kP; x += 256) {
    const int r = x / 64, c = x % 64;
    if (I0 + r < n && J0 + c < n)
      A[(int64_t)(I0 + r) * n + J0 + c] = (bi == bj && r > c) ? sX[c][r] : sX[r][c];
    if (bi != bj && J0 + r < n && I0 + c < n) A[(int64_t)(J0 + r) * n + I0 + c] = sX[c][r];
  }
}

}  // namespace

void launch_assemble_dense(const Grid& g, const CoarseOrder& o, const double* Ke, double* A,
                           hipStream_t s) {
  k_assemble_dense<<<(unsigned)((3 * g.nn + 3) / 4), 256, 0, s>>>(g.nx, g.ny, g.nz, o, Ke, A);
}

int64_t inv_scratch_doubles(const InvPlan& plan) {
  return (2 * (int64_t)plan.max_pivots * kInvBlock + 4 * (int64_t)plan.n) * plan.max_rows;
}

void launch_invert(const InvPlan& plan, const InvTask* tasks, double* A, double* scratch, hipStream_t s) {
  // pivot inverses and panels alternate between two buffers each
  const int64_t ps = (int64_t)plan.max_pivots * plan.max_rows * kInvBlock;
  const int64_t cs = 2 * (int64_t)plan.max_rows * plan.n;
  double* P[2] = {scratch, scratch + ps};
  double* C[2] = {scratch + 2 * ps, scratch + 2 * ps + cs};
  for (int st = 0; st < (int)plan.steps.size(); ++st) {
    const InvStep& S = plan.steps[st];
    const int b = st & 1;
    k_inv_step<<<S.ntask, 256, 0, s>>>(plan.n, plan.max_rows, A, tasks + S.task0, P[b], P[b ^ 1], C[b],
                                       C[b ^ 1]);
  }
  const unsigned nb = (unsigned)((plan.n + kInvBlock - 1) / kInvBlock);
  k_inv_finish<<<dim3(nb, nb), 256, 0, s>>>(plan.n, A);
}

}  // namespace aarmr
