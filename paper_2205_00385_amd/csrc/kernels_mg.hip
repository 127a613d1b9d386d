// Transfers and small pieces of the V-cycle (Algorithm 2): restriction P^T and
// interpolation P (trilinear, 2:1 per axis), damped-Jacobi sweeps from a stored
// product, and the coarsest solve's product with the explicit inverse
// (kernels_inv.hip).
#include <algorithm>

#include "chunks.hpp"
#include "internal.hpp"

namespace aarmr {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

__device__ inline int64_t node_of(int nx, int ny, int i, int j, int k) {
  return (int64_t)i + (int64_t)(nx + 1) * ((int64_t)j + (int64_t)(ny + 1) * k);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Workgroup w of `total` is given slot (w % 8) * (total / 8) + w / 8
// (the remainder spread over the first XCDs), so every XCD walks one
// contiguous range of slots and data shared by neighbouring slots meets in
// one L2.
__device__ __forceinline__ int xcd_slot(int w, int total) {
  const int xcd = w & 7, pos = w >> 3, q = total >> 3, r = total & 7;
  return (xcd < r) ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
}

// bc = P^T Df (bf - tf) (tf == nullptr: bf alone), weights (1/2, 1, 1/2)
// per axis.  One thread per (coarse node, fine z-offset) and component
// (grid.y); the three z-planes of a coarse node are summed in LDS.  On the
// plane grid (cnz = 0) only the middle offset lies in the grid.
// mask == nullptr: no fine fixed DOFs.
// With xc non-null also the coarse level's first Jacobi sweep from zero,
// xc = omega dc bc.  o: the order of the coarse vector.
// These levels are bound by latency, not by bytes: a thread issues its nine
// (with tf eighteen) values, the masks and dc at once, at clamped indexes
// whose terms are left out of the sum by a select, and node numbers are
// divided in 32 bits (average over the levels: 24x12x12, FP64 5.0 -> 3.4 us;
// 96x48x48, FP64 6.9 -> 4.5 us; 56x40x64 x 4, FP32 8.8 -> 6.9 us).
template <typename T>
__global__ void __launch_bounds__(192) k_restrict(int cnx, int cny, int cnz,
                                                  const T* __restrict__ bf,
                                                  const T* __restrict__ tf,
                                                  const uint8_t* __restrict__ mask,
                                                  T* __restrict__ bc,
                                                  const T* __restrict__ dc, T omega,
                                                  T* __restrict__ xc, CoarseOrder o,
                                                  int64_t fs = 0, int64_t cs = 0) {
  __shared__ T part[3][64];
  const int lane = threadIdx.x & 63, dzi = threadIdx.x >> 6;
  const int c = blockIdx.y;
  const uint32_t cxp = cnx + 1, cyp = cny + 1, cnn = cxp * cyp * (cnz + 1);
  const uint32_t fxp = 2 * cnx + 1, fyp = 2 * cny + 1;
  const int fnz = 2 * cnz;
  {  // load case blockIdx.z (fs, cs: fine and coarse vector strides), component c
    const int64_t fnn = (int64_t)fxp * fyp * (fnz + 1);
    const int64_t fo = (int64_t)blockIdx.z * fs + c * fnn, co = (int64_t)blockIdx.z * cs;
    bf += fo;
    if (tf) tf += fo;
    bc += co;
    if (xc) xc += co;
  }
  const uint32_t n = blockIdx.x * 64 + lane, nc = n < cnn ? n : cnn - 1;
  const uint32_t rest = nc / cxp, K = rest / cyp;
  const int I = (int)(nc - rest * cxp), J = (int)(rest - K * cyp);
  const int dst = c * o.sc + I * o.si + J * o.sj + (int)K * o.sk;
  const int fk = 2 * (int)K + dzi - 1;
  const bool zok = fk >= 0 && fk <= fnz;
  const T d = (xc && dzi == 0) ? dc[dst] : T(0);
  uint32_t f[9];
  T val[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int fi = min(max(2 * I + q % 3 - 1, 0), (int)fxp - 1);
    const int fj = min(max(2 * J + q / 3 - 1, 0), (int)fyp - 1);
    f[q] = (uint32_t)fi + fxp * ((uint32_t)fj + fyp * (uint32_t)(zok ? fk : 0));
    val[q] = bf[f[q]];
  }
  uint32_t fixed = 0;  // bit q: node q's DOF is fixed
  if (mask) {
    uint32_t m[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) m[q] = mask[f[q]];
#pragma unroll
    for (int q = 0; q < 9; ++q) fixed |= ((m[q] >> c) & 1u) << q;
  }
  if (tf) {
    T t[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) t[q] = tf[f[q]];
#pragma unroll
    for (int q = 0; q < 9; ++q) val[q] -= t[q];
  }
  T acc = 0;
  const T wz = dzi == 1 ? T(1) : T(0.5);
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int fi = 2 * I + q % 3 - 1, fj = 2 * J + q / 3 - 1;
    const T w = (q % 3 != 1 ? T(0.5) : T(1)) * ((q / 3 != 1 ? T(0.5) : T(1)) * wz);
    const bool use = zok && fi >= 0 && fi < (int)fxp && fj >= 0 && fj < (int)fyp &&
                     !((fixed >> q) & 1u);
    acc = use ? fma(w, val[q], acc) : acc;
  }
  part[dzi][lane] = acc;
  __syncthreads();
  if (dzi == 0 && n < cnn) {
    const T v = part[0][lane] + part[1][lane] + part[2][lane];
    bc[dst] = v;
    if (xc) xc[dst] = omega * d * v;
  }
}

// Lane i of a wavefront takes lane i-1's (wave_shr:1) or lane i+1's
// (wave_shl:1) value through DPP; the end lanes read 0.
template <int CTRL>
__device__ inline double wave_shift(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ inline float wave_shift(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// The same restriction on large 3D grids, separably and as a z-march: a
// workgroup takes a tile of kRsCI x kRsCJ coarse columns and a chunk of
// coarse planes [K0, K1), and reads each fine plane of the chunk once (the
// tile's 2 kRsCJ + 1 fine rows, one fine node per lane, 63 nodes of a row on
// lanes 0..62: whole rows, coalesced).  A fine plane is restricted along x in
// registers (DPP neighbours) and along y through LDS; every coarse node
// keeps the xy sum of the last odd fine plane and forms plane K along z as
// sy(2K) + (sy(2K-1) + sy(2K+1)) / 2.  Per coarse node the sum is thus
// m + (l + r) / 2 along x, then y, then z: a fixed order, so results are
// deterministic, and equal to the per-node sum of the small-grid kernel up
// to rounding.  All three components in one workgroup (one mask load per
// fine node).  Eight wavefronts take three of the 17 fine rows each.  Two
// raw-plane buffers: a buffer is reloaded with the plane two ahead as soon
// as its values are read, so each plane's loads have two planes of work to
// arrive in.  blockIdx.x: (tile, chunk) with tiles fastest, in XCD-contiguous
// order; blockIdx.z: load case.
constexpr int kRsCI = 31;
constexpr int kRsCJ = 8;
constexpr int kRsRows = 2 * kRsCJ + 1;
constexpr int kRmWaves = 8;
constexpr int kRmRowsPerWave = (kRsRows + kRmWaves - 1) / kRmWaves;
template <typename T>
struct RmRaw {
  T b[3][kRmRowsPerWave], t[3][kRmRowsPerWave];
  uint32_t m[kRmRowsPerWave];
};
template <typename T>
__global__ void __launch_bounds__(64 * kRmWaves) k_restrict_zm(
    int cnx, int cny, int cnz, int gx, int gy, int TK, const T* __restrict__ bf,
    const T* __restrict__ tf, const uint8_t* __restrict__ mask, T* __restrict__ bc,
    const T* __restrict__ dc, T omega, T* __restrict__ xc, int64_t fs, int64_t cs) {
  __shared__ T xr[2][3][kRsRows][32];  // [buffer][component][row][coarse column]
  {  // load case blockIdx.z
    const int64_t fo = (int64_t)blockIdx.z * fs, co = (int64_t)blockIdx.z * cs;
    bf += fo;
    if (tf) tf += fo;
    bc += co;
    if (xc) xc += co;
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int bx, by, K0;
  {
    const int t = xcd_slot(blockIdx.x, gridDim.x);
    bx = t % gx;
    by = (t / gx) % gy;
    K0 = (t / (gx * gy)) * TK;
  }
  const int K1 = min(K0 + TK, cnz + 1);
  const int I0 = bx * kRsCI, J0 = by * kRsCJ;
  const int fnx = 2 * cnx, fny = 2 * cny, fnz = 2 * cnz;
  const int64_t fnn = (int64_t)(fnx + 1) * (fny + 1) * (fnz + 1);
  const int64_t cnn = (int64_t)(cnx + 1) * (cny + 1) * (cnz + 1);
  const int64_t fplane = (int64_t)(fnx + 1) * (fny + 1);
  const int fx = 2 * I0 - 1 + lane;
  const bool xok = lane < 2 * kRsCI + 1 && fx >= 0 && fx <= fnx;
  // raw values of this lane's nodes of rows w + 8 q of fine plane fz; 0 outside
  auto load = [&](int fz, RmRaw<T>& R) {
#pragma unroll
    for (int q = 0; q < kRmRowsPerWave; ++q) {
      const int r = w + kRmWaves * q, fy = 2 * J0 - 1 + r;
      const bool ok = r < kRsRows && xok && fy >= 0 && fy <= fny && fz >= 0 && fz <= fnz;
      const int64_t f = (int64_t)fz * fplane + (int64_t)fy * (fnx + 1) + fx;
      R.m[q] = (mask && ok) ? mask[f] : 0u;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        R.b[c][q] = ok ? bf[c * fnn + f] : T(0);
        R.t[c][q] = (tf && ok) ? tf[c * fnn + f] : T(0);
      }
    }
  };
  const int ci = threadIdx.x & 31, cj = threadIdx.x >> 5;  // output thread's coarse node
  const bool out = threadIdx.x < 32 * kRsCJ && ci < kRsCI && I0 + ci <= cnx && J0 + cj <= cny;
  int buf = 0;
  // Df (b - t) of a loaded plane, then its x sums into LDS; after the
  // barrier the output threads form the y sums sy
  auto values = [&](const RmRaw<T>& R, T (&v)[3][kRmRowsPerWave]) {
#pragma unroll
    for (int q = 0; q < kRmRowsPerWave; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        T val = R.b[c][q];
        if (tf) val -= R.t[c][q];
        v[c][q] = ((R.m[q] >> c) & 1u) ? T(0) : val;
      }
  };
  auto xy = [&](const T (&v)[3][kRmRowsPerWave], T (&sy)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int q = 0; q < kRmRowsPerWave; ++q) {
        const int r = w + kRmWaves * q;
        const T l = wave_shift<0x138>(v[c][q]), rr = wave_shift<0x130>(v[c][q]);
        const T sx = v[c][q] + T(0.5) * (l + rr);
        if (r < kRsRows && (lane & 1) && lane < 2 * kRsCI) xr[buf][c][r][lane >> 1] = sx;
      }
    __syncthreads();
    if (out) {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        sy[c] = xr[buf][c][2 * cj + 1][ci] +
                T(0.5) * (xr[buf][c][2 * cj][ci] + xr[buf][c][2 * cj + 2][ci]);
    }
    buf ^= 1;
  };
  RmRaw<T> RA, RB;
  T carry[3] = {T(0), T(0), T(0)}, s0[3] = {T(0), T(0), T(0)}, s1[3] = {T(0), T(0), T(0)};
  {
    RmRaw<T> R0;
    load(2 * K0 - 1, R0);
    load(2 * K0, RA);
    load(2 * K0 + 1, RB);
    T v[3][kRmRowsPerWave];
    values(R0, v);
    xy(v, carry);
  }
  for (int K = K0; K < K1; ++K) {
    T v[3][kRmRowsPerWave];
    values(RA, v);
    load(K + 1 < K1 ? 2 * K + 2 : -1, RA);
    xy(v, s0);
    values(RB, v);
    load(K + 1 < K1 ? 2 * K + 3 : -1, RB);
    xy(v, s1);
    if (out) {
      const int64_t n =
          (int64_t)K * (cnx + 1) * (cny + 1) + (int64_t)(J0 + cj) * (cnx + 1) + I0 + ci;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const T acc = s0[c] + T(0.5) * (carry[c] + s1[c]);
        bc[c * cnn + n] = acc;
        if (xc) xc[c * cnn + n] = omega * dc[c * cnn + n] * acc;
        carry[c] = s1[c];
      }
    }
  }
}

// xf += Df P xc: thread per fine node and NC components (from NC grid.y on),
// branch-free over the (up to) 8 parent nodes: along an axis an even fine index takes its
// parent with weight 1, an odd one both neighbours with weight 1/2.  On the
// plane grid (fnz = 0) the z pair is (0, 0) with weights (1, 0).  o: the
// order of the coarse vector.  As in k_restrict every load is issued before
// the first is used, and the indexes are 32-bit.
template <typename T, int NC>
__global__ void __launch_bounds__(256) k_prolong_add(int fnx, int fny, int fnz,
                                                     const T* __restrict__ xc,
                                                     const uint8_t* __restrict__ mask,
                                                     T* __restrict__ xf, CoarseOrder o,
                                                     int64_t cs = 0, int64_t fs = 0) {
  const int c0 = blockIdx.y * NC;
  const uint32_t fxp = fnx + 1, fyp = fny + 1, fnn = fxp * fyp * (fnz + 1);
  const uint32_t n = blockIdx.x * 256 + threadIdx.x;
  if (n >= fnn) return;
  xc += (int64_t)blockIdx.z * cs + (int64_t)c0 * o.sc;  // load case blockIdx.z
  xf += (int64_t)blockIdx.z * fs + (int64_t)c0 * fnn;
  T old[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) old[c] = xf[(int64_t)c * fnn + n];
  const uint32_t m = mask ? mask[n] : 0u;
  const uint32_t rest = n / fxp, fk = rest / fyp;
  const int fi = (int)(n - rest * fxp), fj = (int)(rest - fk * fyp);
  const int ix[2] = {fi >> 1, (fi + 1) >> 1};
  const int iy[2] = {fj >> 1, (fj + 1) >> 1};
  const int iz[2] = {(int)fk >> 1, ((int)fk + 1) >> 1};
  const T wx[2] = {(fi & 1) ? T(0.5) : T(1), (fi & 1) ? T(0.5) : T(0)};
  const T wy[2] = {(fj & 1) ? T(0.5) : T(1), (fj & 1) ? T(0.5) : T(0)};
  const T wz[2] = {(fk & 1) ? T(0.5) : T(1), (fk & 1) ? T(0.5) : T(0)};
  T x[NC][8];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int q = 0; q < 8; ++q)
      x[c][q] = xc[c * o.sc + ix[q & 1] * o.si + iy[(q >> 1) & 1] * o.sj + iz[q >> 2] * o.sk];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    T s = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s = fma(wx[q & 1] * wy[(q >> 1) & 1] * wz[q >> 2], x[c][q], s);
    if (!((m >> (c0 + c)) & 1u)) xf[(int64_t)c * fnn + n] = old[c] + s;
  }
}

// The same interpolation on large 3D grids with the coarse values staged in
// LDS: a workgroup takes a 64 x 16 tile of the fine planes 2K and 2K+1 (one
// fine node per lane and row, rows w, w+4, w+8, w+12 on wavefront w, whole
// rows per load), which interpolate from the coarse planes K and K+1 only.
// It issues its fine loads, stages the 33 x 9 coarse nodes of both planes
// in LDS, and forms each node's sum with the weights and order of
// k_prolong_add, so the results are the same bits.  blockIdx.x: (tile, K)
// with K fastest, in XCD-contiguous order; blockIdx.z: load case.
constexpr int kPzX = 64, kPzY = 16;
constexpr int kPzCX = kPzX / 2 + 1, kPzCY = kPzY / 2 + 1;
constexpr int kPzRows = kPzY / 4;  // rows per wavefront
template <typename T>
__global__ void __launch_bounds__(256) k_prolong_z(int fnx, int fny, int fnz, int gx,
                                                   const T* __restrict__ xc,
                                                   const uint8_t* __restrict__ mask,
                                                   T* __restrict__ xf, int64_t cs, int64_t fs) {
  __shared__ T sx[3][2][kPzCY][kPzCX];
  xc += (int64_t)blockIdx.z * cs;  // load case blockIdx.z
  xf += (int64_t)blockIdx.z * fs;
  const int cnx = fnx / 2, cny = fny / 2, cnz = fnz / 2;
  const int64_t fnn = (int64_t)(fnx + 1) * (fny + 1) * (fnz + 1);
  const int64_t cnn = (int64_t)(cnx + 1) * (cny + 1) * (cnz + 1);
  int bx, by, K;
  {
    const int total = gridDim.x, wg = blockIdx.x;
    const int xcd = wg & 7, pos = wg >> 3, q = total >> 3, r = total & 7;
    const int t = (xcd < r) ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
    K = t % (cnz + 1);
    const int tile = t / (cnz + 1);
    bx = tile % gx;
    by = tile / gx;
  }
  const int cx0 = bx * (kPzX / 2), cy0 = by * (kPzY / 2);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int fi = bx * kPzX + lane;
  // this thread's fine values first: planes 2K + dz, rows w + 4 q4
  T old[2][kPzRows][3];
  uint8_t msk[2][kPzRows];
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int q4 = 0; q4 < kPzRows; ++q4) {
      const int fj = by * kPzY + w + 4 * q4, fz = 2 * K + dz;
      const bool ok = fi <= fnx && fj <= fny && fz <= fnz;
      const int64_t n = ok ? node_of(fnx, fny, fi, fj, fz) : 0;
      msk[dz][q4] = (ok && mask) ? mask[n] : 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) old[dz][q4][c] = ok ? xf[c * fnn + n] : T(0);
    }
  for (int x = threadIdx.x; x < 3 * 2 * kPzCY * kPzCX; x += 256) {
    const int ci = x % kPzCX, cj = (x / kPzCX) % kPzCY, pz = (x / (kPzCX * kPzCY)) % 2,
              c = x / (2 * kPzCX * kPzCY);
    const int I = cx0 + ci, J = cy0 + cj, Kz = K + pz;
    T val = T(0);
    if (I <= cnx && J <= cny && Kz <= cnz) val = xc[c * cnn + node_of(cnx, cny, I, J, Kz)];
    sx[c][pz][cj][ci] = val;
  }
  __syncthreads();
  if (fi > fnx) return;  // no barrier below
  const int ixl[2] = {(fi >> 1) - cx0, ((fi + 1) >> 1) - cx0};
  const T wx[2] = {(fi & 1) ? T(0.5) : T(1), (fi & 1) ? T(0.5) : T(0)};
#pragma unroll
  for (int dz = 0; dz < 2; ++dz) {
    const int fz = 2 * K + dz;
    if (fz > fnz) break;
    // local coarse planes of fz: {fz >> 1, (fz + 1) >> 1} - K
    const int izl[2] = {(fz >> 1) - K, ((fz + 1) >> 1) - K};
    const T wz[2] = {(fz & 1) ? T(0.5) : T(1), (fz & 1) ? T(0.5) : T(0)};
#pragma unroll
    for (int q4 = 0; q4 < kPzRows; ++q4) {
      const int fj = by * kPzY + w + 4 * q4;
      if (fj > fny) break;
      const int iyl[2] = {(fj >> 1) - cy0, ((fj + 1) >> 1) - cy0};
      const T wy[2] = {(fj & 1) ? T(0.5) : T(1), (fj & 1) ? T(0.5) : T(0)};
      const int64_t n = node_of(fnx, fny, fi, fj, fz);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        T sum = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q)
          sum = fma(wx[q & 1] * wy[(q >> 1) & 1] * wz[q >> 2],
                    sx[c][izl[q >> 2]][iyl[(q >> 1) & 1]][ixl[q & 1]], sum);
        if (!((msk[dz][q4] >> c) & 1)) xf[c * fnn + n] = old[dz][q4][c] + sum;
      }
    }
  }
}

template <typename T>
__global__ void k_jacobi_first(int64_t n3, const T* __restrict__ b, const T* __restrict__ dinv,
                               T omega, T* __restrict__ x, int64_t rs = 0) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ro = (int64_t)blockIdx.z * rs;  // load case blockIdx.z
  if (i < n3) x[ro + i] = omega * dinv[i] * b[ro + i];
}

template <typename T>
__global__ void k_jacobi_update(int64_t n3, const T* __restrict__ b, const T* __restrict__ t,
                                const T* __restrict__ dinv, T omega, T* __restrict__ x,
                                int64_t rs = 0) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ro = (int64_t)blockIdx.z * rs;  // load case blockIdx.z
  if (i < n3) x[ro + i] += omega * dinv[i] * (b[ro + i] - t[ro + i]);
}

// y = A x for the dense (symmetric) inverse; one wavefront per row.
template <typename TX, typename TY>
__global__ void __launch_bounds__(256) k_gemv(int n, const double* __restrict__ A,
                                              const TX* __restrict__ x, TY* __restrict__ y,
                                              int64_t rs = 0) {
  x += (int64_t)blockIdx.z * rs;  // load case blockIdx.z
  y += (int64_t)blockIdx.z * rs;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const double* a = A + (int64_t)row * n;
  // four independent accumulators: eight loads in flight per lane
  double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
  int j = lane;
  for (; j + 192 < n; j += 256) {
    acc0 = fma(a[j], (double)x[j], acc0);
    acc1 = fma(a[j + 64], (double)x[j + 64], acc1);
    acc2 = fma(a[j + 128], (double)x[j + 128], acc2);
    acc3 = fma(a[j + 192], (double)x[j + 192], acc3);
  }
  for (; j < n; j += 64) acc0 = fma(a[j], (double)x[j], acc0);
  double acc = (acc0 + acc1) + (acc2 + acc3);
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) y[row] = (TY)acc;
}

}  // namespace

// 3D restriction launch: one workgroup per (tile, chunk of coarse planes,
// case).  Used from kRsMinNodes coarse nodes up; on smaller grids, where a
// launch is a few microseconds either way, the per-node kernel measured
// faster than the separable form (256x128x128, FP32, as one workgroup per
// coarse plane: fine level 90 -> 68 us, second level 13.1 -> 11.0 us, third
// to fifth level 6.1/5.2/4.7 -> 8.2/6.9/5.2).  As a z-march the fine level
// takes 79.5 us (FP64) and 39.1 us (FP32).
constexpr int64_t kRsMinNodes = 100000;

// The order of a level's vectors: [component][node], x fastest.
static CoarseOrder natural(const Grid& g) {
  CoarseOrder o;
  o.si = 1;
  o.sj = g.nx + 1;
  o.sk = (g.nx + 1) * (g.ny + 1);
  o.sc = (int)g.nn;
  return o;
}
template <typename T>
static void restrict_z(const Grid& coarse, const T* bf, const T* tf, const uint8_t* mask, T* bc,
                       const T* dc, T omega, T* xc, hipStream_t s, int nr, int64_t fs,
                       int64_t cs) {
  const int gx = (coarse.nx + 1 + kRsCI - 1) / kRsCI;
  const int gy = (coarse.ny + 1 + kRsCJ - 1) / kRsCJ;
  // z-march in chunks sized by the device's resident workgroups (one per CU
  // in FP64, two in FP32; 256x128x128 fine level: 79.5 and 39.1 us, three
  // per CU in FP32 46.3 us).  A chunk of t coarse planes reads 2 t + 1 fine
  // planes, and the launch takes about ceil(workgroups / slots) rounds of
  // them: the chunk length with the fewest fine-plane reads in sequence is
  // taken (one round where the tiles fit; results do not depend on it)
  static const int slots = [] {
    int dev = 0, n = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_restrict_zm<T>,
                                                        64 * kRmWaves, 0);
    return (n > 0 && per_cu > 0) ? n * per_cu : 256;
  }();
  const int planes = coarse.nz + 1, tiles = gx * gy;
  int tk = planes;
  int64_t best = -1;
  for_chunk_lengths(planes, 1, [&](int t) {
    const int64_t chunks = (planes + t - 1) / t;
    const int64_t cost = ((int64_t)tiles * chunks + slots - 1) / slots * (2 * t + 1);
    if (best < 0 || cost < best) {
      best = cost;
      tk = t;
    }
  });
  const int gz = (planes + tk - 1) / tk;
  k_restrict_zm<T><<<dim3((unsigned)(tiles * gz), 1, (unsigned)nr), 64 * kRmWaves, 0, s>>>(
      coarse.nx, coarse.ny, coarse.nz, gx, gy, tk, bf, tf, mask, bc, dc, omega, xc, fs, cs);
}

void launch_restrict_jacobi_f32(const Grid& coarse, const float* bf, const float* tf,
                                const uint8_t* mask, float* bc, const float* dinv_c, float omega,
                                float* xc, hipStream_t s, int nr) {
  const int64_t fnn = (int64_t)(2 * coarse.nx + 1) * (2 * coarse.ny + 1) * (2 * coarse.nz + 1);
  if (coarse.nz > 0 && coarse.nn >= kRsMinNodes) {
    restrict_z<float>(coarse, bf, tf, mask, bc, dinv_c, omega, xc, s, nr, 3 * fnn, 3 * coarse.nn);
    return;
  }
  k_restrict<float><<<dim3(nblk(coarse.nn, 64), 3, nr), 192, 0, s>>>(
      coarse.nx, coarse.ny, coarse.nz, bf, tf, mask, bc, dinv_c, omega, xc, natural(coarse),
      3 * fnn, 3 * coarse.nn);
}

void launch_restrict_f32(const Grid& coarse, const float* bf, const float* tf,
                         const uint8_t* mask, float* bc, hipStream_t s, int nr,
                         const CoarseOrder* o) {
  const int64_t fnn = (int64_t)(2 * coarse.nx + 1) * (2 * coarse.ny + 1) * (2 * coarse.nz + 1);
  if (!o && coarse.nz > 0 && coarse.nn >= kRsMinNodes) {
    restrict_z<float>(coarse, bf, tf, mask, bc, nullptr, 0.0f, nullptr, s, nr, 3 * fnn,
                      3 * coarse.nn);
    return;
  }
  k_restrict<float><<<dim3(nblk(coarse.nn, 64), 3, nr), 192, 0, s>>>(
      coarse.nx, coarse.ny, coarse.nz, bf, tf, mask, bc, nullptr, 0.0f, nullptr,
      o ? *o : natural(coarse), 3 * fnn, 3 * coarse.nn);
}

// Interpolation with the coarse values in LDS on 3D grids from kPzMinNodes
// fine nodes up (256x128x128 fine level: 87.5 -> 61 us FP64, 39 -> 36 us
// FP32; on the smaller levels the per-node kernel's few microseconds stand).
constexpr int64_t kPzMinNodes = 1000000;
template <typename T>
static void prolong_z(const Grid& fine, const T* xc, const uint8_t* mask, T* xf, hipStream_t s,
                      int nr, int64_t cs, int64_t fs) {
  const int gx = (fine.nx + 1 + kPzX - 1) / kPzX, gy = (fine.ny + 1 + kPzY - 1) / kPzY;
  k_prolong_z<T><<<dim3((unsigned)(gx * gy * (fine.nz / 2 + 1)), 1, (unsigned)nr), 256, 0, s>>>(
      fine.nx, fine.ny, fine.nz, gx, xc, mask, xf, cs, fs);
}

// The per-node kernel: one component per thread where three would leave
// compute units without a workgroup (25x13x13 nodes, FP64: 4.2 -> 3.2 us),
// all three from one workgroup per compute unit up, where the shared index
// work and masks count (97x49x49 nodes, FP64: 6.6 against 7.4 us; 57x41x65
// nodes x 4, FP32: 6.6 against 8 us).
constexpr int64_t kPnBlocks = 256;
template <typename T>
static void prolong_nodes(const Grid& fine, const T* xc, const uint8_t* mask, T* xf, int ncomp,
                          const CoarseOrder* o, hipStream_t s, int nr) {
  const Grid cg = make_grid(fine.nx / 2, fine.ny / 2, fine.nz / 2);
  const CoarseOrder co = o ? *o : natural(cg);
  const unsigned nb = nblk(fine.nn, 256);
  const int64_t cs = ncomp * cg.nn, fs = ncomp * fine.nn;
  if (ncomp == 3 && (int64_t)nb * nr >= kPnBlocks)
    k_prolong_add<T, 3><<<dim3(nb, 1, nr), 256, 0, s>>>(fine.nx, fine.ny, fine.nz, xc, mask, xf,
                                                        co, cs, fs);
  else
    k_prolong_add<T, 1><<<dim3(nb, ncomp, nr), 256, 0, s>>>(fine.nx, fine.ny, fine.nz, xc, mask,
                                                            xf, co, cs, fs);
}

void launch_prolong_add_f32(const Grid& fine, const float* xc, const uint8_t* mask, float* xf,
                            hipStream_t s, int nr, const CoarseOrder* o) {
  if (!o && fine.nz > 0 && fine.nn >= kPzMinNodes) {
    const int64_t cnn = make_grid(fine.nx / 2, fine.ny / 2, fine.nz / 2).nn;
    prolong_z<float>(fine, xc, mask, xf, s, nr, 3 * cnn, 3 * fine.nn);
    return;
  }
  prolong_nodes<float>(fine, xc, mask, xf, 3, o, s, nr);
}

void launch_jacobi_first_f32(int64_t n3, const float* b, const float* dinv, float omega, float* x,
                             hipStream_t s, int nr) {
  k_jacobi_first<float><<<dim3(nblk(n3, 256), 1, nr), 256, 0, s>>>(n3, b, dinv, omega, x, n3);
}

void launch_jacobi_update_f32(int64_t n3, const float* b, const float* t, const float* dinv,
                              float omega, float* x, hipStream_t s, int nr) {
  k_jacobi_update<float><<<dim3(nblk(n3, 256), 1, nr), 256, 0, s>>>(n3, b, t, dinv, omega, x, n3);
}

void launch_gemv_f32(int n, const double* A, const float* x, float* y, hipStream_t s, int nr) {
  k_gemv<float, float><<<dim3(nblk(n, 4), 1, nr), 256, 0, s>>>(n, A, x, y, n);
}

void launch_restrict(const Grid& coarse, const double* bf, const double* tf, const uint8_t* mask,
                     double* bc, hipStream_t s, int ncomp, const CoarseOrder* o) {
  if (!o && coarse.nz > 0 && ncomp == 3 && coarse.nn >= kRsMinNodes) {
    restrict_z<double>(coarse, bf, tf, mask, bc, nullptr, 0.0, nullptr, s, 1, 0, 0);
    return;
  }
  k_restrict<double><<<dim3(nblk(coarse.nn, 64), ncomp), 192, 0, s>>>(coarse.nx, coarse.ny, coarse.nz,
                                                                  bf, tf, mask, bc, nullptr, 0.0,
                                                                  nullptr, o ? *o : natural(coarse));
}

void launch_restrict_jacobi(const Grid& coarse, const double* bf, const double* tf,
                            const uint8_t* mask, double* bc, const double* dinv_c, double omega,
                            double* xc, hipStream_t s, int ncomp) {
  if (coarse.nz > 0 && coarse.nn >= kRsMinNodes) {
    restrict_z<double>(coarse, bf, tf, mask, bc, dinv_c, omega, xc, s, 1, 0, 0);
    return;
  }
  k_restrict<double><<<dim3(nblk(coarse.nn, 64), ncomp), 192, 0, s>>>(coarse.nx, coarse.ny, coarse.nz,
                                                                  bf, tf, mask, bc, dinv_c, omega,
                                                                  xc, natural(coarse));
}

void launch_prolong_add(const Grid& fine, const double* xc, const uint8_t* mask, double* xf,
                        hipStream_t s, int ncomp, const CoarseOrder* o) {
  if (!o && fine.nz > 0 && ncomp == 3 && fine.nn >= kPzMinNodes) {
    prolong_z<double>(fine, xc, mask, xf, s, 1, 0, 0);
    return;
  }
  prolong_nodes<double>(fine, xc, mask, xf, ncomp, o, s, 1);
}

void launch_jacobi_first(int64_t n3, const double* b, const double* dinv, double omega, double* x,
                         hipStream_t s) {
  k_jacobi_first<double><<<nblk(n3, 256), 256, 0, s>>>(n3, b, dinv, omega, x);
}

void launch_jacobi_update(int64_t n3, const double* b, const double* t, const double* dinv,
                          double omega, double* x, hipStream_t s) {
  k_jacobi_update<double><<<nblk(n3, 256), 256, 0, s>>>(n3, b, t, dinv, omega, x);
}

void launch_gemv(int n, const double* A, const double* x, double* y, hipStream_t s) {
  k_gemv<double, double><<<nblk(n, 4), 256, 0, s>>>(n, A, x, y);
}

}  // namespace aarmr
