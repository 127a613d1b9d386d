// Density filter (eqs. 31-32), its adjoint (eq. 33) and the device-side
// bisection of the optimality-criteria update.
#include <cmath>

#include <algorithm>

#include "internal.hpp"

namespace aarmr {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Hs_e = sum of in-domain cone weights max(0, r - |d|) around element e.
__global__ void k_filter_rowsum(int nx, int ny, int nz, double r, int R, double* __restrict__ Hs) {
  const int64_t ne = (int64_t)nx * ny * nz;
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  const int i = (int)(e % nx);
  const int64_t rest = e / nx;
  const int j = (int)(rest % ny), k = (int)(rest / ny);
  double s = 0.0;
  for (int dk = -R; dk <= R; ++dk) {
    if (k + dk < 0 || k + dk >= nz) continue;
    for (int dj = -R; dj <= R; ++dj) {
      if (j + dj < 0 || j + dj >= ny) continue;
      for (int di = -R; di <= R; ++di) {
        if (i + di < 0 || i + di >= nx) continue;
        const double w = r - sqrt((double)(di * di + dj * dj + dk * dk));
        if (w > 0.0) s += w;
      }
    }
  }
  Hs[e] = s;
}

// mode 0: out_e = sum_j w_ej in_j / Hs_e;  mode 1: out_e = sum_i w_ie in_i / Hs_i.
// W holds the cone weights max(0, r - |d|) of the (2R+1)^3 offsets
// (dk, dj, di), di fastest.  Any reach; thread per element.
__global__ void __launch_bounds__(256) k_filter(int nx, int ny, int nz, int R, int mode,
                                                const double* __restrict__ W,
                                                const double* __restrict__ Hs,
                                                const double* __restrict__ in,
                                                double* __restrict__ out) {
  const int D = 2 * R + 1;
  const int64_t ne = (int64_t)nx * ny * nz;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= ne) return;
  const int i = (int)(e % nx);
  const int64_t rest = e / nx;
  const int j = (int)(rest % ny), k = (int)(rest / ny);
  const int64_t sy = nx, sz = (int64_t)nx * ny;
  double s = 0.0;
  for (int dk = -R; dk <= R; ++dk) {
    const int kk = k + dk;
    if (kk < 0 || kk >= nz) continue;
    for (int dj = -R; dj <= R; ++dj) {
      const int jj = j + dj;
      if (jj < 0 || jj >= ny) continue;
      for (int di = -R; di <= R; ++di) {
        const int ii = i + di;
        if (ii < 0 || ii >= nx) continue;
        const double w = W[((dk + R) * D + (dj + R)) * D + (di + R)];
        const int64_t nb = e + di + sy * dj + sz * dk;
        s = mode == 0 ? fma(w, in[nb], s) : fma(w, in[nb] / Hs[nb], s);
      }
    }
  }
  out[e] = mode == 0 ? s / Hs[e] : s;
}

// The same sums for a small reach, from LDS: a workgroup takes a tile of
// kFtX x kFtY x TZ elements and stages it with its halo (0 outside the grid:
// a term of 0 leaves the sum's bits), in mode 1 already divided by Hs, so an
// element is divided two to four times and not once per tap.  Read directly,
// the taps cost a pass of bounds checks in every wavefront that holds an
// element on a side of the grid, which on rows of 96 is nearly all of them.
// PLANE: one layer, whose sums have no z offsets.  Per call, both modes,
// R = 1: 96x48x48 12.9 -> 4.9 us, 24x12x12 7.7 -> 4.1 us; R = 2: plane
// 320x160 8.8 -> 3.8 us.
constexpr int kFtX = 32, kFtY = 8;
template <int R, int TZ, bool PLANE>
__global__ void __launch_bounds__(kFtX * kFtY) k_filter_tile(int nx, int ny, int nz, int gx, int gy,
                                                             int mode,
                                                             const double* __restrict__ W,
                                                             const double* __restrict__ Hs,
                                                             const double* __restrict__ in,
                                                             double* __restrict__ out) {
  constexpr int D = 2 * R + 1, RZ = PLANE ? 0 : R;
  constexpr int SX = kFtX + 2 * R, SY = kFtY + 2 * R, SZ = TZ + 2 * RZ, N = SX * SY * SZ;
  constexpr int kPer = (N + kFtX * kFtY - 1) / (kFtX * kFtY);
  __shared__ double tile[N];
  const int b = blockIdx.x, by = b / gx, bz = by / gy;
  const int i0 = (b - by * gx) * kFtX, j0 = (by - bz * gy) * kFtY, k0 = bz * TZ;
  double v[kPer], h[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int t = threadIdx.x + q * kFtX * kFtY;
    const int i = i0 + t % SX - R, j = j0 + t / SX % SY - R, k = k0 + t / (SX * SY) - RZ;
    const bool ok = t < N && i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz;
    const int64_t e = ok ? i + (int64_t)nx * (j + (int64_t)ny * k) : 0;
    v[q] = in[e];
    h[q] = mode ? Hs[e] : 1.0;
    if (!ok) v[q] = 0.0;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int t = threadIdx.x + q * kFtX * kFtY;
    if (t < N) tile[t] = mode ? v[q] / h[q] : v[q];
  }
  const int li = threadIdx.x % kFtX, lj = threadIdx.x / kFtX;
  const int i = i0 + li, j = j0 + lj;
  const bool col = i < nx && j < ny;
  double hs[TZ];
#pragma unroll
  for (int z = 0; z < TZ; ++z)
    hs[z] = (!mode && col && k0 + z < nz) ? Hs[i + (int64_t)nx * (j + (int64_t)ny * (k0 + z))]
                                          : 1.0;
  __syncthreads();
  if (!col) return;
#pragma unroll
  for (int z = 0; z < TZ; ++z) {
    if (k0 + z >= nz) break;
    double s = 0.0;
#pragma unroll
    for (int dk = -RZ; dk <= RZ; ++dk)
#pragma unroll
      for (int dj = -R; dj <= R; ++dj)
#pragma unroll
        for (int di = -R; di <= R; ++di)
          s = fma(W[((dk + R) * D + (dj + R)) * D + (di + R)],
                  tile[((z + dk + RZ) * SY + lj + dj + R) * SX + li + di + R], s);
    out[i + (int64_t)nx * (j + (int64_t)ny * (k0 + z))] = mode ? s : s / hs[z];
  }
}

// The OC update of one element at multiplier lmid.
__device__ inline double oc_x(double xe, double B, double lmid, double move, double eta) {
  double v = xe * (eta == 0.5 ? sqrt(B / lmid) : pow(B / lmid, eta));
  v = fmin(v, fmin(1.0, xe + move));
  return fmax(v, fmax(0.0, xe - move));
}

// State of the bisection: the bracket, the last multiplier evaluated, whether
// the end is reached ((l2 - l1)/(l1 + l2) <= 1e-3, or the 200th step) and the
// steps taken.  As doubles l1, l2, lmid, done, steps in memory (kOcState
// apart).
struct OcState {
  double l1, l2, lmid, done, steps;
};

// Launch `round` of the bisection finishes the volumes that launch round - 1
// left as partials for kOcTrials multipliers, in heap order (node t: midpoint
// of its interval, 2t + 1 and 2t + 2: its left and right halves), and takes up
// to kOcLevels steps along the path that the decisions take.  Every workgroup
// does so for itself, in the same order, so no launch is needed in between;
// workgroup 0 also stores the state.  States and partials alternate between
// two buffers, so a launch reads only what the launch before it wrote.
// 16 lanes sum each trial's partials.
__device__ inline OcState oc_walk(int round, double* __restrict__ state,
                                  const double* __restrict__ partial, double target,
                                  double* vol) {
  OcState st{0.0, 1e9, 0.5e9, 0.0, 0.0};
  if (round > 0) {
    const double* from = state + ((round - 1) & 1) * kOcState;
    st = {from[0], from[1], from[2], from[3], from[4]};
    if (st.done == 0.0) {  // workgroup-uniform
      const double* p = partial + (int64_t)((round - 1) & 1) * kOcTrials * kOcParts;
      const int t = threadIdx.x >> 4, part = threadIdx.x & 15;
      if (t < kOcTrials) {
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < kOcParts / 16; ++q) acc += p[t * kOcParts + q * 16 + part];
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (part == 0) vol[t] = acc;
      }
      __syncthreads();
      int h = 0;
#pragma unroll
      for (int level = 0; level < kOcLevels; ++level) {
        if (st.done != 0.0) break;
        st.lmid = 0.5 * (st.l1 + st.l2);
        const bool right = vol[h] > target;
        (right ? st.l1 : st.l2) = st.lmid;
        h = 2 * h + (right ? 2 : 1);
        st.steps += 1.0;
        if ((st.l2 - st.l1) / (st.l1 + st.l2) <= 1e-3 || st.steps >= 200.0) st.done = 1.0;
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double* to = state + (round & 1) * kOcState;
    to[0] = st.l1;
    to[1] = st.l2;
    to[2] = st.lmid;
    to[3] = st.done;
    to[4] = st.steps;
  }
  return st;
}

// One launch of the bisection: the steps that the previous launch's volumes
// decide, then partials of sum_j c_j x_new_j, the volume of the filtered x_new
// (c = H^T (1 / Hs), the column weights of the normalised filter), for the
// kOcTrials multipliers that the next kOcLevels steps can visit.  The update's
// root splits, x (B / l)^eta = (x B^eta) l^-eta, so an element costs one root
// and a product and two clamps per trial.  The launches are a serial chain of
// a few microseconds each, so what counts is their number: five levels here
// (31 trials, 62 accumulator registers) against three per pair of launches
// (96x48x48: 15 pairs of 11.8 us before, 9 launches of 8 us now).  The trial
// sums of a wavefront are added by halving: 32 values in 32 exchanges.
template <bool HALF>
__global__ void __launch_bounds__(kOcThreads) k_oc_round(
    int64_t ne, const double* __restrict__ x, const double* __restrict__ dc,
    const double* __restrict__ dv, const double* __restrict__ cw, double move, double eta,
    double target, int round, double* __restrict__ state, double* __restrict__ partial) {
  __shared__ double vol[kOcTrials + 1], rl[kOcTrials + 1], red[kOcTrials + 1][kOcThreads / 64];
  const int64_t stride = (int64_t)kOcParts * kOcThreads;
  int64_t e = (int64_t)blockIdx.x * kOcThreads + threadIdx.x;
  // the first element's values arrive while the state is walked
  const bool any = e < ne;
  double xe = any ? x[e] : 0.0, ge = any ? dc[e] : 0.0, ve = any ? dv[e] : 1.0,
         c = any ? cw[e] : 0.0;
  const OcState st = oc_walk(round, state, partial, target, vol);
  if (st.done != 0.0) return;  // workgroup-uniform
  if (threadIdx.x < kOcTrials) {  // the trial multipliers: walk down to node t
    const int n = threadIdx.x + 1;  // heap index from 1: its bits below the top one are the path
    double l1 = st.l1, l2 = st.l2;
    for (int bit = 30 - __clz(n); bit >= 0; --bit) {
      const double lm = 0.5 * (l1 + l2);
      if ((n >> bit) & 1)
        l1 = lm;
      else
        l2 = lm;
    }
    const double lm = 0.5 * (l1 + l2);
    rl[threadIdx.x] = HALF ? 1.0 / sqrt(lm) : pow(lm, -eta);
  }
  __syncthreads();
  double acc[kOcTrials + 1];
#pragma unroll
  for (int t = 0; t <= kOcTrials; ++t) acc[t] = 0.0;
  while (e < ne) {
    const double B = fmax(0.0, -ge) / ve;
    const double xb = xe * (HALF ? sqrt(B) : pow(B, eta));
    const double hi = fmin(1.0, xe + move), lo = fmax(0.0, xe - move);
#pragma unroll
    for (int t = 0; t < kOcTrials; ++t) acc[t] = fma(c, fmax(fmin(xb * rl[t], hi), lo), acc[t]);
    e += stride;
    if (e < ne) {
      xe = x[e];
      ge = dc[e];
      ve = dv[e];
      c = cw[e];
    }
  }
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int half = (kOcTrials + 1) / 2; half > 0; half >>= 1) {
    const bool up = lane & (2 * half);
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const double send = up ? acc[i] : acc[i + half], keep = up ? acc[i + half] : acc[i];
      acc[i] = keep + __shfl_xor(send, 2 * half, 64);
    }
  }
  acc[0] += __shfl_xor(acc[0], 1, 64);
  if (!(lane & 1)) red[lane >> 1][threadIdx.x >> 6] = acc[0];  // lane bits 5..1 are the trial's
  __syncthreads();
  if (threadIdx.x < kOcTrials) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kOcThreads / 64; ++w) s += red[threadIdx.x][w];
    partial[(int64_t)(round & 1) * kOcTrials * kOcParts + threadIdx.x * kOcParts + blockIdx.x] = s;
  }
}

// The last launch's volumes decided, then, if they end the bisection, x_new
// at the last multiplier it evaluated.
__global__ void __launch_bounds__(kOcThreads) k_oc_final(
    int64_t ne, const double* __restrict__ x, const double* __restrict__ dc,
    const double* __restrict__ dv, double move, double eta, double target, int round,
    double* __restrict__ state, const double* __restrict__ partial, double* __restrict__ xnew) {
  __shared__ double vol[kOcTrials + 1];
  const OcState st = oc_walk(round, state, partial, target, vol);
  if (st.done == 0.0) return;
  const int64_t stride = (int64_t)gridDim.x * kOcThreads;
  for (int64_t e = (int64_t)blockIdx.x * kOcThreads + threadIdx.x; e < ne; e += stride)
    xnew[e] = oc_x(x[e], fmax(0.0, -dc[e]) / dv[e], st.lmid, move, eta);
}

template <typename T>
__global__ void k_fill(int64_t n, T v, T* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = v;
}

}  // namespace

static int filter_reach(double r) { return (int)ceil(r) - 1; }

void filter_weights(double r, double* W) {
  const int R = filter_reach(r), D = 2 * R + 1;
  for (int dk = -R; dk <= R; ++dk)
    for (int dj = -R; dj <= R; ++dj)
      for (int di = -R; di <= R; ++di) {
        const double w = r - std::sqrt((double)(di * di + dj * dj + dk * dk));
        W[((dk + R) * D + (dj + R)) * D + (di + R)] = w > 0.0 ? w : 0.0;
      }
}

int filter_taps(double r) {
  const int D = 2 * filter_reach(r) + 1;
  return D * D * D;
}

void launch_filter_rowsum(const Grid& g, double r, double* Hs, hipStream_t s) {
  k_filter_rowsum<<<nblk(g.ne, 256), 256, 0, s>>>(g.nx, g.ny, g.nz, r, filter_reach(r), Hs);
}

template <int R, int TZ, bool PLANE>
static void filter_tile(const Grid& g, const double* W, int mode, const double* Hs,
                        const double* in, double* out, hipStream_t s) {
  const int gx = (g.nx + kFtX - 1) / kFtX, gy = (g.ny + kFtY - 1) / kFtY, gz = (g.nz + TZ - 1) / TZ;
  k_filter_tile<R, TZ, PLANE><<<(unsigned)((int64_t)gx * gy * gz), kFtX * kFtY, 0, s>>>(
      g.nx, g.ny, g.nz, gx, gy, mode, W, Hs, in, out);
}

// Tiles for the reaches 1 and 2 (radii up to 3), whose halo is a small
// multiple of the tile; larger ones per element.
void launch_filter(const Grid& g, double r, const double* W, int mode, const double* Hs,
                   const double* in, double* out, hipStream_t s) {
  const int R = filter_reach(r);
  if (R == 1 && g.nz == 1)
    filter_tile<1, 1, true>(g, W, mode, Hs, in, out, s);
  else if (R == 2 && g.nz == 1)
    filter_tile<2, 1, true>(g, W, mode, Hs, in, out, s);
  else if (R == 1)
    filter_tile<1, 2, false>(g, W, mode, Hs, in, out, s);
  else if (R == 2)
    filter_tile<2, 4, false>(g, W, mode, Hs, in, out, s);
  else
    k_filter<<<nblk(g.ne, 256), 256, 0, s>>>(g.nx, g.ny, g.nz, R, mode, W, Hs, in, out);
}

void launch_fill(int64_t n, double v, double* out, hipStream_t s) {
  k_fill<double><<<nblk(n, 256), 256, 0, s>>>(n, v, out);
}

void launch_fill_f32(int64_t n, float v, float* out, hipStream_t s) {
  k_fill<float><<<nblk(n, 256), 256, 0, s>>>(n, v, out);
}

void launch_oc_round(int64_t ne, const double* x, const double* dc, const double* dv,
                     const double* cw, double move, double eta, double target, int round,
                     double* scratch, hipStream_t s) {
  double* partial = scratch + 2 * kOcState;
  if (eta == 0.5)
    k_oc_round<true><<<kOcParts, kOcThreads, 0, s>>>(ne, x, dc, dv, cw, move, eta, target, round,
                                                     scratch, partial);
  else
    k_oc_round<false><<<kOcParts, kOcThreads, 0, s>>>(ne, x, dc, dv, cw, move, eta, target, round,
                                                      scratch, partial);
}

void launch_oc_final(int64_t ne, const double* x, const double* dc, const double* dv, double move,
                     double eta, double target, int round, double* scratch, double* xnew,
                     hipStream_t s) {
  const unsigned nb = std::min(nblk(ne, kOcThreads), 1024u);
  k_oc_final<<<nb, kOcThreads, 0, s>>>(ne, x, dc, dv, move, eta, target, round, scratch,
                                       scratch + 2 * kOcState, xnew);
}

}  // namespace aarmr
