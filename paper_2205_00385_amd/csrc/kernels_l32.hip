// FP32 products of the coarse levels, for the refinement form's V-cycle.
//
// They are not in the moment form (kernels_level.hip), though it is the faster
// one: 6 us against two launches of 4.5 and 5.5 us for a level-1 product of
// 56x40x64, 33 against 48 us on level 1 of 256x128x128; a refinement solve of
// 256x128x128 took 13.9 ms with it when it took 15.4 ms with these.  Another
// rounding of any FP32 product moves the returned displacement by some 1e-10, by
// 1e-9 where an inner iteration more or less is taken: within cg_rtol, but no
// longer the values that were checked, so that change is a step of its own.
#include "internal.hpp"

namespace aarmr {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

typedef double f64x4 __attribute__((ext_vector_type(4)));
__host__ __device__ constexpr int sidx(int r, int c) { return sym_index(r, c); }

// XCD-contiguous order of the workgroups (see kernels_mg.hip).
__device__ __forceinline__ int xcd_slot(int w, int total) {
  const int xcd = w & 7, pos = w >> 3, q = total >> 3, r = total & 7;
  return (xcd < r) ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
}

// FP32 element matrices of a level >= 2 from its moments: K[entry] = sum_m
// C[entry][m] M_m, formed in FP64 and rounded once.  As a product
// [300 x 28] x [28 x elements] on FP64 MFMA: each wavefront takes 16 elements
// (their moments as the B operand, in registers) and walks the 19 tiles of 16
// entries, 7 MFMA steps of k = 4 each; a lane holds result rows g + 4v (g = lane
// / 16) of column lane % 16, so each store writes 16 consecutive elements of one
// entry.  Exact for unflagged elements; the flagged ones are overwritten.
__global__ void __launch_bounds__(256) k_elemmat_moments(int64_t ne, const double* __restrict__ C,
                                                         const double* __restrict__ mom,
                                                         float* __restrict__ K) {
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int64_t p0 = (int64_t)blockIdx.x * 64 + 16 * (threadIdx.x >> 6);
  if (p0 >= ne) return;  // a whole wavefront past the end (no LDS, no barriers)
  const int64_t e = p0 + j;
  const bool live = e < ne;
  double bop[7];  // B[k = g][col = j] of step s: moment 4 s + g of element e
#pragma unroll
  for (int st = 0; st < 7; ++st)
    bop[st] = (live && 4 * st + g < 27) ? mom[(int64_t)(4 * st + g) * ne + e] : 0.0;
  for (int e0 = 0; e0 < kSymEntries; e0 += 16) {
    const int ea = e0 + j;  // A[row = j][k = g] = C[e0 + j][4 s + g]
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int st = 0; st < 7; ++st) {
      const double a = ea < kSymEntries ? C[ea * 28 + 4 * st + g] : 0.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bop[st], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ent = e0 + g + 4 * v;
      if (live && ent < kSymEntries) K[(int64_t)ent * ne + e] = (float)acc[v];
    }
  }
}

// The stored matrices of the listed elements over them.
__global__ void __launch_bounds__(256) k_elemmat_stored(int64_t ne, const double* __restrict__ Kst,
                                                        const int* __restrict__ list,
                                                        const int* __restrict__ count,
                                                        float* __restrict__ K) {
  const int n = *count;
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < (int64_t)n * kSymEntries;
       t += (int64_t)gridDim.x * 256) {
    const int64_t w = t % n, q = t / n;
    K[q * ne + list[w]] = (float)Kst[q * ne + w];
  }
}

// y = sum_e L_e^T Ke_e L_e v on a coarse level (levels >= 2) from the stored
// packed element matrices.  Block: 64 consecutive nodes x 8 waves; wave a
// takes each node as local corner a of the element e = node - offset(a) and
// forms rows 3a..3a+2 of Ke_e v_e; the 8 partial rows are summed in LDS in a
// fixed order.  Blocks in XCD-contiguous order: the two
// copies of a symmetric entry are read by the waves of two corners, for
// nodes up to a plane apart, and are then fetched into one L2 only.
// mode 0: y = A v; 1: y = v + omega jd (jb - A v), a damped-Jacobi sweep; 2:
// y = jb - A v, the residual (y distinct from v).
__global__ void __launch_bounds__(512) k_apply_elemmat(int nx, int ny, int nz, int mode,
                                                       const float* __restrict__ Ke,
                                                       const float* __restrict__ v,
                                                       float* __restrict__ y,
                                                       const float* __restrict__ jb,
                                                       const float* __restrict__ jd, float omega,
                                                       int64_t rs) {
  typedef float T;
  __shared__ T red[8][3][64];
  {  // load case blockIdx.z of a lock-step multi-vector (rs: vector stride)
    const int64_t ro = (int64_t)blockIdx.z * rs;
    v += ro;
    y += ro;
    if (mode) jb += ro;
  }
  const int a = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int nn = (nx + 1) * (ny + 1) * (nz + 1);
  const int64_t ne = (int64_t)nx * ny * nz;
  const int n = xcd_slot(blockIdx.x, gridDim.x) * 64 + lane;
  T acc0 = 0, acc1 = 0, acc2 = 0;
  if (n < nn) {
    const int i = n % (nx + 1), rest = n / (nx + 1);
    const int j = rest % (ny + 1), k = rest / (ny + 1);
    const int ex = i - (a & 1), ey = j - ((a >> 1) & 1), ez = k - (a >> 2);
    if (ex >= 0 && ex < nx && ey >= 0 && ey < ny && ez >= 0 && ez < nz) {
      const int e = ex + nx * (ey + ny * ez);
      T ve[24];
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int nb = ex + (b & 1) + (nx + 1) * (ey + ((b >> 1) & 1) + (ny + 1) * (ez + (b >> 2)));
#pragma unroll
        for (int c = 0; c < 3; ++c) ve[3 * b + c] = v[c * nn + nb];
      }
#pragma unroll
      for (int q = 0; q < 24; ++q) {
        acc0 = fma(Ke[(int64_t)sidx(3 * a + 0, q) * ne + e], ve[q], acc0);
        acc1 = fma(Ke[(int64_t)sidx(3 * a + 1, q) * ne + e], ve[q], acc1);
        acc2 = fma(Ke[(int64_t)sidx(3 * a + 2, q) * ne + e], ve[q], acc2);
      }
    }
  }
  red[a][0][lane] = acc0;
  red[a][1][lane] = acc1;
  red[a][2][lane] = acc2;
  __syncthreads();
  if (a < 3 && n < nn) {
    T sum = red[0][a][lane];
#pragma unroll
    for (int q = 1; q < 8; ++q) sum += red[q][a][lane];
    const int64_t d = (int64_t)a * nn + n;
    y[d] = mode == 0 ? sum : mode == 1 ? v[d] + omega * jd[d] * (jb[d] - sum) : jb[d] - sum;
  }
}

// 8-point Walsh-Hadamard transform x[k] <- sum_a (-1)^popcount(k & a) x[a]
// of the entries 3a + s (one component s) of a 24-vector.
typedef float T;
__device__ __forceinline__ void wht8(T* x, int s) {
#pragma unroll
  for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
    for (int a = 0; a < 8; ++a)
      if (!(a & bit)) {
        const T p = x[3 * a + s], q = x[3 * (a | bit) + s];
        x[3 * a + s] = p + q;
        x[3 * (a | bit) + s] = p - q;
      }
}

// Level-1 element products, pass 1: Y[q][e] = (Ke_e v_e)[q].  SO = 0..2: one
// thread per parent element e and output component SO, which writes the
// entries q = 3a + SO; SO = 3: one thread per parent, all 24 entries (the
// inputs, their transforms and the moduli's are then formed once, not three
// times; on large levels that is faster, on small ones three times the
// threads fill the chip better).  Parents without a fixed DOF among their fine nodes have
// Ke_e = sum_c E_c M_c with M_c = R_c M_0 R_c (R_c the mirror map of child c).
// In the Walsh basis over the 8 corners (index 3k + s), R_c is the diagonal
// sign (-1)^popcount(c & mu), mu(k, s) = k ^ (1 << s), so
//   W Ke_e W / 64 = B'[kappa][lambda] * Ehat[mu(kappa) ^ mu(lambda)]
// with B' = W M_0 W / 64 and Ehat the Walsh transform of the 8 child moduli:
// y = W ((B' o Ehat) (W v)), about 256 FMA per thread.  Parents with eflag 1
// are left to l1_masked_rows, so no wave carries both paths.
template <int SO>
__device__ __forceinline__ void l1_elem(int nx, int ny, int nz,
                                        const T* __restrict__ Bw, const T* __restrict__ Ef,
                                        const uint8_t* __restrict__ eflag,
                                        const T* __restrict__ v, T* __restrict__ Y, int nbe) {
  const int nn = (nx + 1) * (ny + 1) * (nz + 1), ne = nx * ny * nz;
  const int e = SO == 3 ? (blockIdx.y * nbe + blockIdx.x) * 256 + threadIdx.x
                        : blockIdx.x * 256 + threadIdx.x;
  if (e >= ne || eflag[e]) return;  // flagged parents: l1_masked_rows
  const int ex = e % nx, rest = e / nx, ey = rest % ny, ez = rest / ny;
  T x[24];
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const int nb = ex + (b & 1) + (nx + 1) * (ey + ((b >> 1) & 1) + (ny + 1) * (ez + (b >> 2)));
#pragma unroll
    for (int c = 0; c < 3; ++c) x[3 * b + c] = v[c * nn + nb];
  }
  {
    T Eh[8];
    const int fnx = 2 * nx, fny = 2 * ny;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      Eh[c] = Ef[(int64_t)(2 * ex + (c & 1)) +
                 (int64_t)fnx * ((2 * ey + ((c >> 1) & 1)) + (int64_t)fny * (2 * ez + (c >> 2)))];
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (!(c & bit)) {
          const T p = Eh[c], q = Eh[c | bit];
          Eh[c] = p + q;
          Eh[c | bit] = p - q;
        }
#pragma unroll
    for (int s = 0; s < 3; ++s) wht8(x, s);
#pragma unroll
    for (int so = 0; so < 3; ++so) {  // output component: entries 3a + so
      if (SO != 3 && so != SO) continue;
      const T* B = Bw + so * 24;       // row kappa = 3k + so starts at B + 72k
      T y[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int muk = k ^ (1 << so);
        T acc = 0;
#pragma unroll
        for (int mm = 0; mm < 8; ++mm) {
          T t = 0;
#pragma unroll
          for (int s2 = 0; s2 < 3; ++s2) {
            const int la = 3 * (muk ^ mm ^ (1 << s2)) + s2;
            t = fma(B[72 * k + la], x[la], t);
          }
          acc = fma(Eh[mm], t, acc);
        }
        y[k] = acc;
      }
#pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
        for (int a = 0; a < 8; ++a)
          if (!(a & bit)) {
            const T p = y[a], q = y[a | bit];
            y[a] = p + q;
            y[a | bit] = p - q;
          }
#pragma unroll
      for (int a = 0; a < 8; ++a) Y[(int64_t)(3 * a + so) * ne + e] = y[a];
    }
  }
}

// Level-1 element products of the flagged parents from their stored Galerkin
// matrices (elist[0..cnt), of which only the flagged ones are written): rows
// r0..r0 + 2.  r0 is uniform per wavefront; its lanes take 16 list entries w
// (from chunk * 16 in steps of nchunk * 16), four lanes per entry, each lane two
// corners (six columns q = 3b + c); the four sums are then added in a fixed
// order.  The matrix entries need only w, so the chain is the element's number
// and then everything else at once, the flag included.  Three rows a wavefront
// and not one, with a third of the workgroups, and the flag no longer ahead of
// the operands: 56x40x64's level 1 with 4 cases 11.9 -> 10.7 us for the launch.
__device__ __forceinline__ void l1_masked_rows(int nx, int ny, int nz,
                                               const double* __restrict__ Kst,
                                               const uint8_t* __restrict__ eflag,
                                               const int* __restrict__ list, int cnt,
                                               const T* __restrict__ v, T* __restrict__ Y,
                                               int chunk, int nchunk, int r0) {
  const int nn = (nx + 1) * (ny + 1) * (nz + 1);
  const int64_t ne = (int64_t)nx * ny * nz;
  const int lane = threadIdx.x & 63, quarter = lane >> 4;
  // the loop bound is uniform per wavefront, so every lane reaches the shuffles
  for (int base = chunk * 16; base < cnt; base += nchunk * 16) {
    const int w = base + (lane & 15), wc = min(w, cnt - 1);
    const int e = list[wc];
    double K[3][6];
    T x[6];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int t = 0; t < 3; ++t)
          K[t][3 * h + c] = Kst[(int64_t)sidx(r0 + t, 3 * (2 * quarter + h) + c) * ne + wc];
    const bool live = eflag[e] != 0 && w < cnt;
    const int ex = e % nx, rest = e / nx, ey = rest % ny, ez = rest / ny;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = 2 * quarter + h;
      const int nb = ex + (b & 1) + (nx + 1) * (ey + ((b >> 1) & 1) + (ny + 1) * (ez + (b >> 2)));
#pragma unroll
      for (int c = 0; c < 3; ++c) x[3 * h + c] = v[c * nn + nb];
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      T acc = 0;
#pragma unroll
      for (int q = 0; q < 6; ++q) acc = fma((T)K[t][q], x[q], acc);
      acc += __shfl_down(acc, 32, 64);  // corners 0-3 + 4-7
      acc += __shfl_down(acc, 16, 64);
      if (quarter == 0 && live) Y[(int64_t)(r0 + t) * ne + e] = acc;
    }
  }
}

// Pass 1 in one launch: workgroups x < nbe run the element path (grid.y:
// output component, or with all3 a third of the elements each); the rest,
// counted over grid.y, run the flagged parents: two workgroups per 16-entry
// chunk of the list, twelve rows each.  (Those first: 11.2 against 10.7 us.)
__global__ void __launch_bounds__(256) k_l1_elem(int nx, int ny, int nz,
                                                 const double* __restrict__ Kst,
                                                 const T* __restrict__ Bw,
                                                 const T* __restrict__ Ef,
                                                 const uint8_t* __restrict__ eflag,
                                                 const T* __restrict__ v, T* __restrict__ Y,
                                                 int nbe, const int* __restrict__ list, int cnt,
                                                 int all3, int64_t rs, int64_t Ys) {
  v += (int64_t)blockIdx.z * rs;  // load case blockIdx.z
  Y += (int64_t)blockIdx.z * Ys;
  if ((int)blockIdx.x >= nbe) {  // workgroup-uniform
    const int per = (int)gridDim.x - nbe, mb = (int)blockIdx.x - nbe + per * (int)blockIdx.y;
    if (mb >= 3 * per / 2 * 2) return;  // an odd one out has no partner
    l1_masked_rows(nx, ny, nz, Kst, eflag, list, cnt, v, Y, mb >> 1, 3 * per >> 1,
                   12 * (mb & 1) + 3 * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)));
    return;
  }
  if (all3) {
    l1_elem<3>(nx, ny, nz, Bw, Ef, eflag, v, Y, nbe);
    return;
  }
  switch (blockIdx.y) {  // output component
    case 0: l1_elem<0>(nx, ny, nz, Bw, Ef, eflag, v, Y, nbe); break;
    case 1: l1_elem<1>(nx, ny, nz, Bw, Ef, eflag, v, Y, nbe); break;
    default: l1_elem<2>(nx, ny, nz, Bw, Ef, eflag, v, Y, nbe); break;
  }
}

// Pass 2: y[c][n] = sum over the (up to 8) elements around node n, taken in
// corner order a = 0..7, of Y[3a + c][e(n, a)].
// mode 1: y = v + omega jd (jb - A v), the damped-Jacobi sweep; mode 2: y =
// jb - A v, the residual.  All 24 entries and the epilogue's operands are
// loaded at once, at clamped elements whose terms a select leaves out (with a
// branch per corner 6.4 us on 56x40x64's level 1 with 4 cases and 16.8 us on
// 256x128x128's, 4.1 and 13.8 us so).
__global__ void __launch_bounds__(256) k_l1_gather(int nx, int ny, int nz, int mode,
                                                   const T* __restrict__ Y,
                                                   const T* __restrict__ v, T* __restrict__ y,
                                                   const T* __restrict__ jb,
                                                   const T* __restrict__ jd, T omega,
                                                   int64_t rs, int64_t Ys) {
  const int nn = (nx + 1) * (ny + 1) * (nz + 1);
  const int64_t ne = (int64_t)nx * ny * nz;
  const int n = blockIdx.x * 256 + threadIdx.x;
  Y += (int64_t)blockIdx.z * Ys;  // load case blockIdx.z
  v += (int64_t)blockIdx.z * rs;
  y += (int64_t)blockIdx.z * rs;
  if (mode) jb += (int64_t)blockIdx.z * rs;
  if (n >= nn) return;
  T vn[3] = {}, bn[3] = {}, dn[3] = {};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int64_t d = (int64_t)c * nn + n;
    if (mode) bn[c] = jb[d];
    if (mode == 1) {
      vn[c] = v[d];
      dn[c] = jd[d];
    }
  }
  const int i = n % (nx + 1), rest = n / (nx + 1), j = rest % (ny + 1), k = rest / (ny + 1);
  T t[8][3];
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int ex = min(max(i - (a & 1), 0), nx - 1), ey = min(max(j - ((a >> 1) & 1), 0), ny - 1);
    const int ez = min(max(k - (a >> 2), 0), nz - 1), e = ex + nx * (ey + ny * ez);
#pragma unroll
    for (int c = 0; c < 3; ++c) t[a][c] = Y[(int64_t)(3 * a + c) * ne + e];
  }
  T acc[3] = {0, 0, 0};
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int ex = i - (a & 1), ey = j - ((a >> 1) & 1), ez = k - (a >> 2);
    const bool in = ex >= 0 && ex < nx && ey >= 0 && ey < ny && ez >= 0 && ez < nz;
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = in ? acc[c] + t[a][c] : acc[c];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    y[(int64_t)c * nn + n] = mode == 0 ? acc[c]
                             : mode == 1 ? vn[c] + omega * dn[c] * (bn[c] - acc[c])
                                         : bn[c] - acc[c];
}

constexpr int64_t kL1All3 = 200000;

}  // namespace

void launch_elemmat_f32(const Grid& g, const double* C, const double* mom, const double* Kst,
                        const int* list, const int* count, float* K, hipStream_t s) {
  k_elemmat_moments<<<nblk(g.ne, 64), 256, 0, s>>>(g.ne, C, mom, K);
  k_elemmat_stored<<<512, 256, 0, s>>>(g.ne, Kst, list, count, K);
}

void launch_apply_elemmat_f32(const Grid& g, const float* Ke, int mode, const float* v, float* y,
                              const float* jb, const float* jd, float omega, int nr,
                              hipStream_t s) {
  k_apply_elemmat<<<dim3(nblk(g.nn, 64), 1, nr), 512, 0, s>>>(g.nx, g.ny, g.nz, mode, Ke, v, y, jb,
                                                              jd, omega, 3 * g.nn);
}

void launch_apply_l1_f32(const Grid& g, const double* Kst, const float* Bw, const float* Ef,
                         const uint8_t* eflag, const int* list, int nlist, int mode,
                         const float* v, float* Y, float* y, const float* jb, const float* jd,
                         float omega, int nr, hipStream_t s) {
  // one thread per element from kL1All3 elements up (256x128x128, level 1:
  // 41.6 -> 33.2 us per call); per (element, component) below, where the
  // 96x48x48 loop's level 1 measured faster
  const int all3 = g.ne >= kL1All3 ? 1 : 0;
  const int nbe = (int)nblk(g.ne, all3 ? 3 * 256 : 256);
  const int chunks = (int)nblk(nlist, 16);
  const int nbm = nlist > 0 ? (2 * (chunks < 1024 ? chunks : 1024) + 2) / 3 : 0;  // per grid.y
  const int64_t rs = 3 * g.nn, Ys = 24 * g.ne;
  k_l1_elem<<<dim3(nbe + nbm, 3, nr), 256, 0, s>>>(g.nx, g.ny, g.nz, Kst, Bw, Ef, eflag, v, Y, nbe,
                                                   list, nlist, all3, rs, Ys);
  k_l1_gather<<<dim3(nblk(g.nn, 256), 1, nr), 256, 0, s>>>(g.nx, g.ny, g.nz, mode, Y, v, y, jb, jd,
                                                           omega, rs, Ys);
}

}  // namespace aarmr
