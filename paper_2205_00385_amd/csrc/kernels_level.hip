// Coarse levels of the hierarchy (Algorithm 2): Galerkin operators in moment
// form (moment.hpp), their Jacobi diagonals and products.
//
// An element of level l >= 1 that contains no fixed fine DOF is applied from
// the moments of its moduli: the 8 child moduli on level 1, 27 stored numbers
// on the levels below.  An element that does ("flagged") has the masked
// operator (Df P)^T K (Df P), which is stored as a packed 24x24 matrix.  Nodes
// of flagged elements ("special" nodes) are computed from stored matrices
// alone, so the elements around them are stored too, unless the level is split
// (k_lists).  On the coarsest level every element is stored: its matrices are
// assembled into the dense operator.
//
// A level-1 product used to write its element products to a [24][ne] buffer and
// gather them in a second launch, and a product below read the 300 stored entries
// of every element.  Per product, from those to this form (FP64): 256x128x128
// level 1 73 -> 43 us, level 2 44 -> 17, levels 3 and 4 10 -> 8; 96x48x48 level 1
// 14.8 -> 7.5, level 2 9.9 -> 7.5; 24x12x12 level 1 10 -> 6 us.
#include <type_traits>

#include "chunks.hpp"
#include "internal.hpp"
#include "moment.hpp"

namespace aarmr {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

__host__ __device__ constexpr int sidx(int r, int c) { return sym_index(r, c); }

// Weight of parent corner A (0/1) at position pos (0, 1, 2) inside the parent.
__device__ inline double phi1(int pos, int A) {
  return pos == 1 ? 0.5 : ((pos >> 1) == A ? 1.0 : 0.0);
}

// Whether one of the elements x - 1 .. x + N - 2 (and so in y and z) is flagged.
// Outside the grid the index is clamped to an element of the set, which leaves
// the answer, so all N^3 loads are independent (in a loop over the elements
// inside the grid each waited for the one before: 14 us a list pass on 96x48x48,
// 7.3 to 8.2 us so).
template <int N>
__device__ __forceinline__ bool flagged_near(const uint8_t* f, int nx, int ny, int nz, int x, int y,
                                             int z) {
  unsigned any = 0;
#pragma unroll
  for (int dz = -1; dz < N - 1; ++dz)
#pragma unroll
    for (int dy = -1; dy < N - 1; ++dy)
#pragma unroll
      for (int dx = -1; dx < N - 1; ++dx)
        any |= f[min(max(x + dx, 0), nx - 1) +
                 nx * (min(max(y + dy, 0), ny - 1) + ny * min(max(z + dz, 0), nz - 1))];
  return any != 0;
}

// ---- flags and lists -------------------------------------------------------

// Level-1 elements with a fixed DOF among their 27 fine nodes.
__global__ void __launch_bounds__(256) k_flags1(int nx, int ny, int nz,
                                                const uint8_t* __restrict__ mask,
                                                uint8_t* __restrict__ eflag) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= nx * ny * nz) return;
  const int x = e % nx, r = e / nx, y = r % ny, z = r / ny;
  const int fx = 2 * nx + 1, fy = 2 * ny + 1;
  const uint8_t* p = mask + 2 * x + (int64_t)fx * (2 * y + fy * (2 * z));
  unsigned any = 0;
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const uint8_t* q = p + (t % 3) * fx + (t / 3) * fx * fy;
    any |= q[0] | q[1] | q[2];
  }
  eflag[e] = any ? 1 : 0;
}

// Levels >= 2 in one launch, one wavefront per element: flagged if one of its
// level-1 descendants is.  A row of descendants along x is n = 2^(l - 1) bytes
// at an offset that is a multiple of n, so rows are read in words of up to 16
// bytes, eight a lane in flight (byte by byte the few elements of the deepest
// levels set the launch's time: setup of 128x128x128 in eight levels 807 -> 368 us).
template <typename W>
__device__ __forceinline__ bool any_in(const W& w) {
  if constexpr (sizeof(W) == 16)
    return (w.x | w.y | w.z | w.w) != 0;
  else if constexpr (sizeof(W) == 8)
    return (w.x | w.y) != 0;
  else
    return w != 0;
}
template <typename W>
__device__ __forceinline__ bool flagged_below(const uint8_t* f, int nx1, int ny1, int s, int x, int y,
                                              int z, int lane) {
  const int n = 1 << s, lw = s - (31 - __builtin_clz((unsigned)sizeof(W)));  // words of a row: 2^lw
  const int words = n << (s + lw);
  const uint8_t* p = f + x * n + (int64_t)nx1 * (y * n + (int64_t)ny1 * (z * n));
  bool any = false;
  for (int d0 = lane; d0 < words; d0 += 8 * 64) {
    W w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int d = min(d0 + 64 * q, words - 1);  // a word of the element again past its end
      const int dx = d & ((1 << lw) - 1), dy = (d >> lw) & (n - 1), dz = d >> (lw + s);
      w[q] = *reinterpret_cast<const W*>(p + dx * (int)sizeof(W) + (int64_t)nx1 * (dy + (int64_t)ny1 * dz));
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) any |= any_in(w[q]);
  }
  return any;
}
__global__ void __launch_bounds__(256) k_flags_deep(LevelTable T) {
  int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int l = 2;
  while (l < T.nlev && item >= T.ne[l]) item -= T.ne[l++];  // wave-uniform
  if (l >= T.nlev) return;
  const int nx = T.nx[l], ny = T.ny[l];
  const int x = item % nx, r = item / nx, y = r % ny, z = r / ny;
  const int s = l - 1, nx1 = T.nx[1], ny1 = T.ny[1];
  const uint8_t* f = T.eflag[1];
  const bool any = s == 1   ? flagged_below<uint16_t>(f, nx1, ny1, s, x, y, z, lane)
                   : s == 2 ? flagged_below<uint32_t>(f, nx1, ny1, s, x, y, z, lane)
                   : s == 3 ? flagged_below<uint2>(f, nx1, ny1, s, x, y, z, lane)
                            : flagged_below<uint4>(f, nx1, ny1, s, x, y, z, lane);
  const bool flag = __any(any);
  if (lane == 0) T.eflag[l][item] = flag ? 1 : 0;
}

// The stored elements and the special nodes of every level, in index order
// (neighbouring entries then lie side by side in the stored matrices).  Items
// are the elements, then the nodes, of level 1, 2, ..; a block takes 1024 of
// one segment.  Pass 0 counts a block's hits, pass 1 adds up the counts before
// it and writes its part of the list.
//
// A level is split where kSplitElements elements or more have a special node but
// no flag: its list then holds the flagged elements alone, the march takes what
// they would add as 0 (moments, on level 1 moduli) and k_level_add adds it.  Below
// that the stored rows of all elements around a special node, in the march's own
// launch, are the faster form (256x128x128 with one clamped face, 4096 such
// elements: level 1 30 against 35 us); above, supports spread over a grid had ten
// stored elements to a flagged one (256x128x128 with 0.1% of the nodes fixed: setup
// 2.93 -> 0.93 ms, level 1 126 -> 60 us, solve 21.2 -> 16.2 ms).  Levels of less
// than kSplitLevel elements are left as they are, without a second launch.
// A count of part[] is near elements (low half) and flagged ones.
constexpr int kChunk = 1024;
constexpr int kSplitElements = 16384, kSplitLevel = 32768;
template <int PASS>
__global__ void __launch_bounds__(256) k_lists(LevelTable T) {
  __shared__ int sh[256];
  __shared__ int2 sb[256];
  int blk = blockIdx.x, first = 0, l = 1, nodes = 0, nb;
  for (;;) {  // the segment of this block (uniform)
    const int n = nodes ? T.nn[l] : T.ne[l];
    nb = (n + kChunk - 1) / kChunk;
    if (blk < first + nb) break;
    first += nb;
    l += nodes;
    nodes ^= 1;
  }
  const int n = nodes ? T.nn[l] : T.ne[l];
  const int nx = T.nx[l], ny = T.ny[l], nz = T.nz[l];
  const bool all = l == T.nlev - 1;  // the coarsest level is stored whole
  const bool can = !nodes && !all && n >= kSplitLevel;
  const uint8_t* f = T.eflag[l];
  unsigned hit = 0, hitf = 0;
  const int i0 = (blk - first) * kChunk + 4 * (int)threadIdx.x;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = min(i0 + q, n - 1);
    const int wx = nodes ? nx + 1 : nx, wy = nodes ? ny + 1 : ny;
    const int x = i % wx, r = i / wx, y = r % wy, z = r / wy;
    const bool near = all || (nodes ? flagged_near<2>(f, nx, ny, nz, x, y, z)
                                    : flagged_near<3>(f, nx, ny, nz, x, y, z));
    if (near && i0 + q < n) hit |= 1u << q;
    if (can && f[i] && i0 + q < n) hitf |= 1u << q;
  }
  int base = 0;
  bool split = false;
  if (PASS == 1) {  // near but unflagged elements of the level; both counts of the blocks before
    int saved = 0;
    int2 s = {0, 0};
    for (int b = first + (int)threadIdx.x; b < (can ? first + nb : blk); b += 256) {
      const int p = T.part[b];
      saved += (p & 0xFFFF) - (p >> 16);
      if (b < blk) {
        s.x += p & 0xFFFF;
        s.y += p >> 16;
      }
    }
    sh[threadIdx.x] = saved;
    sb[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) {
        sh[threadIdx.x] += sh[threadIdx.x + off];
        sb[threadIdx.x].x += sb[threadIdx.x + off].x;
        sb[threadIdx.x].y += sb[threadIdx.x + off].y;
      }
      __syncthreads();
    }
    split = can && sh[0] >= kSplitElements;
    base = split ? sb[0].y : sb[0].x;
    if (split) hit = hitf;
    __syncthreads();
  }
  const int cnt = __popc(hit) | (PASS == 0 ? __popc(hitf) << 16 : 0);
  sh[threadIdx.x] = cnt;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {  // inclusive scan
    const int t = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  if (PASS == 0) {
    if (threadIdx.x == 255) T.part[blk] = sh[255];
    return;
  }
  int w = base + sh[threadIdx.x] - cnt;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + q;
    if (i >= n) break;
    const bool h = (hit >> q) & 1;
    if (nodes) {
      T.special[l][i] = h ? 1 : 0;
      if (h) T.nlist[l][w++] = i;
    } else {
      T.eidx[l][i] = h ? w : -1;
      if (h) T.elist[l][w++] = i;
    }
  }
  if (threadIdx.x == 0 && i0 + kChunk >= n) {
    T.counts[2 * l + nodes] = base + sh[255];
    if (!nodes) T.counts[kCountSplit + l] = split ? 1 : 0;
  }
}

// The place among the stored elements of the element that has a special node
// as corner a, -1 outside the grid: corner[a][place of the node in its list].
__global__ void __launch_bounds__(256) k_corners(LevelTable T) {
  int t = blockIdx.x * 256 + threadIdx.x, l = 1;
  while (l < T.nlev && t >= 8 * T.nn[l]) t -= 8 * T.nn[l++];
  if (l >= T.nlev) return;
  const int a = t & 7, i = t >> 3;
  if (i >= T.counts[2 * l + 1]) return;
  const int n = T.nlist[l][i], nx = T.nx[l], ny = T.ny[l], nz = T.nz[l];
  const int x = n % (nx + 1) - (a & 1), r = n / (nx + 1);
  const int y = r % (ny + 1) - ((a >> 1) & 1), z = r / (ny + 1) - (a >> 2);
  const bool in = x >= 0 && x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
  T.corner[l][(int64_t)a * T.nn[l] + i] = in ? T.eidx[l][x + nx * (y + ny * z)] : -1;
}

// ---- moments ---------------------------------------------------------------

// Level 2 from the 64 fine moduli, axis by axis; descendant position p along
// an axis has tau = 3 - 2 p.
__global__ void __launch_bounds__(64) k_moments2(int nx, int ny, int nz, const double* __restrict__ E,
                                                 const uint8_t* __restrict__ zero,
                                                 double* __restrict__ mom) {
  const int ne = nx * ny * nz;
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= ne) return;
  const int x = e % nx, r = e / nx, y = r % ny, z = r / ny;
  const int64_t sy = 4 * nx, sz = sy * 4 * ny;
  const double* p = E + 4 * x + sy * (4 * y) + sz * (4 * z);
  double v[16][4];
#pragma unroll
  for (int q = 0; q < 16; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) v[q][t] = p[t + sy * (q & 3) + sz * (q >> 2)];
  double m[27];
#pragma unroll
  for (int a = 0; a < 27; ++a) m[a] = 0.0;
#pragma unroll
  for (int dz = 0; dz < 4; ++dz) {
    double yz[3][3] = {};  // [a][b] of one z layer
#pragma unroll
    for (int dy = 0; dy < 4; ++dy) {
      const double* q = v[dy + 4 * dz];
      const double s03 = q[0] + q[3], s12 = q[1] + q[2];
      const double x0 = s03 + s12, x1 = fma(3.0, q[0] - q[3], q[1] - q[2]), x2 = fma(9.0, s03, s12);
      const double ty = 3.0 - 2.0 * dy;
      const double xa[3] = {x0, x1, x2};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        yz[a][0] += xa[a];
        yz[a][1] = fma(ty, xa[a], yz[a][1]);
        yz[a][2] = fma(ty * ty, xa[a], yz[a][2]);
      }
    }
    const double tz = 3.0 - 2.0 * dz;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        m[a + 3 * b] += yz[a][b];
        m[a + 3 * b + 9] = fma(tz, yz[a][b], m[a + 3 * b + 9]);
        m[a + 3 * b + 18] = fma(tz * tz, yz[a][b], m[a + 3 * b + 18]);
      }
  }
  const bool none = zero && zero[e];  // a flagged element of a level that may be split
#pragma unroll
  for (int a = 0; a < 27; ++a) mom[(int64_t)a * ne + e] = none ? 0.0 : m[a];
}

// The fine moduli with those of flagged level-1 elements 0, for a split level 1.
__global__ void __launch_bounds__(256) k_split_moduli(int nx, int ny, int64_t ne,
                                                      const double* __restrict__ E,
                                                      const uint8_t* __restrict__ eflag,
                                                      const int* __restrict__ split,
                                                      double* __restrict__ Es) {
  if (!*split) return;
  const uint32_t e = blockIdx.x * 256 + threadIdx.x;
  if (e >= ne) return;
  const uint32_t r = e / (2 * nx), x = e - r * (2 * nx), z = r / (2 * ny), y = r - z * (2 * ny);
  const double v = E[e];
  Es[e] = eflag[(x >> 1) + nx * ((y >> 1) + ny * (z >> 1))] ? 0.0 : v;
}

// Level l >= 3 from level l - 1, eight lanes per element, one per child: the
// child's moments about the parent's centre (shift = +-2^(l-1) per axis), summed
// over the children in a fixed order.
__global__ void __launch_bounds__(256) k_moments_up(int nx, int ny, int nz, double shift,
                                                    const double* __restrict__ child,
                                                    const uint8_t* __restrict__ zero,
                                                    double* __restrict__ mom) {
  const int ne = nx * ny * nz;
  const int t = blockIdx.x * 256 + threadIdx.x, e = t >> 3, c = t & 7;
  const bool live = e < ne;
  const int x = e % nx, r = e / nx, y = r % ny, z = r / ny;
  const int64_t cne = 8 * (int64_t)ne;
  const int64_t ce = 2 * x + (c & 1) + (int64_t)(2 * nx) * (2 * y + ((c >> 1) & 1) + (int64_t)(2 * ny) * (2 * z + (c >> 2)));
  double m[3][3][3];  // [z][y][x]
#pragma unroll
  for (int a = 0; a < 27; ++a) m[a / 9][(a / 3) % 3][a % 3] = live ? child[a * cne + ce] : 0.0;
  const double sx = (c & 1) ? -shift : shift, sy = (c & 2) ? -shift : shift, sz = (c & 4) ? -shift : shift;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      m[a][b][2] = fma(sx * sx, m[a][b][0], fma(2.0 * sx, m[a][b][1], m[a][b][2]));
      m[a][b][1] = fma(sx, m[a][b][0], m[a][b][1]);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      m[a][2][b] = fma(sy * sy, m[a][0][b], fma(2.0 * sy, m[a][1][b], m[a][2][b]));
      m[a][1][b] = fma(sy, m[a][0][b], m[a][1][b]);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      m[2][a][b] = fma(sz * sz, m[0][a][b], fma(2.0 * sz, m[1][a][b], m[2][a][b]));
      m[1][a][b] = fma(sz, m[0][a][b], m[1][a][b]);
    }
  const bool none = live && zero && zero[e];  // as on level 2 (a parent of it is flagged too)
#pragma unroll
  for (int a = 0; a < 27; ++a) {
    double s = m[a / 9][(a / 3) % 3][a % 3];
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 4, 64);
    if (live && c == (a & 7)) mom[(int64_t)a * ne + e] = none ? 0.0 : s;
  }
}

// ---- stored matrices -------------------------------------------------------

// Row and column of packed entry s (upper triangle, row-major, 24 x 24).
__device__ inline void sym_unpack(int s, int& r, int& q) {
  int a = (int)((49.0f - sqrtf((float)(2401 - 8 * s))) * 0.5f);
  if (a < 23 && sidx(a + 1, a + 1) <= s) ++a;
  if (sidx(a, a) > s) --a;
  r = a;
  q = a + (s - sidx(a, a));
}

// In-place 8-point Walsh transform.
__device__ inline void wht8(double (&x)[8]) {
#pragma unroll
  for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
    for (int a = 0; a < 8; ++a)
      if (!(a & bit)) {
        const double p = x[a], q = x[a | bit];
        x[a] = p + q;
        x[a | bit] = p - q;
      }
}

__device__ inline Moments8<double> load_moments8(const double* E, int x, int y, int z, int nx, int ny) {
  Moments8<double> M;
  const int64_t sy = 2 * nx, sz = sy * 2 * ny;
  const double* p = E + 2 * x + sy * (2 * y) + sz * (2 * z);
#pragma unroll
  for (int c = 0; c < 8; ++c) M.m[c] = p[(c & 1) + sy * ((c >> 1) & 1) + sz * (c >> 2)];
  wht8(M.m);
  return M;
}

__device__ inline Moments27<double> load_moments27(const double* mom, int64_t ne, int64_t e) {
  Moments27<double> M;
#pragma unroll
  for (int a = 0; a < 27; ++a) M.m[a] = mom[a * ne + e];
  return M;
}

// Matrices of the listed elements of level l, one workgroup of 8 x 24 threads
// each: thread (child c, column) interpolates the column's unit vector to the
// child's corners, applies the child and restricts the result; the eight
// children are summed in order.  A child is, on level 1 (LV 1), a fine element
// with the fixed DOFs removed on both sides; on level 2 (LV 2) a stored level-1
// matrix or the moduli of an unflagged one; below (LV 3) a stored matrix or
// moments.  The stored children go through LDS.
template <int LV>
__global__ void __launch_bounds__(192, 2) k_store(int nx, int ny, int nz, double gam, WalshConsts K,
                                               const double* __restrict__ E,
                                               const uint8_t* __restrict__ mask,
                                               const double* __restrict__ mom_c,
                                               const double* __restrict__ Kst_c,
                                               const int* __restrict__ eidx_c,
                                               const int* __restrict__ list,
                                               const int* __restrict__ count,
                                               double* __restrict__ Kst) {
  __shared__ double sK[8][24][25];
  __shared__ int sw[8];  // the children's places among the stored elements of level l - 1
  const int ch = threadIdx.x / 24, col = threadIdx.x % 24, A = col / 3, s = col % 3;
  const int dx = ch & 1, dy = (ch >> 1) & 1, dz = ch >> 2;
  const int n = *count;
  const int64_t ne = (int64_t)nx * ny * nz, cne = 8 * ne;
  // interpolation of the column's unit vector to the child's low and high
  // corner along each axis
  const double wx[2] = {phi1(dx, A & 1), phi1(dx + 1, A & 1)};
  const double wy[2] = {phi1(dy, (A >> 1) & 1), phi1(dy + 1, (A >> 1) & 1)};
  const double wz[2] = {phi1(dz, A >> 2), phi1(dz + 1, A >> 2)};
  for (int w = blockIdx.x; w < n; w += gridDim.x) {  // uniform
    const int e = list[w];
    const int x = e % nx, r = e / nx, y = r % ny, z = r / ny;
    const int cx = 2 * x + dx, cy = 2 * y + dy, cz = 2 * z + dz;
    const int64_t ce = cx + (int64_t)(2 * nx) * (cy + (int64_t)(2 * ny) * cz);
    double yc[24];
    if (LV > 1) {  // the stored children into LDS
      if (col == 0) sw[ch] = eidx_c[ce];
      __syncthreads();
      for (int t = threadIdx.x; t < 8 * kSymEntries; t += 192) {
        const int c = t / kSymEntries, q = t % kSymEntries;
        if (sw[c] < 0) continue;
        int a, b;
        sym_unpack(q, a, b);
        const double k = Kst_c[(int64_t)q * cne + sw[c]];
        sK[c][a][b] = k;
        sK[c][b][a] = k;
      }
      __syncthreads();
    }
    if (LV > 1 && sw[ch] >= 0) {
#pragma unroll
      for (int q = 0; q < 24; ++q) {
        double acc = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b)
          acc = fma(sK[ch][q][3 * b + s], wx[b & 1] * wy[(b >> 1) & 1] * wz[b >> 2], acc);
        yc[q] = acc;
        if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // few reads in flight, few registers
      }
    } else {
      double h[8][3], zz[8][3], sc[8], v[8];
      unsigned fixed = 0;  // bit 3 b + c: component c of the child's corner b
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        v[b] = wx[b & 1] * wy[(b >> 1) & 1] * wz[b >> 2];
        if (LV == 1) {
          const unsigned m = mask[cx + (b & 1) + (int64_t)(2 * nx + 1) * (cy + ((b >> 1) & 1) + (int64_t)(2 * ny + 1) * (cz + (b >> 2)))];
          fixed |= (m & 7u) << (3 * b);
          if ((m >> s) & 1) v[b] = 0.0;
        }
      }
      const double gc = LV == 1 ? 1.0 : 2.0 * gam;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        sc[k] = __popc(k) == 0 ? 1.0 : __popc(k) == 1 ? gc : __popc(k) == 2 ? gc * gc : gc * gc * gc;
      wht8(v);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) h[k][c] = c == s ? sc[k] * v[k] : 0.0;
      if (LV == 1)
        walsh_blocks<double>(K, E[ce], h, zz);
      else if (LV == 2)
        moment_apply(K, load_moments8(E, cx, cy, cz, 2 * nx, 2 * ny), h, zz);
      else
        moment_apply(K, load_moments27(mom_c, cne, ce), h, zz);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) t[k] = sc[k] * zz[k][c];
        wht8(t);
#pragma unroll
        for (int a = 0; a < 8; ++a) yc[3 * a + c] = (LV == 1 && ((fixed >> (3 * a + c)) & 1)) ? 0.0 : t[a];
      }
    }
    // restriction, axis by axis: (lo, hi) <- (lo + hi / 2, hi / 2) for a child
    // on the low side, (lo / 2, lo / 2 + hi) on the high one
#pragma unroll
    for (int axis = 0; axis < 3; ++axis) {
      const bool hi_side = axis == 0 ? dx : axis == 1 ? dy : dz;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        if (b & (1 << axis)) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          double& lo = yc[3 * b + c];
          double& hi = yc[3 * (b | (1 << axis)) + c];
          const double half = 0.5 * (hi_side ? lo : hi);
          const double l2 = hi_side ? half : lo + half, h2 = hi_side ? half + hi : half;
          lo = l2;
          hi = h2;
        }
      }
    }
    __syncthreads();  // the children are read
#pragma unroll
    for (int q = 0; q < 24; ++q) sK[ch][q][col] = yc[q];
    __syncthreads();
    for (int t = threadIdx.x; t < 576; t += 192) {
      const int q = t / 24, c = t % 24;
      if (q > c) continue;
      double acc = sK[0][q][c];
#pragma unroll
      for (int k = 1; k < 8; ++k) acc += sK[k][q][c];
      Kst[(int64_t)sidx(q, c) * ne + w] = acc;
    }
    __syncthreads();  // sK and sw are reused
  }
}

// ---- Jacobi diagonals ------------------------------------------------------

// Inverse Jacobi diagonal of level l >= 1.  Flagged elements: the stored
// diagonal.  Others: for a unit vector at corner a, component c, the Walsh
// coefficient k on a descendant is n^-|k| prod over the axes outside k of
// (1 + sigma t), so the entry is sum_k B_kk n^-2|k| F_k with F_k the moments
// contracted with (1, 2 sigma, 1) along those axes and (1, 0, 0) along k's.
// Eight threads per node, one per corner, the corners' shares added in order
// (one thread per node took the eight elements one after another: 96x48x48 13.2
// -> 4.8 us a level, 256x128x128 19.4 -> 13.2 us).
constexpr int kDiagNodes = 32;
__global__ void __launch_bounds__(8 * kDiagNodes) k_diag_level(
    int l, int nx, int ny, int nz, double gam, WalshConsts K, const double* __restrict__ E,
    const double* __restrict__ mom, const double* __restrict__ Kst,
    const uint8_t* __restrict__ eflag, const int* __restrict__ eidx, double* __restrict__ dinv,
    float* __restrict__ dinv32) {
  const int nxp = nx + 1, nyp = ny + 1, nn = nxp * nyp * (nz + 1);
  __shared__ double part[8][3][kDiagNodes];
  const int lane = threadIdx.x % kDiagNodes, a = threadIdx.x / kDiagNodes;
  const int first = blockIdx.x * kDiagNodes, n = min(first + lane, nn - 1);
  const int64_t ne = (int64_t)nx * ny * nz;
  const int i = n % nxp, r = n / nxp, j = r % nyp, k = r / nyp;
  double d[3] = {0.0, 0.0, 0.0};
  const double ga = K.a1mb1 + K.b1, ga4 = K.a4mb4 + K.b4;
  const double g2 = gam * gam, g4 = g2 * g2, g6 = g4 * g2;
  const int ex = i - (a & 1), ey = j - ((a >> 1) & 1), ez = k - (a >> 2);
  const bool in = ex >= 0 && ex < nx && ey >= 0 && ey < ny && ez >= 0 && ez < nz;
  const int64_t e = in ? ex + (int64_t)nx * (ey + (int64_t)ny * ez) : 0;
  if (in && eflag[e]) {
    const int64_t w = eidx[e];
    for (int c = 0; c < 3; ++c) d[c] = Kst[(int64_t)sidx(3 * a + c, 3 * a + c) * ne + w];
  } else if (in) {
    const double sx = (a & 1) ? -2.0 * gam : 2.0 * gam, sy = (a & 2) ? -2.0 * gam : 2.0 * gam,
                 sz = (a & 4) ? -2.0 * gam : 2.0 * gam;
    // P[axis set kept as derivative][remaining]: contract x, then y, then z
    double X[2][9];
    if (l == 1) {
      const Moments8<double> M = load_moments8(E, ex, ey, ez, nx, ny);
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int b = q % 3, c = q / 3;
        X[1][q] = M(0, b, c);
        X[0][q] = fma(sx, M(1, b, c), fma(g2, M(2, b, c), M(0, b, c)));
      }
    } else {
      const Moments27<double> M = load_moments27(mom, ne, e);
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int b = q % 3, c = q / 3;
        X[1][q] = M(0, b, c);
        X[0][q] = fma(sx, M(1, b, c), fma(g2, M(2, b, c), M(0, b, c)));
      }
    }
    double F[8];  // by axis set k
#pragma unroll
    for (int kx = 0; kx < 2; ++kx) {
      double Y[2][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Y[1][c] = X[kx][3 * c];
        Y[0][c] = fma(sy, X[kx][3 * c + 1], fma(g2, X[kx][3 * c + 2], X[kx][3 * c]));
      }
#pragma unroll
      for (int ky = 0; ky < 2; ++ky) {
        F[kx + 2 * ky + 4] = Y[ky][0];
        F[kx + 2 * ky] = fma(sz, Y[ky][1], fma(g2, Y[ky][2], Y[ky][0]));
      }
    }
    const double f1 = g2 * F[1], f2 = g2 * F[2], f4 = g2 * F[4], f3 = g4 * F[3], f5 = g4 * F[5],
                 f6 = g4 * F[6], f7 = K.h * g6 * F[7];
    d[0] = ga * f1 + K.g * (f2 + f4) + K.d * (f3 + f5) + ga4 * f6 + f7;
    d[1] = ga * f2 + K.g * (f1 + f4) + K.d * (f3 + f6) + ga4 * f5 + f7;
    d[2] = ga * f4 + K.g * (f1 + f2) + K.d * (f5 + f6) + ga4 * f3 + f7;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) part[a][c][lane] = d[c];
  __syncthreads();
  if (a < 3 && first + lane < nn) {  // component a
    double sum = part[0][a][lane];
#pragma unroll
    for (int q = 1; q < 8; ++q) sum += part[q][a][lane];
    const double di = sum == 0.0 ? 1.0 : 1.0 / sum;  // dead coarse DOF: identity row
    dinv[(int64_t)a * nn + n] = di;
    if (dinv32) dinv32[(int64_t)a * nn + n] = (float)di;
  }
}

// ---- the product -----------------------------------------------------------

template <int CTRL>
__device__ inline double lane_shift(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
constexpr int kShl1 = 0x130, kShr1 = 0x138;  // lane i <- lane i + 1, lane i - 1

constexpr uint32_t kOutside = 0x80000000u;  // see the fine-grid product
__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ inline void ld(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff, double& x) {
  x = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)soff, 0));
}
__device__ inline void st(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff, double x) {
  __builtin_amdgcn_raw_buffer_store_b64(
      __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), x), r, (int)off,
      (int)soff, 0);
}
constexpr int kLanes = 32;
// x-rows of a workgroup, two per wavefront.  Sixteen (one workgroup a CU) measured
// slower on every level: 256x128x128 level 1 48 / 44 us against 43 / 40, level 2
// 18 / 15 against 19 / 17 but level 3 14 / 11 against 9 / 7; 96x48x48 level 1 11
// to 12 against 8.
constexpr int kRows = 8;
// Lanes of an x-row on levels of up to kNarrow elements along x, where 32-lane
// rows would hold at most 12 nodes: a tile is then one wavefront of eight 8-lane
// rows, and the four wavefronts of a workgroup take four tiles (or chunks), each
// for itself.  Thin grids have many planes for few columns: wide tiles left nearly
// all lanes idle and, with one chunk a workgroup, gave a chunk several layers
// (16x16x8192 with a single support, levels 1 to 3: 49.2, 21.8 and 15.6 us with
// wide tiles, 28.1, 12.2 and 8.9 us so; 64x64x64's 8x8x8 level the same either way).
constexpr int kNarrowLanes = 8, kNarrow = 11;

// Slot of workgroup w of `total` in XCD-contiguous order (see kernels_mg.hip).
__device__ __forceinline__ int xcd_slot(int w, int total) {
  const int xcd = w & 7, pos = w >> 3, q = total >> 3, r = total & 7;
  return (xcd < r) ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
}

// Special nodes from the stored matrices, eight threads per node: thread
// (corner a, node) takes the node as corner a of its element and forms the
// node's three rows; the eight partial rows are summed in LDS in a fixed order.
// One corner a thread keeps the chain short (node and matrix index, then all
// operands at once, 72 matrix entries in flight): it sets the time of the small
// levels' launches.
template <int MODE, int NODES, bool ADD>
__device__ __forceinline__ void special_nodes(const LevelArgs& L, const double* v, double* y,
                                              const double* jb, const double* jd, double omega,
                                              int blk, double* lds) {
  double (*red)[3][NODES] = reinterpret_cast<double (*)[3][NODES]>(lds);
  const int lane = threadIdx.x % NODES, a = threadIdx.x / NODES;
  const int nx = L.nx, ny = L.ny, nz = L.nz, nxp = nx + 1, nyp = ny + 1, nn = nxp * nyp * (nz + 1);
  const int64_t ne = (int64_t)nx * ny * nz;
  int total = L.count ? *L.count : L.nspecial;
  if (L.gate && (*L.gate != 0) != ADD) total = 0;  // the other form's launch
  const int nb = (total + NODES - 1) / NODES;
  if (blk >= nb) return;  // workgroup-uniform
  const int idx = xcd_slot(blk, nb) * NODES + lane;
  const bool live = idx < total;
  const int n = live ? L.nlist[idx] : 0;
  const int64_t w = live ? L.corner[(int64_t)a * nn + idx] : -1;
  double acc[3] = {0.0, 0.0, 0.0};
  if (w >= 0) {
    const int n0 = n - (a & 1) - nxp * ((a >> 1) & 1) - nxp * nyp * (a >> 2);
    const double* K = L.Kst + w;
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double x = v[c * nn + n0 + (b & 1) + nxp * ((b >> 1) & 1) + nxp * nyp * (b >> 2)];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const int r = 3 * a + q, col = 3 * b + c, lo = min(r, col), hi = max(r, col);
          acc[q] = fma(K[(lo * 24 - (lo * (lo - 1)) / 2 + hi - lo) * ne], x, acc[q]);
        }
      }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) red[a][q][lane] = acc[q];
  __syncthreads();
  const int q = threadIdx.x / NODES;
  if (q < 3 && live) {
    double sum = red[0][q][lane];
#pragma unroll
    for (int t = 1; t < 8; ++t) sum += red[t][q][lane];
    const int d = q * nn + n;
    if (ADD)
      y[d] = MODE == 0 ? y[d] + sum : MODE == 1 ? fma(-omega * jd[d], sum, y[d]) : y[d] - sum;
    else
      y[d] = MODE == 0 ? sum : MODE == 1 ? v[d] + omega * jd[d] * (jb[d] - sum) : jb[d] - sum;
  }
}

// On a split level: what the flagged elements add to the marched product.
template <int MODE>
__global__ void __launch_bounds__(256) k_level_add(LevelArgs L, const double* __restrict__ v,
                                                   double* __restrict__ y,
                                                   const double* __restrict__ jd, double omega) {
  __shared__ double red[8 * 3 * 32];
  special_nodes<MODE, 32, true>(L, v, y, nullptr, jd, omega, (int)blockIdx.x, red);
}

// y = A_l v (MODE 0), v + omega jd (jb - A_l v) (MODE 1, a damped-Jacobi sweep)
// or jb - A_l v (MODE 2, the residual) on level l >= 1; y distinct from v.
// The tiles, the march along z, the exchanges between neighbouring columns and
// the out-of-range rule are those of the fine-grid product (k_ebe_z); the
// element operator is moment_apply with the 8 child moduli (LV1) or 27 stored
// moments.  FP64, one load case (the refinement form's FP32 products:
// kernels_l32.hip).  The first gridDim.x - nmarch workgroups take special nodes
// instead; SPLIT: there are none, and every node is marched.
template <bool LV1, int MODE, int LANES, bool SPLIT>
__global__ void __launch_bounds__(kLanes * kRows, 2) k_level_z(
    LevelArgs L, int gx, int gy, int ntile, int TZ, int nmarch, WalshConsts K, const double* __restrict__ E,
    const double* __restrict__ v, double* __restrict__ y, const double* __restrict__ jb,
    const double* __restrict__ jd, double omega) {
  constexpr int kTileX = LANES - 2, kTileY = kRows - 1;
  constexpr int kSub = kLanes / LANES, kTile = LANES * kRows;  // tiles of a workgroup, their threads
  __shared__ double xs[2 * 3 * kRows * kLanes];  // special nodes: 8 x 3 x 4 kRows of it
  const int nsp = SPLIT ? 0 : (int)gridDim.x - nmarch;
  if (!SPLIT && (int)blockIdx.x < nsp) {
    special_nodes<MODE, 4 * kRows, false>(L, v, y, jb, jd, omega, (int)blockIdx.x, xs);
    return;
  }
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  const double gam = L.gam;
  const int sub = kSub > 1 ? (int)threadIdx.x / kTile : 0;
  const int tx = threadIdx.x & (LANES - 1), ty = (int)threadIdx.x % kTile / LANES;
  int bx, by, bz;
  {  // XCD-contiguous tile order
    const int t = kSub * xcd_slot((int)blockIdx.x - nsp, nmarch) + sub;
    if (kSub > 1 && t >= ntile) return;  // a whole wavefront: no barrier below waits for it
    bx = t % gx;
    by = (t / gx) % gy;
    bz = t / (gx * gy);
  }
  const int i = bx * kTileX - 1 + tx, j = by * kTileY - 1 + ty;
  const int kz0 = bz * TZ, kz1 = min(kz0 + TZ, nz + 1);
  const int nxp = nx + 1, nyp = ny + 1, plane = nxp * nyp, nn = plane * (nz + 1), ne = nx * ny * nz;
  const uint32_t TS = 8u, cstride = (uint32_t)nn * TS;
  const auto rv = make_rsrc(v, 3u * cstride);
  const auto ry = make_rsrc(y, 3u * cstride);
  const auto rjb = make_rsrc(jb, MODE != 0 ? 3u * cstride : 0u);
  const auto rjd = make_rsrc(jd, MODE == 1 ? 3u * cstride : 0u);
  const auto rsp = make_rsrc(L.special, (uint32_t)nn);
  const auto rE = make_rsrc(E, LV1 ? 8u * ne * TS : 0u);
  const auto rM = make_rsrc(L.mom, LV1 || !L.mom ? 0u : 27u * ne * 8u);
  const bool col_ok = tx < LANES - 1 && i >= 0 && i < nx && j >= 0 && j < ny;
  const bool xi_ok = i >= 0 && i <= nx, yj_ok = j >= 0 && j <= ny, yj1_ok = j + 1 >= 0 && j + 1 <= ny;
  const bool own = tx >= 1 && tx < LANES - 1 && ty >= 1 && i <= nx && j <= ny;
  const int off00 = i + nxp * j;

  double q0[3], q2[3];
  auto load_plane = [&](int k) {
    const bool kin = k >= 0 && k <= nz;
    const uint32_t o0 = kin && xi_ok && yj_ok ? (uint32_t)(k * plane + off00) * TS : kOutside;
    const uint32_t o2 = kin && xi_ok && yj1_ok ? (uint32_t)(k * plane + off00 + nxp) * TS : kOutside;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      ld(rv, o0, (uint32_t)c * cstride, q0[c]);
      ld(rv, o2, (uint32_t)c * cstride, q2[c]);
    }
  };
  // x-y Walsh transform of the loaded plane, scaled by gam per axis
  auto transform = [&](double (&P)[4][3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double a0 = q0[c], a2 = q2[c];
      const double ye = a0 + a2, yo = gam * (a0 - a2);
      const double ye1 = lane_shift<kShl1>(ye), yo1 = lane_shift<kShl1>(yo);
      P[0][c] = ye + ye1;
      P[1][c] = gam * (ye - ye1);
      P[2][c] = yo + yo1;
      P[3][c] = gam * (yo - yo1);
    }
  };
  typename std::conditional<LV1, Moments8<double>, Moments27<double>>::type M;
  auto load_moments = [&](int k) {
    const bool ok = col_ok && k >= 0 && k < nz;
    if constexpr (LV1) {
      const int fx = 2 * nx;
      const uint32_t sy = (uint32_t)fx * TS, sz = sy * 2u * ny;
      const uint32_t o = ok ? ((uint32_t)(2 * k) * (2 * ny) * fx + (uint32_t)(2 * j) * fx + 2 * i) * TS : kOutside;
#pragma unroll
      for (int c = 0; c < 8; ++c)
        ld(rE, o + (c & 1) * TS, (c & 2 ? sy : 0u) + (c & 4 ? sz : 0u), M.m[c]);
    } else {
      const uint32_t o = ok ? (uint32_t)(i + nx * j + nx * ny * k) * 8u : kOutside;
#pragma unroll
      for (int a = 0; a < 27; ++a) ld(rM, o, (uint32_t)a * ((uint32_t)ne * 8u), M.m[a]);
    }
  };

  // The form that the device chose.  Asked here, not first: a branch on one
  // argument holds back the loads of the others (0.8 us of a 7.7 us launch, on
  // 96x48x48's levels).
  if (L.gate && (*L.gate != 0) != SPLIT) return;
  double P[4][3], carry[4][3];
  load_plane(kz0 - 1);
  load_moments(kz0 - 1);
  transform(P);
  load_plane(kz0);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < 3; ++c) carry[q][c] = 0;
  double own_v[3] = {0, 0, 0};
  int buf = 0;
#pragma unroll 1
  for (int k = kz0 - 1; k < kz1; ++k) {
    double Pt[4][3];
    double v_next[3];
    transform(Pt);
    if (MODE == 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) v_next[c] = q0[c];
    }
    load_plane(k + 2 <= kz1 ? k + 2 : -2);
    // plane k's own values; the first layer of a chunk only primes the carry
    const bool wr = own && k >= kz0;
    const uint32_t on = wr ? (uint32_t)(k * plane + off00) : kOutside;
    const uint32_t sp = SPLIT ? 0 : __builtin_amdgcn_raw_buffer_load_b8(rsp, (int)on, 0, 0);
    double ob[3], od[3];
    if (MODE != 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) ld(rjb, wr ? on * TS : kOutside, (uint32_t)c * cstride, ob[c]);
    }
    if (MODE == 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) ld(rjd, wr ? on * TS : kOutside, (uint32_t)c * cstride, od[c]);
    }
    double h[8][3], z[8][3];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        h[q][c] = P[q][c] + Pt[q][c];
        h[q + 4][c] = gam * (P[q][c] - Pt[q][c]);
        P[q][c] = Pt[q][c];
      }
    if constexpr (LV1) {
      Moments8<double> W = M;
#pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (!(c & bit)) {
            const double p0 = W.m[c], r0 = W.m[c | bit];
            W.m[c] = p0 + r0;
            W.m[c | bit] = p0 - r0;
          }
      load_moments(k + 1 < kz1 ? k + 1 : -1);
      moment_apply(K, W, h, z);
    } else {
      moment_apply(K, M, h, z);
      load_moments(k + 1 < kz1 ? k + 1 : -1);
    }
    // as in the fine-grid product, with the outputs' scaling by gam per axis
    double X0[3];
    double (*xb)[kRows][LANES] =
        reinterpret_cast<double (*)[kRows][LANES]>(xs + (2 * sub + buf) * 3 * kTile);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      using std::fma;
      const double a0 = carry[0][c] + fma(gam, z[4][c], z[0][c]);
      const double a1 = carry[1][c] + fma(gam, z[5][c], z[1][c]);
      const double a2 = carry[2][c] + fma(gam, z[6][c], z[2][c]);
      const double a3 = carry[3][c] + fma(gam, z[7][c], z[3][c]);
      carry[0][c] = fma(-gam, z[4][c], z[0][c]);
      carry[1][c] = fma(-gam, z[5][c], z[1][c]);
      carry[2][c] = fma(-gam, z[6][c], z[2][c]);
      carry[3][c] = fma(-gam, z[7][c], z[3][c]);
      const double u = fma(gam, a1, a0) + lane_shift<kShr1>(fma(-gam, a1, a0));
      const double w = gam * (fma(gam, a3, a2) + lane_shift<kShr1>(fma(-gam, a3, a2)));
      X0[c] = u + w;
      xb[c][ty][tx] = u - w;
    }
    if constexpr (kSub == 1) {
      __syncthreads();
    } else {  // one wavefront writes and reads: its LDS accesses stay in this order
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const uint32_t oy = wr && !sp ? on * TS : kOutside;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double out = (X0[c] + xb[c][ty > 0 ? ty - 1 : 0][tx]);
      if (MODE == 1) out = own_v[c] + omega * od[c] * (ob[c] - out);
      if (MODE == 2) out = ob[c] - out;
      st(ry, oy, (uint32_t)c * cstride, out);
    }
    buf ^= 1;
    if (MODE == 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) own_v[c] = v_next[c];
    }
  }
}

template <bool LV1, int MODE, int LANES, bool SPLIT>
void level_march(const LevelArgs& L, const WalshConsts& K, const double* E, const double* v, double* y,
                 const double* jb, const double* jd, double omega, hipStream_t s) {
  // resident workgroups of this kernel on the device (thread-safe one-time init)
  static const int slots = [] {
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_level_z<LV1, MODE, LANES, SPLIT>,
                                                        kLanes * kRows, 0);
    return (cus > 0 && per_cu > 0) ? cus * per_cu : 256;
  }();
  constexpr int kSub = kLanes / LANES;
  const int gx = (L.nx + 1 + LANES - 3) / (LANES - 2), gy = (L.ny + 1 + kRows - 2) / (kRows - 1);
  const int planes = L.nz + 1;
  // a chunk of t planes is t + 1 layers, and the launch takes about
  // ceil(workgroups / slots) rounds of them
  const int64_t tiles = (int64_t)gx * gy;
  int tz = planes;
  int64_t best = -1;
  for_chunk_lengths(planes, 1, [&](int t) {
    const int64_t groups = (tiles * ((planes + t - 1) / t) + kSub - 1) / kSub;
    const int64_t cost = (groups + slots - 1) / slots * (t + 1);
    if (best < 0 || cost < best) {
      best = cost;
      tz = t;
    }
  });
  // the coarsest level is special as a whole and has no moments: nothing to march
  const bool whole = !SPLIT && !L.count && L.nspecial == (L.nx + 1) * (L.ny + 1) * (L.nz + 1);
  const int ntile = whole ? 0 : gx * gy * ((planes + tz - 1) / tz);
  const int nmarch = (ntile + kSub - 1) / kSub;
  const int nsp = (L.nspecial + 4 * kRows - 1) / (4 * kRows);
  k_level_z<LV1, MODE, LANES, SPLIT><<<(unsigned)(nmarch + (SPLIT ? 0 : nsp)), kLanes * kRows, 0, s>>>(
      L, gx, gy, ntile, tz, nmarch, K, E, v, y, jb, jd, omega);
  if (SPLIT && nsp > 0) k_level_add<MODE><<<(unsigned)nsp, 256, 0, s>>>(L, v, y, jd, omega);
}

template <bool LV1, int MODE, int LANES>
void level_form(const LevelArgs& L, const WalshConsts& K, const double* E, const double* v, double* y,
                const double* jb, const double* jd, double omega, hipStream_t s) {
  // both forms where only the device knows which one the lists are for
  if (L.gate || !L.split) level_march<LV1, MODE, LANES, false>(L, K, E, v, y, jb, jd, omega, s);
  if (L.gate || L.split)
    level_march<LV1, MODE, LANES, true>(L, K, LV1 ? L.Esplit : E, v, y, jb, jd, omega, s);
}

template <bool LV1, int MODE>
void level_launch(const LevelArgs& L, const WalshConsts& K, const double* E, const double* v,
                  double* y, const double* jb, const double* jd, double omega, hipStream_t s) {
  if (L.nx <= kNarrow)
    level_form<LV1, MODE, kNarrowLanes>(L, K, E, v, y, jb, jd, omega, s);
  else
    level_form<LV1, MODE, kLanes>(L, K, E, v, y, jb, jd, omega, s);
}

}  // namespace

bool level_may_split(int nx, int ny, int nz) { return (int64_t)nx * ny * nz >= kSplitLevel; }

int64_t level_list_blocks(const Grid* lg, int nlev) {
  int64_t nb = 0;
  for (int l = 1; l < nlev; ++l) nb += nblk(lg[l].ne, kChunk) + nblk(lg[l].nn, kChunk);
  return nb;
}

void launch_level_lists(const LevelTable& T, const uint8_t* mask, hipStream_t s) {
  k_flags1<<<nblk(T.ne[1], 256), 256, 0, s>>>(T.nx[1], T.ny[1], T.nz[1], mask, T.eflag[1]);
  int64_t deep = 0, nb = 0;
  for (int l = 1; l < T.nlev; ++l) {
    if (l > 1) deep += T.ne[l];
    nb += nblk(T.ne[l], kChunk) + nblk(T.nn[l], kChunk);
  }
  if (deep > 0) k_flags_deep<<<nblk(deep, 4), 256, 0, s>>>(T);
  k_lists<0><<<(unsigned)nb, 256, 0, s>>>(T);
  k_lists<1><<<(unsigned)nb, 256, 0, s>>>(T);
  int64_t nodes = 0;
  for (int l = 1; l < T.nlev; ++l) nodes += T.nn[l];
  k_corners<<<nblk(8 * nodes, 256), 256, 0, s>>>(T);
}

void launch_level_moments(const LevelTable& T, int level, const double* E, hipStream_t s) {
  const int nx = T.nx[level], ny = T.ny[level], nz = T.nz[level], ne = T.ne[level];
  const uint8_t* zero = level_may_split(nx, ny, nz) ? T.eflag[level] : nullptr;
  if (level == 2)
    k_moments2<<<nblk(ne, 64), 64, 0, s>>>(nx, ny, nz, E, zero, T.mom[2]);
  else
    k_moments_up<<<nblk(8 * (int64_t)ne, 256), 256, 0, s>>>(nx, ny, nz, (double)(1 << (level - 1)),
                                                            T.mom[level - 1], zero, T.mom[level]);
}

void launch_level_moduli(const LevelTable& T, const double* E, hipStream_t s) {
  if (!T.Esplit) return;
  const int64_t ne = 8 * (int64_t)T.ne[1];
  k_split_moduli<<<nblk(ne, 256), 256, 0, s>>>(T.nx[1], T.ny[1], ne, E, T.eflag[1],
                                               T.counts + kCountSplit + 1, T.Esplit);
}

void launch_level_store(const LevelTable& T, int level, const WalshConsts& K, const double* E,
                        const uint8_t* mask, hipStream_t s) {
  const int l = level, ne = T.ne[l];
  const unsigned grid = (unsigned)(ne < 2048 ? ne : 2048);
  auto kernel = l == 1 ? k_store<1> : l == 2 ? k_store<2> : k_store<3>;
  kernel<<<grid, 192, 0, s>>>(T.nx[l], T.ny[l], T.nz[l], 1.0 / (1 << l), K, E, mask, T.mom[l - 1],
                              T.Kst[l - 1], T.eidx[l - 1], T.elist[l], T.counts + 2 * l, T.Kst[l]);
}

void launch_level_diag(const LevelTable& T, int level, const WalshConsts& K, const double* E,
                       double* dinv, float* dinv32, hipStream_t s) {
  k_diag_level<<<nblk(T.nn[level], kDiagNodes), 8 * kDiagNodes, 0, s>>>(
      level, T.nx[level], T.ny[level], T.nz[level], 1.0 / (1 << level), K, E, T.mom[level],
      T.Kst[level], T.eflag[level], T.eidx[level], dinv, dinv32);
}

void launch_level_product(const LevelArgs& L, const WalshConsts& K, const double* E, int mode,
                          const double* v, double* y, const double* jb, const double* jd,
                          double omega, hipStream_t s) {
  if (L.level == 1) {
    if (mode == 0) level_launch<true, 0>(L, K, E, v, y, jb, jd, omega, s);
    else if (mode == 1) level_launch<true, 1>(L, K, E, v, y, jb, jd, omega, s);
    else level_launch<true, 2>(L, K, E, v, y, jb, jd, omega, s);
  } else {
    if (mode == 0) level_launch<false, 0>(L, K, E, v, y, jb, jd, omega, s);
    else if (mode == 1) level_launch<false, 1>(L, K, E, v, y, jb, jd, omega, s);
    else level_launch<false, 2>(L, K, E, v, y, jb, jd, omega, s);
  }
}

}  // namespace aarmr
