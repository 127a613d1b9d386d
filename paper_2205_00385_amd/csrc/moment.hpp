// Galerkin operators of the coarse levels from moments of the fine moduli.
//
// A coarse element is a cube of n = 2^l fine elements (descendants) per axis.
// With one coordinate per axis that runs over the coarse element, +1 at its
// low corner and -1 at its high one, the trilinear interpolation is affine per
// axis, so in the Walsh basis of the corners (h_k, k a set of axes) the
// values on the descendant d centred at tau / n (tau: odd integers, |tau| < n,
// per axis) have the coefficients
//   g_k = sum_{j >= k} tau^{j \ k} hs_j,   hs_j = n^-|j| h_j.
// Its stiffness is E_d W^T B W with B the block pattern of walsh_blocks(), so
// the Galerkin matrix sum_d E_d P_d^T KE P_d depends on the moduli only
// through the 27 moments
//   M[a][b][c] = sum_d E_d tau_x^a tau_y^b tau_z^c,   a, b, c in {0, 1, 2}:
// every block of B contributes a polynomial in tau (the sum of the g's it
// couples), whose coefficients are multiplied by the moment (Hankel) matrix
// of its monomials.  287 multiply-adds with moments and about 150 other
// operations besides the transforms, against 576 multiply-adds with the 300
// stored entries of the matrix, and 27 numbers an element to read instead
// of 300.  On level 1 tau = +-1, tau^2 = 1, and the moments are the Walsh
// transform of the 8 child moduli.
#pragma once

#include "walsh.hpp"

namespace aarmr {

// Moments of an element on level >= 2, M[a + 3 b + 9 c].
template <typename T>
struct Moments27 {
  T m[27];
  __host__ __device__ T operator()(int a, int b, int c) const { return m[a + 3 * b + 9 * c]; }
};

// Moments of a level-1 element: the Walsh transform of its 8 child moduli.
template <typename T>
struct Moments8 {
  T m[8];
  __host__ __device__ T operator()(int a, int b, int c) const {
    return m[(a & 1) + 2 * (b & 1) + 4 * (c & 1)];
  }
};

// Exponents of the monomials 1, x, y, z, xy, xz, yz: two bits per axis, so
// that the sum of two is the exponent of their product.
enum : int { kOne = 0, kX = 1, kY = 4, kZ = 16, kXY = 5, kXZ = 17, kYZ = 20 };

// q_i = sum_j M(mono_i mono_j) s_j
template <typename T, typename MOM, int N>
__host__ __device__ inline void hankel(const MOM& M, const int (&mono)[N], const T (&s)[N], T (&q)[N]) {
  using std::fma;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T acc = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int e = mono[i] + mono[j];
      const T w = M(e & 3, (e >> 2) & 3, e >> 4);
      acc = j == 0 ? w * s[0] : fma(w, s[j], acc);
    }
    q[i] = acc;
  }
}

// z = sum_d E_d G_d^T B G_d h, h and z scaled by n^-|k| (the caller's part).
template <typename T, typename MOM>
__host__ __device__ inline void moment_apply(const WalshConsts& K, const MOM& M, const T (&h)[8][3],
                                             T (&z)[8][3]) {
  const T a1 = (T)K.a1mb1, b1 = (T)K.b1, g = (T)K.g, e = (T)K.e, dme = (T)(K.d - K.e), a4 = (T)K.a4mb4,
          b4 = (T)K.b4;
  z[0][0] = z[0][1] = z[0][2] = 0;
  {  // g_1x + g_2y + g_4z
    const int mono[7] = {kOne, kX, kY, kZ, kXY, kXZ, kYZ};
    const T s[7] = {b1 * (h[1][0] + h[2][1] + h[4][2]), b1 * (h[3][1] + h[5][2]),
                    b1 * (h[3][0] + h[6][2]),           b1 * (h[5][0] + h[6][1]),
                    b1 * h[7][2],                       b1 * h[7][1],
                    b1 * h[7][0]};
    T q[7];
    hankel(M, mono, s, q);
    z[1][0] = z[2][1] = z[4][2] = q[0];
    z[3][1] = z[5][2] = q[1];
    z[3][0] = z[6][2] = q[2];
    z[5][0] = z[6][1] = q[3];
    z[7][2] = q[4];
    z[7][1] = q[5];
    z[7][0] = q[6];
  }
  // a pair of one axis' own polynomial: (1, u, v, uv) over the other two axes
  auto own4 = [&](const int (&mono)[4], int k0, int k1, int k2, int c) {
    const T s[4] = {a1 * h[k0][c], a1 * h[k1][c], a1 * h[k2][c], a1 * h[7][c]};
    T q[4];
    hankel(M, mono, s, q);
    z[k0][c] += q[0];
    z[k1][c] += q[1];
    z[k2][c] += q[2];
    z[7][c] += q[3];
  };
  {
    const int mx[4] = {kOne, kY, kZ, kYZ}, my[4] = {kOne, kX, kZ, kXZ}, mz[4] = {kOne, kX, kY, kXY};
    own4(mx, 1, 3, 5, 0);
    own4(my, 2, 3, 6, 1);
    own4(mz, 4, 5, 6, 2);
  }
  {  // g_1y + g_2x
    const int mono[6] = {kOne, kX, kY, kZ, kXZ, kYZ};
    const T s[6] = {g * (h[1][1] + h[2][0]), g * h[3][0], g * h[3][1],
                    g * (h[5][1] + h[6][0]), g * h[7][0], g * h[7][1]};
    T q[6];
    hankel(M, mono, s, q);
    z[1][1] = q[0];
    z[2][0] = q[0];
    z[3][0] += q[1];
    z[3][1] += q[2];
    z[5][1] = q[3];
    z[6][0] = q[3];
    z[7][0] += q[4];
    z[7][1] += q[5];
  }
  {  // g_1z + g_4x
    const int mono[6] = {kOne, kX, kY, kZ, kXY, kYZ};
    const T s[6] = {g * (h[1][2] + h[4][0]), g * h[5][0], g * (h[3][2] + h[6][0]),
                    g * h[5][2],             g * h[7][0], g * h[7][2]};
    T q[6];
    hankel(M, mono, s, q);
    z[1][2] = q[0];
    z[4][0] = q[0];
    z[5][0] += q[1];
    z[3][2] = q[2];
    z[6][0] += q[2];
    z[5][2] += q[3];
    z[7][0] += q[4];
    z[7][2] += q[5];
  }
  {  // g_2z + g_4y
    const int mono[6] = {kOne, kX, kY, kZ, kXY, kXZ};
    const T s[6] = {g * (h[2][2] + h[4][1]), g * (h[3][2] + h[5][1]), g * h[6][1],
                    g * h[6][2],             g * h[7][1],             g * h[7][2]};
    T q[6];
    hankel(M, mono, s, q);
    z[2][2] = q[0];
    z[4][1] = q[0];
    z[3][2] += q[1];
    z[5][1] += q[1];
    z[6][1] += q[2];
    z[6][2] += q[3];
    z[7][1] += q[4];
    z[7][2] += q[5];
  }
  {  // g_3z + g_5y + g_6x
    const int mono[4] = {kOne, kX, kY, kZ};
    const T s[4] = {b4 * (h[3][2] + h[5][1] + h[6][0]), b4 * h[7][0], b4 * h[7][1], b4 * h[7][2]};
    T q[4];
    hankel(M, mono, s, q);
    z[3][2] += q[0];
    z[5][1] += q[0];
    z[6][0] += q[0];
    z[7][0] += q[1];
    z[7][1] += q[2];
    z[7][2] += q[3];
  }
  // a two-axis term's own polynomial (1, u) over the third axis
  auto own2 = [&](int mono1, int k, int c, T w) {
    const int mono[2] = {kOne, mono1};
    const T s[2] = {w * h[k][c], w * h[7][c]};
    T q[2];
    hankel(M, mono, s, q);
    z[k][c] += q[0];
    z[7][c] += q[1];
  };
  own2(kZ, 3, 2, a4);
  own2(kY, 5, 1, a4);
  own2(kX, 6, 0, a4);
  // pairs [[d, e], [e, d]]: e times the sum's polynomial, d - e times each own
  auto pair = [&](int m1, int k1, int c1, int m2, int k2, int c2) {
    const int mono[3] = {kOne, m1, m2};
    const T s[3] = {e * (h[k1][c1] + h[k2][c2]), e * h[7][c1], e * h[7][c2]};
    T q[3];
    hankel(M, mono, s, q);
    z[k1][c1] += q[0];
    z[k2][c2] += q[0];
    z[7][c1] += q[1];
    z[7][c2] += q[2];
    own2(m1, k1, c1, dme);
    own2(m2, k2, c2, dme);
  };
  pair(kZ, 3, 0, kX, 6, 2);
  pair(kZ, 3, 1, kY, 5, 2);
  pair(kY, 5, 0, kX, 6, 1);
  const T eta = (T)K.h * M(0, 0, 0);
#pragma unroll
  for (int c = 0; c < 3; ++c) z[7][c] += eta * h[7][c];
}

}  // namespace aarmr
