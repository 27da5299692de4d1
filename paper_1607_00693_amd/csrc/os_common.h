// Pieces shared by the oversampled Petrov-Galerkin kernels (Sec. 2.2 remark on
// oversampling): where a patch lies, and the recombination of a pair's Schur
// products into its 4 x 4 stiffness.
#pragma once
#include "band_rows.h"

namespace stomsfem {

struct OsRowsArgs {
  UpArgs up;
  int32_t o;
  // optional: solve only the pairs list[i], i < nlist, into S[i], status[i]
  const int64_t* list;
  int64_t nlist;
};

// first fine cell (one axis) of the patch of coarse element k
__device__ __forceinline__ int os_patch_origin(int k, int m, int o, int nf) {
  int x0 = k * m - o;
  if (x0 > nf - (m + 2 * o)) x0 = nf - (m + 2 * o);
  return x0 < 0 ? 0 : x0;
}

// The ten right-hand sides at the interior patch node (ix, iy) with element
// coefficients q4 (SW, SE, NW, NE): lifts f^0..2 = -(K p^j) on the patch, the
// unit vectors of K's corners, r^0..2 = K^K p^l (only the elements of K
// count).
__device__ __forceinline__ void os_right_hand_sides(const double* q4, int ix, int iy, int M, int m, int cx, int cy,
                                                    double* rhs) {
  const double rM = 1.0 / M, rm = 1.0 / m;
  const int px = ix + 1, py = iy + 1;
  double f[3];
  bilinear_load(q4[0], q4[1], q4[2], q4[3], (ix + 0.5) * rM, (iy + 0.5) * rM, rM, f);
#pragma unroll
  for (int l = 0; l < 3; ++l) rhs[l] = -f[l];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int kpx = cx + ((k == 1 || k == 2) ? m : 0), kpy = cy + (k >= 2 ? m : 0);
    rhs[3 + k] = (px == kpx && py == kpy) ? 1.0 : 0.0;
  }
  const bool w = px > cx && px <= cx + m, e = px >= cx && px < cx + m;
  const bool s = py > cy && py <= cy + m, n = py >= cy && py < cy + m;
  bilinear_load(w && s ? q4[0] : 0.0, e && s ? q4[1] : 0.0, w && n ? q4[2] : 0.0, e && n ? q4[3] : 0.0,
                (ix + 0.5 - cx) * rm, (iy + 0.5 - cy) * rm, rm, f);
#pragma unroll
  for (int l = 0; l < 3; ++l) rhs[7 + l] = f[l];
}

// Bilinear functions on a square: grad p^l = (GA[l] + GB[l] y, HA[l] + HB[l] x),
// twist GT[l], l = 0..2.
struct Bilinear {
  static __host__ __device__ constexpr double ga(int l) { return l == 0 ? -1.0 : l == 1 ? 1.0 : 0.0; }
  static __host__ __device__ constexpr double gb(int l) { return l == 1 ? -1.0 : 1.0; }
  static __host__ __device__ constexpr double ha(int l) { return l == 0 ? -1.0 : 0.0; }
  static __host__ __device__ constexpr double hb(int l) { return l == 1 ? -1.0 : 1.0; }
  static __host__ __device__ constexpr double tw(int l) { return l == 1 ? -1.0 : 1.0; }
};

// S[4][4] of one pair.  Patch of M cells, K = m x m cells from patch node
// (cx, cy).  mo: sums over K's elements of a, a x, a y, a x^2, a y^2 (element
// centres in K's coordinates).  G(jv, t): w^jv . t = f^jv . K_II^{-1} t for
// the patch lift jv and test t (corners of K 0..3, r^0..2 = K^K p^l 4..6).
// psi^j = p^j + w^j; Psi_kj = psi^j(x_k), A_jl = psi^j . K^K p^l,
// S = Psi^{-T} A.  Returns false when Psi is singular.
template <typename GF>
__device__ __forceinline__ bool os_recombine(int M, int m, int cx, int cy, const double* mo, GF&& G, double* out) {
  const double rM = 1.0 / M, rm = 1.0 / m;
  const double X0 = cx * rM, Y0 = cy * rM, rho = m * rM;
  double Psi[4][4], A[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int kpx = cx + ((k == 1 || k == 2) ? m : 0), kpy = cy + (k >= 2 ? m : 0);
    const bool onb = kpx == 0 || kpx == M || kpy == 0 || kpy == M;
    const double x = kpx * rM, y = kpy * rM;
    const double p[3] = {(1.0 - x) * (1.0 - y), x * (1.0 - y), x * y};
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Psi[k][j] = p[j] + (onb ? 0.0 : G(j, k));
      sum += Psi[k][j];
    }
    Psi[k][3] = 1.0 - sum;
  }
  const double s0 = mo[0], sx = mo[1], sy = mo[2], sxx = mo[3], syy = mo[4];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double ga = Bilinear::ga(j) + Bilinear::gb(j) * Y0, gb = Bilinear::gb(j) * rho;
    const double ha = Bilinear::ha(j) + Bilinear::hb(j) * X0, hb = Bilinear::hb(j) * rho;
    double rs = 0.0;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const double la = Bilinear::ga(l), lb = Bilinear::gb(l), ma = Bilinear::ha(l), mb = Bilinear::hb(l);
      const double e = (ga * la) * s0 + (ga * lb + gb * la) * sy + (gb * lb) * syy + (ha * ma) * s0 +
                       (ha * mb + hb * ma) * sx + (hb * mb) * sxx +
                       (Bilinear::tw(j) * Bilinear::tw(l)) * (s0 * rM * rm * (1.0 / 6.0));
      A[j][l] = e * (rM * rm) + G(j, 4 + l);
      rs += A[j][l];
    }
    A[j][3] = -rs;
  }
#pragma unroll
  for (int l = 0; l < 4; ++l) A[3][l] = -(A[0][l] + A[1][l] + A[2][l]);
  // C = (Psi^T)^{-1}: Gauss-Jordan with partial pivoting on [Psi^T | I]
  // (every index compile-time: the row interchange is a select per entry)
  double B[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < 8; ++c) B[i][c] = c < 4 ? Psi[c][i] : (c - 4 == i ? 1.0 : 0.0);
  bool sing = false;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int pr = c;
    double best = fabs(B[c][c]);
#pragma unroll
    for (int i = c + 1; i < 4; ++i)
      if (fabs(B[i][c]) > best) {
        best = fabs(B[i][c]);
        pr = i;
      }
#pragma unroll
    for (int i = c + 1; i < 4; ++i) {
      const bool sw = i == pr;
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) {
        const double t = B[c][cc];
        B[c][cc] = sw ? B[i][cc] : t;
        B[i][cc] = sw ? t : B[i][cc];
      }
    }
    sing = sing || !(fabs(B[c][c]) > 0.0);
    const double iv = 1.0 / B[c][c];
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) B[c][cc] *= iv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i == c) continue;
      const double f = B[i][c];
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) B[i][cc] -= f * B[c][cc];
    }
  }
#pragma unroll
  for (int l = 0; l < 4; ++l)
#pragma unroll
    for (int lp = 0; lp < 4; ++lp) {
      double v = 0.0;
#pragma unroll
      for (int j = 0; j < 4; ++j) v += B[l][4 + j] * A[j][lp];
      out[4 * l + lp] = v;
    }
  return !sing;
}

}  // namespace stomsfem
