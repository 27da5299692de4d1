// Offline stage of the reduced basis (rb.hip): from the snapshots phi of
// N_train coefficient samples to the modes and the element table of every
// patch.  With Psi the nI x ns matrix of centred snapshots (ns = 3 N_train,
// column c = 3 s + l) and E = K_II(abar) = L_E L_E^T, abar the training mean of
// the coefficient, the KL expansion in the energy inner product is
//   primal (ns >= nI): C = L_E^T Psi Psi^T L_E = V Lambda V^T,
//                      Z = L_E^{-T} V_r (so that Z^T E Z = I),
//   dual (ns < nI, the method of snapshots): C = Psi^T E Psi = V Lambda V^T
//                      (the same nonzero eigenvalues), z_q = Psi v_q / sqrt(lambda_q).
// Steps over all patches:
//   rb_means_kernel    abar and the snapshot means phibar
//   rb_energy_kernel   dual: W = E Psi
//   rb_gram_kernel     H = Psi Psi^T (primal) or C = Psi^T W (dual) in 64 x 64
//                      tiles, the primal sum over the snapshots in `parts` parts
//   rb_eigen_kernel    one workgroup per patch: C, its eigenpairs (pivoted
//                      Cholesky, then one-sided Jacobi), the tail rule for r,
//                      the modes Z
//   rb_table_kernel    the element table G
#include "rb.h"

namespace stomsfem {
namespace {

constexpr int RB_THREADS = 256;
constexpr int RB_NMAX = 1024;       // largest eigenproblem (primal nI or dual 3 ntrain)
constexpr int RB_EIGEN = 1024;      // most threads of the eigen kernel
constexpr double RB_RANK_TOL = 1e-12;
constexpr size_t RB_LDS = 160 * 1024 - 512;  // less the static variables
constexpr int RB_MANY = 256;        // patches that fill the GPU with a workgroup each
constexpr int RB_TABLE_BLOCKS = 8192;
constexpr int RB_TINY = 4;          // unknowns of the patches with their own Gram kernel

// Buffers of a build.  The eigenproblem has n = nI (primal) or ns (dual)
// unknowns.
struct RbWork {
  int ns, n, parts;
  double* abar;  // [M][m*m]
  double* W;     // dual: [M][ns][nI]
  double* C;     // [M][parts][n][n]
  double* L;     // primal: [M][nI][m + 1] Cholesky band where it does not fit LDS
};

// The eigen kernel holds its matrix in LDS up to this size (16 lanes take a
// column of at most 8 values each) and works in memory beyond.
constexpr int RB_LDS_N = 128;
inline int rb_lda(int n) { return n <= RB_LDS_N ? n | 1 : n; }
inline size_t rb_eigen_lds(bool dual, int m, int n, int rmax) {
  const size_t nI = (size_t)(m - 1) * (m - 1);
  size_t d = 4 * (size_t)n + 1 + n;  // diagonal (two), values, tails; pivots and order
  if (!dual) d += (n <= RB_LDS_N ? nI * (m + 1) : 0) + (size_t)rmax * nI;
  if (n <= RB_LDS_N) d += (size_t)n * rb_lda(n);
  return d * sizeof(double);
}

// Carve the buffers of a build out of work (NULL: sizes only); returns the
// doubles taken.
int64_t rb_work_layout(int ncx, int ncy, int m, int ntrain, double* work, RbWork* w) {
  const int64_t Mc = (int64_t)ncx * ncy, nI = (int64_t)(m - 1) * (m - 1);
  const bool dual = rb_dual(m, ntrain);
  RbWork d{};
  d.ns = 3 * ntrain;
  d.n = dual ? d.ns : (int)nI;
  // a patch has few tiles: where the patches are few too the snapshots are summed
  // in parts, which the eigen kernel adds as it fills LDS (in memory it works on
  // the sum in place)
  d.parts = dual || d.n > RB_LDS_N || d.n <= RB_TINY || Mc >= RB_MANY ? 1 : 3;
  int64_t off = 0;
  auto take = [&](int64_t count) {
    double* p = work ? work + off : nullptr;
    off += count;
    return p;
  };
  d.abar = take(Mc * m * m);
  if (dual) d.W = take(Mc * d.ns * nI);
  d.C = take(Mc * d.parts * d.n * d.n);
  if (!dual && d.n > RB_LDS_N) d.L = take(Mc * nI * (m + 1));
  if (w) *w = d;
  return off;
}

// Training means of the coefficient (abar, m*m values) and of the snapshots
// (phibar, 3 nI values): 32 values per workgroup, the samples in eight
// interleaved parts.
template <typename TA>
__global__ __launch_bounds__(RB_THREADS) void rb_means_kernel(RbBuildArgs b, RbWork d) {
  __shared__ double part[8][33];
  const int K = blockIdx.x, m = b.m, nI = (m - 1) * (m - 1), Mc = b.ncx * b.ncy;
  const int x = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int v = blockIdx.y * 32 + x, i = v - m * m;
  const int64_t lda = (int64_t)b.ncx * m;
  double acc = 0.0;
  if (v < m * m) {
    const int64_t at = (int64_t)((K / b.ncx) * m + v / m) * lda + (K % b.ncx) * m + v % m;
    for (int s = g; s < b.ntrain; s += 8) acc += ld((const TA*)b.a + (int64_t)s * (b.ncy * m) * lda, at);
  } else if (i < 3 * nI) {
    for (int s = g; s < b.ntrain; s += 8) acc += b.phi[((int64_t)s * Mc + K) * 3 * nI + i];
  }
  part[g][x] = acc;
  __syncthreads();
  if (g != 0) return;
#pragma unroll
  for (int k = 1; k < 8; ++k) acc += part[k][x];
  if (v < m * m)
    d.abar[(int64_t)K * m * m + v] = acc / b.ntrain;
  else if (i < 3 * nI)
    b.phibar[(int64_t)K * 3 * nI + i] = acc / b.ntrain;
}

// The 9-point row of K_II(abar) at interior node r: diagonal in ks[8]'s
// companion kc, the eight neighbour couplings ks[q] at offsets (dxs, dys).
struct Stencil9 {
  double kc, ks[8];
};
__device__ constexpr int RB_DX[8] = {-1, 1, 0, 0, -1, 1, -1, 1};
__device__ constexpr int RB_DY[8] = {0, 0, -1, 1, -1, -1, 1, 1};
__device__ __forceinline__ Stencil9 rb_stencil(const double* abar, int m, int ix, int iy) {
  const double aSW = abar[iy * m + ix], aSE = abar[iy * m + ix + 1];
  const double aNW = abar[(iy + 1) * m + ix], aNE = abar[(iy + 1) * m + ix + 1];
  Stencil9 st;
  st.kc = (2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE));
  st.ks[0] = -(aSW + aNW) / 6.0;
  st.ks[1] = -(aSE + aNE) / 6.0;
  st.ks[2] = -(aSW + aSE) / 6.0;
  st.ks[3] = -(aNW + aNE) / 6.0;
  st.ks[4] = -aSW / 3.0;
  st.ks[5] = -aSE / 3.0;
  st.ks[6] = -aNW / 3.0;
  st.ks[7] = -aNE / 3.0;
  return st;
}

__device__ __forceinline__ double rb_psi(const RbBuildArgs& b, int K, int c, int i, int nI) {
  const int s = c / 3, l = c - 3 * (c / 3);
  const int Mc = b.ncx * b.ncy;
  return b.phi[(((int64_t)s * Mc + K) * 3 + l) * nI + i] - b.phibar[((int64_t)K * 3 + l) * nI + i];
}

// W[c][i] = (E Psi)_{i c}: one thread per interior node i, all columns c.
__global__ __launch_bounds__(RB_THREADS) void rb_energy_kernel(RbBuildArgs b, RbWork d) {
  const int K = blockIdx.x, m = b.m, n = m - 1, nI = n * n;
  const int i = blockIdx.y * RB_THREADS + threadIdx.x;
  if (i >= nI) return;
  const int ix = i % n, iy = i / n, px = ix + 1, py = iy + 1;
  const Stencil9 st = rb_stencil(d.abar + (int64_t)K * m * m, m, ix, iy);
  int nb[8];
  for (int q = 0; q < 8; ++q) {
    const int qx = px + RB_DX[q], qy = py + RB_DY[q];
    nb[q] = (qx >= 1 && qx <= n && qy >= 1 && qy <= n) ? (qy - 1) * n + (qx - 1) : -1;
  }
  double* W = d.W + (int64_t)K * d.ns * nI;
  for (int c = 0; c < d.ns; ++c) {
    double v = st.kc * rb_psi(b, K, c, i, nI);
    for (int q = 0; q < 8; ++q)
      if (nb[q] >= 0) v += st.ks[q] * rb_psi(b, K, c, nb[q], nI);
    W[(int64_t)c * nI + i] = v;
  }
}

// Gram matrices in 64 x 64 tiles (upper tiles computed, mirrored), the
// contraction in chunks of 32 staged in LDS; each thread accumulates a 4 x 4
// block of its tile.
//   DUAL:  C[c][e] = sum_i Psi[i][c] W[e][i] over the interior nodes
//   else:  part z of H[i][j] = sum_c Psi[i][c] Psi[j][c] over the snapshots
constexpr int RBG_T = 64, RBG_K = 32;
template <bool DUAL>
__global__ __launch_bounds__(RB_THREADS) void rb_gram_kernel(RbBuildArgs b, RbWork d) {
  const int K = blockIdx.x, m = b.m, nI = (m - 1) * (m - 1), ns = d.ns, n = d.n;
  const int nt = (n + RBG_T - 1) / RBG_T;
  int t = blockIdx.y, tc = 0;
  while (t >= nt - tc) {  // upper-triangle tile index -> (tc, td), tc <= td
    t -= nt - tc;
    ++tc;
  }
  const int td = tc + t;
  __shared__ double Ps[RBG_K][RBG_T + 1], Ws[RBG_K][RBG_T + 1];
  const int tid = threadIdx.x, ty = tid / 16, tx = tid % 16;
  const double* W = DUAL ? d.W + (int64_t)K * ns * nI : nullptr;
  const int depth = DUAL ? nI : ns;
  const int share = ((depth + RBG_K - 1) / RBG_K + d.parts - 1) / d.parts * RBG_K;
  const int first = (int)blockIdx.z * share, last = first + share < depth ? first + share : depth;
  double acc[4][4] = {};
  for (int k0 = first; k0 < last; k0 += RBG_K) {
    for (int idx = tid; idx < RBG_K * RBG_T; idx += RB_THREADS) {
      if (DUAL) {
        const int kk = idx % RBG_K, cc = idx / RBG_K;
        const int c = tc * RBG_T + cc, dd = td * RBG_T + cc, i = k0 + kk;
        Ps[kk][cc] = (c < ns && i < nI) ? rb_psi(b, K, c, i, nI) : 0.0;
        Ws[kk][cc] = (dd < ns && i < nI) ? W[(int64_t)dd * nI + i] : 0.0;
      } else {
        const int cc = idx % RBG_T, kk = idx / RBG_T;
        const int i = tc * RBG_T + cc, j = td * RBG_T + cc, c = k0 + kk;
        Ps[kk][cc] = (i < nI && c < last) ? rb_psi(b, K, c, i, nI) : 0.0;
        if (tc != td) Ws[kk][cc] = (j < nI && c < last) ? rb_psi(b, K, c, j, nI) : 0.0;
      }
    }
    __syncthreads();
    const double(*Q)[RBG_T + 1] = DUAL || tc != td ? Ws : Ps;
    for (int kk = 0; kk < RBG_K; ++kk) {
      double pv[4], wv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        pv[u] = Ps[kk][4 * ty + u];
        wv[u] = Q[kk][4 * tx + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] += pv[u] * wv[v];
    }
    __syncthreads();
  }
  const int64_t ld = n;
  double* C = d.C + ((int64_t)K * d.parts + blockIdx.z) * ld * ld;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = tc * RBG_T + 4 * ty + u, c = td * RBG_T + 4 * tx + v;
      if (r < n && c < n && r <= c) {
        C[r * ld + c] = acc[u][v];
        C[c * ld + r] = acc[u][v];
      }
    }
}

// H of patches with at most RB_TINY unknowns, where a tile would be nearly empty:
// an entry per wavefront, its lanes along the snapshots (1024 patches of one
// unknown 17 us in tiles).
__global__ __launch_bounds__(RB_THREADS) void rb_gram_tiny_kernel(RbBuildArgs b, RbWork d) {
  const int K = blockIdx.x, n = d.n, lane = threadIdx.x & 63;
  double* C = d.C + (int64_t)K * d.parts * n * n;
  for (int e = threadIdx.x >> 6; e < n * n; e += RB_THREADS / 64) {
    const int i = e / n, j = e - i * n;
    if (j < i) continue;
    double v = 0.0;
    for (int c = lane; c < d.ns; c += 64) v += rb_psi(b, K, c, i, n) * rb_psi(b, K, c, j, n);
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) C[i * n + j] = C[j * n + i] = v;
  }
}

// sum over the 16 lanes of a DPP row, the same bits in all of them
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
  union { double d; int w[2]; } x{v}, y;
  y.w[0] = __builtin_amdgcn_update_dpp(0, x.w[0], 0x120 + N, 0xf, 0xf, false);
  y.w[1] = __builtin_amdgcn_update_dpp(0, x.w[1], 0x120 + N, 0xf, 0xf, false);
  return y.d;
}
__device__ __forceinline__ double row_sum(double v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  return v + row_rotate<1>(v);
}

// largest value of the wavefront, the same in all lanes
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  auto larger = [](unsigned a, unsigned b) { return a > b ? a : b; };
  v = larger(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, false));
  v = larger(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, false));
  return larger(larger(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                larger(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// 1 / sqrt(x) for normal x: one third-order step from the instruction's 2^-23
__device__ __forceinline__ double inv_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// The rotation of the symmetric Schur pair (Golub and Van Loan): c, s with
// the smaller angle that make the (p, q) entry of J^T A J vanish.  From the
// double angle, cos 2t = |d| / h and sin 2t = sign(d) e / h with d = a_qq -
// a_pp, e = 2 a_pq, h = sqrt(d^2 + e^2): two reciprocal roots instead of a chain
// of three divisions and two roots, then one correction of c^2 + s^2 to 1.
__device__ __forceinline__ void schur_pair(double app, double aqq, double apq, double* c, double* s) {
  *c = 1.0;
  *s = 0.0;
  if (apq == 0.0) return;
  const double d = aqq - app, e = 2.0 * apq, h2 = fma(d, d, e * e);
  if (h2 > 1e-280 && h2 < 1e280) {
    const double g = inv_sqrt(h2);
    const double c2 = 1.0 + fabs(d) * g, s2 = (d >= 0.0 ? e : -e) * g;
    const double y = inv_sqrt(2.0 * c2);
    const double c1 = c2 * y, s1 = s2 * y;
    const double f = 0.5 * fma(-c1, c1, fma(-s1, s1, 1.0));
    *c = fma(c1, f, c1);
    *s = fma(s1, f, s1);
  } else {  // squares out of range, or not finite
    const double tau = d / e;
    const double t = (tau >= 0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
    *c = 1.0 / sqrt(1.0 + t * t);
    *s = t * *c;
  }
}

// Pivoted Cholesky factor of the symmetric positive semidefinite n x n matrix
// A, C = F F^T, in place: pivot k's column of F replaces row piv[k] of A.  Left
// looking (a pivot's row of A is read only when it is chosen), 16 lanes to a
// row of F, one barrier per pivot; diag holds the Schur complement's diagonal
// for this pivot and the next.  The largest remaining diagonal value (to 2^-10)
// is the pivot; below 1e-15 of the first one it is rounding of C, the factor
// ends and the rows left over are zero columns.  Returns the rank; *d0 is the
// first pivot.  Whole workgroup.
__device__ __forceinline__ int rb_pivoted_cholesky(double* A, int lda, int n, double* diag, int* piv, double* d0) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, l = tid & 15;
  const double dead = -INFINITY;
  for (int i = tid; i < n; i += nt) diag[i] = A[i * lda + i];
  __syncthreads();
  double floor = 0.0;
  *d0 = 0.0;
  int k = 0;
  for (; k < n; ++k) {
    const double* dk = diag + (k & 1) * n;
    double* dn = diag + (1 - (k & 1)) * n;
    unsigned key = 0;
    for (int i = lane; i < n; i += 64) {
      const double v = dk[i];
      const unsigned c = v > 0.0 ? ((unsigned)__double2hiint(v) & ~1023u) | (unsigned)i : 0u;
      key = c > key ? c : key;
    }
    key = wave_max(key);
    const int p = key & 1023u;
    const double d = key != 0 ? dk[p] : 0.0;
    if (k == 0) {
      *d0 = d;
      floor = 1e-15 * d;
    }
    if (!(d > floor)) break;
    const double y = inv_sqrt(d);
    for (int i = tid >> 4; i < n; i += nt >> 4) {
      double v = 0.0;
      for (int j = l; j < k; j += 16) {
        const double* F = A + piv[j] * lda;
        v += F[i] * F[p];
      }
      v = row_sum(v);
      if (l == 0) {
        const double di = dk[i];
        double f = 0.0, dd = dead;
        if (i == p) {
          f = d * y;
        } else if (di != dead) {
          f = (A[p * lda + i] - v) * y;
          dd = di - f * f;
        }
        A[p * lda + i] = f;
        dn[i] = dd;
      }
    }
    if (tid == 0) piv[k] = p;
    __syncthreads();
  }
  // the rows left over
  const double* dk = diag + (k & 1) * n;
  for (int i = tid >> 6; i < n; i += nt >> 6)
    if (dk[i] != dead)
      for (int j = lane; j < n; j += 64) A[i * lda + j] *= 0.0;  // what is not a number stays one
  if (tid == 0)
    for (int i = 0, j = k; i < n; ++i)
      if (dk[i] != dead) piv[j++] = i;
  __syncthreads();
  return k;
}

// One-sided Jacobi on the first k columns of F (column j: row piv[j] of A):
// C = F F^T is unchanged by rotations of the columns, and when they are
// orthogonal they are its eigenvectors times the roots of their eigenvalues.
// A sweep is k - 1 rounds of k / 2 disjoint pairs (the round-robin pairing, k
// rounded up to even), 16 lanes to a pair, one barrier per round; a column is
// in registers (RT values per lane) or, RT = 0, read a second time.  Ends
// after a sweep in which every inner product was below 1e-14 of the two norms
// (below 1e-15 of the first pivot where an eigenvalue is below 1e-14 of it).  The pivoted factor is graded, so that the decaying spectra of
// the snapshots take about half the sweeps of the two-sided iteration, and
// there are no eigenvectors to update.  Whole workgroup.
template <int RT>
__device__ __forceinline__ void rb_jacobi(double* A, int lda, int n, int k, const int* piv, double d0, int max_sweeps) {
  const int nt = blockDim.x, g = threadIdx.x >> 4, l = threadIdx.x & 15, groups = nt >> 4;
  const int ke = k + (k & 1), np = ke / 2;
  const double tiny = 1e-30 * d0 * d0, low = 1e-14 * d0;
  auto rows = [&](int r, int i, int* rp, int* rq) {  // rows of A of pair i in round r; -1 for the dummy
    int p = r + i, q = r - i;
    p -= p >= ke - 1 ? ke - 1 : 0;
    q += q < 0 ? ke - 1 : 0;
    if (i == 0) q = ke - 1;
    *rp = p < k ? piv[p] : -1;
    *rq = q < k ? piv[q] : -1;
  };
  auto open = [&](double a, double b, double c) { return c * c > (a > low && b > low ? 1e-28 * a * b : tiny); };
  for (int sweep = 0; sweep < max_sweeps && k > 1; ++sweep) {
    bool more = false;
    int rp = -1, rq = -1;
    if (RT > 0 && g < np) rows(0, g, &rp, &rq);
    for (int r = 0; r < ke - 1; ++r) {
      if constexpr (RT > 0) {
        if (rp >= 0 && rq >= 0) {
          double *P = A + rp * lda, *Q = A + rq * lda;
          double x[RT], y[RT], a = 0.0, b = 0.0, c = 0.0;
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            const int i = l + 16 * t;
            x[t] = i < n ? P[i] : 0.0;
            y[t] = i < n ? Q[i] : 0.0;
          }
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            a = fma(x[t], x[t], a);
            b = fma(y[t], y[t], b);
            c = fma(x[t], y[t], c);
          }
          a = row_sum(a);
          b = row_sum(b);
          c = row_sum(c);
          more = more || open(a, b, c);
          if (c * c > 1e-30 * a * b) {  // below, a rotation is rounding of the columns
            double cs, sn;
            schur_pair(a, b, c, &cs, &sn);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
              const int i = l + 16 * t;
              if (i < n) {
                P[i] = cs * x[t] - sn * y[t];
                Q[i] = sn * x[t] + cs * y[t];
              }
            }
          }
        }
        if (g < np) rows(r + 1 < ke - 1 ? r + 1 : 0, g, &rp, &rq);
      } else {
        for (int i0 = g; i0 < np; i0 += groups) {
          rows(r, i0, &rp, &rq);
          if (rp < 0 || rq < 0) continue;
          double *P = A + (int64_t)rp * lda, *Q = A + (int64_t)rq * lda, a = 0.0, b = 0.0, c = 0.0;
          for (int i = l; i < n; i += 16) {
            const double x = P[i], y = Q[i];
            a = fma(x, x, a);
            b = fma(y, y, b);
            c = fma(x, y, c);
          }
          a = row_sum(a);
          b = row_sum(b);
          c = row_sum(c);
          more = more || open(a, b, c);
          double cs, sn;
          schur_pair(a, b, c, &cs, &sn);
          for (int i = l; i < n; i += 16) {
            const double x = P[i], y = Q[i];
            P[i] = cs * x - sn * y;
            Q[i] = sn * x + cs * y;
          }
        }
      }
      __syncthreads();
    }
    if (!__syncthreads_or(more)) break;
  }
}

// Eigenvalues (raw, by column) in descending order into order[], val[] and
// lambda[0..nlam) (zeros beyond n), and the number of modes: r = min(rcap, rmax,
// n, smallest r whose relative tail sqrt(sum_{q>r} lambda_q / sum lambda_q) <=
// tail_tol, number of eigenvalues above RB_RANK_TOL lambda_max).  Whole
// workgroup.  tail: n + 1 values, first: one, of LDS.
__device__ __forceinline__ int rb_sort_tail(const double* raw, int n, double* val, double* tail, int* order, int* first,
                                            double tail_tol, int rcap, int rmax, double* lambda, int nlam) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double x = raw[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {  // a permutation also with values that are not numbers
      const double y = raw[j];
      rank += y > x || (!(y < x) && j < i && (y == x || (x != x && y != y))) || (x != x && y == y);
    }
    order[rank] = i;
    val[rank] = x;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nlam; i += blockDim.x) lambda[i] = i < n ? val[i] : 0.0;
  double tot = 0.0;
  if (threadIdx.x == 0) {
    for (int i = 0; i < n; ++i) tot += fmax(val[i], 0.0);
    double t = tot;
    for (int i = 0; i < n; ++i) tail[i] = t -= fmax(val[i], 0.0);
    tail[n] = tot;
    *first = n;
  }
  __syncthreads();
  tot = tail[n];
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double rel = tot > 0 ? sqrt(fmax(tail[i], 0.0) / tot) : 0.0;
    if (rel <= tail_tol) atomicMin(first, i + 1);
  }
  __syncthreads();
  int r = *first;
  if (r > rcap) r = rcap;
  if (r > rmax) r = rmax;
  if (r > n) r = n;
  // numerical rank of the snapshots: eigenvalues at or below 1e-12 of the
  // largest are rounding, not modes (the method of snapshots would divide by
  // their square roots); r = 0 when the centred snapshots vanish
  const double lmax = n > 0 ? val[0] : 0.0;
  int rank = 0;
  while (rank < n && rank < r && val[rank] > RB_RANK_TOL * lmax) ++rank;
  return r > rank ? rank : r;
}

// Cholesky band of E = K_II(abar), one wavefront: L[r][d] = L_E(r, r - d), half
// bandwidth m.  Right looking; the rank-one update of a column in 8 x 8 pieces.
__device__ __forceinline__ void rb_cholesky_band(double* L, const double* abar, int m) {
  const int n = m - 1, nI = n * n, LB = m + 1, lane = threadIdx.x & 63;
  auto fence = [] { __threadfence_block(); };
  for (int i = lane; i < nI * LB; i += 64) L[i] = 0.0;
  fence();
  for (int r = lane; r < nI; r += 64) {
    const int ix = r % n, iy = r / n;
    const Stencil9 st = rb_stencil(abar, m, ix, iy);
    L[r * LB] = st.kc;
    for (int q = 0; q < 8; ++q) {
      const int qx = ix + RB_DX[q], qy = iy + RB_DY[q], dd = r - (qy * n + qx);
      if (qx >= 0 && qx < n && qy >= 0 && qy < n && dd > 0) L[r * LB + dd] = st.ks[q];
    }
  }
  fence();
  const int x0 = lane >> 3, y0 = lane & 7;
  for (int j = 0; j < nI; ++j) {
    const double djj = sqrt(L[j * LB]);
    fence();
    const int h = nI - 1 - j < m ? nI - 1 - j : m;
    for (int l = lane; l <= h; l += 64) L[(j + l) * LB + l] = l == 0 ? djj : L[(j + l) * LB + l] / djj;
    fence();
    for (int x = 1 + x0; x <= h; x += 8) {
      const double lx = L[(j + x) * LB + x];
      for (int y = 1 + y0; y <= x; y += 8) L[(j + x) * LB + x - y] -= lx * L[(j + y) * LB + y];
    }
    fence();
  }
}

// One workgroup per patch, 16 lanes for each pair of columns.  RT: values of a
// column per lane with the matrix in LDS, 0 with the matrix in memory.  At n = 49
// (64 patches, ranks 15 to 49) the phases took 20 us (factor of E), 25 (C), 56
// (pivoted Cholesky), 64 to 310 (Jacobi: 7 sweeps, 0.9 us a round: the columns
// through LDS and the latency of the reductions and of the rotation), 13 (order)
// and 20 (modes), the kernel 515 us; with C formed in registers, the pivot's
// maximum by DPP, the tails' roots in parallel and rotations below rounding
// left out 466.  With the two-sided iteration, one rotation after the other in
// memory, the build of the 64 patches took 20.5 ms, with its rounds in parallel
// in LDS 0.93 ms (13 sweeps).  A build with the FP64 online stage, end to end:
// n = 49 21.9 -> 0.85 ms, n = 121 190 -> 2.8 ms.
template <int RT, bool DUAL>
__global__ __launch_bounds__(RB_EIGEN) void rb_eigen_kernel(RbBuildArgs b, RbWork d) {
  extern __shared__ double smem[];
  __shared__ int rsel;
  const int K = blockIdx.x, tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6, m = b.m, nI = (m - 1) * (m - 1), LB = m + 1;
  const int n = d.n, rmax = b.rmax;
  const int64_t nn = (int64_t)n * n;
  double* lds = smem;
  auto take = [&](int count) {
    double* p = lds;
    lds += count;
    return p;
  };
  double* diag = take(2 * n);
  double* val = take(n);
  double* tail = take(n + 1);
  int* piv = (int*)take(n);  // pivots, then the order of the eigenvalues
  int* order = piv + n;
  double* L = DUAL ? nullptr : RT > 0 ? take(nI * LB) : d.L + (int64_t)K * nI * LB;
  double* zb = DUAL ? nullptr : take(rmax * nI);
  const int lda = RT > 0 ? n | 1 : n;
  double* C = d.C + (int64_t)K * d.parts * nn;
  double* A = RT > 0 ? take(n * lda) : C;

  // the Gram matrix, its parts added; the first wavefront factors E meanwhile
  const int w0 = DUAL ? 0 : 1;
  if (!DUAL && tid < 64) rb_cholesky_band(L, d.abar + (int64_t)K * m * m, m);
  if (RT > 0 && tid >= 64 * w0)
    for (int i = tid / 64 - w0; i < n; i += nw - w0)
      for (int j = tid % 64; j < n; j += 64) {
        double v = 0.0;
        for (int z = 0; z < d.parts; ++z) v += C[z * nn + (int64_t)i * n + j];
        A[i * lda + j] = v;
      }
  __syncthreads();
  if (!DUAL) {
    // C = L_E^T H L_E in place: H L_E by rows (a wavefront has read what it
    // needs of its row before it writes), then the upper part of L_E^T (H L_E),
    // formed in registers before any of it is written (in memory: by columns),
    // and mirrored
    for (int i = tid / 64; i < n; i += nw)
      for (int j0 = 0; j0 < n; j0 += 64) {
        const int j = j0 + tid % 64;
        double v = 0.0;
        if (j < n)
          for (int k = j; k < n && k <= j + m; ++k) v += A[(int64_t)i * lda + k] * L[k * LB + k - j];
        __threadfence_block();
        if (j < n) A[(int64_t)i * lda + j] = v;
        __threadfence_block();
      }
    __syncthreads();
    if constexpr (RT > 0) {
      constexpr int PER = 2 * RT;  // n^2 entries over 16 ceil(n / 2) threads or more
      double v[PER];
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int i = (tid + e * nt) / n, j = (tid + e * nt) - i * n;
        v[e] = 0.0;
        if (i <= j && i < n)
          for (int k = i; k < n && k <= i + m; ++k) v[e] += L[k * LB + k - i] * A[k * lda + j];
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int i = (tid + e * nt) / n, j = (tid + e * nt) - i * n;
        if (i <= j && i < n) {
          A[i * lda + j] = v[e];
          A[j * lda + i] = v[e];
        }
      }
    } else {
      for (int j = tid; j < n; j += nt)
        for (int i = 0; i <= j; ++i) {
          double v = 0.0;
          for (int k = i; k < n && k <= i + m; ++k) v += L[k * LB + k - i] * A[(int64_t)k * lda + j];
          A[(int64_t)i * lda + j] = v;
        }
      __syncthreads();
      for (int i = tid / 64; i < n; i += nw)
        for (int j = i + 1 + tid % 64; j < n; j += 64) A[(int64_t)j * lda + i] = A[(int64_t)i * lda + j];
    }
    __syncthreads();
  }
  double d0;
  const int k = rb_pivoted_cholesky(A, lda, n, diag, piv, &d0);
  rb_jacobi<RT>(A, lda, n, k, piv, d0, b.max_sweeps);
  // eigenvalues: the squared norms of the columns (of a matrix that is not
  // finite: not numbers)
  double* raw = diag;
  __syncthreads();
  for (int c = tid >> 4; c < n; c += nt >> 4) {
    const double* F = A + (int64_t)piv[c] * lda;
    double v = 0.0;
    for (int i = tid & 15; i < n; i += 16) v = fma(F[i], F[i], v);
    v = row_sum(v);
    if ((tid & 15) == 0) raw[c] = v;
  }
  __syncthreads();
  const int rs = rb_sort_tail(raw, n, val, tail, order, &rsel, b.tail_tol, b.rcap, rmax, b.lambda + (int64_t)K * nI, nI);
  if (tid == 0) b.rK[K] = rs;
  const int r = rs;
  double* Zk = b.Z + (int64_t)K * nI * rmax;
  if (DUAL) {
    for (int iq = tid; iq < nI * rmax; iq += nt) {
      const int i = iq / rmax, q = iq % rmax;
      double v = 0.0;
      if (q < r) {
        const double* F = A + (int64_t)piv[order[q]] * lda;
        for (int c = 0; c < n; ++c) v += rb_psi(b, K, c, i, nI) * F[c];
        v = val[q] > 0.0 ? v / val[q] : 0.0;
      }
      Zk[iq] = v;
    }
    return;
  }
  // Z = L_E^{-T} V_r, zero beyond r: a wavefront per column, right looking
  for (int q = tid >> 6; q < rmax; q += nw) {
    const int lane = tid & 63;
    double* z = zb + q * nI;
    const double root = q < r ? sqrt(val[q]) : 1.0;
    for (int i = lane; i < nI; i += 64) z[i] = q < r ? A[(int64_t)piv[order[q]] * lda + i] / root : 0.0;
    __threadfence_block();
    if (q < r)
      for (int i = nI - 1; i >= 0; --i) {
        const double zi = z[i] / L[i * LB];
        __threadfence_block();
        for (int l = lane; l <= m && l <= i; l += 64) z[i - l] = l == 0 ? zi : z[i - l] - L[i * LB + l] * zi;
        __threadfence_block();
      }
    for (int i = lane; i < nI; i += 64) Zk[i * rmax + q] = z[i];
  }
}

// Element table G of patch K from its modes Zk [nI][rmax] and means pbar
// [3][nI] (the P coefficients: rb.hip), one coefficient per thread.
__global__ __launch_bounds__(RB_THREADS) void rb_table_kernel(RbBuildArgs b) {
  const int K = blockIdx.x;
  const int m = b.m, n = m - 1, nI = n * n, rmax = b.rmax;
  const double* Zk = b.Z + (int64_t)K * nI * rmax;
  const double* pbar = b.phibar + (int64_t)K * 3 * nI;
  const int PP = b.PP, KD = b.KD, NA = rb_na(rmax);
  for (int ep = blockIdx.y * RB_THREADS + threadIdx.x; ep < KD * PP; ep += gridDim.y * RB_THREADS) {
    const int e = ep / PP, pidx = ep % PP;
    double val = 0.0;
    if (e < m * m && pidx < rb_p(rmax)) {
      const int ex = e % m, ey = e / m;
      int nid[4];
      int pxs[4] = {ex, ex + 1, ex + 1, ex}, pys[4] = {ey, ey, ey + 1, ey + 1};
      for (int c = 0; c < 4; ++c) {
        const bool inner = pxs[c] > 0 && pxs[c] < m && pys[c] > 0 && pys[c] < m;
        nid[c] = inner ? (pys[c] - 1) * n + (pxs[c] - 1) : -1;
      }
      auto zeta = [&](int q, int c) { return nid[c] >= 0 ? Zk[nid[c] * rmax + q] : 0.0; };
      auto pb = [&](int l, int c) { return nid[c] >= 0 ? pbar[l * nI + nid[c]] : pcorner(l, pxs[c], pys[c], m); };
      if (pidx < NA) {
        int q = 0, rem = pidx;
        while (rem >= rmax - q) {
          rem -= rmax - q;
          ++q;
        }
        const int qp = q + rem;
        for (int al = 0; al < 4; ++al)
          for (int be = 0; be < 4; ++be) val += zeta(q, al) * kref(al, be) * zeta(qp, be);
      } else if (pidx < NA + 3 * rmax) {
        const int l = (pidx - NA) / rmax, q = (pidx - NA) % rmax;
        for (int al = 0; al < 4; ++al)
          for (int be = 0; be < 4; ++be) val += zeta(q, al) * kref(al, be) * pb(l, be);
      } else {
        const int t = pidx - NA - 3 * rmax;
        const int ls[6] = {0, 0, 0, 1, 1, 2}, lps[6] = {0, 1, 2, 1, 2, 2};
        for (int al = 0; al < 4; ++al)
          for (int be = 0; be < 4; ++be) val += pb(ls[t], al) * kref(al, be) * pb(lps[t], be);
      }
    }
    b.G64[((int64_t)K * KD + e) * PP + pidx] = val;
    b.G32[((int64_t)K * KD + e) * PP + pidx] = (float)val;
  }
}


template <int RT, bool DUAL>
hipError_t launch_eigen(const RbBuildArgs& b, const RbWork& d, hipStream_t st) {
  const size_t lds = rb_eigen_lds(DUAL, b.m, d.n, b.rmax);
  if (lds > RB_LDS) return hipErrorInvalidValue;
  if (lds > 65536) {  // above 64 KB the dynamic-LDS limit is raised on the current device
    hipError_t e = hipFuncSetAttribute((const void*)rb_eigen_kernel<RT, DUAL>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int lanes = (d.n + 1) / 2 * 16;  // one group per pair: a barrier costs by the wavefronts
  const int nt = lanes <= 256 ? 256 : lanes >= RB_EIGEN ? RB_EIGEN : (lanes + 63) / 64 * 64;
  hipLaunchKernelGGL((rb_eigen_kernel<RT, DUAL>), dim3(b.ncx * b.ncy), dim3(nt), lds, st, b, d);
  return hipGetLastError();
}

template <bool DUAL>
hipError_t launch_eigen_any(const RbBuildArgs& b, const RbWork& d, hipStream_t st) {
  if (d.n <= 64) return launch_eigen<4, DUAL>(b, d, st);
  if (d.n <= RB_LDS_N) return launch_eigen<8, DUAL>(b, d, st);
  return launch_eigen<0, DUAL>(b, d, st);
}

}  // namespace

int64_t rb_work_doubles(int ncx, int ncy, int m, int ntrain) {
  return rb_work_layout(ncx, ncy, m, ntrain, nullptr, nullptr);
}

bool rb_dual(int m, int ntrain) { return 3 * ntrain < (m - 1) * (m - 1); }

hipError_t launch_rb_build(const RbBuildArgs& b, hipStream_t st) {
  const int Mc = b.ncx * b.ncy, m = b.m, nI = (m - 1) * (m - 1);
  const bool dual = rb_dual(m, b.ntrain);
  RbWork d;
  rb_work_layout(b.ncx, b.ncy, m, b.ntrain, b.work, &d);
  if (d.n > RB_NMAX) return hipErrorInvalidValue;
  const dim3 means(Mc, (m * m + 3 * nI + 31) / 32);
  if (b.a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL(rb_means_kernel<float>, means, dim3(RB_THREADS), 0, st, b, d);
  else
    hipLaunchKernelGGL(rb_means_kernel<double>, means, dim3(RB_THREADS), 0, st, b, d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nt = (d.n + RBG_T - 1) / RBG_T;
  const dim3 tiles(Mc, nt * (nt + 1) / 2, d.parts);
  if (dual) {
    hipLaunchKernelGGL(rb_energy_kernel, dim3(Mc, (nI + RB_THREADS - 1) / RB_THREADS), dim3(RB_THREADS), 0, st, b, d);
    hipLaunchKernelGGL(rb_gram_kernel<true>, tiles, dim3(RB_THREADS), 0, st, b, d);
  } else if (d.n <= RB_TINY) {
    hipLaunchKernelGGL(rb_gram_tiny_kernel, dim3(Mc), dim3(RB_THREADS), 0, st, b, d);
  } else {
    hipLaunchKernelGGL(rb_gram_kernel<false>, tiles, dim3(RB_THREADS), 0, st, b, d);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = dual ? launch_eigen_any<true>(b, d, st) : launch_eigen_any<false>(b, d, st);
  if (e != hipSuccess) return e;
  // a coefficient per thread, several where the patches are many: workgroups of
  // one coefficient take longer to launch than to run (1024 patches at m = 2: 77 us)
  const int most = (b.KD * b.PP + RB_THREADS - 1) / RB_THREADS, blocks = RB_TABLE_BLOCKS / Mc;
  hipLaunchKernelGGL(rb_table_kernel, dim3(Mc, blocks < 1 ? 1 : blocks > most ? most : blocks), dim3(RB_THREADS), 0, st, b);
  return hipGetLastError();
}

}  // namespace stomsfem
