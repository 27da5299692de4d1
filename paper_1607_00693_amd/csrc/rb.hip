// Reduced-basis upscaling (Sec. 3.2, eqs. KLphi, localRB, localRBsystem,
// RBaffine / localAF; Algorithms 3 and 4).
//
// Offline (per patch K, from N_train coefficient samples):
//   cell_phi_kernel  -- the cell-problem solutions phi^l(xi_s), l = 0..2, on
//                       the interior nodes (banded LDL^T in LDS, one
//                       wavefront per pair, forward and backward solves);
//                       where that band does not fit LDS the refined
//                       FP32/FP64 kernel of upscale_mixed.hip supplies them;
//   rb_build.hip     -- means, energy matrix, KL eigenpairs (primal or dual
//                       form), modes Z with Z^T E Z = I and the element table G.
// The Q1 stiffness is affine in the per-element coefficient values
// (K(a) = sum_e a_e K_e), which is the paper's affine structure taken at
// element level: every quantity of the online Galerkin system is a linear
// function of the patch's m*m coefficient values,
//     A_qq'  = sum_e a_e zeta_q . K_e zeta_q'           (r(r+1)/2 values)
//     Fh_lq  = sum_e a_e zeta_q . K_e phibar^l          (3 r values)
//     B_ll'  = sum_e a_e phibar^l . K_e phibar^l'       (6 values)
// (phibar^l carries the Dirichlet data g^l on the boundary).  G holds these
// P per-element coefficients, so the online stage is one GEMM
// [pairs x m*m] x [m*m x P] per patch, then an r x r Cholesky per pair and
//     S_ll' = B_ll' - Fh_l . A^{-1} Fh_l'
// (Galerkin identity: phi_rb = phibar + Z c with A c = -Fh).
//
// Online: rb_apply_mfma_kernel (FP32 MFMA 16x16x4, FP32 accumulation, FP32
// r x r solve) and rb_apply_f64_kernel (FP64 throughout, for parity checks).
#include "rb.h"
#include "rb_os_dev.h"

#include <type_traits>

namespace stomsfem {

// ---------------------------------------------------------------------------
// Cell-problem solutions (snapshots)
// ---------------------------------------------------------------------------
struct PhiArgs {
  UpArgs up;
  double* phi;  // [npairs][3][nI]
};

// LDS latency and the issue of the band updates bound it; a lane's place in the
// triangle below a pivot is worked out once (it took a square root per pivot),
// and the backward pass spreads a solved value over the rows before it.  PHI_Q,
// PHI_F: entries and right-hand sides of a pivot's update per lane, from m <= 10
// (55 entries) and m <= 21 (63 right-hand sides) on.  16 384 pairs at m = 8:
// 245 -> 119 us.
template <typename TA, int PHI_Q, int PHI_F>
__global__ __launch_bounds__(64) void cell_phi_kernel(PhiArgs pa) {
  extern __shared__ double smem[];
  const UpArgs& args = pa.up;
  const int m = args.m, n = m - 1, nI = n * n, B = m;
  double* A = smem;            // m*m
  double* Bd = A + m * m;      // nI*(B+1): Bd[i*(B+1)+d] = K(i, i-d), column j kept unscaled
  double* F = Bd + nI * (B + 1);  // 3*nI
  const int tid = threadIdx.x;
  const int Mc = args.ncx * args.ncy;
  const int64_t lda = (int64_t)args.ncx * m;
  // this lane's entries (io, ko) of the triangle below a pivot, and its rows
  // fi and right-hand sides fl
  int io[PHI_Q], ko[PHI_Q], fi[PHI_F], fl[PHI_F];
#pragma unroll
  for (int k = 0; k < PHI_Q; ++k) {
    // row i of entry q: 8 q + 1 runs from (2 i + 1)^2 to 8 below (2 i + 3)^2; one
    // more leaves the root's rounding no say
    const int q = tid + 64 * k, i = (int)((sqrtf((float)(8 * q + 2)) - 1.0f) * 0.5f);
    io[k] = i;
    ko[k] = q - i * (i + 1) / 2;
  }
#pragma unroll
  for (int k = 0; k < PHI_F; ++k) {
    fi[k] = (tid + 64 * k) / 3;
    fl[k] = (tid + 64 * k) % 3;
  }
  for (int64_t p = blockIdx.x; p < args.npairs; p += gridDim.x) {
    const int64_t s = p / Mc;
    const int K = (int)(p - s * Mc);
    const TA* a = (const TA*)args.a + block_offset(s, K, args.ncx, args.ncy, m);
    __syncthreads();
    for (int i = tid; i < m * m; i += blockDim.x) A[i] = ld(a, (i / m) * lda + (i % m));
    __syncthreads();
    for (int r = tid; r < nI; r += blockDim.x) {
      const int ix = r % n, iy = r / n, px = ix + 1, py = iy + 1;
      const double aSW = A[iy * m + ix], aSE = A[iy * m + ix + 1];
      const double aNW = A[(iy + 1) * m + ix], aNE = A[(iy + 1) * m + ix + 1];
      double* row = Bd + r * (B + 1);
      for (int d = 0; d <= B; ++d) row[d] = 0.0;
      row[0] = (2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE));
      const int dxs[8] = {-1, 1, 0, 0, -1, 1, -1, 1};
      const int dys[8] = {0, 0, -1, 1, -1, -1, 1, 1};
      const double ks[8] = {-(aSW + aNW) / 6.0, -(aSE + aNE) / 6.0, -(aSW + aSE) / 6.0, -(aNW + aNE) / 6.0,
                            -aSW / 3.0,         -aSE / 3.0,         -aNW / 3.0,         -aNE / 3.0};
      double f[3] = {0, 0, 0};
      for (int q = 0; q < 8; ++q) {
        const int qx = px + dxs[q], qy = py + dys[q];
        if (qx == 0 || qx == m || qy == 0 || qy == m) {
          for (int l = 0; l < 3; ++l) f[l] -= ks[q] * pcorner(l, qx, qy, m);
        } else {
          const int c = (qy - 1) * n + (qx - 1);
          if (c < r) row[r - c] = ks[q];
        }
      }
      for (int l = 0; l < 3; ++l) F[l * nI + r] = f[l];
    }
    __syncthreads();
    // right-looking LDL^T, column j kept unscaled (W_ij = l_ij d_j)
    for (int j = 0; j < nI; ++j) {
      const double inv = 1.0 / Bd[j * (B + 1)];
      const int cnt = (j + B < nI - 1 ? j + B : nI - 1) - j;
      double* next = Bd + (j + 1) * (B + 1);
#pragma unroll
      for (int k = 0; k < PHI_Q; ++k)
        if (io[k] < cnt) {
          const double *x = next + io[k] * (B + 1), *y = next + ko[k] * (B + 1);
          next[io[k] * (B + 1) + io[k] - ko[k]] -= x[io[k] + 1] * inv * y[ko[k] + 1];
        }
#pragma unroll
      for (int k = 0; k < PHI_F; ++k) {
        const int t = tid + 64 * k, i = fi[k];
        if (i < cnt && t < 3 * B) F[fl[k] * nI + j + 1 + i] -= next[i * (B + 1) + i + 1] * inv * F[fl[k] * nI + j];
      }
      __syncthreads();
    }
    // backward, right looking: x_j = v_j / d_j (v stays), v_{j-t} -= W_{j,j-t} x_j
    for (int j = nI - 1; j >= 0; --j) {
      const double d = Bd[j * (B + 1)];
#pragma unroll
      for (int k = 0; k < PHI_F; ++k) {
        const int t = tid + 64 * k, i = fi[k] + 1, l = fl[k];
        if (t < 3 * B && i <= j) F[l * nI + j - i] -= Bd[j * (B + 1) + i] * (F[l * nI + j] / d);
      }
      __syncthreads();
    }
    __syncthreads();
    for (int i = tid; i < 3 * nI; i += blockDim.x) pa.phi[p * 3 * nI + i] = F[i] / Bd[(i % nI) * (B + 1)];
  }
}

size_t cell_phi_lds_bytes(int m) {
  const int nI = (m - 1) * (m - 1);
  return sizeof(double) * ((size_t)m * m + (size_t)nI * (m + 1) + 3 * (size_t)nI);
}

template <typename TA, int PHI_Q, int PHI_F>
static hipError_t launch_phi(const PhiArgs& pa, unsigned blocks, size_t lds, hipStream_t st) {
  // above 64 KB the kernel's dynamic-LDS limit is raised on the current
  // device before the launch
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)cell_phi_kernel<TA, PHI_Q, PHI_F>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((cell_phi_kernel<TA, PHI_Q, PHI_F>), dim3(blocks), dim3(64), lds, st, pa);
  return hipGetLastError();
}

hipError_t launch_cell_phi(const UpArgs& args, int a_dtype, double* phi, hipStream_t st) {
  const PhiArgs pa{args, phi};
  const int64_t blocks = args.npairs < 65536 ? args.npairs : 65536;
  if (blocks == 0) return hipSuccess;
  const size_t lds = cell_phi_lds_bytes(args.m);
  if (lds > CELL_PHI_LDS_MAX) return hipErrorInvalidValue;
  const unsigned g = (unsigned)blocks;
  const bool f32 = a_dtype == STOMSFEM_F32;
  if (args.m <= 10) return f32 ? launch_phi<float, 1, 1>(pa, g, lds, st) : launch_phi<double, 1, 1>(pa, g, lds, st);
  if (args.m <= 15) return f32 ? launch_phi<float, 2, 1>(pa, g, lds, st) : launch_phi<double, 2, 1>(pa, g, lds, st);
  return f32 ? launch_phi<float, 6, 2>(pa, g, lds, st) : launch_phi<double, 6, 2>(pa, g, lds, st);
}

// Snapshots of cells whose band does not fit a workgroup's LDS (used for
// m > 32, past the refined kernel).  One wavefront per pair.  The band rows
// j .. j+B of the elimination window sit in a circular LDS ring of B+1 rows
// (row i in slot i mod (B+1), entry d = K(i, i-d), column j kept unscaled as
// in cell_phi_kernel); the three lifts are forward-substituted in the same
// pivot loop.  A row leaves the ring after its pivot, finished, to the
// workgroup's global row store with its forward-substituted right-hand
// sides, and the backward substitution reads the stored rows in reverse: the
// B products of a step are taken by the lanes and reduced over the
// wavefront, the next step's entries fetched one step ahead.
struct PhiBandArgs {
  UpArgs up;
  double* phi;   // [npairs][3][nI]
  double* rows;  // [gridDim.x][nI][B+1] finished rows
  double* ys;    // [gridDim.x][3][nI] forward-substituted right-hand sides
};

#define RB_WAVE_SYNC()                                     \
  do {                                                     \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); \
    __builtin_amdgcn_wave_barrier();                       \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); \
  } while (0)

template <typename TA>
__global__ __launch_bounds__(64) void cell_phi_band_kernel(PhiBandArgs pa) {
  extern __shared__ double smem[];
  const UpArgs& args = pa.up;
  const int m = args.m, n = m - 1, nI = n * n, B = m, W = B + 1;
  double* Wn = smem;          // [W][W] ring of band rows
  double* Fr = Wn + W * W;    // [3][W] right-hand sides of the ring rows
  double* Xr = Fr + 3 * W;    // [3][W] solution values of the last B rows (backward pass)
  const int lane = threadIdx.x;
  const int Mc = args.ncx * args.ncy;
  const int64_t lda = (int64_t)args.ncx * m;
  double* rows = pa.rows + (int64_t)blockIdx.x * nI * W;
  double* ys = pa.ys + (int64_t)blockIdx.x * 3 * nI;
  for (int64_t p = blockIdx.x; p < args.npairs; p += gridDim.x) {
    const int64_t s = p / Mc;
    const int K = (int)(p - s * Mc);
    const TA* a = (const TA*)args.a + block_offset(s, K, args.ncx, args.ncy, m);
    // row r of K_II into slot r mod W and its lifts (the stencil of cell_phi_kernel)
    auto build = [&](int r) {
      double* row = Wn + (r % W) * W;
      for (int d = lane; d <= B; d += 64) row[d] = 0.0;
      RB_WAVE_SYNC();
      if (lane == 0) {
        const int ix = r % n, iy = r / n, px = ix + 1, py = iy + 1;
        const double aSW = ld(a, (int64_t)iy * lda + ix), aSE = ld(a, (int64_t)iy * lda + ix + 1);
        const double aNW = ld(a, (int64_t)(iy + 1) * lda + ix), aNE = ld(a, (int64_t)(iy + 1) * lda + ix + 1);
        row[0] = (2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE));
        const int dxs[8] = {-1, 1, 0, 0, -1, 1, -1, 1};
        const int dys[8] = {0, 0, -1, 1, -1, -1, 1, 1};
        const double ks[8] = {-(aSW + aNW) / 6.0, -(aSE + aNE) / 6.0, -(aSW + aSE) / 6.0, -(aNW + aNE) / 6.0,
                              -aSW / 3.0,         -aSE / 3.0,         -aNW / 3.0,         -aNE / 3.0};
        double f[3] = {0, 0, 0};
        for (int q = 0; q < 8; ++q) {
          const int qx = px + dxs[q], qy = py + dys[q];
          if (qx == 0 || qx == m || qy == 0 || qy == m) {
            for (int l = 0; l < 3; ++l) f[l] -= ks[q] * pcorner(l, qx, qy, m);
          } else {
            const int c = (qy - 1) * n + (qx - 1);
            if (c < r) row[r - c] = ks[q];
          }
        }
        for (int l = 0; l < 3; ++l) Fr[l * W + r % W] = f[l];
      }
      RB_WAVE_SYNC();
    };
    for (int r = 0; r < W && r < nI; ++r) build(r);
    for (int j = 0; j < nI; ++j) {
      const int sj = j % W;
      const double inv = 1.0 / Wn[sj * W];
      const int cnt = (j + B < nI - 1 ? j + B : nI - 1) - j;
      const int npr = cnt * (cnt + 1) / 2;
      for (int q = lane; q < npr; q += 64) {
        int io = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
        while (io * (io + 1) / 2 > q) --io;
        while ((io + 1) * (io + 2) / 2 <= q) ++io;
        const int ko = q - io * (io + 1) / 2;
        const int i = j + 1 + io, k = j + 1 + ko;
        Wn[(i % W) * W + (i - k)] -= Wn[(i % W) * W + (i - j)] * inv * Wn[(k % W) * W + (k - j)];
      }
      for (int t = lane; t < 3 * cnt; t += 64) {
        const int i = j + 1 + t / 3, l = t % 3;
        Fr[l * W + i % W] -= Wn[(i % W) * W + (i - j)] * inv * Fr[l * W + sj];
      }
      RB_WAVE_SYNC();
      // row j is finished: to the row store, its slot to the row entering at j + W
      for (int d = lane; d <= B; d += 64) rows[(int64_t)j * W + d] = Wn[sj * W + d];
      if (lane < 3) ys[(int64_t)lane * nI + j] = Fr[lane * W + sj];
      RB_WAVE_SYNC();
      if (j + W < nI) build(j + W);
    }
    // the stored rows are read back by other lanes of the wavefront
    __threadfence();
    __syncthreads();
    // backward: x_j = (y_j - sum_{t=1..B} W_{j+t,j} x_{j+t}) / d_j; lane t
    // takes t (lane 0 takes t = 64 when B = 64)
    const int t = lane == 0 ? 64 : lane;
    const bool tl = t <= B;
    auto fetch = [&](int j) { return (j >= 0 && tl && j + t < nI) ? rows[(int64_t)(j + t) * W + t] : 0.0; };
    double wc = fetch(nI - 1);
    double* out = pa.phi + p * 3 * nI;
    for (int j = nI - 1; j >= 0; --j) {
      const double wn = fetch(j - 1);
      double v[3];
      const bool on = tl && j + t < nI;
#pragma unroll
      for (int l = 0; l < 3; ++l) v[l] = on ? wc * Xr[l * W + (j + t) % W] : 0.0;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int l = 0; l < 3; ++l) v[l] += __shfl_xor(v[l], off, 64);
      if (lane < 3) {
        const double x = (ys[(int64_t)lane * nI + j] - v[lane]) / rows[(int64_t)j * W];
        Xr[lane * W + j % W] = x;
        out[(int64_t)lane * nI + j] = x;
      }
      RB_WAVE_SYNC();
      wc = wn;
    }
    __syncthreads();  // the ring and the row store are reused by the next pair
  }
}

size_t cell_phi_band_lds_bytes(int m) {
  const size_t W = (size_t)m + 1;
  return sizeof(double) * (W * W + 6 * W);
}

int64_t cell_phi_band_ws_doubles(int m) {
  const int64_t nI = (int64_t)(m - 1) * (m - 1);
  return nI * (m + 1) + 3 * nI;
}

hipError_t launch_cell_phi_band(const UpArgs& args, int a_dtype, double* phi, double* ws, int64_t blocks,
                                hipStream_t st) {
  if (args.npairs == 0) return hipSuccess;
  if (args.m < 2 || args.m > 64 || blocks < 1) return hipErrorInvalidValue;
  const int64_t nI = (int64_t)(args.m - 1) * (args.m - 1);
  if (blocks > args.npairs) blocks = args.npairs;
  PhiBandArgs pa{args, phi, ws, ws + blocks * nI * (args.m + 1)};
  const size_t lds = cell_phi_band_lds_bytes(args.m);
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL(cell_phi_band_kernel<float>, dim3((unsigned)blocks), dim3(64), lds, st, pa);
  else
    hipLaunchKernelGGL(cell_phi_band_kernel<double>, dim3((unsigned)blocks), dim3(64), lds, st, pa);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Online stage
// ---------------------------------------------------------------------------
// r x r LDL^T of A (packed upper in v), forward solves with the three Fh
// columns, S_ll' = B_ll' - Fh_l . A^{-1} Fh_l' = B_ll' - sum_i y_l[i] y_l'[i] / d_i
// with L y_l = Fh_l (unit L), in the arithmetic of T (FP64 for the reference
// stage, FP32 after the FP32 matrix-core products: A is close to the
// identity, since the modes are orthonormal in the energy of the training
// mean).  No square roots, and one reciprocal per pivot (FP32: the hardware
// reciprocal, within an ulp, far below the FP32 products' error).  Returns
// false on a non-positive pivot.
template <typename T>
__device__ __forceinline__ T rb_recip(T d) {
  return T(1) / d;
}
template <>
__device__ __forceinline__ float rb_recip<float>(float d) {
  return __builtin_amdgcn_rcpf(d);
}
template <int RMAX, typename T>
__device__ __forceinline__ bool rb_small_solve(const T* v, int r, double S3[3][3]) {
  constexpr int NA = RMAX * (RMAX + 1) / 2;
  T L[RMAX][RMAX];  // lower part: A, then the unit factor's l_ij (i > j)
  T U[RMAX][RMAX];  // u_ij = l_ij d_j (i > j)
  T dinv[RMAX];
  T X[3][RMAX];
  bool ok = true;
#pragma unroll
  for (int q = 0; q < RMAX; ++q)
#pragma unroll
    for (int qp = q; qp < RMAX; ++qp) {
      // identity on the unused modes keeps the factorisation well defined
      const T a = v[q * RMAX - q * (q - 1) / 2 + (qp - q)];
      L[qp][q] = (q < r && qp < r) ? a : (q == qp ? T(1) : T(0));
    }
  // Crout LDL^T: u_ij = a_ij - sum_k u_ik l_jk, d_j = a_jj - sum_k u_jk l_jk
#pragma unroll
  for (int j = 0; j < RMAX; ++j) {
    T d = L[j][j];
#pragma unroll
    for (int k = 0; k < j; ++k) d -= U[j][k] * L[j][k];
    ok = ok && d > T(0);
    const T inv = rb_recip<T>(d);
    dinv[j] = inv;
#pragma unroll
    for (int i = j + 1; i < RMAX; ++i) {
      T u = L[i][j];
#pragma unroll
      for (int k = 0; k < j; ++k) u -= U[i][k] * L[j][k];
      U[i][j] = u;
      L[i][j] = u * inv;
    }
  }
#pragma unroll
  for (int l = 0; l < 3; ++l)
#pragma unroll
    for (int i = 0; i < RMAX; ++i) {
      T t = (i < r) ? v[NA + l * RMAX + i] : T(0);
#pragma unroll
      for (int k = 0; k < i; ++k) t -= L[i][k] * X[l][k];
      X[l][i] = t;
    }
  const int ls[6] = {0, 0, 0, 1, 1, 2}, lps[6] = {0, 1, 2, 1, 2, 2};
  T Z[3][RMAX];
#pragma unroll
  for (int l = 0; l < 3; ++l)
#pragma unroll
    for (int i = 0; i < RMAX; ++i) Z[l][i] = X[l][i] * dinv[i];
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    T acc = v[NA + 3 * RMAX + t];
#pragma unroll
    for (int i = 0; i < RMAX; ++i) acc -= Z[ls[t]][i] * X[lps[t]][i];
    S3[ls[t]][lps[t]] = (double)acc;
    S3[lps[t]][ls[t]] = (double)acc;
  }
  return ok;
}

// FP64 reference online stage: one thread per pair.  SAMPLES: the 64 samples of a
// wavefront on one patch, so that the table is read at uniform addresses
// (scalar loads): 65 536 pairs at m = 8 took 260 us with the lanes along the
// patches, 66 gathers per coefficient; 55 us so.  Few samples leave most of those
// lanes idle; on many patches they go along the patches.  Both do the same
// operations, hence the same bits.
typedef __attribute__((address_space(4))) const double rb_table_t;
template <int RMAX, typename TA, bool SAMPLES>
__global__ __launch_bounds__(64) void rb_apply_f64_kernel(RbApplyArgs ra, int64_t nsamples, unsigned groups) {
  const UpArgs& args = ra.up;
  const int m = args.m, Mc = args.ncx * args.ncy;
  int64_t s = (int64_t)blockIdx.x * 64 + threadIdx.x;
  int K;
  if constexpr (SAMPLES) {
    K = (int)(blockIdx.x / groups);
    s = (int64_t)(blockIdx.x % groups) * 64 + threadIdx.x;
  } else {
    const int64_t i = s;
    s = i / Mc;
    K = (int)(i - s * Mc);
  }
  if (s >= nsamples) return;
  const int64_t p = s * Mc + K;
  const TA* a = (const TA*)args.a + block_offset(s, K, args.ncx, args.ncy, m);
  const int64_t lda = (int64_t)args.ncx * m;
  constexpr int P = RMAX * (RMAX + 1) / 2 + 3 * RMAX + 6;
  double v[P];
#pragma unroll
  for (int q = 0; q < P; ++q) v[q] = 0.0;
  using Table = std::conditional_t<SAMPLES, const rb_table_t*, const double*>;
  Table G = (Table)(ra.G64 + (int64_t)K * ra.KD * ra.PP);
  for (int ey = 0; ey < m; ++ey)
    for (int ex = 0; ex < m; ++ex, G += ra.PP) {
      const double ae = ld(a, ey * lda + ex);
      if constexpr (SAMPLES) {
#pragma unroll
        for (int q = 0; q < P; ++q) v[q] += ae * G[q];
      } else {
        // each lane has cache lines of its own: a batch of loads takes what a line
        // holds before other wavefronts drive it out (8 samples of 96 x 96 patches
        // 487 us with loads and sums mixed, 362 so)
        constexpr int BATCH = 8;
#pragma unroll
        for (int q0 = 0; q0 < P; q0 += BATCH) {
          double t[BATCH];
#pragma unroll
          for (int q = q0; q < q0 + BATCH && q < P; ++q) t[q - q0] = G[q];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = q0; q < q0 + BATCH && q < P; ++q) v[q] += ae * t[q - q0];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  double S3[3][3];
  const bool ok = rb_small_solve<RMAX, double>(v, ra.rK[K], S3);
  store_packed(args.S + p * 10, S3);
  if (args.status) args.status[p] = ok ? STOMSFEM_OK : STOMSFEM_ENOTSPD;
}

// FP32 MFMA online stage.  Workgroup = 4 wavefronts = 128 samples of one
// patch.  C[128 x PP] = A[128 x KD] G[KD x PP] with v_mfma_f32_16x16x4f32 and
// FP32 accumulation (wavefront w computes rows 32w..32w+31, two row tiles,
// all PP/16 column tiles), the k dimension (the patch's m*m fine elements,
// padded to KD, a multiple of 64) in chunks of 64 staged in LDS: the chunk's
// coefficients of the 128 samples and its 64 rows of the patch's table,
// the next chunk's coefficients loaded into registers while the current one
// is multiplied.  Then one lane per sample does the FP32 r x r solve (the
// result rows pass through LDS, in the space of the staging buffers).
constexpr int RBA_SAMPLES = 128;
constexpr int RBA_KC = 64;
constexpr int RBA_LDA = RBA_KC + 4;
constexpr int RBA_PF = RBA_SAMPLES * RBA_KC / 256;  // coefficients per thread and chunk

// Workgroup order: one-dimensional grid of ntiles x M workgroups.  When a
// patch's coefficient row is shorter than a 128-byte cache line, the patch
// index runs fastest, so that neighbouring patches, which share the lines of
// a sample, are read by one L2: the hardware deals consecutive workgroups
// round-robin to the eight XCDs (each with its own L2), and the logical index
// L = (b mod 8) (n / 8) + b / 8 gives each XCD a contiguous range.
// Otherwise the sample tile runs fastest and consecutive workgroups share
// the patch's table.
//
// OS = true: the oversampled patches (rb_os.hip).  The block of element K is
// its patch (side m + 2 os_o, origin rbo_origin), the table is GO32 (PP =
// RBO_PO columns: A, Fh and the element sums U), and the per-sample epilogue
// is the FP64 solve for c and the recombination at K's corners (16 entries
// per pair).  vec_ok: every patch row starts on a 16-byte boundary.
//
// MT = true (plain variant, single-chunk tiles): a workgroup takes tpw
// consecutive sample tiles of its patch and the (tile, chunk) steps form one
// loop, so the next tile's coefficients are in flight during the current
// tile's products and solves (two wavefronts per SIMD kept for the extra
// prefetch registers).  MT = false: one tile per workgroup (tpw = 1).
template <int RMAX, int PP, typename TA, bool OS = false, bool MT = false>
__global__ __launch_bounds__(256, MT ? 2 : 1) void rb_apply_mfma_kernel(RbApplyArgs ra, int64_t ntiles,
                                                                       int patch_fast, int vec_ok, int tpw) {
  using f4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;
  const UpArgs& args = ra.up;
  const int m = args.m, Mc = args.ncx * args.ncy, KD = ra.KD;
  const int bs = OS ? m + 2 * ra.os_o : m, mm = bs * bs;  // block side and elements
  const int64_t ngroups = (ntiles + tpw - 1) / tpw, nb = ngroups * Mc, b = blockIdx.x;
  const int64_t L = (patch_fast && nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
  const int K = (int)(patch_fast ? L % Mc : L / ngroups);
  const int64_t tile0 = (patch_fast ? L / Mc : L % ngroups) * tpw;
  const int64_t lda = (int64_t)args.ncx * m;
  constexpr int AS_FLOATS = RBA_SAMPLES * RBA_LDA, GS_FLOATS = RBA_KC * PP;
  constexpr int CS_FLOATS = RBA_SAMPLES * (PP + 1);
  constexpr int SM_FLOATS = (AS_FLOATS + GS_FLOATS) > CS_FLOATS ? (AS_FLOATS + GS_FLOATS) : CS_FLOATS;
  __shared__ __align__(16) float smem[SM_FLOATS];
  float(*As)[RBA_LDA] = reinterpret_cast<float(*)[RBA_LDA]>(smem);
  float(*Gs)[PP] = reinterpret_cast<float(*)[PP]>(smem + AS_FLOATS);
  float(*Cs)[PP + 1] = reinterpret_cast<float(*)[PP + 1]>(smem);
  const int tid = threadIdx.x;
  const int kx = K % args.ncx, ky = K / args.ncx;
  const int bx0 = OS ? rbo_origin(kx, m, ra.os_o, args.ncx * m) : kx * m;
  const int by0 = OS ? rbo_origin(ky, m, ra.os_o, args.ncy * m) : ky * m;
  const int w = tid / 64, lane = tid % 64;
  constexpr int NTILE = PP / 16;
  f4 acc[2][NTILE];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < NTILE; ++t) acc[h][t] = f4{0.f, 0.f, 0.f, 0.f};
  const float* G = ra.G32 + (int64_t)K * KD * PP;
  // thread tid loads coefficient (i, e0 + c) of the tile starting at sample
  // s0 for idx = tid + 256 q, i = idx / KC
  auto load_chunk = [&](int64_t s0, int e0, float (&v)[RBA_PF]) {
#pragma unroll
    for (int q = 0; q < RBA_PF; ++q) {
      const int idx = tid + 256 * q, i = idx / RBA_KC, e = e0 + idx % RBA_KC;
      const int64_t s = s0 + i;
      float x = 0.0f;
      if (s < args.nsamples && e < mm) {
        const TA* a = (const TA*)args.a + s * (int64_t)(args.ncy * m) * lda;
        x = (float)ld(a, (int64_t)(by0 + e / bs) * lda + bx0 + e % bs);
      }
      v[q] = x;
    }
  };
  // block side in {8, 16, 32} with FP32 coefficients: a chunk of 64
  // elements is 64 / bs whole rows of the block, so each sample's share comes
  // in 16-byte loads (16 per sample and chunk: thread tid takes float4
  // f = idx % 16 of sample idx / 16, idx = tid + 256 q)
  const bool vec = std::is_same<TA, float>::value && vec_ok && (bs == 8 || bs == 16 || bs == 32);
  const int lm = bs == 8 ? 3 : bs == 16 ? 4 : 5;
  auto load_chunk_vec = [&](int64_t s0, int e0, float (&v)[RBA_PF]) {
#pragma unroll
    for (int q = 0; q < RBA_PF / 4; ++q) {
      const int idx = tid + 256 * q, i = idx >> 4, e = e0 + 4 * (idx & 15);
      const int64_t s = s0 + i;
      f4 x = f4{0.f, 0.f, 0.f, 0.f};
      if (s < args.nsamples && e < mm) {
        const float* a = (const float*)args.a + s * (int64_t)(args.ncy * m) * lda;
        x = *reinterpret_cast<const f4*>(a + (int64_t)(by0 + (e >> lm)) * lda + bx0 + (e & (bs - 1)));
      }
      v[4 * q] = x[0];
      v[4 * q + 1] = x[1];
      v[4 * q + 2] = x[2];
      v[4 * q + 3] = x[3];
    }
  };
  const int nch = KD / RBA_KC, nit = (MT ? tpw : 1) * nch;
  auto load_step = [&](int it, float (&v)[RBA_PF]) {
    const int64_t s0 = (tile0 + it / nch) * RBA_SAMPLES;
    const int e0 = (it % nch) * RBA_KC;
    if (vec)
      load_chunk_vec(s0, e0, v);
    else
      load_chunk(s0, e0, v);
  };
  float pf[RBA_PF];
  // one (tile, chunk) step: stage the coefficients and the table chunk, start
  // the next step's loads, accumulate the products
  auto step = [&](int it) {
    const int e0 = (it % nch) * RBA_KC;
    __syncthreads();  // the previous step's readers (products or solves) are done
    if (vec) {
#pragma unroll
      for (int q = 0; q < RBA_PF / 4; ++q) {
        const int idx = tid + 256 * q;
        *reinterpret_cast<f4*>(&As[idx >> 4][4 * (idx & 15)]) =
            f4{pf[4 * q], pf[4 * q + 1], pf[4 * q + 2], pf[4 * q + 3]};
      }
    } else {
#pragma unroll
      for (int q = 0; q < RBA_PF; ++q) {
        const int idx = tid + 256 * q;
        As[idx / RBA_KC][idx % RBA_KC] = pf[q];
      }
    }
    // the chunk's 64 table rows: contiguous, PP a multiple of 4, 16-byte loads
    static_assert(PP % 4 == 0 && (RBA_KC * PP) % (4 * 256) == 0, "table chunk in float4 per thread");
#pragma unroll
    for (int q = 0; q < RBA_KC * PP / (4 * 256); ++q) {
      const int idx = 4 * (tid + 256 * q);
      *reinterpret_cast<f4*>(&Gs[0][0] + idx) = *reinterpret_cast<const f4*>(G + (int64_t)e0 * PP + idx);
    }
    __syncthreads();
    if (it + 1 < nit) load_step(it + 1, pf);  // in flight during the products (and the solves)
#pragma unroll 4
    for (int kk = 0; kk < RBA_KC / 4; ++kk) {
      const float av0 = As[32 * w + (lane & 15)][4 * kk + (lane >> 4)];
      const float av1 = As[32 * w + 16 + (lane & 15)][4 * kk + (lane >> 4)];
#pragma unroll
      for (int t = 0; t < NTILE; ++t) {
        const float bv = Gs[4 * kk + (lane >> 4)][16 * t + (lane & 15)];
        acc[0][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av0, bv, acc[0][t], 0, 0, 0);
        acc[1][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av1, bv, acc[1][t], 0, 0, 0);
      }
    }
  };
  // a complete tile: its rows through LDS, then one lane per sample
  auto finish_tile = [&](int64_t tile) {
    __syncthreads();  // Cs overlays the staging buffers
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < NTILE; ++t) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Cs[32 * w + 16 * h + 4 * (lane >> 4) + v][16 * t + (lane & 15)] = acc[h][t][v];
        acc[h][t] = f4{0.f, 0.f, 0.f, 0.f};
      }
    __syncthreads();
    const int64_t s = tile * RBA_SAMPLES + tid;
    if (tid < RBA_SAMPLES && s < args.nsamples) {
      const int64_t p = s * Mc + K;
      if constexpr (OS) {
        double c[3][RMAX];
        const bool ok = rbo_coeffs<RMAX>(&Cs[tid][0], ra.rK[K], c);
        double S[4][4];
        const bool nonsing = rbo_recombine<RMAX>(c, &Cs[tid][RBO_H], ra.Pc + (int64_t)K * 4 * RBO_NF, S);
        double* out = args.S + p * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int lp = 0; lp < 4; ++lp) out[4 * i + lp] = S[i][lp];
        if (args.status) args.status[p] = (ok && nonsing) ? STOMSFEM_OK : STOMSFEM_ENOTSPD;
      } else {
        constexpr int P = RMAX * (RMAX + 1) / 2 + 3 * RMAX + 6;
        float v[P];
#pragma unroll
        for (int q = 0; q < P; ++q) v[q] = Cs[tid][q];
        double S3[3][3];
        const bool ok = rb_small_solve<RMAX, float>(v, ra.rK[K], S3);
        store_packed(args.S + p * 10, S3);
        if (args.status) args.status[p] = ok ? STOMSFEM_OK : STOMSFEM_ENOTSPD;
      }
    }
  };
  load_step(0, pf);
  if constexpr (!MT) {
    for (int it = 0; it < nch; ++it) step(it);
    finish_tile(tile0);
  } else {
    for (int it = 0; it < nit; ++it) {
      step(it);
      if (it % nch == nch - 1) finish_tile(tile0 + it / nch);
    }
  }
}

// Tiles per workgroup.  Where a tile is a single chunk (m <= 8) nothing
// overlaps its loads otherwise: about four workgroups per CU (1024) when the
// batch has that many tiles, at most eight tiles each (8x8 mesh, 16 384
// samples: 0.205 ms with one tile per workgroup, 0.175 ms with four, 0.170 ms
// with eight).  Longer tiles already overlap chunk with chunk, and grouping
// them only costs parallelism (32x32 mesh, H/h = 32: 6.2 ms with one, 6.8 ms
// with eight).
static int rba_tiles_per_workgroup(int64_t ntiles, int Mc, int KD) {
  if (KD > RBA_KC) return 1;
  const int64_t t = ntiles * Mc / 1024;
  return (int)(t < 1 ? 1 : t > 8 ? 8 : t);
}

int rb_pad_p(int rmax) { return ((rb_p(rmax) + 15) / 16) * 16; }
int rb_pad_kd(int m) { return ((m * m + RBA_KC - 1) / RBA_KC) * RBA_KC; }

hipError_t launch_rb_apply(const RbApplyArgs& ra, int a_dtype, bool f64, hipStream_t st) {
  const UpArgs& u = ra.up;
  if (u.npairs == 0) return hipSuccess;
  if (ra.rmax != 8) return hipErrorInvalidValue;
  if (f64) {
    const int64_t Mc = (int64_t)u.ncx * u.ncy, n = u.npairs / Mc, groups = (n + 63) / 64;
    // 1 and 8 samples along the samples / the patches, us: 96 x 96 patches at m = 8
    // 447 / 259, 452 / 361; 128 x 128 at m = 4 149 / 55, 151 / 126; 200 x 200 at m = 4
    // 447 / 104, 459 / 605; 64 x 64 at m = 8 179 / 171, 180 / 188; 32 x 32 63 / 170
    const bool patches = n <= 8 && Mc > 4096;
    const dim3 g((unsigned)(patches ? (u.npairs + 63) / 64 : groups * Mc)), block(64);
    const unsigned gr = (unsigned)groups;
    const bool f32 = a_dtype == STOMSFEM_F32;
    if (patches && f32)
      hipLaunchKernelGGL((rb_apply_f64_kernel<8, float, false>), g, block, 0, st, ra, n, gr);
    else if (patches)
      hipLaunchKernelGGL((rb_apply_f64_kernel<8, double, false>), g, block, 0, st, ra, n, gr);
    else if (f32)
      hipLaunchKernelGGL((rb_apply_f64_kernel<8, float, true>), g, block, 0, st, ra, n, gr);
    else
      hipLaunchKernelGGL((rb_apply_f64_kernel<8, double, true>), g, block, 0, st, ra, n, gr);
    return hipGetLastError();
  }
  if (ra.PP != 80 || ra.KD % RBA_KC != 0 || ra.KD < u.m * u.m) return hipErrorInvalidValue;
  const int Mc = u.ncx * u.ncy;
  const int64_t ntiles = (u.nsamples + RBA_SAMPLES - 1) / RBA_SAMPLES;
  const int tpw = rba_tiles_per_workgroup(ntiles, Mc, ra.KD);
  const int64_t nb = (ntiles + tpw - 1) / tpw * Mc;
  if (nb > 0x7fffffff) return hipErrorInvalidValue;
  const int elem = a_dtype == STOMSFEM_F32 ? 4 : 8;
  const int patch_fast = u.m * elem < 128 ? 1 : 0;
  // single-chunk tiles take the multi-tile variant
  if (ra.KD == RBA_KC) {
    if (a_dtype == STOMSFEM_F32)
      hipLaunchKernelGGL((rb_apply_mfma_kernel<8, 80, float, false, true>), dim3((unsigned)nb), dim3(256), 0, st, ra,
                         ntiles, patch_fast, 1, tpw);
    else
      hipLaunchKernelGGL((rb_apply_mfma_kernel<8, 80, double, false, true>), dim3((unsigned)nb), dim3(256), 0, st,
                         ra, ntiles, patch_fast, 1, tpw);
  } else {
    if (a_dtype == STOMSFEM_F32)
      hipLaunchKernelGGL((rb_apply_mfma_kernel<8, 80, float>), dim3((unsigned)nb), dim3(256), 0, st, ra, ntiles,
                         patch_fast, 1, tpw);
    else
      hipLaunchKernelGGL((rb_apply_mfma_kernel<8, 80, double>), dim3((unsigned)nb), dim3(256), 0, st, ra, ntiles,
                         patch_fast, 1, tpw);
  }
  return hipGetLastError();
}

hipError_t launch_rb_os_apply_mfma(const RbApplyArgs& ra, int a_dtype, hipStream_t st) {
  const UpArgs& u = ra.up;
  if (u.npairs == 0) return hipSuccess;
  const int bs = u.m + 2 * ra.os_o;
  if (ra.rmax != 8 || ra.PP != RBO_PO || ra.KD % RBA_KC != 0 || ra.KD < bs * bs || !ra.Pc)
    return hipErrorInvalidValue;
  const int Mc = u.ncx * u.ncy;
  const int64_t ntiles = (u.nsamples + RBA_SAMPLES - 1) / RBA_SAMPLES;
  const int tpw = 1;  // one tile per workgroup (the kernel's OS variant)
  const int64_t nb = ntiles * Mc;
  if (nb > 0x7fffffff) return hipErrorInvalidValue;
  const int elem = a_dtype == STOMSFEM_F32 ? 4 : 8;
  const int patch_fast = bs * elem < 128 ? 1 : 0;
  // patch rows on 16-byte boundaries: every origin is a multiple of 4 cells
  const int vec_ok = (u.m % 4 == 0 && ra.os_o % 4 == 0 && (u.ncx * u.m) % 4 == 0) ? 1 : 0;
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL((rb_apply_mfma_kernel<8, RBO_PO, float, true>), dim3((unsigned)nb), dim3(256), 0, st, ra,
                       ntiles, patch_fast, vec_ok, tpw);
  else
    hipLaunchKernelGGL((rb_apply_mfma_kernel<8, RBO_PO, double, true>), dim3((unsigned)nb), dim3(256), 0, st, ra,
                       ntiles, patch_fast, vec_ok, tpw);
  return hipGetLastError();
}

}  // namespace stomsfem
