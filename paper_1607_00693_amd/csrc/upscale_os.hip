// Oversampled local upscaling with the Petrov-Galerkin stiffness (Sec. 2.2,
// remark on oversampling; eq. stiffness_local_petrov).
//
// For the coarse element K the cell problems (eq. MsFEB) are solved on a
// patch of M = m + 2o fine cells per side around K (moved inside the domain
// at its edges), with the bilinear nodal functions g^j of the patch corners
// as boundary data: psi^j, j = 0..3, psi^3 = 1 - psi^0 - psi^1 - psi^2.  All
// the Petrov-Galerkin stiffness needs of them is linear in psi^j, so it comes
// out of the same sliding-window LDL^T as the plain path, with test vectors
// carried through the forward substitution beside the three data sets
// f^j = -K_IB g^j:
//   psi^j(x_k) = e_k . K_II^{-1} f^j          (corner x_k of K inside the patch)
//   A[j][l]    = psi^j . r^l,  r^l = K^K p^l  (K^K: fine stiffness of K's
//                elements; p^l: K's bilinear nodal functions)
// and, with K_II = L D L^T, u . K_II^{-1} v = sum_k (L^{-1}u)_k (L^{-1}v)_k / d_k.
// C = Psi^{-T} makes phi^i = sum_j C[i][j] psi^j nodal at K's corners, and
// S[l][l'] = int_K a grad phi^l . grad p^l' = (C A)[l][l'].
//
// Three kernels: upscale_os_rows.hip (patches of 4 to 32 cells, four pairs per
// wavefront), upscale_os_wide.hip (33 to 64 cells, one pair per wavefront) and
// the one below for the two smallest patches (one and four unknowns), one pair
// per lane.
#include "band_rows.h"
#include "os_common.h"

namespace stomsfem {

template <int M, typename TA>
__global__ __launch_bounds__(64) void upscale_os_small_kernel(OsRowsArgs args) {
  constexpr int n = M - 1, NI = n * n, NV = 10;
  const int64_t io = linear_block() * 64 + threadIdx.x;
  if (io >= (args.list ? args.nlist : args.up.npairs)) return;
  const int64_t p = args.list ? args.list[io] : io;
  const int m = args.up.m, o = args.o;
  const int ncx = args.up.ncx, ncy = args.up.ncy, Mc = ncx * ncy;
  const int64_t s = p / Mc;
  const int K = (int)(p - s * Mc), kx = K % ncx, ky = K / ncx;
  const int nfx = ncx * m, nfy = ncy * m;
  const int x0 = os_patch_origin(kx, m, o, nfx), y0 = os_patch_origin(ky, m, o, nfy);
  const int cx = kx * m - x0, cy = ky * m - y0;
  const TA* a = (const TA*)args.up.a + s * (int64_t)nfy * nfx + (int64_t)y0 * nfx + x0;
  double A[NI][NI], F[NI][NV];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int ix = i % n, iy = i / n;
    const TA* at = a + (int64_t)iy * nfx + ix;
    const double q4[4] = {ld(at, 0), ld(at, 1), ld(at, nfx), ld(at, (int64_t)nfx + 1)};
    os_right_hand_sides(q4, ix, iy, M, m, cx, cy, F[i]);
    NodeRow e;
    e.set(q4, ix, iy, n);
#pragma unroll
    for (int k = 0; k <= i; ++k) {
      const int dx = k % n - ix, dy = k / n - iy;
      A[i][k] = dy == 0 ? (dx == 0 ? e.D : e.W) : dx == 0 ? e.S : dx < 0 ? e.SW : e.SE;
    }
  }
  bool bad = false;
  double G[21];
#pragma unroll
  for (int t = 0; t < 21; ++t) G[t] = 0.0;
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    bad = bad || !(A[j][j] > 0.0);
    const double inv = 1.0 / A[j][j];
#pragma unroll
    for (int t = 0; t < 21; ++t) G[t] += F[j][t / 7] * inv * F[j][3 + t % 7];
#pragma unroll
    for (int i = j + 1; i < NI; ++i) {
      const double l = A[i][j] * inv;
#pragma unroll
      for (int k = j + 1; k <= i; ++k) A[i][k] -= l * A[k][j];
#pragma unroll
      for (int v = 0; v < NV; ++v) F[i][v] -= l * F[j][v];
    }
  }
  double mo[5] = {0, 0, 0, 0, 0};
  const double rm = 1.0 / m;
  for (int ey = 0; ey < m; ++ey)
    for (int ex = 0; ex < m; ++ex) {
      const double x = (ex + 0.5) * rm, y = (ey + 0.5) * rm, c = ld(a, (int64_t)(cy + ey) * nfx + cx + ex);
      mo[0] += c;
      mo[1] += c * x;
      mo[2] += c * y;
      mo[3] += c * (x * x);
      mo[4] += c * (y * y);
    }
  double out[16];
  const bool ok = os_recombine(M, m, cx, cy, mo, [&](int jv, int t) { return G[7 * jv + t]; }, out);
#pragma unroll
  for (int t = 0; t < 16; ++t) args.up.S[io * 16 + t] = out[t];
  if (args.up.status) args.up.status[io] = (bad || !ok) ? STOMSFEM_ENOTSPD : STOMSFEM_OK;
}

bool upscale_os_supports(int m, int o) { return m >= 1 && o >= 0 && m + 2 * o >= 2 && m + 2 * o <= 64; }

hipError_t launch_upscale_os_rows(const OsRowsArgs& args, int a_dtype, hipStream_t st);
hipError_t launch_upscale_os_wide(const OsRowsArgs& args, int a_dtype, hipStream_t st);

template <int M>
static void launch_small(const OsRowsArgs& args, int64_t n, int a_dtype, hipStream_t st) {
  const dim3 grid = grid_of_blocks((n + 63) / 64), block(64);
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL((upscale_os_small_kernel<M, float>), grid, block, 0, st, args);
  else
    hipLaunchKernelGGL((upscale_os_small_kernel<M, double>), grid, block, 0, st, args);
}

// list != nullptr: only the pairs list[i] (i < nlist) of the batch, their
// S and status written compactly at i.
hipError_t launch_upscale_os(const UpArgs& up, int o, int a_dtype, hipStream_t st, const int64_t* list,
                             int64_t nlist) {
  if (!upscale_os_supports(up.m, o)) return hipErrorInvalidValue;
  const int64_t n = list ? nlist : up.npairs;
  if (n <= 0) return hipSuccess;
  const OsRowsArgs args{up, o, list, nlist};
  const int M = up.m + 2 * o;
  // 16 rows per lane group hold the window of up to 32 cells in registers;
  // beyond, a pair needs the wavefront's 64 lanes
  if (M > 32) return launch_upscale_os_wide(args, a_dtype, st);
  if (M > 3) return launch_upscale_os_rows(args, a_dtype, st);
  if (M == 3) launch_small<3>(args, n, a_dtype, st);
  else launch_small<2>(args, n, a_dtype, st);
  return hipGetLastError();
}

}  // namespace stomsfem
