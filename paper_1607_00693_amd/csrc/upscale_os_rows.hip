// Oversampled Petrov-Galerkin local upscaling for patches of M = m + 2o = 4
// ... 32 cells per side, row-distributed (band_rows.h; Sec. 2.2 remark on
// oversampling, eq. stiffness_local_petrov).
//
// The quantities of upscale_os.hip: psi^j = p^j + w^j with K_II w^j = f^j =
// -(K p^j)_I on the patch, and the values w^j(x_k) at K's corners and w^j . r^l,
// r^l = K^K p^l, as Schur products f^j . K_II^{-1} t with seven test vectors
// t, so the patch solutions are never formed.  p^j is the bilinear function on
// the whole patch (not a lift of its boundary values), so f^j and r^l come
// from coefficient differences in closed form and psi's part from p^j is a
// handful of moments of the coefficient over K.
//
// Four pairs per wavefront.  The ten right-hand sides (three lifts, four
// corner units, r^0..2) ride along as one more row block whose lane v is
// right-hand side v and whose columns are the unknowns: the update by a pivot
// is the same broadcast multiply-add per column, and lane v accumulates its
// products with the three lifts from the broadcast of its own pivot entry.
//
// FP64-issue bound: at M = 24 a pivot costs 40 window instructions on average,
// 28 for the right-hand sides and about 20 for the pivot and the products.
// Measured at M = 24, 131 072 pairs: 12.2 -> 3.4 ms (22.9 TFLOP/s) against the
// ten-lane tile layout it replaced, which moved panel columns and right-hand
// sides through LDS.
#include "band_rows.h"
#include "os_common.h"

namespace stomsfem {

constexpr int OR_NV = 10;    // right-hand sides
constexpr int OR_LD = 11;    // LDS row of the entering right-hand sides (entry 10 stays 0)
constexpr int OR_PAIRS = 4;  // pairs per wavefront

template <int NS, int MC, typename TA>
__global__ __launch_bounds__(64, (NS == 1 ? 3 : 2)) void upscale_os_rows_kernel(OsRowsArgs args) {
  __shared__ double img[OR_PAIRS * RowImage<NS, MC>::SIZE];
  __shared__ double rhs_all[OR_PAIRS][16][OR_LD];
  const int m = args.up.m, o = args.o;
  const int M = MC ? MC : m + 2 * o;
  const int n = M - 1, NI = n * n, NP = (NI + 15) / 16;
  const int lane = threadIdx.x & 63, q = lane >> 4, r = lane & 15;

  const int64_t nout = args.list ? args.nlist : args.up.npairs;
  int64_t io = linear_block() * OR_PAIRS + q;  // output slot
  const bool valid = io < nout;
  if (!valid) io = nout - 1;
  const int64_t p = args.list ? args.list[io] : io;
  const int ncx = args.up.ncx, ncy = args.up.ncy, Mc = ncx * ncy;
  const int64_t s = p / Mc;
  const int K = (int)(p - s * Mc), kx = K % ncx, ky = K / ncx;
  const int nfx = ncx * m, nfy = ncy * m;
  const int x0 = os_patch_origin(kx, m, o, nfx), y0 = os_patch_origin(ky, m, o, nfy);
  const int cx = kx * m - x0, cy = ky * m - y0;  // K's lower-left node in patch nodes
  const TA* a = (const TA*)args.up.a + s * (int64_t)nfy * nfx + (int64_t)y0 * nfx + x0;

  RowImage<NS, MC> im;
  im.init(img + q * RowImage<NS, MC>::SIZE, r, M);
  double(*rhs)[OR_LD] = rhs_all[q];
  rhs[r][OR_NV] = 0.0;
  const int v = r < OR_NV ? r : OR_NV;  // this lane's right-hand side

  int ix = r % n, iy = r / n;
  double q4[4];
  auto load_quad = [&]() {
    if (iy < n) {
      const TA* at = a + (int64_t)iy * nfx + ix;
      q4[0] = ld(at, 0);
      q4[1] = ld(at, 1);
      q4[2] = ld(at, nfx);
      q4[3] = ld(at, (int64_t)nfx + 1);
    } else {
      q4[0] = q4[1] = q4[2] = q4[3] = 0.0;
    }
  };
  load_quad();

  RowWindow<NS> W;
  W.zero();
  double R[NS][16];  // columns of block k at (k + phase) mod NS; block NS in the place of block 0
#pragma unroll
  for (int k = 0; k < NS; ++k)
#pragma unroll
    for (int c = 0; c < 16; ++c) R[k][c] = 0.0;
  double acc[3] = {0.0, 0.0, 0.0};  // -f^jv . K_II^{-1} (this lane's right-hand side)
  unsigned long long bad = 0;  // lanes whose pair met a pivot that is not positive
  NodeRow e;

  // row 16 (P + NS) + r: couplings to the image, right-hand sides to LDS
  auto stage_row = [&]() {
    e.set(q4, ix, iy, n);
    im.put_left(e.SW, e.S, e.SE);
    double f[OR_NV];
    os_right_hand_sides(q4, ix, iy, M, m, cx, cy, f);
#pragma unroll
    for (int t = 0; t < OR_NV; ++t) rhs[r][t] = f[t];
    WAVE_SYNC();
  };
  auto stage_diag = [&]() {
    WAVE_SYNC();
    im.put_diag(e.SW, e.S, e.SE, e.W, e.D);
    WAVE_SYNC();
    ix += 16;
    while (ix >= n) {
      ix -= n;
      ++iy;
    }
    load_quad();
  };

  // ---- initial window: the first NS row blocks ----
  static_for<0, NS>([&](auto bc) {
    constexpr int b = decltype(bc)::value;
    stage_row();
#pragma unroll
    for (int k = NS - b; k < NS; ++k)
#pragma unroll
      for (int c = 0; c < 16; ++c) W.template block<b>(NS, k)[c] = im.left(16 * k + c, e.W);
    stage_diag();
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      W.template block<b>(NS, NS)[c] = im.diag(c);
      R[b][c] = rhs[c][v];
    }
    WAVE_SYNC();
  });

  auto panel = [&](auto phase) {
    constexpr int PH = decltype(phase)::value;
    stage_row();
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int c = 0; c < 16; ++c) W.template block<PH>(NS, k)[c] = im.left(16 * k + c, e.W);
    stage_diag();
    double d = row_bcast<0>(W.template block<PH>(0, 0)[0]);
    static_for<0, 16>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      bad |= __builtin_amdgcn_ballot_w64(!(d > 0.0));
      asm volatile("" : "+s"(bad));  // test the pivot here: it need not stay live
      const double ninv = neg_recip(d);
      double col[NS + 1], nl[NS + 1];
#pragma unroll
      for (int b = 0; b <= NS; ++b) {
        col[b] = W.template block<PH>(b, 0)[j];
        nl[b] = col[b] * ninv;
      }
      row_updates<j + 1, 16>(W.template block<PH>(0, 0), col[0], nl[0]);
      if constexpr (j < 15) d = row_bcast<j + 1>(W.template block<PH>(0, 0)[j + 1]);
      W.template block<PH>(NS, NS)[j] = im.diag(j);
      const double y = R[PH][j], nr = y * ninv;
      row_lifts3(acc, y, nr);
      R[PH][j] = rhs[j][v];
      row_updates<j + 1, 16>(R[PH], col[0], nr);
      static_for<1, NS + 1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        // with m known, the entering rows need no update before they are reached
        constexpr bool reached = b < NS || MC == 0 || j >= 16 * NS - MC;
        if constexpr (reached) {
          row_updates<j + 1, 16>(W.template block<PH>(b, 0), col[0], nl[b]);
          static_for<1, b + 1>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int c1 = k < NS ? 16 : j + 1 - (MC ? 16 * NS - MC : 0);
            row_updates<0, c1>(W.template block<PH>(b, k), col[k], nl[b]);
          });
        }
        constexpr int c1 = b < NS ? 16 : j + 1 - (MC ? 16 * NS - MC : 0);
        if constexpr (c1 > 0) row_updates<0, c1>(R[(b + PH) % NS], col[b], nr);
      });
    });
    WAVE_SYNC();
  };
#pragma unroll 1
  for (int P = 0; P < NP; P += NS) {
    panel(std::integral_constant<int, 0>{});
    if constexpr (NS == 2) {
      if (P + 1 < NP) panel(std::integral_constant<int, 1>{});
    }
  }

  // ---- moments of the coefficient over K ----
  double mo[5] = {0, 0, 0, 0, 0};
  {
    const TA* ak = a + (int64_t)cy * nfx + cx;
    const double rm = 1.0 / m;
#pragma unroll 1
    for (int i = r; i < m * m; i += 16) {
      const int ey = i / m, ex = i - ey * m;
      const double x = (ex + 0.5) * rm, y = (ey + 0.5) * rm, c = ld(ak, (int64_t)ey * nfx + ex);
      mo[0] += c;
      mo[1] += c * x;
      mo[2] += c * y;
      mo[3] += c * (x * x);
      mo[4] += c * (y * y);
    }
  }
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) mo[t] += __shfl_xor(mo[t], d, 16);
  WAVE_SYNC();
  if (r < OR_NV)
    for (int jv = 0; jv < 3; ++jv) rhs[jv][r] = -acc[jv];
  WAVE_SYNC();
  if (r == 0 && valid) {
    double out[16];
    const bool ok = os_recombine(M, m, cx, cy, mo, [&](int jv, int t) { return rhs[jv][3 + t]; }, out);
    double* dst = args.up.S + io * 16;
#pragma unroll
    for (int t = 0; t < 16; ++t) dst[t] = out[t];
    if (args.up.status) args.up.status[io] = (((bad >> lane) & 1) || !ok) ? STOMSFEM_ENOTSPD : STOMSFEM_OK;
  }
}

template <int NS, int MC>
static void launch_or(const OsRowsArgs& args, int a_dtype, hipStream_t st) {
  const int64_t n = args.list ? args.nlist : args.up.npairs;
  const dim3 grid = grid_of_blocks((n + OR_PAIRS - 1) / OR_PAIRS), block(64);
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL((upscale_os_rows_kernel<NS, MC, float>), grid, block, 0, st, args);
  else
    hipLaunchKernelGGL((upscale_os_rows_kernel<NS, MC, double>), grid, block, 0, st, args);
}

hipError_t launch_upscale_os_rows(const OsRowsArgs& args, int a_dtype, hipStream_t st) {
  const int M = args.up.m + 2 * args.o;
  if (M < 4 || M > 32) return hipErrorInvalidValue;
  // sizes of the ratios 2 and 3 at H/h = 8, 10, 12 and 16 have their bandwidth compiled in
  if (M == 16) launch_or<1, 16>(args, a_dtype, st);
  else if (M < 16) launch_or<1, 0>(args, a_dtype, st);
  else if (M == 20) launch_or<2, 20>(args, a_dtype, st);
  else if (M == 24) launch_or<2, 24>(args, a_dtype, st);
  else if (M == 30) launch_or<2, 30>(args, a_dtype, st);
  else if (M == 32) launch_or<2, 32>(args, a_dtype, st);
  else launch_or<2, 0>(args, a_dtype, st);
  return hipGetLastError();
}

}  // namespace stomsfem
