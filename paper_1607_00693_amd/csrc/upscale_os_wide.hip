// Oversampled Petrov-Galerkin local upscaling for patches of M = m + 2o = 33
// ... 64 cells per side: row-distributed elimination (band_rows.h) with one
// pair per wavefront.  The quantities are those of upscale_os_rows.hip.
//
// The live (M+1) x (M+1) window holds row blocks b = 0 (the panel's 16 pivots)
// ... NS = ceil(M / 16), each in one DPP row of 16 lanes: block b in DPP row
// b for b < 4.  A lane keeps its row's columns, block k of them in
// w[k][0..15].  At NS = 4 the entering block 4 shares DPP row 0 with the
// pivots: their columns 16.. are not needed below the diagonal, so w[1..3] of
// those lanes are block 4's, its first 16 columns have registers of their own
// (z0), and its diagonal block takes the registers that the pivot columns
// leave (as in band_rows.h).  Per pivot the column of 64 entries is replicated
// over the DPP rows with three permlane swaps per half, after which every
// update is a row-broadcast multiply-add within the DPP row.
//
// Right-hand sides: lane = row, ten registers.  The panel's own rows are
// substituted forward with the ten spread over the four DPP rows (three per
// DPP row, the pivot column being there in replica); the other rows take the
// panel's 16 pivots at its end, and the 21 Schur products are formed by 21
// lanes, both from the panel's y in LDS.  After each panel the window moves up
// by one DPP row and left by one column block through LDS, and the lanes of
// the entering block read its image.
//
// FP64-issue bound: at NS = 4 about 110 instructions per pivot (71 window
// updates, of them 32 useful by lane count) and 10 for the deferred
// right-hand sides.  Measured at 60 cells, 12 800 pairs: 50.6 -> 13.8 ms (15.9
// TFLOP/s) against the 55-lane tile layout it replaced.  The window's move is
// masked to the lanes that hold each block: all lanes taking part (LDS then
// busy 85% of the time) measured 17.5 ms.
#include "band_rows.h"
#include "os_common.h"

namespace stomsfem {

constexpr int OW_NV = 10;      // right-hand sides: lifts 0..2, corner units 0..3, r^0..2 (10, 11 unused)
constexpr int OW_SLD = 17;     // shift buffer row
constexpr int OW_SHIFT = 64 * OW_SLD;

template <int NS>
struct OwLds {
  static constexpr int LD = 16 * (NS + 1) + 2;
  double shift[OW_SHIFT];  // also the panel's right-hand sides: [v][row], from 192 on times -1/d
  double img[16 * LD];     // entering rows over the panel's columns; unused entries stay zero
};

// The vectors of the four DPP rows of v, each replicated over all rows.
__device__ __forceinline__ void replicate(double v, double* rep) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  uint32_t part[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t x = (uint32_t)(b >> (32 * h));
    const auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(s[0], s[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(s[1], s[1], false, false);
    part[h][0] = lo[0];
    part[h][1] = lo[1];
    part[h][2] = hi[0];
    part[h][3] = hi[1];
  }
#pragma unroll
  for (int d = 0; d < 4; ++d)
    rep[d] = __builtin_bit_cast(double, ((uint64_t)part[1][d] << 32) | part[0][d]);
}

constexpr unsigned long long OW_ROW0 = 0xffffull;

template <int NS, typename TA>
__global__ __launch_bounds__(64, 2) void upscale_os_wide_kernel(OsRowsArgs args) {
  static_assert(NS == 3 || NS == 4, "33 to 64 cells");
  __shared__ __attribute__((aligned(16))) OwLds<NS> sh;
  const int m = args.up.m, o = args.o, M = m + 2 * o;
  const int n = M - 1, NI = n * n, NP = (NI + 15) / 16;
  const int lane = threadIdx.x & 63, r = lane & 15;
  const bool zrow = NS == 4 ? lane < 16 : lane >= 48;  // lanes of the entering block

  const int64_t nout = args.list ? args.nlist : args.up.npairs, io = linear_block();  // output slot
  if (io >= nout) return;
  const int64_t p = args.list ? args.list[io] : io;
  const int ncx = args.up.ncx, ncy = args.up.ncy, Mc = ncx * ncy;
  const int64_t s = p / Mc;
  const int K = (int)(p - s * Mc), kx = K % ncx, ky = K / ncx;
  const int nfx = ncx * m, nfy = ncy * m;
  const int x0 = os_patch_origin(kx, m, o, nfx), y0 = os_patch_origin(ky, m, o, nfy);
  const int cx = kx * m - x0, cy = ky * m - y0;  // K's lower-left node in patch nodes
  const TA* a = (const TA*)args.up.a + s * (int64_t)nfy * nfx + (int64_t)y0 * nfx + x0;

  for (int i = lane; i < 16 * OwLds<NS>::LD; i += 64) sh.img[i] = 0.0;
  double* irow = sh.img + r * OwLds<NS>::LD;

  // every DPP row forms the entering row r (the same values)
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
  // couplings of row 16 (P + NS) + r into the image
  auto stage_row = [&]() {
    NodeRow e;
    e.set(q4, ix, iy, n);
    const int q0 = 16 * NS - M + r;
    irow[q0] = e.SW;
    irow[q0 + 1] = e.S;
    irow[q0 + 2] = e.SE;
    irow[16 * NS + r - 1] = e.W;
    irow[16 * NS + r] = e.D;
    WAVE_SYNC();
  };

  double w[NS][16], z0[16];
  double f[OW_NV];
#pragma unroll
  for (int k = 0; k < NS; ++k)
#pragma unroll
    for (int c = 0; c < 16; ++c) w[k][c] = 0.0;
#pragma unroll
  for (int c = 0; c < 16; ++c) z0[c] = 0.0;
#pragma unroll
  for (int v = 0; v < OW_NV; ++v) f[v] = 0.0;
  double G = 0.0;  // lane 7 jv + t < 21: -w^jv . t
  unsigned long long bad = 0;

  // right-hand sides of the entering row, where it lives
  auto stage_rhs = [&]() {
    double e[OW_NV];
    os_right_hand_sides(q4, ix, iy, M, m, cx, cy, e);
#pragma unroll
    for (int v = 0; v < OW_NV; ++v) f[v] = zrow ? e[v] : f[v];
    ix += 16;
    while (ix >= n) {
      ix -= n;
      ++iy;
    }
    load_quad();
  };

  // the next panel's window: DPP row d takes row d + 1's (mod 4), column block
  // k block k + 1's; block 0's registers hold the entering diagonal block
  double* put = sh.shift + lane * OW_SLD;
  const double* get = sh.shift + ((lane + 16) & 63) * OW_SLD;
  auto shift = [&]() {
    // block k + 1 is held from DPP row k + 1 on (and by the entering rows):
    // only those lanes take part
    double t0[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) t0[c] = w[0][c];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      WAVE_SYNC();
      if (NS == 4 ? (((lane + 48) & 63) >= 16 * k) : lane >= 16 * (k + 1)) {
#pragma unroll
        for (int c = 0; c < 16; ++c) put[c] = k + 1 < NS ? w[k + 1 < NS ? k + 1 : 0][c] : t0[c];
      }
      WAVE_SYNC();
      if (NS == 4 ? lane >= 16 * k : (lane >= 16 * k && lane < 48)) {
#pragma unroll
        for (int c = 0; c < 16; ++c) w[k][c] = get[c];
      }
    }
    WAVE_SYNC();
#pragma unroll
    for (int v = 0; v < OW_NV; ++v) put[v] = f[v];
    WAVE_SYNC();
#pragma unroll
    for (int v = 0; v < OW_NV; ++v) f[v] = get[v];
    WAVE_SYNC();
  };
  // columns of the entering rows from the image
  auto enter_left = [&]() {
    if constexpr (NS == 4) {
#pragma unroll
      for (int c = 0; c < 16; ++c) z0[c] = 0.0;
    }
    if (zrow) {
      if constexpr (NS == 4) {
#pragma unroll
        for (int c = 0; c < 16; ++c) z0[c] = irow[c];
      }
#pragma unroll
      for (int k = NS == 4 ? 1 : 0; k < NS; ++k)
#pragma unroll
        for (int c = 0; c < 16; ++c) w[k][c] = irow[16 * k + c];
    }
  };

  // ---- initial window: the first NS row blocks ----
#pragma unroll 1
  for (int b = 0; b < NS; ++b) {
    stage_row();
    enter_left();
    // diagonal block in the place of block 0, whose columns lie outside the
    // matrix until the window is full
#pragma unroll
    for (int c = 0; c < 16; ++c) w[0][c] = irow[16 * NS + c];
    WAVE_SYNC();
    stage_rhs();
    shift();
  }

#pragma unroll 1
  for (int P = 0; P < NP; ++P) {
    stage_row();
    enter_left();
    // the panel rows' right-hand sides v = 4 i + d in DPP row d
    double fx[3];
    if (lane < 16) {
#pragma unroll
      for (int v = 0; v < OW_NV; ++v) sh.shift[v * 16 + r] = f[v];
    }
    WAVE_SYNC();
#pragma unroll
    for (int i = 0; i < 3; ++i) fx[i] = sh.shift[i * 64 + lane];
    WAVE_SYNC();
    double own = 0.0;  // -1/d of pivot row r, in every DPP row
    double cc[16];     // pivot columns at the rows below the panel
    static_for<0, 16>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const double col = w[0][j];
      double rep[4];
      replicate(col, rep);
      const double d = row_bcast<j>(rep[0]);
      bad |= __builtin_amdgcn_ballot_w64(!(d > 0.0));
      asm volatile("" : "+s"(bad));  // test the pivot here: it need not stay live
      const double ninv = neg_recip(d);
      own = __builtin_amdgcn_inverse_ballot_w64(row_mask_at(j)) ? ninv : own;
      const double nl0 = col * ninv;
      const double up = rep[0] * (__builtin_amdgcn_inverse_ballot_w64(row_mask_above(j)) ? ninv : 0.0);
      const double dg = irow[16 * NS + j];
      if constexpr (NS == 4) {
        const double nz = z0[j] * ninv;
        cc[j] = __builtin_amdgcn_inverse_ballot_w64(OW_ROW0) ? z0[j] : col;
        const double nlc = cc[j] * ninv;
        w[0][j] = __builtin_amdgcn_inverse_ballot_w64(OW_ROW0) ? dg : col;
        row_updates<j + 1, 16>(w[0], rep[0], nl0);
        row_updates<j + 1, 16>(z0, rep[0], nz);
        row_updates<0, 16>(w[1], rep[1], nlc);
        row_updates<0, 16>(w[2], rep[2], nlc);
        row_updates<0, 16>(w[3], rep[3], nlc);
        row_updates<0, j + 1>(w[0], z0[j], nz);
      } else {
        cc[j] = col;
        w[0][j] = dg;
        row_updates<j + 1, 16>(w[0], rep[0], nl0);
        row_updates<0, 16>(w[1], rep[1], nl0);
        row_updates<0, 16>(w[2], rep[2], nl0);
        row_updates<0, j + 1>(w[0], col, nl0);
      }
      row_rhs3_own<j>(fx, up);
    });
    WAVE_SYNC();
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      sh.shift[i * 64 + lane] = fx[i];
      sh.shift[192 + i * 64 + lane] = fx[i] * own;
    }
    WAVE_SYNC();
    double z[OW_NV];
#pragma unroll
    for (int v = 0; v < OW_NV; ++v) z[v] = sh.shift[192 + v * 16 + r];
    if (lane < 21) {
      const double* zl = sh.shift + 192 + (lane / 7) * 16;
      const double* yt = sh.shift + (3 + lane % 7) * 16;
#pragma unroll
      for (int i = 0; i < 16; ++i) G += zl[i] * yt[i];
    }
    stage_rhs();
    static_for<0, 16>([&](auto jc) { row_rhs10<decltype(jc)::value>(f, z, cc[decltype(jc)::value]); });
    shift();
  }

  // ---- moments of the coefficient over K ----
  double mo[5] = {0, 0, 0, 0, 0};
  {
    const TA* ak = a + (int64_t)cy * nfx + cx;
    const double rm = 1.0 / m;
#pragma unroll 1
    for (int i = lane; i < m * m; i += 64) {
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
    for (int i = 32; i > 0; i >>= 1) mo[t] += __shfl_xor(mo[t], i, 64);
  WAVE_SYNC();
  if (lane < 21) sh.shift[lane] = -G;
  WAVE_SYNC();
  if (lane == 0) {
    double out[16];
    const bool ok = os_recombine(M, m, cx, cy, mo, [&](int jv, int t) { return sh.shift[7 * jv + t]; }, out);
    double* dst = args.up.S + io * 16;
#pragma unroll
    for (int t = 0; t < 16; ++t) dst[t] = out[t];
    if (args.up.status) args.up.status[io] = (bad != 0 || !ok) ? STOMSFEM_ENOTSPD : STOMSFEM_OK;
  }
}

template <int NS>
static void launch_ow(const OsRowsArgs& args, int a_dtype, hipStream_t st) {
  const int64_t n = args.list ? args.nlist : args.up.npairs;
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL((upscale_os_wide_kernel<NS, float>), grid_of_blocks(n), dim3(64), 0, st, args);
  else
    hipLaunchKernelGGL((upscale_os_wide_kernel<NS, double>), grid_of_blocks(n), dim3(64), 0, st, args);
}

hipError_t launch_upscale_os_wide(const OsRowsArgs& args, int a_dtype, hipStream_t st) {
  const int M = args.up.m + 2 * args.o;
  if (M <= 32 || M > 64) return hipErrorInvalidValue;
  if (M <= 48) launch_ow<3>(args, a_dtype, st);
  else launch_ow<4>(args, a_dtype, st);
  return hipGetLastError();
}

}  // namespace stomsfem
