// Batched coarse solve of the symmetric system for 4 <= ncx <= 32
// (eq. upscaleSUF): row-distributed LDL^T (band_rows.h), sixteen lanes per
// sample, four samples per wavefront, forward and backward pass in one
// launch.
//
// The interior coarse nodes in natural order give the nine-point band of the
// cell problems with n = ncx - 1 nodes per row, so the forward pass is theirs
// with the node's couplings read from the four element matrices around it (a
// panel ahead) and one right-hand side.  Pivot j's column of -L (rows j + 1
// ... j + ncx) goes to the workspace as it is formed, z = D^{-1} y to U.
//
// Backward pass L^T x = z by panels from the last: lane j takes its column
// (consecutive doubles, a panel ahead), adds the rows of the later blocks with
// x broadcast from the lane that holds it, and the panel's own 16 unknowns
// follow one by one.
//
// A batch of a few hundred samples leaves most SIMDs one wavefront or none, so
// the time is that of one wavefront's instruction stream: about 85 vector
// instructions per pivot at 17 <= ncx, 45 below.  Measured with both passes at
// 32 x 32, 1024 samples: 2.58 -> 0.38 ms; 16 x 16, 256 samples: 0.49 -> 0.06 ms
// (against one workgroup and a barrier per pivot).
#include "band_rows.h"
#include "coarse.h"

namespace stomsfem {

constexpr int CR_SAMPLES = 4;  // samples per wavefront

template <int NS, int MC>
__global__ __launch_bounds__(64, 2) void coarse_rows_kernel(CoarseArgs args) {
  __shared__ double img[CR_SAMPLES * RowImage<NS, MC>::SIZE];
  const int M = MC ? MC : args.ncx;
  const int ncy = args.ncy, n = M - 1, ny = ncy - 1, NI = n * ny, NP = (NI + 15) / 16;
  const int lane = threadIdx.x & 63, q = lane >> 4, r = lane & 15;

  int64_t s = (int64_t)blockIdx.x * CR_SAMPLES + q;
  const bool valid = s < args.nsamples;
  if (!valid) s = args.nsamples - 1;
  const double* S = args.S + s * (int64_t)M * ncy * 10;
  double* U = args.U + s * (int64_t)NI;
  // column j of -L at j M (rows j + 1 ... j + M); columns past the last
  // unknown share one more.  Lanes past the last sample repeat it and write
  // the same values to its slice.
  double* Lw = args.work + s * ((int64_t)NI * (M + 1) + 1);
  // whether row 16 b + r of the window (relative to the panel) lies in column j
  auto in_column = [&](int b, int j) { return MC == 16 * NS || 16 * b + r - j - 1 < M; };
  const double H = 1.0 / M;

  RowImage<NS, MC> im;
  im.init(img + q * RowImage<NS, MC>::SIZE, r, M);

  // the element-matrix entries around node (ix, iy) that its row needs:
  // elements SW, SE, NW, NE see it as local node 2, 3, 1, 0; packed indices
  // (0,0)=0 (0,1)=1 (0,2)=2 (0,3)=3 (1,1)=4 (1,2)=5 (1,3)=6 (2,2)=7 (2,3)=8 (3,3)=9
  int ix = r % n, iy = r / n;
  double e[10], fl;
  auto load_node = [&]() {
    if (iy < ny) {
      const double* sw = S + ((int64_t)iy * M + ix) * 10;
      const double* se = sw + 10;
      const double* nw = sw + (int64_t)M * 10;
      const double* ne = nw + 10;
      e[0] = sw[7];
      e[1] = se[9];
      e[2] = nw[4];
      e[3] = ne[0];
      e[4] = sw[8];
      e[5] = nw[1];
      e[6] = se[6];
      e[7] = sw[5];
      e[8] = se[3];
      e[9] = sw[2];
      fl = H * H;  // four elements, int_K p^l = H^2/4 each
      if (args.load) {
        const double* L = args.load + ((int64_t)iy * M + ix) * 4;
        fl = (L[2] + L[4 + 3]) + (L[(int64_t)M * 4 + 1] + L[((int64_t)M + 1) * 4 + 0]);
      }
    }
  };
  load_node();

  RowWindow<NS> W;
  W.zero();
  double f[NS + 1];
#pragma unroll
  for (int b = 0; b <= NS; ++b) f[b] = 0.0;
  unsigned long long bad = 0;  // lanes whose sample met a pivot that is not positive
  double cSW, cS, cSE, cW, cD;

  // row 16 (P + NS) + r: couplings to the image, load to f[NS]; then the
  // image's second turn, and the next row's entries on their way
  auto stage_row = [&]() {
    const bool in = iy < ny, w = ix >= 1, so = iy >= 1;
    cD = in ? (e[0] + e[1]) + (e[2] + e[3]) : 1.0;
    cW = in && w ? e[4] + e[5] : 0.0;
    cSE = in && so && ix <= n - 2 ? e[6] : 0.0;
    cS = in && so ? e[7] + e[8] : 0.0;
    cSW = in && so && w ? e[9] : 0.0;
    f[NS] = in ? fl : 0.0;
    im.put_left(cSW, cS, cSE);
    WAVE_SYNC();
  };
  auto stage_diag = [&]() {
    WAVE_SYNC();
    im.put_diag(cSW, cS, cSE, cW, cD);
    WAVE_SYNC();
    ix += 16;
    while (ix >= n) {
      ix -= n;
      ++iy;
    }
    load_node();
  };
  auto next_rhs = [&]() {
#pragma unroll
    for (int i = 0; i < NS; ++i) f[i] = f[i + 1];
  };

  // ---- initial window: the first NS row blocks ----
  static_for<0, NS>([&](auto bc) {
    constexpr int b = decltype(bc)::value;
    stage_row();
#pragma unroll
    for (int k = NS - b; k < NS; ++k)
#pragma unroll
      for (int c = 0; c < 16; ++c) W.template block<b>(NS, k)[c] = im.left(16 * k + c, cW);
    stage_diag();
#pragma unroll
    for (int c = 0; c < 16; ++c) W.template block<b>(NS, NS)[c] = im.diag(c);
    WAVE_SYNC();
    next_rhs();
  });

  auto panel = [&](auto phase, int P) {
    constexpr int PH = decltype(phase)::value;
    stage_row();
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int c = 0; c < 16; ++c) W.template block<PH>(NS, k)[c] = im.left(16 * k + c, cW);
    stage_diag();
    double own = 0.0;  // -1/d of the pivot row this lane holds
    double d = row_bcast<0>(W.template block<PH>(0, 0)[0]);
    static_for<0, 16>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      bad |= __builtin_amdgcn_ballot_w64(!(d > 0.0));
      asm volatile("" : "+s"(bad));  // test the pivot here: it need not stay live
      const double ninv = neg_recip(d);
      own = __builtin_amdgcn_inverse_ballot_w64(row_mask_at(j)) ? ninv : own;
      double col[NS + 1], nl[NS + 1];
#pragma unroll
      for (int b = 0; b <= NS; ++b) {
        col[b] = W.template block<PH>(b, 0)[j];
        nl[b] = col[b] * ninv;
      }
      // a pivot's own row and the rows above it keep their right-hand sides
      const bool below = __builtin_amdgcn_inverse_ballot_w64(row_mask_above(j));
      const double up = below ? nl[0] : 0.0;
      row_updates<j + 1, 16>(W.template block<PH>(0, 0), col[0], nl[0]);
      if constexpr (j < 15) d = row_bcast<j + 1>(W.template block<PH>(0, 0)[j + 1]);
      W.template block<PH>(NS, NS)[j] = im.diag(j);
      double* Lj = Lw + (int64_t)(16 * P + j < NI ? 16 * P + j : NI) * M + (r - j - 1);
      if (below ? in_column(0, j) : in_column(NS, j)) Lj[below ? 0 : 16 * NS] = below ? nl[0] : nl[NS];
      static_for<1, NS + 1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if constexpr (b < NS) {
          if (in_column(b, j)) Lj[16 * b] = nl[b];
        }
        row_updates<j + 1, 16>(W.template block<PH>(b, 0), col[0], nl[b]);
        row_rhs1<j>(f[b], f[0], nl[b]);
        static_for<1, b + 1>([&](auto kc) {
          constexpr int k = decltype(kc)::value;
          row_updates<0, (k == NS ? j + 1 : 16)>(W.template block<PH>(b, k), col[k], nl[b]);
        });
      });
      row_rhs1_own<j>(f[0], up);
    });
    if (valid && 16 * P + r < NI) U[16 * P + r] = -f[0] * own;
    WAVE_SYNC();
    next_rhs();
  };
#pragma unroll 1
  for (int P = 0; P < NP; P += RowWindow<NS>::PERIOD) {
    panel(std::integral_constant<int, 0>{}, P);
    if constexpr (NS == 2) {
      if (P + 1 < NP) panel(std::integral_constant<int, 1>{}, P + 1);
    }
  }
  if (args.status && r == 0 && valid) args.status[s] = ((bad >> lane) & 1) ? STOMSFEM_ENOTSPD : STOMSFEM_OK;

  // ---- backward pass ----
  __threadfence_block();  // the wavefront reads back what its lanes wrote
  double x[NS + 1];       // x of row blocks P + b, one per lane
#pragma unroll
  for (int b = 0; b <= NS; ++b) x[b] = 0.0;
  // lane j's column: rows of block 0 after j and of block NS up to j in
  // Ln[0], rows of block 1 in Ln[1] (0 where the column does not reach)
  double Ln[NS][16], zn = 0.0;
  auto load_panel = [&](int P) {
    const int j = 16 * P + r < NI ? 16 * P + r : NI;
    const double* at = Lw + (int64_t)j * M;
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int off = (b == 0 && i <= r ? 16 * NS : 16 * b) + i - r - 1;
        const bool in = MC == 16 * NS || off < M;
        const double v = at[in ? off : 0];
        Ln[b][i] = in ? v : 0.0;
      }
    zn = 16 * P + r < NI ? U[16 * P + r] : 0.0;
  };
  load_panel(NP - 1);
#pragma unroll 1
  for (int P = NP - 1; P >= 0; --P) {
    double L[NS][16], t = zn;
#pragma unroll
    for (int b = 0; b < NS; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) L[b][i] = Ln[b][i];
    if (P > 0) load_panel(P - 1);
#pragma unroll
    for (int b = NS; b > 0; --b) x[b] = x[b - 1];
    // rows of block NS (on and above the diagonal of the shared block), of
    // the blocks between, then the panel's own, last to first
    static_for<0, 16>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const bool below = __builtin_amdgcn_inverse_ballot_w64(~row_mask_above(i) & ~row_mask_at(i));  // lane < i
      row_rhs1<i>(t, x[NS], below ? 0.0 : L[0][i]);
      if constexpr (NS == 2) row_rhs1<i>(t, x[1], L[1][i]);
    });
    static_for<0, 15>([&](auto ic) {
      constexpr int i = 15 - decltype(ic)::value;
      const bool below = __builtin_amdgcn_inverse_ballot_w64(~row_mask_above(i) & ~row_mask_at(i));
      row_rhs1_own<i>(t, below ? L[0][i] : 0.0);
    });
    x[0] = 16 * P + r < NI ? t : 0.0;
    if (valid && 16 * P + r < NI) U[16 * P + r] = t;
  }
}

bool coarse_rows_supports(int ncx) { return ncx >= 4 && ncx <= 32; }

hipError_t launch_coarse_rows(const CoarseArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)((a.nsamples + CR_SAMPLES - 1) / CR_SAMPLES)), block(64);
  if (a.ncx == 8) hipLaunchKernelGGL((coarse_rows_kernel<1, 8>), grid, block, 0, st, a);
  else if (a.ncx == 16) hipLaunchKernelGGL((coarse_rows_kernel<1, 16>), grid, block, 0, st, a);
  else if (a.ncx < 16) hipLaunchKernelGGL((coarse_rows_kernel<1, 0>), grid, block, 0, st, a);
  else if (a.ncx == 32) hipLaunchKernelGGL((coarse_rows_kernel<2, 32>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((coarse_rows_kernel<2, 0>), grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace stomsfem
