// Local upscaling for 9 <= m <= 32: row-distributed sliding-window LDL^T.
//
// Mathematics (Sec. 2.2 eqs. MsFEB and stiffness_local): with phi^l = p^l + w,
// p^l the bilinear corner function on the whole coarse element and w = 0 on
// its boundary, K_II w = f^l := -(K p^l)_I and
//     S_ll' = p^l . K p^l'  -  f^l . K_II^{-1} f^l' .
// K_II = L D L^T in natural order (half-bandwidth m), y = L^{-1} f, and the
// second term is sum_j y_j^l y_j^l' / d_j, so the factor is consumed as it is
// produced and never stored.  (p^l on the whole element instead of a lift of
// the boundary values alone: f^l then needs the coefficient differences
// around a node only, with no test for the boundary, and the two terms of S
// are of the size of S instead of m times larger.)
//
// Layout (band_rows.h).  Sixteen lanes per (element, sample) pair, four pairs
// per wavefront; the live (m+1) x (m+1) window sits in registers, lane r
// holding the rows i = r (mod 16), and is eliminated in panels of 16 pivots
// with compile-time register indices.  NS = ceil(m / 16) row blocks follow
// the panel's own.  Per panel each lane forms one entering row from the four
// coefficients around its node (loaded a panel ahead) and spreads its five
// nonzeros over the columns through LDS, whose zeros are written once.
//
// FP64-issue bound: per pivot at m = 32, 63 update instructions (33 of 63
// lane-FMAs useful: the triangles of the 16 x 16 blocks and the rows not yet
// reached cost the rest), 9 for the right-hand sides and about 15 for the
// pivot itself, shared by four pairs.  Measured on 1 048 576 pairs against the
// ten-lane tile layout it replaced (T x T tiles, panel columns and triangular
// solves through LDS): m = 32, 102.1 -> 46.4 ms (27.9 TFLOP/s); m = 16 from
// FP32 coefficients, 13.6 -> 6.2 ms.  Copying the window between panels
// instead of taking turns cost 49.5 ms at m = 32.
#include "band_rows.h"

namespace stomsfem {

constexpr int RW_PAIRS = 4;  // pairs per wavefront

// One wavefront's four pairs wtile * 4 + q.  MC: m at compile time, or 0
// (m from the arguments, any 16 (NS - 1) < m <= 16 NS).  img: the wavefront's
// LDS images.
template <int NS, int MC, typename TA>
__device__ __forceinline__ void rows_wave(const UpArgs& args, int64_t wtile, int lane, double* img) {
  const int M = MC ? MC : args.m;
  const int n = M - 1, NI = n * n, NP = (NI + 15) / 16;
  const int r = lane & 15;

  int64_t p = wtile * RW_PAIRS + (lane >> 4);
  const bool valid = p < args.npairs;
  if (!valid) p = args.npairs - 1;
  const int Mc = args.ncx * args.ncy;
  const int64_t s = p / Mc;
  const int K = (int)(p - s * Mc);
  const TA* a = (const TA*)args.a + block_offset(s, K, args.ncx, args.ncy, M);
  const int64_t lda = (int64_t)args.ncx * M;
  const double rm = 1.0 / M;
  RowImage<NS, MC> im;
  im.init(img + (lane >> 4) * RowImage<NS, MC>::SIZE, r, M);

  // node of the row entering next, (ix, iy), and its four coefficients
  int ix = r % n, iy = r / n;
  double q4[4];
  auto load_quad = [&]() {
    if (iy < n) {
      const TA* at = a + iy * lda + ix;
      q4[0] = ld(at, 0);
      q4[1] = ld(at, 1);
      q4[2] = ld(at, lda);
      q4[3] = ld(at, lda + 1);
    } else {
      q4[0] = q4[1] = q4[2] = q4[3] = 0.0;
    }
  };
  load_quad();

  RowWindow<NS> W;
  W.zero();
  double f[NS + 1][3];
#pragma unroll
  for (int b = 0; b <= NS; ++b) f[b][0] = f[b][1] = f[b][2] = 0.0;
  double sc[6] = {0, 0, 0, 0, 0, 0};
  unsigned long long bad = 0;  // lanes whose pair met a pivot that is not positive
  NodeRow e;

  // row 16 (P + NS) + r: couplings to the image, right-hand sides to f[NS];
  // then the image's second turn, and the next row's coefficients on their way
  auto stage_row = [&]() {
    e.set(q4, ix, iy, n);
    im.put_left(e.SW, e.S, e.SE);
    bilinear_load(q4[0], q4[1], q4[2], q4[3], (ix + 0.5) * rm, (iy + 0.5) * rm, rm, f[NS]);
#pragma unroll
    for (int l = 0; l < 3; ++l) f[NS][l] = -f[NS][l];
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
  auto next_rhs = [&]() {
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int l = 0; l < 3; ++l) f[i][l] = f[i + 1][l];
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
    for (int c = 0; c < 16; ++c) W.template block<b>(NS, NS)[c] = im.diag(c);
    WAVE_SYNC();
    next_rhs();
  });

  auto panel = [&](auto phase) {
    constexpr int PH = decltype(phase)::value;
    stage_row();
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int c = 0; c < 16; ++c) W.template block<PH>(NS, k)[c] = im.left(16 * k + c, e.W);
    stage_diag();
    double own = 0.0;  // -1/d of the pivot row this lane holds
    double d = row_bcast<0>(W.template block<PH>(0, 0)[0]);
    static_for<0, 16>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      bad |= __builtin_amdgcn_ballot_w64(!(d > 0.0));
      asm volatile("" : "+s"(bad));  // test the pivot here: it need not stay live
      const double ninv = neg_recip(d);
      own = __builtin_amdgcn_inverse_ballot_w64(row_mask_at(j)) ? ninv : own;
      // a pivot's own row and the rows above it keep their right-hand sides
      const double up = __builtin_amdgcn_inverse_ballot_w64(row_mask_above(j)) ? ninv : 0.0;
      double col[NS + 1], nl[NS + 1];
#pragma unroll
      for (int b = 0; b <= NS; ++b) {
        col[b] = W.template block<PH>(b, 0)[j];
        nl[b] = col[b] * (b == 0 ? up : ninv);
      }
      row_updates<j + 1, 16>(W.template block<PH>(0, 0), col[0], nl[0]);
      if constexpr (j < 15) d = row_bcast<j + 1>(W.template block<PH>(0, 0)[j + 1]);
      W.template block<PH>(NS, NS)[j] = im.diag(j);
      static_for<1, NS + 1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        row_updates<j + 1, 16>(W.template block<PH>(b, 0), col[0], nl[b]);
        row_rhs3<j>(f[b], f[0], nl[b]);
        static_for<1, b + 1>([&](auto kc) {
          constexpr int k = decltype(kc)::value;
          row_updates<0, (k == NS ? j + 1 : 16)>(W.template block<PH>(b, k), col[k], nl[b]);
        });
      });
      row_rhs3_own<j>(f[0], nl[0]);
    });
    // -y y^T / d of the panel's 16 rows, one per lane
    const double z0 = f[0][0] * own, z1 = f[0][1] * own, z2 = f[0][2] * own;
    sc[0] += z0 * f[0][0];
    sc[1] += z0 * f[0][1];
    sc[2] += z0 * f[0][2];
    sc[3] += z1 * f[0][1];
    sc[4] += z1 * f[0][2];
    sc[5] += z2 * f[0][2];
    WAVE_SYNC();
    next_rhs();
  };
#pragma unroll 1
  for (int P = 0; P < NP; P += RowWindow<NS>::PERIOD) {
    panel(std::integral_constant<int, 0>{});
    if constexpr (NS == 2) {
      if (P + 1 < NP) panel(std::integral_constant<int, 1>{});
    }
  }

  // ---- p^l . K p^l' over the elements: moments of a about the element
  //      centres (the gradients of p^l are linear in them) ----
  double mo[5] = {0, 0, 0, 0, 0};  // sum of a, a x, a y, a x^2, a y^2
#pragma unroll 1
  for (int ey = 0; ey < M; ++ey) {
    const double y = (ey + 0.5) * rm;
    double r0 = 0.0;
    for (int ex = r; ex < M; ex += 16) {
      const double x = (ex + 0.5) * rm, v = ld(a, ey * lda + ex);
      r0 += v;
      mo[1] += v * x;
      mo[3] += v * (x * x);
    }
    mo[0] += r0;
    mo[2] += r0 * y;
    mo[4] += r0 * (y * y);
  }
  {
    // grad p^0 = -(1-y, 1-x), grad p^1 = (1-y, -x), grad p^2 = (y, x); twists
    // +, -, + with energy rm^2 / 6 each (per element, unit coefficient, rm^2
    // outside)
    const double s0 = mo[0], sx = mo[1], sy = mo[2], sxx = mo[3], syy = mo[4];
    const double u2 = s0 - 2.0 * sy + syy, v2 = s0 - 2.0 * sx + sxx;  // sums of a (1-y)^2, a (1-x)^2
    const double uy = sy - syy, vx = sx - sxx;                       // sums of a y (1-y), a x (1-x)
    const double tw = s0 * (rm * rm / 6.0);
    const double e[6] = {u2 + v2 + tw, vx - u2 - tw, tw - uy - vx, u2 + sxx + tw, uy - sxx - tw, syy + sxx + tw};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      double v = rm * rm * e[t] + sc[t];  // sc holds -sum y y^T / d
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 16);
      sc[t] = v;
    }
  }
  if (r == 0 && valid) {
    const double s3[3][3] = {{sc[0], sc[1], sc[2]}, {sc[1], sc[3], sc[4]}, {sc[2], sc[4], sc[5]}};
    store_packed(args.S + p * 10, s3);
    if (args.status) args.status[p] = ((bad >> lane) & 1) ? STOMSFEM_ENOTSPD : STOMSFEM_OK;
  }
}

// Registers allow two wavefronts per SIMD at NS = 2 and three at NS = 1; at
// m = 16 the image leaves room for four, and the cap of 128 registers (two to
// four spilled outside the panel loop) measured 6.2 against 6.45 ms.
template <int NS, int MC, typename TA, int WV>
__global__ __launch_bounds__(64 * WV, (NS == 1 ? (MC == 16 ? 4 : 3) : 2)) void upscale_rows_kernel(UpArgs args) {
  // WV independent wavefronts per workgroup (a launch-shape choice only)
  __shared__ __attribute__((aligned(16))) double img[WV][RW_PAIRS * RowImage<NS, MC>::SIZE];
  const int wave = threadIdx.x >> 6;
  rows_wave<NS, MC, TA>(args, linear_block() * WV + wave, threadIdx.x & 63, img[wave]);
}
bool rows_supports(int m) { return m >= 9 && m <= 32; }

template <int NS, int MC, int WV>
static hipError_t launch_r(const UpArgs& args, int a_dtype, hipStream_t st) {
  const int64_t per_block = (int64_t)RW_PAIRS * WV;
  const int64_t blocks = (args.npairs + per_block - 1) / per_block;
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL((upscale_rows_kernel<NS, MC, float, WV>), grid_of_blocks(blocks), dim3(64 * WV), 0, st, args);
  else
    hipLaunchKernelGGL((upscale_rows_kernel<NS, MC, double, WV>), grid_of_blocks(blocks), dim3(64 * WV), 0, st, args);
  return hipGetLastError();
}

template <int NS, int MC>
static hipError_t launch_rw(const UpArgs& args, int a_dtype, hipStream_t st, int waves) {
  if (waves == 2) return launch_r<NS, MC, 2>(args, a_dtype, st);
  return launch_r<NS, MC, 1>(args, a_dtype, st);
}

hipError_t launch_upscale_rows(const UpArgs& args, int a_dtype, hipStream_t st, int waves) {
  if (!rows_supports(args.m)) return hipErrorInvalidValue;
  if (args.m == 16) return launch_rw<1, 16>(args, a_dtype, st, waves);
  if (args.m == 32) return launch_rw<2, 32>(args, a_dtype, st, waves);
  // other m: the bandwidth is a kernel argument, the window that of 16 or 32
  if (args.m < 16) return launch_r<1, 0, 1>(args, a_dtype, st);
  return launch_r<2, 0, 1>(args, a_dtype, st);
}

// ---- one persistent launch over batches of several m (8, 16, 32) ----
//
// A single queue of work items spans every batch; each wavefront takes the
// next item with one atomic increment and loops until the queue is empty.  An
// item is one wavefront's work: four pairs for m = 16 and 32 (the
// row-distributed elimination above), 64 pairs for m = 8 (one pair per lane,
// small_cell.h).  Items are numbered by decreasing cost -- every m = 32 item
// first, then m = 16, then m = 8 -- so the costliest items are taken first and
// the launch ends on the cheapest ones (longest-processing-time-first list
// scheduling on the CUs).  Every pair runs the same device code as in the
// per-m kernels, so S and the status are bitwise those of stomsfem_upscale.
// Registers and LDS are the maximum over the three paths: two wavefronts per
// SIMD, the m = 32 limits (m = 16 tiles run at half their own kernel's
// occupancy, m = 8 lanes at their register limit).
struct QueueBatch {
  UpArgs args;
  int64_t first;  // number of the batch's first item
  int32_t m;
};
constexpr int QUEUE_MAXB = 8;
struct QueueArgs {
  QueueBatch b[QUEUE_MAXB];  // in item order: m = 32, then 16, then 8
  int32_t nb;
  int64_t total;             // items in all
  unsigned long long* counter;
};

__global__ void queue_reset_kernel(unsigned long long* counter) {
  if (threadIdx.x == 0) *counter = 0ull;
}

template <typename TA>
__global__ __launch_bounds__(128, 2) void upscale_queue_kernel(QueueArgs qa) {
  // the image has one size for every m
  __shared__ __attribute__((aligned(16))) double lds[2][RW_PAIRS * RowImage<2, 32>::SIZE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (;;) {
    unsigned long long it = 0;
    if (lane == 0) it = atomicAdd(qa.counter, 1ull);
    // the item number is wavefront-uniform: keep it (and what follows from
    // it) in scalar registers
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)it);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(it >> 32));
    const int64_t item = (int64_t)(((uint64_t)hi << 32) | lo);
    if (item >= qa.total) break;
    int b = 0;
    while (b + 1 < qa.nb && item >= qa.b[b + 1].first) ++b;
    const UpArgs args = qa.b[b].args;
    const int64_t local = item - qa.b[b].first;
    const int m = qa.b[b].m;
    if (m == 32) {
      rows_wave<2, 32, TA>(args, local, lane, lds[wave]);
    } else if (m == 16) {
      rows_wave<1, 16, TA>(args, local, lane, lds[wave]);
    } else {
      const int64_t p = local * 64 + lane;
      if (p < args.npairs) {
        const int Mc = args.ncx * args.ncy;
        const int64_t s = p / Mc;
        const int K = (int)(p - s * Mc);
        small_cell_solve<8, TA>((const TA*)args.a + block_offset(s, K, args.ncx, args.ncy, 8),
                                (int64_t)args.ncx * 8, args.S + p * 10, args.status ? args.status + p : nullptr);
      }
    }
  }
}

bool queue_supports(int m) { return m == 8 || m == 16 || m == 32; }
int queue_max_batches() { return QUEUE_MAXB; }

// batches: nb <= QUEUE_MAXB, every m in {8, 16, 32}, one coefficient type;
// counter: 8 bytes of device memory, reset here on the stream.
hipError_t launch_upscale_queue(const UpArgs* batches, int nb, int a_dtype, unsigned long long* counter,
                                hipStream_t st) {
  if (nb < 1 || nb > QUEUE_MAXB) return hipErrorInvalidValue;
  QueueArgs qa{};
  int64_t total = 0;
  for (int mm : {32, 16, 8}) {
    for (int i = 0; i < nb; ++i) {
      if (!queue_supports(batches[i].m)) return hipErrorInvalidValue;
      if (batches[i].m != mm || batches[i].npairs == 0) continue;
      QueueBatch& q = qa.b[qa.nb++];
      q.args = batches[i];
      q.first = total;
      q.m = mm;
      const int64_t per = mm == 8 ? 64 : RW_PAIRS;
      total += (batches[i].npairs + per - 1) / per;
    }
  }
  if (total == 0) return hipSuccess;
  qa.total = total;
  qa.counter = counter;
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = a_dtype == STOMSFEM_F32
            ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, upscale_queue_kernel<float>, 128, 0)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, upscale_queue_kernel<double>, 128, 0);
  if (e != hipSuccess) return e;
  int64_t grid = (int64_t)cus * (per_cu > 0 ? per_cu : 1);
  const int64_t waves_needed = (total + 1) / 2;  // two wavefronts per workgroup
  if (grid > waves_needed) grid = waves_needed;
  hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(64), 0, st, counter);
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL(upscale_queue_kernel<float>, dim3((unsigned)grid), dim3(128), 0, st, qa);
  else
    hipLaunchKernelGGL(upscale_queue_kernel<double>, dim3((unsigned)grid), dim3(128), 0, st, qa);
  return hipGetLastError();
}

}  // namespace stomsfem
