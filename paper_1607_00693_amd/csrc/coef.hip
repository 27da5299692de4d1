// Coefficient samples of the synthetic bump family: the exponential
// transform of Sec. 2.1.3 (eq. nonlinear1) applied to an affine sum of
// compactly supported local modes, times a periodic oscillation,
//   a(x, xi) = (base + amp sin(2 pi x1/eps) sin(2 pi x2/eps))
//              * exp(beta * sum_j xi_j psi_j(x)),
//   psi_j(x) = (1 - |x - c_j|^2/rho^2)^2 inside the disc of radius rho.
// One thread per fine element, sampled at the centroid.  Only bumps whose
// centre cell lies within ceil(rho*g) cells of the point are visited, in
// increasing j.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace stomsfem {

struct CoefArgs {
  int64_t nsamples;
  int32_t nfine, nxi, g;
  double rho, eps, base, amp, beta;
  const double* xi;
  void* a;
};

// One workgroup per 16 x 16 tile and `per` consecutive samples.  Neither the
// oscillating factor nor the bump values psi_j(x) depend on the sample, so a
// thread keeps those of its element in registers (sqrt psi_j of the bumps that
// reach the tile at all, up to COEF_KEEP of them) and a sample costs two
// operations per bump, an exponential and the store; the samples' xi_j of the
// kept bumps are shared in LDS.  Tiles that more bumps reach and batches too small
// for the table take the direct kernel, the sum per element and sample; a tile
// whose xi are not finite does so here.  The oscillating factor is separable, so
// its sines are evaluated once per tile row and column.
//
// Bound by the exponential (about 30 vector instructions) and the stores (3.9
// TB/s): 1024 samples of 1024 x 1024 elements 8.4 -> 2.2 ms, 16 384 samples of
// 64 x 64 0.74 -> 0.22 ms against the bump sum per element and sample.
constexpr int COEF_TILE = 16;
constexpr int COEF_KEEP = 16;
constexpr int COEF_PER = 32;  // most samples per workgroup

// The samples of one workgroup at this thread's element, with 2 KP bumps.
template <int KP, typename T>
__device__ __forceinline__ void coef_samples(const double (*xs)[COEF_KEEP], const double* w, int ns, double osc,
                                             double beta, T* out, int64_t step) {
#pragma unroll 4
  for (int t = 0; t < ns; ++t) {
    double field = 0.0;
#pragma unroll
    for (int k = 0; k < 2 * KP; ++k) field = __builtin_fma(xs[t][k] * w[k], w[k], field);
    out[t * step] = (T)(osc * exp(beta * field));
  }
}

// Direct form: one sample per workgroup, the bump sum per element.  NEAR: discs
// that reach one cell at most (a kernel of its own, as the unrolled sum takes the
// registers of a wavefront per SIMD).
template <typename T, bool NEAR>
__global__ __launch_bounds__(256) void coef_bumps_direct_kernel(CoefArgs c, int tiles_x) {
  __shared__ double sx[COEF_TILE], sy[COEF_TILE];
  const int64_t tiles = (int64_t)tiles_x * tiles_x;
  const int64_t nblk = c.nsamples * tiles;
  const double h = 1.0 / c.nfine;
  const int lane = threadIdx.x;
  const BumpParams bp{c.g, c.rho, c.eps, c.base, c.amp, c.beta};
  // workgroup-uniform loop over (sample, tile): the grid is capped so that
  // the launch stays within the per-dispatch thread limit
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int64_t s = b / tiles;
    const int tt = (int)(b - s * tiles);
    const int tx = tt % tiles_x, ty = tt / tiles_x;
    __syncthreads();  // the previous tile's readers are done with sx, sy
    if (lane < 2 * COEF_TILE) {
      const int k = (lane < COEF_TILE ? tx : ty) * COEF_TILE + lane % COEF_TILE;
      const double z = (k + 0.5) * h;
      (lane < COEF_TILE ? sx : sy)[lane % COEF_TILE] = sin(2.0 * M_PI * z / c.eps);
    }
    const int ix = tx * COEF_TILE + (lane % COEF_TILE), iy = ty * COEF_TILE + lane / COEF_TILE;
    const double x = (ix + 0.5) * h, y = (iy + 0.5) * h;
    const double* xi = c.xi + s * c.nxi;
    // a tile in one bump cell has the same candidates for every element: the
    // loop's bounds and the xi loads are then uniform
    const int x1 = min(tx * COEF_TILE + COEF_TILE - 1, c.nfine - 1), y1 = min(ty * COEF_TILE + COEF_TILE - 1, c.nfine - 1);
    const int cx = bump_cell((tx * COEF_TILE + 0.5) * h, c.g), cy = bump_cell((ty * COEF_TILE + 0.5) * h, c.g);
    const bool one_cell = cx == bump_cell((x1 + 0.5) * h, c.g) && cy == bump_cell((y1 + 0.5) * h, c.g);
    double e = 0.0;
    if (ix < c.nfine && iy < c.nfine) {
      if (one_cell)
        e = bump_field_cell(x, y, xi, bp, cx, cy);
      else
        e = NEAR ? bump_field_near(x, y, xi, bp, bump_cell(x, c.g), bump_cell(y, c.g)) : bump_field(x, y, xi, bp);
      e = exp(c.beta * e);
    }
    __syncthreads();
    if (ix < c.nfine && iy < c.nfine)
      ((T*)c.a)[(s * c.nfine + iy) * (int64_t)c.nfine + ix] =
          (T)(bump_osc(bp, sx[lane % COEF_TILE], sy[lane / COEF_TILE]) * e);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void coef_bumps_kernel(CoefArgs c, int tiles_x, int per, int64_t groups) {
  __shared__ double sx[COEF_TILE], sy[COEF_TILE];
  __shared__ __attribute__((aligned(16))) double xs[COEF_PER][COEF_KEEP];
  const int64_t tiles = (int64_t)tiles_x * tiles_x;
  const int64_t nblk = groups * tiles;
  const double h = 1.0 / c.nfine;
  const int lane = threadIdx.x;
  const BumpParams bp{c.g, c.rho, c.eps, c.base, c.amp, c.beta};
  const int reach = (int)ceil(c.rho * c.g);
  // workgroup-uniform loop over (sample group, tile): the grid is capped so
  // that the launch stays within the per-dispatch thread limit
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int64_t s0 = b / tiles * per;
    const int ns = (int)min((int64_t)per, c.nsamples - s0);
    const int tt = (int)(b % tiles);
    const int tx = tt % tiles_x, ty = tt / tiles_x;
    __syncthreads();  // the previous tile's readers are done with the shared arrays
    if (lane < COEF_TILE) {
      const double x = ((tx * COEF_TILE + lane) + 0.5) * h;
      sx[lane] = sin(2.0 * M_PI * x / c.eps);
    } else if (lane < 2 * COEF_TILE) {
      const double y = ((ty * COEF_TILE + lane - COEF_TILE) + 0.5) * h;
      sy[lane - COEF_TILE] = sin(2.0 * M_PI * y / c.eps);
    }
    __syncthreads();
    // the tile's first and last element centroids in each direction
    const int x1 = min(tx * COEF_TILE + COEF_TILE - 1, c.nfine - 1), y1 = min(ty * COEF_TILE + COEF_TILE - 1, c.nfine - 1);
    const int cx0 = bump_cell((tx * COEF_TILE + 0.5) * h, c.g), cx1 = bump_cell((x1 + 0.5) * h, c.g);
    const int cy0 = bump_cell((ty * COEF_TILE + 0.5) * h, c.g), cy1 = bump_cell((y1 + 0.5) * h, c.g);
    const int ix = tx * COEF_TILE + (lane % COEF_TILE), iy = ty * COEF_TILE + lane / COEF_TILE;
    const bool in = ix < c.nfine && iy < c.nfine;
    const double x = (ix + 0.5) * h, y = (iy + 0.5) * h;
    const double osc = bump_osc(bp, sx[lane % COEF_TILE], sy[lane / COEF_TILE]);
    T* out = (T*)c.a + (s0 * c.nfine + iy) * (int64_t)c.nfine + ix;
    const int64_t step = (int64_t)c.nfine * c.nfine;
    int kept = 0;
    double w[COEF_KEEP];
    {
      // every bump within reach of one of the tile's cells, in increasing j;
      // the others' discs miss the tile
      const double ginv = 1.0 / c.g, rinv2 = 1.0 / (c.rho * c.rho);
      bool finite = true;
      for (int jy = max(cy0 - reach, 0); jy <= min(cy1 + reach, c.g - 1) && kept <= COEF_KEEP; ++jy) {
        for (int jx = max(cx0 - reach, 0); jx <= min(cx1 + reach, c.g - 1); ++jx) {
          const double q = in ? bump_root(x, y, jx, jy, ginv, rinv2) : 0.0;
          if (!__syncthreads_or(q != 0.0)) continue;
          if (kept < COEF_KEEP) {
#pragma unroll
            for (int k = 0; k < COEF_KEEP; ++k)
              if (k == kept) w[k] = q;
            if (lane < ns) {
              const double v = c.xi[(s0 + lane) * c.nxi + jy * c.g + jx];
              xs[lane][kept] = v;
              finite = finite && isfinite(v);
            }
          }
          ++kept;
          if (kept > COEF_KEEP) break;
        }
      }
      // an infinite or NaN xi_j counts only inside its disc
      if (__syncthreads_or(!finite)) kept = COEF_KEEP + 1;
    }
    if (kept <= COEF_KEEP) {
      // pairs of bumps; an odd last one is paired with a zero
      const int kp = (kept + 1) / 2;
      if (kept & 1) {
#pragma unroll
        for (int k = 0; k < COEF_KEEP; ++k)
          if (k == kept) w[k] = 0.0;
        if (lane < ns) xs[lane][kept] = 0.0;
      }
      __syncthreads();
      if (in) {
        switch (kp) {
          case 0: coef_samples<0>(xs, w, ns, osc, c.beta, out, step); break;
          case 1: coef_samples<1>(xs, w, ns, osc, c.beta, out, step); break;
          case 2: coef_samples<2>(xs, w, ns, osc, c.beta, out, step); break;
          case 3: coef_samples<3>(xs, w, ns, osc, c.beta, out, step); break;
          case 4: coef_samples<4>(xs, w, ns, osc, c.beta, out, step); break;
          case 5: coef_samples<5>(xs, w, ns, osc, c.beta, out, step); break;
          case 6: coef_samples<6>(xs, w, ns, osc, c.beta, out, step); break;
          case 7: coef_samples<7>(xs, w, ns, osc, c.beta, out, step); break;
          default: coef_samples<8>(xs, w, ns, osc, c.beta, out, step); break;
        }
      }
    } else if (in) {
      const bool one_cell = cx0 == cx1 && cy0 == cy1;
      for (int t = 0; t < ns; ++t) {
        const double* xi = c.xi + (s0 + t) * c.nxi;
        const double field = one_cell ? bump_field_cell(x, y, xi, bp, cx0, cy0) : bump_field(x, y, xi, bp);
        out[t * step] = (T)(osc * exp(c.beta * field));
      }
    }
  }
}

// Most bumps whose discs reach a tile, or more than COEF_KEEP: by the smallest
// distances of the tiles' element centres to the bumps' centres along one axis
// (an upper bound, as the smallest ones need not meet in one tile).
static int coef_reaching(int nfine, int g, double rho) {
  double gap[COEF_KEEP], near[COEF_KEEP];
  int n = 0;
  const int tiles = (nfine + COEF_TILE - 1) / COEF_TILE;
  for (int t = 0; t < tiles; ++t) {
    const double x0 = (t * COEF_TILE + 0.5) / nfine, x1 = (std::min(t * COEF_TILE + COEF_TILE, nfine) - 0.5) / nfine;
    const double lo = std::max(0.0, std::floor((x0 - rho) * g - 0.5)), hi = std::min(g - 1.0, std::ceil((x1 + rho) * g - 0.5));
    int m = 0;
    for (double j = lo; j <= hi; ++j) {
      const double c = (j + 0.5) / g, d = std::max({0.0, x0 - c, c - x1});
      if (!(d < rho * (1.0 + 1e-12))) continue;
      if (m == COEF_KEEP) return COEF_KEEP + 1;
      near[m++] = d;
    }
    std::sort(near, near + m);
    for (int k = 0; k < m; ++k) gap[k] = k < n ? std::min(gap[k], near[k]) : near[k];
    n = std::max(n, m);
  }
  int count = 0;
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < n; ++k) count += gap[i] * gap[i] + gap[k] * gap[k] < rho * rho * (1.0 + 1e-12);
  return count;
}

hipError_t launch_coef_bumps(int64_t nsamples, int nfine, const double* xi, int nxi, int g, double rho, double eps,
                             double base, double amp, double beta, void* a, int a_dtype, hipStream_t st) {
  CoefArgs c{nsamples, nfine, nxi, g, rho, eps, base, amp, beta, xi, a};
  const int tiles_x = (nfine + COEF_TILE - 1) / COEF_TILE;
  const int64_t tiles = (int64_t)tiles_x * tiles_x;
  // enough workgroups to fill the GPU several times over first, then up to
  // COEF_PER samples each to share a tile's table
  int64_t per = std::max<int64_t>(1, std::min<int64_t>(COEF_PER, nsamples * tiles / 8192));
  // The table costs a search over the candidates and a barrier for each, so it
  // pays from a number of samples on that grows with the bumps it holds: per
  // element and sample / with the table, us: 64 x 64 elements, 4 x 4 bumps, 9 to a
  // tile, 3000 samples (5 to a group) 132 / 147, 4096 (8) 180 / 133; 256 x 256,
  // 200 samples (6), 4 to a tile 129 / 100, 16 to a tile 143 / 195; discs of two
  // cells, 16 to a tile, 3000 samples of 64 x 64 (5) 178 / 210, 12 of 1024 x 1024
  // (6) 151 / 138.  Where more than COEF_KEEP reach a tile it never does (64
  // samples of 1024 x 1024, 64 to a tile, 1.55 / 2.36 ms).
  if (per > 1) {
    const int reach = coef_reaching(nfine, g, rho);
    if (reach > COEF_KEEP || per < (rho * g > 1.0 ? 6 : 3 + reach / 2)) per = 1;
  }
  const int64_t groups = (nsamples + per - 1) / per;
  int64_t blocks = groups * tiles;
  if (blocks == 0) return hipSuccess;
  if (blocks > (1 << 20)) blocks = 1 << 20;
  const dim3 grid((unsigned)blocks), block(256);
  const bool f32 = a_dtype == STOMSFEM_F32;
  if (per > 1) {
    if (f32) hipLaunchKernelGGL(coef_bumps_kernel<float>, grid, block, 0, st, c, tiles_x, (int)per, groups);
    else hipLaunchKernelGGL(coef_bumps_kernel<double>, grid, block, 0, st, c, tiles_x, (int)per, groups);
  } else if (rho * g <= 1.0) {
    if (f32) hipLaunchKernelGGL((coef_bumps_direct_kernel<float, true>), grid, block, 0, st, c, tiles_x);
    else hipLaunchKernelGGL((coef_bumps_direct_kernel<double, true>), grid, block, 0, st, c, tiles_x);
  } else {
    if (f32) hipLaunchKernelGGL((coef_bumps_direct_kernel<float, false>), grid, block, 0, st, c, tiles_x);
    else hipLaunchKernelGGL((coef_bumps_direct_kernel<double, false>), grid, block, 0, st, c, tiles_x);
  }
  return hipGetLastError();
}

}  // namespace stomsfem

// ---------------------------------------------------------------------------
// High-contrast channels-and-inclusions medium.  The geometry does not
// depend on the sample, so it is rasterised once per resolution into a
// feature map (index of the highest feature covering each fine element, -1
// for the background); a sample's coefficient is then a gather of its
// feature conductivities theta_j = 10^(decades * sigmoid(xi_j)).
// Coverage (element centroid xc, yc; h = 1/nfine): kind 0 = horizontal
// channel on row floor(y0 nfine) with x0 <= xc <= x0 + size; kind 1 =
// vertical channel on column floor(x0 nfine) with y0 <= yc <= y0 + size;
// kind 2 = square of side `size` centred at (x0, y0), |xc-x0|, |yc-y0| <= size/2.
// ---------------------------------------------------------------------------
namespace stomsfem {

constexpr int FEAT_MAX = 1024;

__global__ __launch_bounds__(256) void feature_map_kernel(int32_t nfine, int32_t nfeat, const int32_t* __restrict__ kind,
                                                          const double* __restrict__ x0, const double* __restrict__ y0,
                                                          const double* __restrict__ size, int32_t* __restrict__ map) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)nfine * nfine) return;
  const int iy = (int)(t / nfine), ix = (int)(t - (int64_t)iy * nfine);
  const double h = 1.0 / nfine;
  const double xc = (ix + 0.5) * h, yc = (iy + 0.5) * h;
  int found = -1;
  for (int j = nfeat - 1; j >= 0 && found < 0; --j) {
    bool cover;
    if (kind[j] == 0) {
      const int row = min((int)floor(y0[j] * nfine), nfine - 1);
      cover = iy == row && xc >= x0[j] && xc <= x0[j] + size[j];
    } else if (kind[j] == 1) {
      const int col = min((int)floor(x0[j] * nfine), nfine - 1);
      cover = ix == col && yc >= y0[j] && yc <= y0[j] + size[j];
    } else {
      cover = fabs(xc - x0[j]) <= 0.5 * size[j] && fabs(yc - y0[j]) <= 0.5 * size[j];
    }
    if (cover) found = j;
  }
  map[t] = found;
}

constexpr int FEAT_TILE = 4096;  // fine elements per workgroup

template <typename T>
__global__ __launch_bounds__(256) void coef_features_kernel(int64_t per, int32_t nfeat, const int32_t* __restrict__ map,
                                                            const double* __restrict__ xi, int32_t nxi, double decades,
                                                            int64_t tiles, int64_t nblk, T* __restrict__ a) {
  __shared__ double th[FEAT_MAX];
  int64_t s_loaded = -1;
  // workgroup-uniform loop over (sample, tile) with a capped grid
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int64_t s = b / tiles;
    const int64_t e0 = (b - s * tiles) * FEAT_TILE;
    if (s != s_loaded) {
      __syncthreads();
      for (int j = threadIdx.x; j < nfeat; j += 256) th[j] = feature_theta(xi[s * nxi + j], decades);
      __syncthreads();
      s_loaded = s;
    }
    T* as = a + s * per;
    const int64_t e1 = min(e0 + FEAT_TILE, per);
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) {
      const int32_t f = map[e];
      as[e] = (T)((unsigned)f < (unsigned)nfeat ? th[f] : 1.0);
    }
  }
}

hipError_t launch_feature_map(int nfine, int nfeat, const int32_t* kind, const double* x0, const double* y0,
                              const double* size, int32_t* map, hipStream_t st) {
  const int64_t n = (int64_t)nfine * nfine;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(feature_map_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, nfine, nfeat, kind, x0,
                     y0, size, map);
  return hipGetLastError();
}

hipError_t launch_coef_features(int64_t nsamples, int nfine, const int32_t* map, int nfeat, const double* xi, int nxi,
                                double decades, void* a, int a_dtype, hipStream_t st) {
  const int64_t per = (int64_t)nfine * nfine;
  const int64_t tiles = (per + FEAT_TILE - 1) / FEAT_TILE;
  const int64_t nblk = nsamples * tiles;
  if (nblk == 0) return hipSuccess;
  const int64_t blocks = nblk < (1 << 20) ? nblk : (1 << 20);
  if (a_dtype == STOMSFEM_F32)
    hipLaunchKernelGGL(coef_features_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, per, nfeat, map, xi,
                       nxi, decades, tiles, nblk, (float*)a);
  else
    hipLaunchKernelGGL(coef_features_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, st, per, nfeat, map, xi,
                       nxi, decades, tiles, nblk, (double*)a);
  return hipGetLastError();
}

}  // namespace stomsfem
