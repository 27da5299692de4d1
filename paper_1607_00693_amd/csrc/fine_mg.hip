// Fine-grid FEM solves for large fine meshes (the u_h of the two-level Monte
// Carlo estimator, Sec. 4.1.1): the global Q1 system K u = b on the
// nfine x nfine mesh of [0,1]^2 with a piecewise-constant coefficient a_e,
// f = 1 (b = h^2 at every interior node) and zero Dirichlet data, solved by
// conjugate gradients preconditioned with one geometric multigrid V-cycle,
// for a batch of samples at once.
//
// Multigrid: level l + 1 halves the element count per side while it is even
// and at least 8; its coefficient is the mean of the four children and its
// operator the Q1 stiffness of that coefficient (rediscretisation).
// Transfers: bilinear interpolation P of the Q1 nodal values and its
// transpose for residuals.  Smoother: damped Jacobi (weight 0.8), two sweeps
// before and two after the coarse correction, the first from zero; the
// coarsest level takes thirty sweeps from zero.  The V-cycle is a fixed
// symmetric positive-definite linear operator (Jacobi is self-adjoint, the
// pre- and post-smoothers are the same, restriction is P^T), as CG needs.
//
// The vectors of a batch are far larger than the caches and every step is a
// short stencil, so memory passes bound the solve.  Kernels of three kinds:
//   streams      a wavefront walks down a strip of 64 columns, keeps the rows
//                it needs in registers, takes its horizontal neighbours by DPP
//                and carries several dependent stencil stages along, each one
//                row behind the other (the strip's edge columns and a few rows
//                at the ends of its segment are computed twice):
//     fmg_down    [r -= alpha A p, u += alpha p,] two sweeps from zero, the
//                 residual and its restriction
//     fmg_up      prolongation, two sweeps, r.z
//     fmg_step    p = z + beta p and p.A p
//                 per iteration 15.5 passes over a level-0 vector instead of
//                 the 36.5 of one kernel per operation
//   fmg_small    all levels of at most 32 elements per side, one workgroup per
//                sample in LDS, 15.6 us (a launch each for 70 sweeps and
//                transfers took 180); the thirty sweeps of at most 49 nodes by
//                one wavefront with its stencil in registers
//   scalars      the sums of the wavefronts' parts, in a fixed order that does
//                not depend on the batch
// Samples that have converged are left alone.  16 samples of 1024 x 1024, 11
// iterations: 19.3 -> 7.5 ms; per iteration fmg_down 234 us, fmg_up 146,
// fmg_step 122 (3.8 to 4.5 TB/s counted without overlap; a copy reaches 5.1),
// the levels below 148.  One sample of 128 x 128: 2.74 -> 0.75 ms.
//
// Layout per level and sample: nodes (n+1) x (n+1), elements n x n; sample s
// of a chunk at offset s (n+1)^2 (nodes) or s n^2 (elements).  Boundary nodes
// are never written and count as zero wherever they are read.  u is updated in
// place in the caller's layout ((n-1)^2 interior nodes).
#include "common.h"

namespace stomsfem {
namespace {

constexpr int FMG_TB = 256;          // threads per block
constexpr double FMG_OMEGA = 0.8;    // Jacobi weight
constexpr int FMG_COARSE_SWEEPS = 30;
constexpr int FMG_SMALL = 32;        // largest level of fmg_small
constexpr int FMG_ROWS = 8;          // shortest segment of a stream
constexpr int FMG_SUM = 4;           // rows to a part of a sum
constexpr int FMG_SUMS = 128;        // most parts of a segment

struct FmgLevel {
  int n;            // elements per side
  const double* a;  // [N][n][n]
  double* x;        // [N][(n+1)^2]: the level's solution (level 0: z = M r)
  double* t;        // after the first two sweeps (coarsest level: Jacobi scratch)
  double* b;        // right-hand side (level 0: the CG residual)
};

struct FmgCg {
  int n;
  int64_t nsamples;
  double* u;         // [N][(n-1)^2]
  double* part;      // [N][parts] partial sums
  double *rz, *rr, *alpha, *beta;  // [N]
  int32_t* active;   // [N]
  int32_t* iters;    // [N] iterations to convergence (or the cap)
  unsigned int* nactive;
  double limit;      // tol^2 b.b
};

// ---- streams ----
// Column of lane l of strip k: H lanes of overlap on both sides.  A segment of
// `rows` node rows from y0 on.
struct Stream {
  int n, W, lane, ix;
  unsigned cx;
  int64_t s;
  int wave, strip, y0, y1;
  bool inner, own;
};
struct StreamGrid {
  int strips, segs, rows;
  int parts;  // of a sum over a sample's rows
};

// Strips of 64 - 2 H columns; segments of at least FMG_ROWS rows, so that about
// `waves` wavefronts are in flight: 4096 for fmg_down and fmg_up (four per SIMD,
// what their registers allow), 5120 for fmg_step.  How many samples share a
// batch decides the segments, so a sum goes by strip and block of FMG_SUM rows:
// a sample's sums, and with them its solution, are the same bits in any batch.
// Segments of whole blocks where there is a sum (whole blocks of 8 rows left
// fmg_up 7% fewer wavefronts at 1024 and 16 samples, 135 -> 146 us; of 4, as
// many), else of an even count (a coarse row belongs to its fine row's segment).
inline StreamGrid stream_grid(int n, int64_t N, int H, int waves, bool sums = true) {
  StreamGrid g;
  g.strips = (n + 63 - 2 * H) / (64 - 2 * H);
  int64_t segs = waves / (g.strips * N);
  const int64_t most = (n + FMG_ROWS - 1) / FMG_ROWS;
  const int64_t least = (n + FMG_SUM * FMG_SUMS - 1) / (FMG_SUM * FMG_SUMS);
  segs = segs < least ? least : segs > most ? most : segs;
  const int unit = sums ? FMG_SUM : 2;
  g.rows = (int)((n + segs - 1) / segs + unit - 1) / unit * unit;
  g.segs = (n + g.rows - 1) / g.rows;
  g.parts = g.strips * ((n + FMG_SUM - 1) / FMG_SUM);
  return g;
}

// the wavefront's stream; false where there is none (or nothing to do)
template <int H>
__device__ __forceinline__ bool stream_of(Stream& t, const StreamGrid& g, int n, int64_t N, const int32_t* active) {
  // (all of it the same in the 64 lanes: row addresses stay in scalar registers)
  auto uniform = [](unsigned v) { return (int)__builtin_amdgcn_readfirstlane(v); };
  t.wave = uniform(threadIdx.x >> 6);
  const unsigned id = blockIdx.x * (FMG_TB / 64) + t.wave, per = g.strips * g.segs;
  if (id >= per * (unsigned)N) return false;
  const int s = uniform(id / per);
  t.s = s;
  if (active && !active[s]) return false;
  const int in_s = uniform(id - s * per);
  const int seg = uniform((unsigned)in_s / (unsigned)g.strips);
  t.strip = uniform(in_s - seg * g.strips);
  t.n = n;
  t.W = n + 1;
  t.lane = threadIdx.x & 63;
  t.ix = t.strip * (64 - 2 * H) + t.lane - H;
  t.cx = t.ix < 0 ? 0 : t.ix > n ? n : t.ix;
  t.inner = t.ix > 0 && t.ix < n;
  t.own = t.inner && t.lane >= H && t.lane < 64 - H;
  t.y0 = seg * g.rows;
  t.y1 = t.y0 + g.rows < n ? t.y0 + g.rows : n;
  return true;
}

// Element of a row: the row's address in scalar registers, the lane's offset
// in bytes in one 32-bit register.
__device__ __forceinline__ double get(const double* row, unsigned bytes) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(row) + bytes);
}
__device__ __forceinline__ void put(double* row, unsigned bytes, double v) {
  *reinterpret_cast<double*>(reinterpret_cast<char*>(row) + bytes) = v;
}

// An offset that the compiler cannot add to an array's address ahead of the loop,
// at two registers each: fmg_up would spill, and a reload waits for every load
// that is on its way (153 us with its sums in LDS, 135 so).
__device__ __forceinline__ unsigned fresh(unsigned bytes) {
  asm("" : "+v"(bytes));
  return bytes;
}

// value of the lane to the left / to the right (zero past the wavefront)
__device__ __forceinline__ double from_left(double v) {
  union { double d; int w[2]; } x{v}, y;
  y.w[0] = __builtin_amdgcn_update_dpp(0, x.w[0], 0x138, 0xf, 0xf, true);
  y.w[1] = __builtin_amdgcn_update_dpp(0, x.w[1], 0x138, 0xf, 0xf, true);
  return y.d;
}
__device__ __forceinline__ double from_right(double v) {
  union { double d; int w[2]; } x{v}, y;
  y.w[0] = __builtin_amdgcn_update_dpp(0, x.w[0], 0x130, 0xf, 0xf, true);
  y.w[1] = __builtin_amdgcn_update_dpp(0, x.w[1], 0x130, 0xf, 0xf, true);
  return y.d;
}

// a / 6 of the elements to the left and to the right of the lane's column in
// one element row, and their sum
struct Elem {
  double w, e, s;
};
__device__ __forceinline__ Elem elem(double a) {
  Elem f;
  f.e = a * (1.0 / 6.0);
  f.w = from_left(f.e);
  f.s = f.w + f.e;
  return f;
}
// weight / k: two Newton steps take the instruction's estimate to full precision
__device__ __forceinline__ double damped(double k) {
  double y = __builtin_amdgcn_rcp(k);
  y = fma(fma(-k, y, 1.0), y, y);
  y = fma(fma(-k, y, 1.0), y, y);
  return FMG_OMEGA * y;
}
// weight / diagonal at a node between element rows f0 and f1
__device__ __forceinline__ double damped_inverse(const Elem& f0, const Elem& f1) { return damped(4.0 * (f0.s + f1.s)); }

// A v row by row: row y of v, between element rows f0 = y - 1 and f1 = y, goes
// to rows y - 1, y and y + 1; returns row y - 1 of A v, which is then complete.
struct Apply {
  double a0 = 0.0, a1 = 0.0;  // rows y and y + 1 so far
  __device__ __forceinline__ double push(double v, const Elem& f0, const Elem& f1) {
    const double l = from_left(v), r = from_right(v);
    const double below = fma(-f0.s, v, fma(-2.0, fma(f0.w, l, f0.e * r), a0));
    double mid = fma(4.0 * (f0.s + f1.s), v, a1);
    mid = fma(-(f0.w + f1.w), l, mid);
    a0 = fma(-(f0.e + f1.e), r, mid);
    a1 = fma(-f1.s, v, -2.0 * fma(f1.w, l, f1.e * r));
    return below;
  }
};

// sum over the wavefront, the same in all lanes: within the DPP rows of 16 by
// rotations, then the four rows' sums
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
  union { double d; int w[2]; } x{v}, y;
  y.w[0] = __builtin_amdgcn_update_dpp(0, x.w[0], 0x120 + N, 0xf, 0xf, false);
  y.w[1] = __builtin_amdgcn_update_dpp(0, x.w[1], 0x120 + N, 0xf, 0xf, false);
  return y.d;
}
__device__ __forceinline__ double lane_of(double v, int lane) {
  union { double d; int w[2]; } x{v}, y;
  y.w[0] = __builtin_amdgcn_readlane(x.w[0], lane);
  y.w[1] = __builtin_amdgcn_readlane(x.w[1], lane);
  return y.d;
}
__device__ __forceinline__ double wave_sum(double v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return (lane_of(v, 0) + lane_of(v, 16)) + (lane_of(v, 32) + lane_of(v, 48));
}

// The sum of a stream's rows by blocks of FMG_SUM, kept in LDS until the segment
// is done (a store to memory in the loop would count among the loads that are on
// their way and shorten them).  OFF: how far the first row of the loop lies
// before y0, AHEAD: rows per turn.
template <int OFF, int AHEAD>
struct BlockSum {
  double* sums;  // FMG_SUMS of LDS
  double acc = 0.0;
  // after row y has been added, in place k of its turn (one place of a turn can
  // end a block)
  __device__ __forceinline__ void row(const Stream& t, int y, int k) {
    if (k != (FMG_SUM - 1 + OFF) % AHEAD || (y & (FMG_SUM - 1)) != FMG_SUM - 1 || y < t.y0 || y >= t.y1) return;
    acc = wave_sum(acc);
    if (t.lane == 0) sums[(y - t.y0) / FMG_SUM] = acc;
    acc = 0.0;
  }
  __device__ __forceinline__ void store(const Stream& t, const StreamGrid& g, double* part) {
    const int blocks = (t.y1 - t.y0 + FMG_SUM - 1) / FMG_SUM;
    if (t.y1 & (FMG_SUM - 1)) {
      acc = wave_sum(acc);
      if (t.lane == 0) sums[blocks - 1] = acc;
    }
    __threadfence_block();
    for (int i = t.lane; i < blocks; i += 64)
      part[t.s * g.parts + (int64_t)(t.y0 / FMG_SUM + i) * g.strips + t.strip] = sums[i];
  }
};

// Two Jacobi sweeps from zero on the right-hand side b, the residual and its
// restriction.
//   SRC 0: b from memory (levels below the first)
//   SRC 1: level 0: b = r - alpha A p, written to r1, and u += alpha p
//   SRC 2: level 0, start: b = h^2, written to r1
// PRE false: without the sweeps (level 0 is the coarsest).  Row y of p (SRC 1)
// or of b is read; the stages follow one row behind each other.
struct DownArgs {
  FmgLevel L;
  StreamGrid g;
  int64_t N;
  const int32_t* active;
  double* bc;           // right-hand side of the next level
  // level 0
  const double *p, *r0;
  double* r1;
  double* u;
  const double* alpha;
  double* part;
  int first;            // u is not read
};
template <int SRC, bool PRE>
__global__ __launch_bounds__(FMG_TB, 4) void fmg_down_kernel(DownArgs d) {
  constexpr int H = PRE ? 4 : 1;
  constexpr int AHEAD = SRC == 1 ? 2 : 4;  // rows on their way while one is worked on
  Stream t;
  if (!stream_of<H>(t, d.g, d.L.n, d.N, d.active)) return;
  const int n = t.n, W = t.W;
  const int64_t node = t.s * W * W;
  const double* a = d.L.a + t.s * n * n;
  const unsigned cb = 8 * t.cx, ca = 8 * (t.cx < (unsigned)n ? t.cx : n - 1);
  const double* src = SRC == 1 ? d.p + node : SRC == 0 ? d.L.b + node : nullptr;
  const double h2 = 1.0 / ((double)n * n);
  const double al = SRC == 1 ? d.alpha[t.s] : 0.0;
  double* u = SRC == 1 ? d.u + t.s * (int64_t)(n - 1) * (n - 1) : nullptr;
  const unsigned cu = t.cx < 1 ? 0 : 8 * (t.cx < (unsigned)n ? t.cx - 1 : n - 2);  // u has the interior columns only
  const bool elem_in = t.ix >= 0 && t.ix < n;
  auto row_in = [&](int y) { return y > 0 && y < n; };
  // raw values of a row (of the nearest one outside the domain); masked when used,
  // not where they are loaded, which would wait for them
  auto load_a = [&](int y) { return get(a + (int64_t)(y < 0 ? 0 : y < n ? y : n - 1) * n, ca); };
  auto load_v = [&](const double* q, int y) { return get(q + (int64_t)(y < 0 ? 0 : y < n ? y : n) * W, cb); };
  auto mask_a = [&](double v, int y) { return elem_in && y >= 0 && y < n ? v : 0.0; };
  auto mask_v = [&](double v, int y) { return t.inner && row_in(y) ? v : 0.0; };
  constexpr int LAG = SRC == 1 ? 1 : 0;  // row of b behind the row that is read
  const int first = t.y0 - (PRE ? 3 : 0) - LAG, last = t.y1 - 1 + (PRE ? 3 : 0) + LAG;
  Elem f0 = elem(mask_a(load_a(first - 1), first - 1)), f1{}, f2{}, f3{};  // in the loop: element rows y, y - 1, y - 2, y - 3
  Apply ap, a1, a2;
  double p1 = 0.0;                       // p of the row before
  double b1 = 0.0, b2 = 0.0;             // b, one and two rows behind its newest
  double x1 = 0.0, i1 = 0.0;             // first sweep and weight / diagonal, one row behind
  double h1 = 0.0, h2r = 0.0;            // rows of the residual, restricted in x
  __shared__ double sums[SRC == 1 ? FMG_TB / 64 : 1][SRC == 1 ? FMG_SUMS : 1];
  BlockSum<(PRE ? 3 : 0) + 2 * LAG, AHEAD> sum{sums[SRC == 1 ? t.wave : 0]};
  auto load_u = [&](int y) { return get(u + (int64_t)(y < 1 ? 0 : y < n ? y - 1 : n - 2) * (n - 1), cu); };
  double ra[AHEAD], rv[AHEAD], rr[AHEAD], ru[AHEAD];
  auto fetch = [&](int k, int y) {
    ra[k] = load_a(y);
    rv[k] = SRC == 2 ? 0.0 : load_v(src, y);
    rr[k] = SRC == 1 ? load_v(d.r0 + node, y - 1) : 0.0;
    ru[k] = SRC == 1 && !d.first ? load_u(y - 1) : 0.0;
  };
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) fetch(k, first + k);
  for (int y8 = first; y8 <= last; y8 += AHEAD)
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) {
    const int y = y8 + k;
    const double va = ra[k], v = SRC == 2 ? 0.0 : mask_v(rv[k], y), vr = rr[k], vu = ru[k];
    fetch(k, y + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    f3 = f2;
    f2 = f1;
    f1 = f0;
    f0 = elem(mask_a(va, y));
    // b of row yb, between element rows fs (below) and fn
    const int yb = y - LAG;
    const Elem &fn = LAG ? f1 : f0, &fs = LAG ? f2 : f1, &fb = LAG ? f3 : f2;
    double b;
    if (SRC == 1) {
      const double q = ap.push(v, f1, f0);
      const bool in = t.inner && row_in(yb);
      const bool mine = t.own && yb >= t.y0 && yb < t.y1 && row_in(yb);
      b = fma(-al, q, vr);
      b = in ? b : 0.0;
      if (mine) {
        put(d.r1 + node + (int64_t)yb * W, cb, b);
        put(u + (int64_t)(yb - 1) * (n - 1), cu, d.first ? al * p1 : fma(al, p1, vu));
        sum.acc = fma(b, b, sum.acc);
      }
      sum.row(t, yb, k);
      p1 = v;
    } else if (SRC == 2) {
      b = t.inner && row_in(yb) ? h2 : 0.0;
      if (t.own && yb >= t.y0 && yb < t.y1 && row_in(yb)) put(d.r1 + node + (int64_t)yb * W, cb, b);
    } else {
      b = v;
    }
    if (PRE) {
      const double inv = damped_inverse(fs, fn);
      const double x = t.inner && row_in(yb) ? inv * b : 0.0;        // first sweep, row yb
      const double ax = a1.push(x, fs, fn);                          // A x, row yb - 1
      const bool in1 = t.inner && row_in(yb - 1);
      const double x2 = in1 ? fma(i1, b1 - ax, x1) : 0.0;            // second sweep, row yb - 1
      if (t.own && yb - 1 >= t.y0 && yb - 1 < t.y1 && row_in(yb - 1)) put(d.L.t + node + (int64_t)(yb - 1) * W, cb, x2);
      const double ax2 = a2.push(x2, fb, fs);                        // row yb - 2
      const double res = t.inner && row_in(yb - 2) ? b2 - ax2 : 0.0;
      const double h = fma(0.5, from_left(res) + from_right(res), res);
      // rows yb - 4, yb - 3, yb - 2 of h make the coarse node of an even row yb - 3
      const int yc = yb - 3;
      if (!(yc & 1) && !(t.ix & 1) && t.own && yc >= t.y0 && yc < t.y1 && row_in(yc)) {
        const int nc = n / 2, Wc = nc + 1;
        d.bc[t.s * Wc * Wc + (int64_t)(yc / 2) * Wc + t.ix / 2] = fma(0.5, h2r + h, h1);
      }
      h2r = h1;
      h1 = h;
      b2 = b1;
      b1 = b;
      x1 = x;
      i1 = inv;
    }
  }
  if (SRC == 1) sum.store(t, d.g, d.part);
}

// x = t + P x_c, two Jacobi sweeps on it; DOT: the part of b.x.
struct UpArgsMg {
  FmgLevel L;
  StreamGrid g;
  int64_t N;
  const int32_t* active;
  const double* xc;
  double* part;
};
template <bool DOT>
__global__ __launch_bounds__(FMG_TB, 4) void fmg_up_kernel(UpArgsMg d) {
  constexpr int H = 2, AHEAD = 4;  // (even)
  Stream t;
  if (!stream_of<H>(t, d.g, d.L.n, d.N, d.active)) return;
  const int n = t.n, W = t.W, nc = n / 2, Wc = nc + 1;
  const int64_t node = t.s * W * W;
  const double* a = d.L.a + t.s * n * n;
  const unsigned cb = 8 * t.cx, ca = 8 * (t.cx < (unsigned)n ? t.cx : n - 1);
  const double *tv = d.L.t + node, *bv = d.L.b + node;
  const unsigned c0 = t.cx < (unsigned)n ? t.cx >> 1 : nc - 1, cc = 8 * c0;
  const double* xc = d.xc + t.s * Wc * Wc;
  const bool elem_in = t.ix >= 0 && t.ix < n, odd = t.ix & 1;
  auto row_in = [&](int y) { return y > 0 && y < n; };
  // raw values of a row (of the nearest one outside the domain); masked when used,
  // not where they are loaded, which would wait for them
  auto load_a = [&](int y) { return get(a + (int64_t)(y < 0 ? 0 : y < n ? y : n - 1) * n, fresh(ca)); };
  auto load_v = [&](const double* q, int y) { return get(q + (int64_t)(y < 0 ? 0 : y < n ? y : n) * W, fresh(cb)); };
  auto mask_a = [&](double v, int y) { return elem_in && y >= 0 && y < n ? v : 0.0; };
  auto mask_v = [&](double v, int y) { return t.inner && row_in(y) ? v : 0.0; };
  auto coarse_row = [&](int yc) { return xc + (int64_t)(yc < 0 ? 0 : yc < nc ? yc : nc) * Wc; };
  auto coarse = [&](double l, double r, int yc) {  // x_c interpolated in x, coarse row yc
    const bool in = yc > 0 && yc < nc;
    const double lv = in && c0 > 0 ? l : 0.0, rv = in && c0 + 1 < (unsigned)nc ? r : 0.0;
    return odd ? 0.5 * (lv + rv) : lv;
  };
  const int first = t.y0 - 2, last = t.y1 - 1 + 2;
  Elem f0 = elem(mask_a(load_a(first - 1), first - 1)), f1{}, f2{};
  Apply a1, a2;
  double v1 = 0.0, w1 = 0.0;              // before and after the first sweep, one row behind
  double b1 = 0.0, b2 = 0.0, i1 = 0.0, i2 = 0.0;
  double low = coarse(get(coarse_row(first >> 1), cc), get(coarse_row(first >> 1), cc + 8), first >> 1);
  __shared__ double sums[DOT ? FMG_TB / 64 : 1][DOT ? FMG_SUMS : 1];
  BlockSum<4, AHEAD> sum{sums[DOT ? t.wave : 0]};
  double ra[AHEAD], rt[AHEAD], rb[AHEAD], rl, rh;
  auto fetch = [&](int k, int y) {
    ra[k] = load_a(y);
    rt[k] = load_v(tv, y);
    rb[k] = load_v(bv, y);
  };
  auto fetch_coarse = [&](int y) {  // for the odd row y: the coarse row above it, one pair of rows ahead
    const double* q = coarse_row((y + 1) >> 1);
    rl = get(q, fresh(cc));
    rh = get(q, fresh(cc) + 8);
  };
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) fetch(k, first + k);
  fetch_coarse(first + 1);  // first is even
  for (int y8 = first; y8 <= last; y8 += AHEAD)
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) {
    const int y = y8 + k;
    const double va = ra[k], vt = rt[k], b = mask_v(rb[k], y);
    const double ul = rl, uh = rh;
    fetch(k, y + AHEAD);
    if (k & 1) fetch_coarse(y + 2);
    __builtin_amdgcn_sched_barrier(0);
    f2 = f1;
    f1 = f0;
    f0 = elem(mask_a(va, y));
    double pc = low;
    if (k & 1) {
      const double up = coarse(ul, uh, (y + 1) >> 1);
      pc = 0.5 * (low + up);
      low = up;
    }
    const double v = t.inner && row_in(y) ? vt + pc : 0.0;
    const double inv = damped_inverse(f1, f0);
    const double av = a1.push(v, f1, f0);                                        // row y - 1
    const double w = t.inner && row_in(y - 1) ? fma(i1, b1 - av, v1) : 0.0;
    const double aw = a2.push(w, f2, f1);                                        // row y - 2
    if (t.own && y - 2 >= t.y0 && y - 2 < t.y1 && row_in(y - 2)) {
      const double z = fma(i2, b2 - aw, w1);
      put(d.L.x + node + (int64_t)(y - 2) * W, fresh(cb), z);
      if (DOT) sum.acc = fma(b2, z, sum.acc);
    }
    if (DOT) sum.row(t, y - 2, k);
    w1 = w;
    v1 = v;
    b2 = b1;
    b1 = b;
    i2 = i1;
    i1 = inv;
  }
  if (DOT) sum.store(t, d.g, d.part);
}

// p1 = z + beta p0 (first: p1 = z) and the part of p1.A p1
struct StepArgs {
  int n;
  StreamGrid g;
  int64_t N;
  const int32_t* active;
  const double *a, *z, *p0, *beta;
  double *p1, *part;
  int first;
};
__global__ __launch_bounds__(FMG_TB, 4) void fmg_step_kernel(StepArgs d) {
  constexpr int H = 1, AHEAD = 4;
  Stream t;
  if (!stream_of<H>(t, d.g, d.n, d.N, d.active)) return;
  const int n = t.n, W = t.W;
  const int64_t node = t.s * W * W;
  const double* a = d.a + t.s * n * n;
  const unsigned cb = 8 * t.cx, ca = 8 * (t.cx < (unsigned)n ? t.cx : n - 1);
  const double *zv = d.z + node, *pv = d.p0 + node;
  const double be = d.first ? 0.0 : d.beta[t.s];
  const bool elem_in = t.ix >= 0 && t.ix < n, with_p = !d.first;
  auto row_in = [&](int y) { return y > 0 && y < n; };
  // raw values of a row (of the nearest one outside the domain); masked when used,
  // not where they are loaded, which would wait for them
  auto load_a = [&](int y) { return get(a + (int64_t)(y < 0 ? 0 : y < n ? y : n - 1) * n, ca); };
  auto load_v = [&](const double* q, int y) { return get(q + (int64_t)(y < 0 ? 0 : y < n ? y : n) * W, cb); };
  auto mask_a = [&](double v, int y) { return elem_in && y >= 0 && y < n ? v : 0.0; };
  auto mask_v = [&](double v, int y) { return t.inner && row_in(y) ? v : 0.0; };
  const int first = t.y0 - 1, last = t.y1;
  Elem f0 = elem(mask_a(load_a(first - 1), first - 1)), f1{};
  Apply ap;
  __shared__ double sums[FMG_TB / 64][FMG_SUMS];
  BlockSum<2, AHEAD> sum{sums[t.wave]};
  double p1 = 0.0;
  double ra[AHEAD], rz[AHEAD], rp[AHEAD];
  auto fetch = [&](int k, int y) {
    ra[k] = load_a(y);
    rz[k] = load_v(zv, y);
    rp[k] = with_p ? load_v(pv, y) : 0.0;
  };
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) fetch(k, first + k);
  for (int y8 = first; y8 <= last; y8 += AHEAD)
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) {
    const int y = y8 + k;
    const double va = ra[k], z = rz[k], p0 = rp[k];
    fetch(k, y + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    f1 = f0;
    f0 = elem(mask_a(va, y));
    const double p = mask_v(fma(be, p0, z), y);
    const double q = ap.push(p, f1, f0);  // row y - 1
    if (t.own && y - 1 >= t.y0 && y - 1 < t.y1) sum.acc = fma(p1, q, sum.acc);
    sum.row(t, y - 1, k);
    if (t.own && y >= t.y0 && y < t.y1 && row_in(y)) put(d.p1 + node + (int64_t)y * W, cb, p);
    p1 = p;
  }
  sum.store(t, d.g, d.part);
}

// ---- small levels ----
// The V-cycle from the level of n <= FMG_SMALL elements per side down, one
// workgroup per sample: x = V-cycle of b.  Right-hand sides, solutions and
// coefficients of all levels in LDS.
constexpr int FMG_SMALL_TB = 512;
struct SmallLevel {
  int n;
  double *a, *x, *b;
};
__device__ __forceinline__ double small_apply(const SmallLevel& L, int ix, int iy, double* inv) {
  const int W = L.n + 1;
  const double* a = L.a + (iy - 1) * L.n + ix - 1;
  const double aSW = a[0], aSE = a[1], aNW = a[L.n], aNE = a[L.n + 1];
  const double kc = (2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE));
  const double* x = L.x + iy * W + ix;
  double v = kc * x[0];
  v -= ((aSW + aNW) * x[-1] + (aSE + aNE) * x[1] + (aSW + aSE) * x[-W] + (aNW + aNE) * x[W]) * (1.0 / 6.0);
  v -= (aSW * x[-W - 1] + aSE * x[-W + 1] + aNW * x[W - 1] + aNE * x[W + 1]) * (1.0 / 3.0);
  *inv = damped(kc);
  return v;
}

__global__ __launch_bounds__(FMG_SMALL_TB) void fmg_small_kernel(FmgLevel top, int nlev, const int32_t* active) {
  constexpr int P0 = (FMG_SMALL + 1) * (FMG_SMALL + 1);
  __shared__ double mem[P0 + (2 * P0 + FMG_SMALL * FMG_SMALL) * 3 / 2];  // residual; levels shrink fourfold
  const int64_t s = blockIdx.x;
  if (active && !active[s]) return;
  const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
  constexpr int TY = FMG_SMALL_TB / 32, NR = FMG_SMALL / TY;  // rows ty, ty + TY, ... of a level
  double* const res = mem;
  double* next = mem + P0;
  auto level = [&](int n) {
    SmallLevel L;
    L.n = n;
    L.a = next;
    L.x = L.a + n * n;
    L.b = L.x + (n + 1) * (n + 1);
    return L;
  };
  auto size = [](int n) { return n * n + 2 * (n + 1) * (n + 1); };
  // f(ix, iy, k) over the interior nodes of a level, k-th of a thread
  auto nodes = [&](int n, auto f) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int ix = 1 + tx, iy = 1 + ty + k * TY;
      if (ix < n && iy < n) f(ix, iy, k);
    }
  };
  auto sweep = [&](const SmallLevel& L) {
    double v[NR];
    nodes(L.n, [&](int ix, int iy, int k) {
      double inv;
      const double ax = small_apply(L, ix, iy, &inv);
      const int i = iy * (L.n + 1) + ix;
      v[k] = L.x[i] + inv * (L.b[i] - ax);
    });
    __syncthreads();
    nodes(L.n, [&](int ix, int iy, int k) { L.x[iy * (L.n + 1) + ix] = v[k]; });
    __syncthreads();
  };
  auto start = [&](const SmallLevel& L) {  // sweep from zero
    nodes(L.n, [&](int ix, int iy, int) {
      const double* a = L.a + (iy - 1) * L.n + ix - 1;
      const double kc = (2.0 / 3.0) * ((a[0] + a[1]) + (a[L.n] + a[L.n + 1]));
      const int i = iy * (L.n + 1) + ix;
      L.x[i] = damped(kc) * L.b[i];
    });
    __syncthreads();
  };
  // first level from memory, the boundary nodes of all levels zero
  for (int i = tid; i < (int)(sizeof(mem) / sizeof(double)); i += FMG_SMALL_TB) mem[i] = 0.0;
  __syncthreads();
  {
    const SmallLevel L = level(top.n);
    const int n = top.n, W = n + 1;
    for (int i = tid; i < n * n; i += FMG_SMALL_TB) L.a[i] = top.a[s * n * n + i];
    nodes(n, [&](int ix, int iy, int) { L.b[iy * W + ix] = top.b[s * W * W + iy * W + ix]; });
  }
  __syncthreads();
  for (int l = 0; l < nlev - 1; ++l) {
    const SmallLevel L = level(top.n >> l);
    next += size(L.n);
    const SmallLevel C = level(L.n >> 1);
    for (int e = tid; e < C.n * C.n; e += FMG_SMALL_TB) {
      const double* f = L.a + 2 * (e / C.n) * L.n + 2 * (e % C.n);
      C.a[e] = 0.25 * ((f[0] + f[1]) + (f[L.n] + f[L.n + 1]));
    }
    start(L);
    sweep(L);
    nodes(L.n, [&](int ix, int iy, int) {
      double inv;
      const double ax = small_apply(L, ix, iy, &inv);
      const int i = iy * (L.n + 1) + ix;
      res[i] = L.b[i] - ax;
    });
    __syncthreads();
    const int W = L.n + 1;
    nodes(C.n, [&](int ix, int iy, int) {
      // interior fine nodes only
      const double* r = res + 2 * iy * W + 2 * ix;
      C.b[iy * (C.n + 1) + ix] = r[0] + 0.5 * ((r[-1] + r[1]) + (r[-W] + r[W])) +
                                 0.25 * ((r[-W - 1] + r[-W + 1]) + (r[W - 1] + r[W + 1]));
    });
    __syncthreads();
  }
  {
    const SmallLevel L = level(top.n >> (nlev - 1));
    start(L);
    if (L.n <= 8) {  // at most 49 nodes: one wavefront, without the workgroup's barriers
      if (tid < 64) {
        // a lane's node, its row of D^{-1} A and its right-hand side in registers
        const int m = L.n - 1, W = L.n + 1;
        const bool on = tid < m * m;
        const int iy = on ? 1 + tid / m : 1, ix = on ? 1 + tid % m : 1, at = iy * W + ix;
        const double* a = L.a + (iy - 1) * L.n + ix - 1;
        const double aSW = a[0], aSE = a[1], aNW = a[L.n], aNE = a[L.n + 1];
        const double inv = damped((2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE))), t = inv * (1.0 / 6.0), u = inv * (1.0 / 3.0);
        const double wW = t * (aSW + aNW), wE = t * (aSE + aNE), wS = t * (aSW + aSE), wN = t * (aNW + aNE);
        const double wSW = u * aSW, wSE = u * aSE, wNW = u * aNW, wNE = u * aNE, rhs = inv * L.b[at];
        double* x = L.x + at;
        double v = x[0];
        for (int k = 1; k < FMG_COARSE_SWEEPS; ++k) {
          // x + w D^{-1} (b - A x) with w D^{-1} A's diagonal w
          double n = fma(wW, x[-1], fma(wE, x[1], rhs)), o = fma(wS, x[-W], wN * x[W]);
          n = fma(wSW, x[-W - 1], fma(wSE, x[-W + 1], n));
          o = fma(wNW, x[W - 1], fma(wNE, x[W + 1], o));
          v = fma(1.0 - FMG_OMEGA, v, n + o);
          __threadfence_block();
          if (on) x[0] = v;
          __threadfence_block();
        }
      }
      __syncthreads();
    } else {
      for (int k = 1; k < FMG_COARSE_SWEEPS; ++k) sweep(L);
    }
  }
  for (int l = nlev - 2; l >= 0; --l) {
    const SmallLevel C = level(top.n >> (l + 1));
    next -= size(top.n >> l);
    const SmallLevel L = level(top.n >> l);
    const int W = L.n + 1, Wc = C.n + 1;
    nodes(L.n, [&](int ix, int iy, int) {
      const double* c = C.x + (iy >> 1) * Wc + (ix >> 1);
      double v;
      if (!(ix & 1) && !(iy & 1)) v = c[0];
      else if (!(iy & 1)) v = 0.5 * (c[0] + c[1]);
      else if (!(ix & 1)) v = 0.5 * (c[0] + c[Wc]);
      else v = 0.25 * ((c[0] + c[1]) + (c[Wc] + c[Wc + 1]));
      L.x[iy * W + ix] += v;
    });
    __syncthreads();
    sweep(L);
    sweep(L);
  }
  {
    const SmallLevel L = level(top.n);
    const int W = top.n + 1;
    nodes(top.n, [&](int ix, int iy, int) { top.x[s * W * W + iy * W + ix] = L.x[iy * W + ix]; });
  }
}

// ---- a coarsest level beyond fmg_small (an odd count of elements) ----
// FIRST: out = w D^{-1} b (a sweep from zero), else out = x + w D^{-1} (b - A x);
// boundary nodes of x read as they are (zero)
template <bool FIRST>
__global__ __launch_bounds__(FMG_TB) void fmg_sweep_kernel(FmgLevel L, const double* __restrict__ x,
                                                           double* __restrict__ out) {
  const int n = L.n, W = n + 1;
  const int node = blockIdx.x * FMG_TB + threadIdx.x;
  if (node >= W * W) return;
  const int iy = node / W, ix = node - iy * W;
  const int64_t s = blockIdx.y, off = s * W * W;
  if (ix == 0 || iy == 0 || ix == n || iy == n) {
    out[off + node] = 0.0;
    return;
  }
  const double* a = L.a + s * n * n + (iy - 1) * n + ix - 1;
  const double aSW = a[0], aSE = a[1], aNW = a[n], aNE = a[n + 1];
  const double kc = (2.0 / 3.0) * ((aSW + aSE) + (aNW + aNE));
  if (FIRST) {
    out[off + node] = FMG_OMEGA * L.b[off + node] / kc;
    return;
  }
  const double* xc = x + off + node;
  double v = kc * xc[0];
  v -= ((aSW + aNW) * xc[-1] + (aSE + aNE) * xc[1] + (aSW + aSE) * xc[-W] + (aNW + aNE) * xc[W]) * (1.0 / 6.0);
  v -= (aSW * xc[-W - 1] + aSE * xc[-W + 1] + aNW * xc[W - 1] + aNE * xc[W + 1]) * (1.0 / 3.0);
  out[off + node] = xc[0] + FMG_OMEGA * (L.b[off + node] - v) / kc;
}

// part of r.z over the interior nodes (level 0 is the coarsest)
__global__ __launch_bounds__(FMG_TB) void fmg_dot_kernel(int n, const double* __restrict__ r,
                                                         const double* __restrict__ z, double* part) {
  __shared__ double red[FMG_TB / 64];
  const int W = n + 1;
  const int64_t s = blockIdx.y;
  double acc = 0.0;
  for (int iy = 1 + blockIdx.x; iy < n; iy += gridDim.x)
    for (int ix = 1 + threadIdx.x; ix < n; ix += FMG_TB) {
      const int64_t i = s * W * W + (int64_t)iy * W + ix;
      acc += r[i] * z[i];
    }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[s * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// coarse element coefficient = mean of its four children
__global__ __launch_bounds__(FMG_TB) void fmg_coef_kernel(const double* __restrict__ af, int nf,
                                                          double* __restrict__ ac) {
  const int nc = nf / 2;
  const int e = blockIdx.x * FMG_TB + threadIdx.x;
  if (e >= nc * nc) return;
  const int64_t s = blockIdx.y;
  const int ey = e / nc, ex = e - ey * nc;
  const double* f = af + s * nf * nf + (2 * ey) * nf + 2 * ex;
  ac[s * nc * nc + e] = 0.25 * ((f[0] + f[1]) + (f[nf] + f[nf + 1]));
}

// per-sample scalar steps (one workgroup per sample: thread t sums the
// parts t, t + 256, ... in order, then a fixed tree; a fixed order)
//   0: active = 1 (no sum);   1: rz = sum, beta = 0 (first direction p = z);
//   2: p.q = sum, alpha = active ? rz / p.q : 0;
//   3: rr = sum, active &= rr > limit (count, iterations);
//   4: beta = active ? sum / rz : 0, rz = sum
template <int STEP>
__global__ __launch_bounds__(FMG_TB) void fmg_scalar_kernel(FmgCg c, int parts, int it) {
  const int64_t s = blockIdx.x;
  if (STEP > 0) {
    if (!c.active[s]) {
      if (threadIdx.x == 0 && STEP == 2) c.alpha[s] = 0.0;
      return;
    }
  }
  __shared__ double red[FMG_TB / 64];
  double v = 0.0;
  if (STEP > 0) {
#pragma unroll 8
    for (int k = threadIdx.x; k < parts; k += FMG_TB) v += c.part[s * parts + k];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = (red[0] + red[1]) + (red[2] + red[3]);
  }
  if (threadIdx.x != 0) return;
  if (STEP == 0) {
    c.active[s] = 1;
    c.iters[s] = 0;
  } else if (STEP == 1) {
    c.rz[s] = v;
    c.beta[s] = 0.0;
  } else if (STEP == 2) {
    c.alpha[s] = v > 0.0 ? c.rz[s] / v : 0.0;
  } else if (STEP == 3) {
    c.rr[s] = v;
    c.iters[s] = it + 1;
    if (!(v > c.limit))
      c.active[s] = 0;
    else
      atomicAdd(c.nactive, 1u);
  } else {
    c.beta[s] = c.rz[s] > 0.0 ? v / c.rz[s] : 0.0;
    c.rz[s] = v;
  }
}

__global__ void fmg_zero_kernel(unsigned int* p) { *p = 0u; }

__global__ void fmg_status_kernel(FmgCg c, int32_t* status) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < c.nsamples) status[s] = c.active[s] ? STOMSFEM_ENOCONV : STOMSFEM_OK;
}

// ---- host side ----
int fmg_levels(int n) {
  int L = 1;
  while (n % 2 == 0 && n >= 8) {
    n /= 2;
    ++L;
  }
  return L;
}

inline unsigned stream_blocks(const StreamGrid& g, int64_t N) {
  const int64_t waves = (int64_t)g.strips * g.segs * N;
  return (unsigned)((waves + FMG_TB / 64 - 1) / (FMG_TB / 64));
}

// x = V-cycle of b on level l (level 0: after its fmg_down); dot: the parts of
// r.z on level 0
hipError_t fmg_vcycle(FmgLevel* lv, int nlev, int l, int64_t N, const int32_t* active, double* part, int* parts,
                      hipStream_t st) {
  FmgLevel& L = lv[l];
  hipError_t e = hipSuccess;
  if (L.n <= FMG_SMALL && (l > 0 || nlev == 1)) {
    hipLaunchKernelGGL(fmg_small_kernel, dim3((unsigned)N), dim3(FMG_SMALL_TB), 0, st, L, nlev - l, active);
  } else if (l == nlev - 1) {
    const int W = L.n + 1;
    const dim3 g((unsigned)((W * W + FMG_TB - 1) / FMG_TB), (unsigned)N), b(FMG_TB);
    hipLaunchKernelGGL(fmg_sweep_kernel<true>, g, b, 0, st, L, (const double*)nullptr, L.x);
    for (int k = 1; k < FMG_COARSE_SWEEPS; ++k) {
      hipLaunchKernelGGL(fmg_sweep_kernel<false>, g, b, 0, st, L, (const double*)L.x, L.t);
      std::swap(L.x, L.t);
    }
  } else {
    if (l > 0) {
      DownArgs d{};
      d.L = L;
      d.g = stream_grid(L.n, N, 4, 4096, false);
      d.N = N;
      d.active = active;
      d.bc = lv[l + 1].b;
      hipLaunchKernelGGL((fmg_down_kernel<0, true>), dim3(stream_blocks(d.g, N)), dim3(FMG_TB), 0, st, d);
    }
    e = hipGetLastError();
    if (e == hipSuccess) e = fmg_vcycle(lv, nlev, l + 1, N, active, nullptr, nullptr, st);
    if (e != hipSuccess) return e;
    UpArgsMg u{};
    u.L = L;
    u.g = stream_grid(L.n, N, 2, 4096, l == 0);
    u.N = N;
    u.active = active;
    u.xc = lv[l + 1].x;
    u.part = part;
    if (l == 0) {
      *parts = u.g.parts;
      hipLaunchKernelGGL(fmg_up_kernel<true>, dim3(stream_blocks(u.g, N)), dim3(FMG_TB), 0, st, u);
    } else {
      hipLaunchKernelGGL(fmg_up_kernel<false>, dim3(stream_blocks(u.g, N)), dim3(FMG_TB), 0, st, u);
    }
    return hipGetLastError();
  }
  e = hipGetLastError();
  if (e == hipSuccess && l == 0) {
    *parts = L.n < 256 ? L.n : 256;
    hipLaunchKernelGGL(fmg_dot_kernel, dim3((unsigned)*parts, (unsigned)N), dim3(FMG_TB), 0, st, L.n,
                       (const double*)L.b, (const double*)L.x, part);
    e = hipGetLastError();
  }
  return e;
}

// most parts per sample of any sum: strips of 56 columns
int64_t fmg_parts(int n) {
  const int64_t streams = (int64_t)((n + 55) / 56) * ((n + FMG_SUM - 1) / FMG_SUM);
  return streams > 256 ? streams : 256;
}

}  // namespace

int64_t fine_pcg_doubles_per_sample(int nfine) {
  const int L = fmg_levels(nfine);
  int64_t d = 0;
  int n = nfine;
  for (int l = 0; l < L; ++l) {
    const int64_t P = (int64_t)(n + 1) * (n + 1);
    d += (l == 0 ? 6 : 3) * P + (l == 0 ? 0 : (int64_t)n * n);  // level 0: r p (two each) z t; others x t b + coef
    n /= 2;
  }
  return d + fmg_parts(nfine) + 8;
}

// Solves one chunk of N samples (reads the active count back every four
// iterations, so it synchronises the stream); work holds
// fine_pcg_doubles_per_sample(n) N doubles.  iters [N] receives the
// iterations each sample took, status [N] (may be NULL) OK or ENOCONV.
hipError_t launch_fine_pcg(const double* a, int n, int64_t N, double tol, int max_iter, double* u, int32_t* iters,
                           int32_t* status, double* work, hipStream_t st) {
  const int nlev = fmg_levels(n);
  const int64_t P0 = (int64_t)(n + 1) * (n + 1);
  double* w = work;
  auto take = [&](int64_t cnt) {
    double* p = w;
    w += cnt;
    return p;
  };
  double* r[2] = {take(P0 * N), take(P0 * N)};
  double* p[2] = {take(P0 * N), take(P0 * N)};
  FmgLevel lv[16];
  int nn = n;
  for (int l = 0; l < nlev; ++l) {
    const int64_t P = (int64_t)(nn + 1) * (nn + 1);
    lv[l].n = nn;
    lv[l].x = take(P * N);
    lv[l].t = take(P * N);
    if (l == 0) {
      lv[l].a = a;
      lv[l].b = r[0];
    } else {
      lv[l].b = take(P * N);
      double* ac = take((int64_t)nn * nn * N);
      if (l == 1 || lv[l - 1].n > FMG_SMALL) {  // fmg_small forms those of its own levels
        const dim3 ge((unsigned)(((int64_t)nn * nn + FMG_TB - 1) / FMG_TB), (unsigned)N);
        hipLaunchKernelGGL(fmg_coef_kernel, ge, dim3(FMG_TB), 0, st, lv[l - 1].a, lv[l - 1].n, ac);
      }
      lv[l].a = ac;
    }
    nn /= 2;
  }
  FmgCg c{};
  c.n = n;
  c.nsamples = N;
  c.u = u;
  c.part = take(fmg_parts(n) * N);
  c.rz = take(N);
  c.rr = take(N);
  c.alpha = take(N);
  c.beta = take(N);
  c.active = (int32_t*)take((N + 1) / 2);
  c.iters = iters;
  c.nactive = (unsigned int*)take(1);
  const double h2 = 1.0 / ((double)n * n);
  c.limit = tol * tol * (h2 * h2 * (double)(n - 1) * (double)(n - 1));
  const dim3 b(FMG_TB);
  const dim3 gs((unsigned)N), bs(FMG_TB);         // scalar steps: one workgroup per sample
  const dim3 gst((unsigned)((N + 63) / 64)), bst(64);  // status: one thread per sample
  const bool pre = nlev > 1;
  DownArgs d{};
  d.L = lv[0];
  d.N = N;
  d.bc = pre ? lv[1].b : nullptr;
  d.u = u;
  d.alpha = c.alpha;
  d.part = c.part;
  hipLaunchKernelGGL(fmg_scalar_kernel<0>, gs, bs, 0, st, c, 0, 0);
  d.r1 = r[0];
  d.g = stream_grid(n, N, pre ? 4 : 1, 4096);
  if (pre)
    hipLaunchKernelGGL((fmg_down_kernel<2, true>), dim3(stream_blocks(d.g, N)), b, 0, st, d);
  else
    hipLaunchKernelGGL((fmg_down_kernel<2, false>), dim3(stream_blocks(d.g, N)), b, 0, st, d);
  int parts = 0;
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = fmg_vcycle(lv, nlev, 0, N, c.active, c.part, &parts, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fmg_scalar_kernel<1>, gs, bs, 0, st, c, parts, 0);
  d.active = c.active;
  StepArgs sa{};
  sa.n = n;
  sa.g = stream_grid(n, N, 1, 5120);
  sa.N = N;
  sa.active = c.active;
  sa.a = a;
  sa.beta = c.beta;
  sa.part = c.part;
  for (int it = 0; it < max_iter; ++it) {
    sa.z = lv[0].x;
    sa.p0 = p[it & 1];
    sa.p1 = p[1 - (it & 1)];
    sa.first = it == 0;
    hipLaunchKernelGGL(fmg_step_kernel, dim3(stream_blocks(sa.g, N)), b, 0, st, sa);
    hipLaunchKernelGGL(fmg_scalar_kernel<2>, gs, bs, 0, st, c, sa.g.parts, it);
    d.L = lv[0];
    d.p = sa.p1;
    d.r0 = r[it & 1];
    d.r1 = r[1 - (it & 1)];
    d.first = it == 0;
    if (pre)
      hipLaunchKernelGGL((fmg_down_kernel<1, true>), dim3(stream_blocks(d.g, N)), b, 0, st, d);
    else
      hipLaunchKernelGGL((fmg_down_kernel<1, false>), dim3(stream_blocks(d.g, N)), b, 0, st, d);
    lv[0].b = d.r1;
    const bool check = (it % 4 == 3) || it == max_iter - 1;
    if (check) hipLaunchKernelGGL(fmg_zero_kernel, dim3(1), dim3(1), 0, st, c.nactive);
    hipLaunchKernelGGL(fmg_scalar_kernel<3>, gs, bs, 0, st, c, d.g.parts, it);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (check) {
      unsigned int na = 0;
      e = hipMemcpyAsync(&na, c.nactive, sizeof(na), hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return e;
      if (na == 0) break;
    }
    e = fmg_vcycle(lv, nlev, 0, N, c.active, c.part, &parts, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fmg_scalar_kernel<4>, gs, bs, 0, st, c, parts, it);
  }
  if (status) hipLaunchKernelGGL(fmg_status_kernel, gst, bst, 0, st, c, status);
  return hipGetLastError();
}

}  // namespace stomsfem
