// Row-distributed banded LDL^T in registers: the pieces shared by the cell
// solvers.  Sixteen lanes (one DPP row) hold one problem, lane r the rows
// i = r (mod 16) of the live window; the pivot column's entries reach the
// other lanes through the row broadcast of the FP64 multiply-add itself
// (v_fmac_f64 with row_newbcast), so a rank-1 update reads neither LDS nor
// scalar registers: one instruction per column updates that column of four
// problems.  On gfx950 this form issues at the rate of a plain v_fma_f64
// (4.5 cycles per SIMD against 4.6 measured with four wavefronts), and FP64
// MFMA shares that pipe (16x16x4: 104 cycles for the work of 16 FMAs), so it
// has nothing to add here.
//
// A DPP operand may be read two wait states after a vector instruction wrote
// it.  The compiler does not look into inline assembly for that, so every
// block below starts with its own s_nop 1 and writes no register that a
// later instruction of the block reads: the accumulators of a block with more
// than one instruction are early-clobber operands, so that an input of the
// same value gets a register of its own.  All 64 lanes must be active.
#pragma once
#include <type_traits>
#include <utility>

#include "small_cell.h"

namespace stomsfem {

#define BR_DPP(w, c, l, n) "v_fmac_f64_dpp " w ", " c ", " l " row_newbcast:" n " row_mask:0xf bank_mask:0xf\n\t"

// columns [C0, C0 + N) of w, N <= 16: w[c] += col(lane c of the row) * nl, in
// one block so that the wait is paid once
template <int C0, int N>
__device__ __forceinline__ void row_update(double* w, double col, double nl) {
  static_assert(N >= 1 && N <= 16 && C0 + N <= 16, "columns of one block");
  if constexpr (N == 16) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%16", "%17", "%18")
            BR_DPP("%1", "%16", "%17", "%19")
            BR_DPP("%2", "%16", "%17", "%20")
            BR_DPP("%3", "%16", "%17", "%21")
            BR_DPP("%4", "%16", "%17", "%22")
            BR_DPP("%5", "%16", "%17", "%23")
            BR_DPP("%6", "%16", "%17", "%24")
            BR_DPP("%7", "%16", "%17", "%25")
            BR_DPP("%8", "%16", "%17", "%26")
            BR_DPP("%9", "%16", "%17", "%27")
            BR_DPP("%10", "%16", "%17", "%28")
            BR_DPP("%11", "%16", "%17", "%29")
            BR_DPP("%12", "%16", "%17", "%30")
            BR_DPP("%13", "%16", "%17", "%31")
            BR_DPP("%14", "%16", "%17", "%32")
            BR_DPP("%15", "%16", "%17", "%33")
        : "+&v"(w[C0]), "+&v"(w[C0 + 1]), "+&v"(w[C0 + 2]), "+&v"(w[C0 + 3]), "+&v"(w[C0 + 4]), "+&v"(w[C0 + 5]),
          "+&v"(w[C0 + 6]), "+&v"(w[C0 + 7]), "+&v"(w[C0 + 8]), "+&v"(w[C0 + 9]), "+&v"(w[C0 + 10]), "+&v"(w[C0 +
          11]), "+&v"(w[C0 + 12]), "+&v"(w[C0 + 13]), "+&v"(w[C0 + 14]), "+&v"(w[C0 + 15])
        : "v"(col), "v"(nl), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3), "n"(C0 + 4), "n"(C0 + 5), "n"(C0
          + 6), "n"(C0 + 7), "n"(C0 + 8), "n"(C0 + 9), "n"(C0 + 10), "n"(C0 + 11), "n"(C0 + 12), "n"(C0 + 13),
          "n"(C0 + 14), "n"(C0 + 15));
  } else if constexpr (N >= 8) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%8", "%9", "%10")
            BR_DPP("%1", "%8", "%9", "%11")
            BR_DPP("%2", "%8", "%9", "%12")
            BR_DPP("%3", "%8", "%9", "%13")
            BR_DPP("%4", "%8", "%9", "%14")
            BR_DPP("%5", "%8", "%9", "%15")
            BR_DPP("%6", "%8", "%9", "%16")
            BR_DPP("%7", "%8", "%9", "%17")
        : "+&v"(w[C0]), "+&v"(w[C0 + 1]), "+&v"(w[C0 + 2]), "+&v"(w[C0 + 3]), "+&v"(w[C0 + 4]), "+&v"(w[C0 + 5]),
          "+&v"(w[C0 + 6]), "+&v"(w[C0 + 7])
        : "v"(col), "v"(nl), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3), "n"(C0 + 4), "n"(C0 + 5), "n"(C0
          + 6), "n"(C0 + 7));
    if constexpr (N > 8) row_update<C0 + 8, N - 8>(w, col, nl);
  } else if constexpr (N >= 4) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%4", "%5", "%6")
            BR_DPP("%1", "%4", "%5", "%7")
            BR_DPP("%2", "%4", "%5", "%8")
            BR_DPP("%3", "%4", "%5", "%9")
        : "+&v"(w[C0]), "+&v"(w[C0 + 1]), "+&v"(w[C0 + 2]), "+&v"(w[C0 + 3])
        : "v"(col), "v"(nl), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3));
    if constexpr (N > 4) row_update<C0 + 4, N - 4>(w, col, nl);
  } else if constexpr (N == 3) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%3", "%4", "%5")
            BR_DPP("%1", "%3", "%4", "%6")
            BR_DPP("%2", "%3", "%4", "%7")
        : "+&v"(w[C0]), "+&v"(w[C0 + 1]), "+&v"(w[C0 + 2])
        : "v"(col), "v"(nl), "n"(C0), "n"(C0 + 1), "n"(C0 + 2));
  } else if constexpr (N == 2) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%2", "%3", "%4")
            BR_DPP("%1", "%2", "%3", "%5")
        : "+&v"(w[C0]), "+&v"(w[C0 + 1])
        : "v"(col), "v"(nl), "n"(C0), "n"(C0 + 1));
  } else if constexpr (N == 1) {
    asm("s_nop 1\n\t"
            BR_DPP("%0", "%1", "%2", "%3")
        : "+v"(w[C0])
        : "v"(col), "v"(nl), "n"(C0));
  }
}

// columns [C0, C1) of w
template <int C0, int C1>
__device__ __forceinline__ void row_updates(double* w, double col, double nl) {
  if constexpr (C0 < C1) row_update<C0, C1 - C0>(w, col, nl);
}

// v of lane L of the row, in every lane of the row
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
  double d;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(v), "n"(L));
  return d;
}

// g += f(lane L of the row) * nl for three right-hand sides; f itself is
// updated by row_rhs_own, after every other block of rows
template <int L>
__device__ __forceinline__ void row_rhs3(double* g, const double* f, double nl) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%3", "%6", "%7") BR_DPP("%1", "%4", "%6", "%7") BR_DPP("%2", "%5", "%6", "%7")
      : "+&v"(g[0]), "+&v"(g[1]), "+&v"(g[2])
      : "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(nl), "n"(L));
}
template <int L>
__device__ __forceinline__ void row_rhs3_own(double* f, double nl) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%0", "%3", "%4") BR_DPP("%1", "%1", "%3", "%4") BR_DPP("%2", "%2", "%3", "%4")
      : "+&v"(f[0]), "+&v"(f[1]), "+&v"(f[2])
      : "v"(nl), "n"(L));
}

// g += f(lane L of the row) * nl, and the same with f in the place of g
template <int L>
__device__ __forceinline__ void row_rhs1(double& g, double f, double nl) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%1", "%2", "%3") : "+v"(g) : "v"(f), "v"(nl), "n"(L));
}
template <int L>
__device__ __forceinline__ void row_rhs1_own(double& f, double nl) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%0", "%1", "%2") : "+v"(f) : "v"(nl), "n"(L));
}

// g[v] += z[v](lane L of the row) * c for ten right-hand sides
template <int L>
__device__ __forceinline__ void row_rhs10(double* g, const double* z, double c) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%10", "%20", "%21") BR_DPP("%1", "%11", "%20", "%21")
          BR_DPP("%2", "%12", "%20", "%21") BR_DPP("%3", "%13", "%20", "%21") BR_DPP("%4", "%14", "%20", "%21")
              BR_DPP("%5", "%15", "%20", "%21") BR_DPP("%6", "%16", "%20", "%21") BR_DPP("%7", "%17", "%20", "%21")
                  BR_DPP("%8", "%18", "%20", "%21") BR_DPP("%9", "%19", "%20", "%21")
      : "+&v"(g[0]), "+&v"(g[1]), "+&v"(g[2]), "+&v"(g[3]), "+&v"(g[4]), "+&v"(g[5]), "+&v"(g[6]), "+&v"(g[7]), "+&v"(g[8]),
        "+&v"(g[9])
      : "v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]), "v"(z[4]), "v"(z[5]), "v"(z[6]), "v"(z[7]), "v"(z[8]), "v"(z[9]),
        "v"(c), "n"(L));
}

// acc[i] += y(lane i of the row) * nl, i < 3
__device__ __forceinline__ void row_lifts3(double* acc, double y, double nl) {
  asm("s_nop 1\n\t" BR_DPP("%0", "%3", "%4", "0") BR_DPP("%1", "%3", "%4", "1") BR_DPP("%2", "%3", "%4", "2")
      : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2])
      : "v"(y), "v"(nl));
}

// Lane masks of the four rows of a wavefront as a scalar constant.
__host__ __device__ constexpr unsigned long long row_mask_at(int r) { return 0x0001000100010001ull << r; }
__host__ __device__ constexpr unsigned long long row_mask_above(int r) {
  return r >= 15 ? 0ull : (0xffffull & ~((2ull << r) - 1)) * 0x0001000100010001ull;
}

// -1/d by Newton's iteration on the hardware reciprocal estimate (two steps
// take the estimate to full double precision).
__device__ __forceinline__ double neg_recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = __builtin_fma(-d, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(-r, e, -r);
}

#define WAVE_SYNC()                                        \
  do {                                                     \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); \
    __builtin_amdgcn_wave_barrier();                       \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); \
  } while (0)

// The live window while a panel of 16 pivots is eliminated: row blocks
// b = 0 (the panel's own rows) ... NS, 16 rows each, with column blocks
// k <= b.  Block NS enters during the panel: its column c is first touched by
// pivot c or later, so block (NS, NS) takes over the registers that the pivot
// columns of block (0, 0) leave, column by column.  From one panel to the
// next every block moves one step up and to the left; instead of copying, the
// arrays of one diagonal (b - k = o) take turns, and the panel code is
// instantiated for each of the PERIOD phases.
template <int NS>
struct RowWindow {
  static_assert(NS == 1 || NS == 2, "phases worked out for one and two row blocks");
  static constexpr int PERIOD = NS;
  double diag[NS][16];  // (b, b), b = 0 .. NS - 1, and (NS, NS) in the place of (0, 0)
  double sub[NS][16];   // (b, b - 1), b = 1 .. NS
  double far[16];       // (2, 0)
  template <int PH>
  __device__ __forceinline__ double* block(int b, int k) {
    return b == k ? diag[(b + PH) % NS] : b == k + 1 ? sub[(k + PH) % NS] : far;
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int c = 0; c < 16; ++c) {
#pragma unroll
      for (int i = 0; i < NS; ++i) diag[i][c] = sub[i][c] = 0.0;
      far[c] = 0.0;
    }
  }
};

// LDS image that spreads the 16 entering rows' couplings over the columns of
// one problem: row 16 (P + NS) + r of a (n = M - 1)-wide nine-point grid has
// SW, S, SE at offsets -M, -M + 1, -M + 2 and W, D at -1, 0.  The columns left
// of block NS and those of block NS take turns in 18 cells per row (column
// OFF + i at cell i + 1, OFF = 16 NS - M; then column 16 NS + c at cell
// c + 1), every unused cell stays zero, cells 0 and 19 always are, and cell 20
// takes what lies outside.  W of row 0 belongs to the block before and is
// added in registers.  M >= 4.
template <int NS, int MC>
struct RowImage {
  static constexpr int LD = 21, SIZE = 16 * LD;  // doubles per problem
  double* row;
  int r, M;
  __device__ __forceinline__ void init(double* img, int r_, int M_) {
    r = r_;
    M = M_;
    row = img + r * LD;
    for (int c = 0; c < LD; ++c) row[c] = 0.0;
  }
  // couplings (of this lane's row) inside block NS: cell, or the dump cell
  __device__ __forceinline__ int inner(int t) const { return r + t >= M ? r + t - M + 1 : 20; }
  __device__ __forceinline__ void put_left(double eSW, double eS, double eSE) {
    row[r] = 0.0;
    if (MC == 0 || MC < 18)
      for (int t = 0; t < 3; ++t) row[inner(t)] = 0.0;
    row[r + 1] = eSW;
    row[r + 2] = eS;
    row[r + 3] = eSE;
  }
  __device__ __forceinline__ void put_diag(double eSW, double eS, double eSE, double eW, double eD) {
    row[r + 2] = row[r + 3] = 0.0;
    row[r + 1] = eD;
    row[r == 0 ? 20 : r] = eW;
    if (MC == 0 || MC < 18) {
      row[inner(0)] = eSW;
      row[inner(1)] = eS;
      row[inner(2)] = eSE;
    }
  }
  // column q < 16 NS (after put_left), eW = this row's W coupling
  __device__ __forceinline__ double left(int q, double eW) const {
    const int i = q - (16 * NS - (MC ? MC : M));
    double v = 0.0;
    if (MC == 0)
      v = row[(i < -1 ? -1 : i > 18 ? 18 : i) + 1];
    else if (i >= 0 && i < 18)
      v = row[i + 1];
    if (q == 16 * NS - 1) v += __builtin_amdgcn_inverse_ballot_w64(row_mask_at(0)) ? eW : 0.0;
    return v;
  }
  // column c of block NS (after put_diag)
  __device__ __forceinline__ double diag(int c) const { return row[c + 1]; }
};

// f += bilinear data: (K p^l) at a node from its four element coefficients,
// l = 0, 1, 2, on a grid of 1/rm cells per side whose element south-west of
// the node has its centre at (xw, ys).  Linear in the coefficients, so
// elements that do not count are passed as 0.
__device__ __forceinline__ void bilinear_load(double aSW, double aSE, double aNW, double aNE, double xw, double ys,
                                              double rm, double* f) {
  const double h2 = 0.5 * rm, t6 = rm * rm * (1.0 / 6.0);
  const double dS = aSW - aSE, dN = aNW - aNE, dW = aSW - aNW, dE = aSE - aNE;
  const double P0 = dS + dN, Q0 = dW + dE;
  const double P1 = ys * P0 + rm * dN, Q1 = xw * Q0 + rm * dE;
  const double T = t6 * (dS - dN);
  f[0] = h2 * ((P1 - P0) + (Q1 - Q0)) + T;
  f[1] = h2 * ((P0 - P1) - Q1) - T;
  f[2] = h2 * (P1 + Q1) + T;
}

// Nine-point couplings of an interior node to its lower neighbours, and its
// diagonal, from the four element coefficients; rows past the grid are
// identity rows.
struct NodeRow {
  double SW, S, SE, W, D;
  __device__ __forceinline__ void set(const double* q4, int ix, int iy, int n) {
    const bool in = iy < n, w = ix >= 1, so = iy >= 1;
    SW = (in && w && so) ? -q4[0] * (1.0 / 3.0) : 0.0;
    S = (in && so) ? -(q4[0] + q4[1]) * (1.0 / 6.0) : 0.0;
    SE = (in && so && ix <= n - 2) ? -q4[1] * (1.0 / 3.0) : 0.0;
    W = (in && w) ? -(q4[0] + q4[2]) * (1.0 / 6.0) : 0.0;
    D = in ? (2.0 / 3.0) * ((q4[0] + q4[1]) + (q4[2] + q4[3])) : 1.0;
  }
};

}  // namespace stomsfem
