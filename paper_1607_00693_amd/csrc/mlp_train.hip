// Training step of the per-patch networks: FP32 forward, hand-written
// backward and the Adam update, one workgroup of four wavefronts per patch.
//
//   mlp_train_kernel<TRAIN>  with TRAIN the Adam update is applied where a
//                            gradient is formed, otherwise the raw gradient
//                            is written (parity checks against the oracle).
//
// Every product of a step is a contraction over 16 x 16 tiles and goes through
// v_mfma_f32_16x16x4_f32 (FP32 operands and sums, twice the rate of
// v_fma_f32).  In its register layouts lane (n, q) = (lane % 16, lane / 16)
// holds
//     A: A[row n][k = q],   B: B[k = q][column n],   C: C[row 4 q + i][column n],
// and a contraction may take its k in any order as long as A and B agree.
// With k = 16 j + 4 q + s in instruction (j, s), a B operand is exactly the
// C layout of a tile: wavefront w owns the 16 output columns of every layer
// from 16 w on, keeps its columns of the weights in the C layout of their
// gradients, and so
//   - a forward product takes its B operand from the registers of the weights,
//   - a weight gradient takes its B operand from the registers of the layer's
//     derivative (and the last layer's A operand from those of H3),
//   - the parameters and both Adam moments stay in registers over all steps
//     (42 of each per lane) and memory is not read for them between the steps.
// LDS holds the activations as A operands (row stride 68 floats: neither the
// float4 nor the column reads of the 16-lane groups meet in a bank), and the
// weights a second time for the products with their transposes.  79 KB: two
// workgroups per CU, so that one's matrix products run beside the other's
// vector work.
//
// Bounds: per step and patch a SIMD has 244 matrix instructions of 32 cycles;
// 24 GELU values with derivatives and 42 Adam updates per lane cost about the
// same again on the vector units.
#include "mlp.h"

namespace stomsfem {
namespace {

constexpr int MB = MLP_BATCH;
constexpr int WD = MLP_WIDTH;
constexpr int NO = MLP_NOUT2;
constexpr int LDH = WD + 4;  // row stride of activations and weights in LDS
static_assert(MB == 32 && WD == 64 && NO == 20 && MLP_KIN == 4, "tiling of the training kernel");

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// GELU z Phi(z) and its derivative Phi + z phi without branches, from one
// exponential e = exp(-z^2 / 2):  |z| < 1: Phi = 1/2 + z P(z^2);  else
// Phi(-|z|) = e Q(|z|), Q(u) = erfcx(u / sqrt 2) / 2 = t R(t), t = 1 / (1 + u / 4).
// P and R are least-maximum-error fits (relative errors 3e-10 and 2e-8).
// Error against FP64 over |z| <= 12: 3.8e-7 and 1.2e-7, as with a correctly
// rounded erf in FP32 (4.5e-7 and 1.3e-7), which takes two branches per value.
__device__ __forceinline__ void gelu_both(float z, float* h, float* g) {
  const float u = fabsf(z), zz = z * z;
  const float e = __builtin_amdgcn_exp2f(zz * -0.72134752f);
  const float t = __builtin_amdgcn_rcpf(fmaf(u, 0.25f, 1.0f));
  float r = -0.04640737920999527f;
  r = fmaf(r, t, 0.10818030685186386f);
  r = fmaf(r, t, -0.020968716591596603f);
  r = fmaf(r, t, 0.0912889912724495f);
  r = fmaf(r, t, 0.07396240532398224f);
  r = fmaf(r, t, 0.09450826793909073f);
  r = fmaf(r, t, 0.09966841340065002f);
  r = fmaf(r, t, 0.09973665326833725f);
  r = r * t * e;
  float p = -7.664680197194684e-06f;
  p = fmaf(p, zz, 0.00011351265857229009f);
  p = fmaf(p, zz, -0.0011863530380651355f);
  p = fmaf(p, zz, 0.009973331354558468f);
  p = fmaf(p, zz, -0.06649035960435867f);
  p = fmaf(p, zz, 0.3989422917366028f);
  asm volatile("" : "+v"(r), "+v"(p));  // both are formed: a select, not a branch
  const float tail = z > 0.0f ? 1.0f - r : r;
  const float Phi = u < 1.0f ? fmaf(z, p, 0.5f) : tail;
  *h = z * Phi;
  *g = fmaf(z, e * 0.39894228040143268f, Phi);
}

struct TrainLds {
  float W2[WD * LDH], W3[WD * LDH], W4[WD * NO];
  float H1[MB * LDH], H2[MB * LDH], H3[MB * LDH], D[MB * LDH];  // H3 becomes the derivative of layer 3
  float dY[MB * NO], X[MB * MLP_KIN], T[MB * 10], red[4];
};
static_assert(sizeof(TrainLds) <= 81920, "two workgroups per CU");

// one parameter with its moments
struct Par {
  float p, m, v;
};
struct Adam {
  float rate;    // lr / (1 - 0.9^t)
  float icorr2;  // 1 / (1 - 0.999^t)
};

// The square root and the reciprocal are the instructions' (within one unit in
// the last place each): an update is rate-sized, so their error is 1e-3 of the
// rounding of p itself.
__device__ __forceinline__ void adam(Par& x, float g, const Adam& c) {
  x.m = 0.9f * x.m + (1.0f - 0.9f) * g;
  x.v = 0.999f * x.v + (1.0f - 0.999f) * g * g;
  x.p -= c.rate * x.m * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(x.v * c.icorr2) + 1e-8f);
}

// sum over the four 16-lane groups; the same bits in all of them
__device__ __forceinline__ float group_sum(float s) {
  s += __shfl_xor(s, 16);
  return s + __shfl_xor(s, 32);
}
__device__ __forceinline__ float sum4(const f4& a) { return (a[0] + a[1]) + (a[2] + a[3]); }

// Places of a lane's parameters: W2, W3 [t][i] = W[16 t + 4 q + i][col], W4 [i] =
// W4[16 w + 4 q + i][n] and W4[col][16 + q], W1[q][col], one bias of each
// layer (of the last one: that of the lane's column in its forward tile).
struct Place {
  unsigned n, q, col, row4, o4, ob4;
  __device__ __forceinline__ Place(unsigned w, unsigned lane)
      : n(lane & 15), q(lane >> 4), col(16 * w + n), row4(4 * q), o4(16 * (w & 1) + n), ob4(o4 < NO ? o4 : NO - 1) {}
  __device__ __forceinline__ unsigned W(unsigned off, int t, int i) const { return (row4 * WD + col) + (off + (16 * t + i) * WD); }
  __device__ __forceinline__ unsigned W4(unsigned w, int i) const { return (row4 * NO + n) + (MLP_OW4 + (16 * w + i) * NO); }
  __device__ __forceinline__ unsigned W4b() const { return col * NO + q + (MLP_OW4 + 16); }
  __device__ __forceinline__ unsigned W1() const { return q * WD + col + MLP_OW1; }
};

template <bool TRAIN>
__global__ __launch_bounds__(256, 2) void mlp_train_kernel(MlpTrainArgs a) {
  __shared__ TrainLds L;
  const int K = blockIdx.x;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned lane = tid & 63;
  Place at(w, lane);
  const unsigned &n = at.n, &q = at.q, &col = at.col, &o4 = at.o4, &ob4 = at.ob4;
  float* const P = a.params + (int64_t)K * MLP_NP;
  float* const P1 = TRAIN ? a.m1 + (int64_t)K * MLP_NP : nullptr;
  float* const P2 = TRAIN ? a.m2 + (int64_t)K * MLP_NP : nullptr;
  auto load = [&](unsigned i) {
    Par x;
    x.p = P[i];
    x.m = TRAIN ? P1[i] : 0.0f;
    x.v = TRAIN ? P2[i] : 0.0f;
    return x;
  };
  Par W1 = load(at.W1()), b1 = load(MLP_OB1 + col), b2 = load(MLP_OB2 + col), b3 = load(MLP_OB3 + col);
  Par b4 = load(MLP_OB4 + ob4), W4b = load(at.W4b());
  Par W2[4][4], W3[4][4], W4[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      W2[t][i] = load(at.W(MLP_OW2, t, i));
      W3[t][i] = load(at.W(MLP_OW3, t, i));
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) W4[i] = load(at.W4(w, i));

  auto put_W = [&](float* dst, const Par(&W)[4][4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[(16 * t + 4 * q + i) * LDH + col] = W[t][i].p;
  };
  auto put_W4 = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) L.W4[(16 * w + 4 * q + i) * NO + n] = W4[i].p;
    L.W4[col * NO + 16 + q] = W4b.p;
  };
  put_W(L.W2, W2);
  put_W(L.W3, W3);
  put_W4();

  // ---- minibatch: thread b + 32 e has entries 2 e and 2 e + 1 of row b's four
  // inputs and ten targets (e < 7); the values of the next step are on their way
  // during a step, the index of the one after it is read with them
  const int vb = tid & 31, ve = tid >> 5;
  const bool gets = ve < 7;
  int64_t pos = (a.t0 * MB + vb) % a.ntrain, idx = 0;
  const int64_t adv = MB % a.ntrain;
  float val[2] = {0.0f, 0.0f};
  auto sample = [&]() {
    idx = a.perm ? a.perm[pos] : pos;
    idx = idx < 0 ? 0 : (idx >= a.ntrain ? a.ntrain - 1 : idx);  // a malformed perm cannot read out of bounds
  };
  auto fetch = [&](const float* x, const float* y, int64_t row) {
    const float* src = ve < 2 ? x + row * MLP_KIN + 2 * ve : y + row * 10 + 2 * (ve - 2);
    val[0] = src[0];
    val[1] = src[1];
  };
  auto prefetch = [&]() {  // the values of idx; then the index after it
    fetch(a.X, a.T, (int64_t)K * a.ntrain + idx);
    pos += adv;
    if (pos >= a.ntrain) pos -= a.ntrain;
    sample();
  };
  if (gets) {
    if (a.xb) {
      fetch(a.xb, a.tb, (int64_t)K * MB + vb);
    } else {
      sample();
      prefetch();
    }
  }

  // A operand of rows 16 t ... of an activation, k = 16 j + 4 q + s, s = 0..3
  auto rowsA = [&](const float* H, int t, int j) {
    return *reinterpret_cast<const f4*>(H + (16 * t + n) * LDH + 16 * j + 4 * q);
  };
  auto store = [&](float* H, const f4(&h)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) H[(16 * t + 4 * q + i) * LDH + col] = h[t][i];
  };
  auto activate = [&](f4(&z)[2], f4(&g)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float h, d;
        gelu_both(z[t][i], &h, &d);
        z[t][i] = h;
        g[t][i] = d;
      }
  };
  // z = H W + b, W's columns from registers
  auto forward = [&](const float* H, const Par(&W)[4][4], float b, f4(&z)[2]) {
    z[0] = z[1] = f4{b, b, b, b};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f4 a0 = rowsA(H, 0, j), a1 = rowsA(H, 1, j);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        z[0] = mma(a0[s], W[j][s].p, z[0]);
        z[1] = mma(a1[s], W[j][s].p, z[1]);
      }
    }
  };
  // d = (D W^T) .* g, W's rows from LDS
  auto backward = [&](const float* Dl, const float* W, const f4(&g)[2], f4(&d)[2]) {
    d[0] = d[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f4 a0 = rowsA(Dl, 0, j), a1 = rowsA(Dl, 1, j);
      const f4 b = *reinterpret_cast<const f4*>(W + col * LDH + 16 * j + 4 * q);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        d[0] = mma(a0[s], b[s], d[0]);
        d[1] = mma(a1[s], b[s], d[1]);
      }
    }
    d[0] *= g[0];
    d[1] *= g[1];
  };
  Adam c;
  auto update = [&](Par& x, float g, unsigned i, bool own) {
    if (TRAIN)
      adam(x, g, c);
    else if (own)
      a.grads[(int64_t)K * MLP_NP + i] = g;
  };
  // gradient of W2 or W3, columns col: sum over the batch of H[b][k] d[b][col]
  auto weights = [&](const float* H, const f4(&d)[2], Par(&W)[4][4], int off) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f4 g = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int s = 0; s < 4; ++s) g = mma(H[(16 * j + 4 * q + s) * LDH + 16 * t + n], d[j][s], g);
#pragma unroll
      for (int i = 0; i < 4; ++i) update(W[t][i], g[i], at.W(off, t, i), true);
    }
  };
  auto bias = [&](const f4(&d)[2], Par& b, int off) { update(b, group_sum(sum4(d[0]) + sum4(d[1])), off + col, q == 0); };

  for (int step = 0; step < a.steps; ++step) {
    // the LDS addresses are formed in each step: 40 of them kept would spill
    asm volatile("" : "+v"(lane));
    at = Place(w, lane);
    const float t = (float)(a.t0 + step + 1);  // Adam step count
    c.rate = a.lr / (1.0f - powf(0.9f, t));
    c.icorr2 = 1.0f / (1.0f - powf(0.999f, t));
    if (gets) {
      float* dst = ve < 2 ? L.X + vb * MLP_KIN + 2 * ve : L.T + vb * 10 + 2 * (ve - 2);
      dst[0] = val[0];
      dst[1] = val[1];
      if (TRAIN) prefetch();
    }
    __syncthreads();

    // ---- forward
    f4 h[2], g1[2], g2[2], g3[2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
      h[r] = mma(L.X[(16 * r + n) * MLP_KIN + q], W1.p, f4{b1.p, b1.p, b1.p, b1.p});
    activate(h, g1);
    store(L.H1, h);
    __syncthreads();
    forward(L.H1, W2, b2.p, h);
    activate(h, g2);
    store(L.H2, h);
    __syncthreads();
    forward(L.H2, W3, b3.p, h);
    activate(h, g3);
    store(L.H3, h);
    __syncthreads();
    // outputs: tile (w / 2, w % 2) of 32 x 32, columns from 20 on unused
    {
      const int rt = w >> 1;
      f4 y = {b4.p, b4.p, b4.p, b4.p};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f4 a0 = rowsA(L.H3, rt, j);
#pragma unroll
        for (int s = 0; s < 4; ++s) y = mma(a0[s], L.W4[(16 * j + 4 * q + s) * NO + ob4], y);
      }
      float lpart = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = 16 * rt + 4 * q + i;
        if (o4 < NO) {
          const float r = y[i] - L.T[b * 10 + (o4 < 10 ? o4 : o4 - 10)];
          lpart += r * r;
          L.dY[b * NO + o4] = 2.0f * r / (float)(MB * NO);
        }
      }
      if (a.loss && step == a.steps - 1) {
        for (int s = 1; s < 64; s <<= 1) lpart += __shfl_xor(lpart, s);
        if ((tid & 63) == 0) L.red[w] = lpart;
      }
    }
    __syncthreads();
    if (a.loss && step == a.steps - 1 && tid == 0)
      a.loss[K] = ((L.red[0] + L.red[1]) + (L.red[2] + L.red[3])) / (float)(MB * NO);

    // ---- backward
    // derivative of layer 3, to the place of H3 (whose columns col are in h)
    f4 d[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      const float b = L.W4[col * NO + 4 * s + q];
#pragma unroll
      for (int r = 0; r < 2; ++r) d[r] = mma(L.dY[(16 * r + n) * NO + 4 * s + q], b, d[r]);
    }
    d[0] *= g3[0];
    d[1] *= g3[1];
    store(L.H3, d);
    __syncthreads();
    // last layer: rows 16 w ... of the first 16 outputs; the other four outputs
    // as rows 0, 4, 8, 12 of a transposed tile, so that lane group q gets output 16 + q
    {
      f4 g = {0.0f, 0.0f, 0.0f, 0.0f}, gb = {0.0f, 0.0f, 0.0f, 0.0f};
      float sb = 0.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float* y = L.dY + (16 * j + 4 * q + s) * NO;
          g = mma(h[j][s], y[n], g);
          gb = mma((n & 3) == 0 ? y[16 + (n >> 2)] : 0.0f, h[j][s], gb);
          sb += y[ob4];
        }
#pragma unroll
      for (int i = 0; i < 4; ++i) update(W4[i], g[i], at.W4(w, i), true);
      update(W4b, gb[0], at.W4b(), true);
      update(b4, group_sum(sb), MLP_OB4 + ob4, w < 2 && q == 0 && o4 < NO);
      if (TRAIN) put_W4();
    }
    f4 d2[2];
    backward(L.H3, L.W3, g2, d2);
    store(L.D, d2);
    __syncthreads();
    weights(L.H2, d, W3, MLP_OW3);
    bias(d, b3, MLP_OB3);
    if (TRAIN) put_W(L.W3, W3);
    backward(L.D, L.W2, g1, d);
    __syncthreads();
    weights(L.H1, d2, W2, MLP_OW2);
    bias(d2, b2, MLP_OB2);
    if (TRAIN) put_W(L.W2, W2);
    {
      f4 g = {0.0f, 0.0f, 0.0f, 0.0f};  // input k as row 4 k: lane group q gets input q
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int s = 0; s < 4; ++s)
          g = mma((n & 3) == 0 ? L.X[(16 * j + 4 * q + s) * MLP_KIN + (n >> 2)] : 0.0f, d[j][s], g);
      update(W1, g[0], at.W1(), true);
      bias(d, b1, MLP_OB1);
    }
    __syncthreads();
  }

  if (!TRAIN) return;
  // the places are formed again here, not kept over the steps
  asm volatile("" : "+v"(lane));
  const Place to(w, lane);
  auto put = [&](const Par& x, unsigned i) {
    P[i] = x.p;
    P1[i] = x.m;
    P2[i] = x.v;
  };
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      put(W2[t][i], to.W(MLP_OW2, t, i));
      put(W3[t][i], to.W(MLP_OW3, t, i));
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) put(W4[i], to.W4(w, i));
  put(W4b, to.W4b());
  put(W1, to.W1());
  if (to.q == 0) {
    put(b1, MLP_OB1 + to.col);
    put(b2, MLP_OB2 + to.col);
    put(b3, MLP_OB3 + to.col);
    if (w < 2 && to.o4 < NO) put(b4, MLP_OB4 + to.o4);
  }
}

}  // namespace

hipError_t launch_mlp_train(const MlpTrainArgs& a, bool train, hipStream_t st) {
  if (train)
    hipLaunchKernelGGL(mlp_train_kernel<true>, dim3(a.npatch), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(mlp_train_kernel<false>, dim3(a.npatch), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace stomsfem
