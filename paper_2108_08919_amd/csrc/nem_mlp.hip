// nem_mlp.hip -- the learned corrector's network on gfx950 matrix cores.
//
// A 12 -> 64 -> 64 -> 5 perceptron (tanh hidden layers, linear output) on
// z-scored inputs and targets. Every product runs on v_mfma_f32_16x16x32_bf16
// (BF16 operands, FP32 accumulation); master weights, Adam moments and all
// element-wise work stay in FP32. Inference keeps a wave's activations in
// registers; training shares 32 samples between the waves of a workgroup, with
// the activations in LDS as BF16.
//
// MFMA 16x16x32 operand layout (wave64, lane l, i = 0..7 / 0..3):
//   A (16 x 32): A[l % 16][8 (l / 16) + i]      B (32 x 16): B[8 (l / 16) + i][l % 16]
//   D (16 x 16): D[4 (l / 16) + i][l % 16]
//
// Flat parameter vector (FP32): W1 (12 x 64, input-major), b1 (64), W2 (64 x 64),
// b2 (64), W3 (64 x 5), b3 (5).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace nem {

typedef __bf16 bf16;
typedef bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NI = 12, NH = 64, NO = 5;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NI * NH, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH;
constexpr int OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH * NO, NPARAM = OFF_B3 + NO;
constexpr int NORM_SLOTS = 64;   // words of the largest-norm reduction
constexpr int ROWS = 32;  // samples per iteration of the backward kernel

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

struct MlpNorm { float xm[NI], xs[NI], xr[NI], ym[NO], ys[NO]; };  // xr = 1 / xs

// tanh(x) = 1 - 2 / (exp(2x) + 1) on the hardware exp2 and reciprocal (about
// 1e-7 absolute error, far below the BF16 rounding of the activations it
// feeds); exp overflow gives +1, underflow -1.
__device__ __forceinline__ float fast_tanh(float x) {
  const float e = __builtin_amdgcn_exp2f(2.8853900817779268f * x);  // 2 log2(e) x
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// ---------------------------------------------------------------- forward
// Y (n x 5): corrections in physical units (denormalised). maxnorm (may be
// NULL): max over samples of the Euclidean norm of the normalised output, as
// float bits, spread over NORM_SLOTS words (cleared by the caller; the result is
// their largest). Atomics on one word from every wave of the grid took ~10 ns each,
// one after another: at 262,144 samples 40 of the kernel's 61 us.
//
// Inference keeps the activations in registers by computing each layer
// transposed, H^T = W^T X^T: the weights are the A operand (fragments in LDS,
// see FwdLds), the 16 samples of an iteration are the N dimension, and the
// output tile D[4g + i][c] (g = l / 16, c = l % 16) holds hidden units
// 16 mt + 4g + i of sample c. The next layer's B operand needs, in lane l,
// K slots 8g..8g+7 of sample c; numbering the hidden units so that K slot
// 8g + i of K tile kc is unit 16 (2 kc + i / 4) + 4g + i % 4 makes that
// operand exactly the lane's own D registers of tiles 2kc and 2kc+1 (the
// weights' K index uses the same numbering), so no data moves between lanes.
__device__ __forceinline__ int unit_of(int kc, int g, int i) { return 16 * (2 * kc + (i >> 2)) + 4 * g + (i & 3); }

// Weight fragments of the inference kernel in LDS, shared by the workgroup's
// four waves (per-wave register copies of all 5184 weights limited the kernel
// to one or two waves per SIMD): fragment f of lane l at frag[f * 64 + l],
// f = 0..3 layer 1 (m tile), 4..11 layer 2 (4 m tiles x 2 K tiles), 12..13
// layer 3 (K tiles). Biases per lane as the four rows it holds, layers 1 and 2
// pre-scaled by 2 log2(e) for the tanh below.
struct FwdLds {
  bf16x8 frag[14 * 64];
  f32x4 b1[4 * 64], b2[4 * 64], b3[64];
};
constexpr float TANH_K = 2.8853900817779268f;   // 2 log2(e)

// tanh(x) with x = d + bias and kb = TANH_K * bias (see fast_tanh)
__device__ __forceinline__ float tanh_kb(float d, float kb) {
  const float e = __builtin_amdgcn_exp2f(fmaf(TANH_K, d, kb));
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// X rows are 48 bytes; VEC reads them as float4 (X 16-byte aligned). clear: words
// for the next kernel of the stream to fill, zeroed here (NULL: none).
template <bool VEC>
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ P, MlpNorm nm,
                                                     const float* __restrict__ X, int64_t n, float* Y,
                                                     unsigned* maxnorm, unsigned* clear, int nclear) {
  constexpr int NB = 2;  // independent 16-sample blocks per iteration (instruction-level parallelism)
  __shared__ FwdLds W;
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, g = l >> 4, c = l & 15;
  if (clear && blockIdx.x == 0)
    for (int t = threadIdx.x; t < nclear; t += 256) clear[t] = 0u;
  // Fill the fragments: A[m][k] = W^T, lane (g, c) holds k = 8 g + i (in the
  // unit numbering of unit_of for layers 2 and 3) of row m = 16 mt + c. Wave wv
  // fills fragments wv, wv + 4, wv + 8, wv + 12, and asks for all its weights
  // before it uses one (waiting for each in turn: 5 us more).
  {
    float f[4][8], fb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * g + i;
      f[0][i] = k < NI ? P[OFF_W1 + k * NH + 16 * wv + c] : 0.0f;
      f[1][i] = P[OFF_W2 + unit_of(wv & 1, g, i) * NH + 16 * (wv >> 1) + c];         // fragments 4 + wv
      f[2][i] = P[OFF_W2 + unit_of(wv & 1, g, i) * NH + 16 * (2 + (wv >> 1)) + c];   // fragments 8 + wv
      f[3][i] = wv < 2 && c < NO ? P[OFF_W3 + unit_of(wv & 1, g, i) * NO + c] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fb[i] = P[OFF_B1 + 16 * wv + 4 * g + i];
      fb[4 + i] = P[OFF_B2 + 16 * wv + 4 * g + i];
    }
    f32x4 v1, v2, v3;
#pragma unroll
    for (int i = 0; i < 4; ++i) v3[i] = 4 * g + i < NO ? P[OFF_B3 + 4 * g + i] : 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bf16x8 v;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (bf16)f[j][i];
      if (j < 3 || wv < 2) W.frag[(4 * j + wv) * 64 + l] = v;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) { v1[i] = TANH_K * fb[i]; v2[i] = TANH_K * fb[4 + i]; }
    W.b1[wv * 64 + l] = v1;
    W.b2[wv * 64 + l] = v2;
    if (wv == 0) W.b3[l] = v3;
  }
  __syncthreads();
  // this lane's input features 8g + i (i < nf) and their normalisation
  const int nf = g == 0 ? 8 : (g == 1 ? NI - 8 : 0);
  float xm8[8], xr8[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    xm8[i] = i < nf ? nm.xm[8 * g + i] : 0.0f;
    xr8[i] = i < nf ? nm.xr[8 * g + i] : 0.0f;
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  float mx = 0.0f;
  const int64_t nblk = (n + 15) / 16;
  for (int64_t b0 = ((int64_t)blockIdx.x * 4 + wv) * NB; b0 < nblk; b0 += (int64_t)gridDim.x * 4 * NB) {
    int64_t s[NB];
    bf16x8 xb[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      s[q] = (b0 + q) * 16 + c;
      const float* xrow = X + (s[q] < n ? s[q] : n - 1) * NI + 8 * g;  // clamped: in bounds for every lane
      float xv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (VEC) {
        if (nf > 0) {
          const float4 v0 = *reinterpret_cast<const float4*>(xrow);
          xv[0] = v0.x; xv[1] = v0.y; xv[2] = v0.z; xv[3] = v0.w;
        }
        if (nf > 4) {
          const float4 v1 = *reinterpret_cast<const float4*>(xrow + 4);
          xv[4] = v1.x; xv[5] = v1.y; xv[6] = v1.z; xv[7] = v1.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (i < nf) xv[i] = xrow[i];
      }
      const float keep = s[q] < n ? 1.0f : 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) xb[q][i] = (bf16)(keep * ((xv[i] - xm8[i]) * xr8[i]));
    }
    // The fragment and bias reads below are the same every iteration; an
    // empty asm statement on the lane index keeps the compiler from hoisting
    // them out of the loop into registers (which would cost the occupancy the
    // LDS copy is for).
    int l_ = l;
    asm volatile("" : "+v"(l_));
    f32x4 d[NB][4];
    bf16x8 hb[NB][2];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 a = W.frag[mt * 64 + l_];
#pragma unroll
      for (int q = 0; q < NB; ++q) d[q][mt] = mfma(a, xb[q], zero);
    }
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const f32x4 k0 = W.b1[(2 * kc) * 64 + l_], k1 = W.b1[(2 * kc + 1) * 64 + l_];
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          hb[q][kc][i] = (bf16)tanh_kb(d[q][2 * kc][i], k0[i]);
          hb[q][kc][4 + i] = (bf16)tanh_kb(d[q][2 * kc + 1][i], k1[i]);
        }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 a0 = W.frag[(4 + 2 * mt) * 64 + l_], a1 = W.frag[(5 + 2 * mt) * 64 + l_];
#pragma unroll
      for (int q = 0; q < NB; ++q) d[q][mt] = mfma(a1, hb[q][1], mfma(a0, hb[q][0], zero));
    }
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const f32x4 k0 = W.b2[(2 * kc) * 64 + l_], k1 = W.b2[(2 * kc + 1) * 64 + l_];
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          hb[q][kc][i] = (bf16)tanh_kb(d[q][2 * kc][i], k0[i]);
          hb[q][kc][4 + i] = (bf16)tanh_kb(d[q][2 * kc + 1][i], k1[i]);
        }
    }
    const bf16x8 a30 = W.frag[12 * 64 + l_], a31 = W.frag[13 * 64 + l_];
    const f32x4 b3 = W.b3[l_];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const f32x4 y = mfma(a31, hb[q][1], mfma(a30, hb[q][0], b3));
      // lane (g, c) holds outputs 4g + i of sample s: g = 0 -> 0..3, g = 1 -> 4
      float sq = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = 4 * g + i;
        if (o < NO) {
          sq += y[i] * y[i];
          if (s[q] < n) Y[s[q] * NO + o] = y[i] * nm.ys[o] + nm.ym[o];
        }
      }
      sq += __shfl_xor(sq, 16, 64);
      sq += __shfl_xor(sq, 32, 64);
      if (s[q] < n) mx = fmaxf(mx, sqrtf(sq));
    }
  }
  if (maxnorm) {
    __shared__ float red[4];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (l == 0) red[wv] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    if (threadIdx.x == 0 && mx > 0.0f) atomicMax(&maxnorm[blockIdx.x & (NORM_SLOTS - 1)], __float_as_uint(mx));
  }
}

// --------------------------------------------------------------- backward
// Minibatch rows: a deterministic shuffle of [0, n) per epoch, row(k) = (k *
// stride + offset) mod n with stride coprime to n; k, stride, offset < n < 2^31.
struct BatchRows { int64_t first, n, stride, offset; double inv_n; };
__device__ __forceinline__ int64_t batch_row(const BatchRows& m, int64_t k) {
  const int64_t v = (m.first + k) * m.stride + m.offset;
  int64_t r = v - (int64_t)((double)v * m.inv_n) * m.n;   // the quotient is at most n: exact to within one
  if (r < 0) r += m.n;
  if (r >= m.n) r -= m.n;
  return r;
}

// Gradient of L = (1/2B) sum_s |y_s - t_s|^2 (normalised units) over a
// minibatch of (X, T): workgroup b takes the 32-sample blocks b, b + gridDim.x,
// ..., accumulates their gradient in registers and writes one partial vector,
// partial[b][0..NPARAM) and its partial loss at [NPARAM].
//
// A batch is a few hundred dependent matrix instructions and three dependent
// global loads, so it is latency and nothing else. Wave w of four owns the
// hidden units 16 w..16 w + 15 of both layers: its columns of every product and
// its rows of the weight gradients. All its weight fragments are loaded into
// registers at once, beside the samples; every activation is kept in LDS twice,
// by sample and by unit, so that each operand of the forward, backward and
// gradient products is one 16-byte read (rows are padded by 8 to spread them over
// the banks). At 4096 samples a call takes 12.4 us; one wave per block with the
// weights copied to LDS and operands read two bytes at a time took 38 us.
constexpr int LDR = NH + 8;     // by sample: [sample][unit]
constexpr int LDT = ROWS + 8;   // by unit: [unit][sample]
struct Act {
  bf16 xr[ROWS * LDT], xt[16 * LDT];   // inputs, units 12.. zero
  bf16 h1r[ROWS * LDR], h1t[NH * LDT];
  bf16 h2r[ROWS * LDR], h2t[NH * LDT];
  bf16 dyr[ROWS * LDT], dyt[16 * LDT]; // dL/dy, outputs 5.. zero
  bf16 d2r[ROWS * LDR], d2t[NH * LDT]; // dL/d(layer 2 before tanh)
  bf16 d1t[NH * LDT];
  int64_t row[ROWS];                   // source rows, -1 past the batch
};

__device__ __forceinline__ bf16x8 frag(const bf16* S, int ld, int r0, int k0, int l) {
  return *reinterpret_cast<const bf16x8*>(S + (r0 + (l & 15)) * ld + k0 + (l >> 4) * 8);
}
// Store a D tile (rows = samples r0 + 4g + i, column = unit n0 + c) both ways.
__device__ __forceinline__ void store_t(bf16* T, int r0, int n0, int l, bf16x4 v) {
  *reinterpret_cast<bf16x4*>(T + (n0 + (l & 15)) * LDT + r0 + (l >> 4) * 4) = v;
}
__device__ __forceinline__ void store_r(bf16* S, int ld, int r0, int n0, int l, bf16x4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) S[(r0 + (l >> 4) * 4 + i) * ld + n0 + (l & 15)] = v[i];
}

__global__ __launch_bounds__(256) void k_mlp_backward(const float* __restrict__ P, MlpNorm nm,
                                                      const float* __restrict__ X, const float* __restrict__ Tg,
                                                      BatchRows rows, int64_t B, float* partial) {
  __shared__ __attribute__((aligned(16))) Act a;
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, g = l >> 4, c = l & 15;
  const int n0 = 16 * wv, col = n0 + c;
  // this thread's part of the staged inputs: two features of one sample
  const int xrow = threadIdx.x >> 3, xc = 2 * (threadIdx.x & 7);
  const float invB = 1.0f / (float)B;
  const int64_t nblk = (B + ROWS - 1) / ROWS;
  auto sample = [&](int64_t b) {
    const int64_t s = b * ROWS + xrow;
    return s < B ? batch_row(rows, s) : (int64_t)-1;
  };
  int64_t src = sample(blockIdx.x);
  float x0 = 0.0f, x1 = 0.0f;
  auto load_x = [&]() {
    if (src >= 0 && xc < NI) { x0 = X[src * NI + xc]; x1 = X[src * NI + xc + 1]; }
  };
  load_x();
  // B operands: lane holds K slots 8g..8g+7 of its column
  bf16x8 w1, w2[2], w3[2], w3t, w2t[2];
  {
    float f1[8], f2[2][8], f3[2][8], f3t[8], f2t[2][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * g + i;
      f1[i] = k < NI ? P[OFF_W1 + k * NH + col] : 0.0f;
      f3t[i] = k < NO ? P[OFF_W3 + col * NO + k] : 0.0f;
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        f2[kc][i] = P[OFF_W2 + (kc * 32 + k) * NH + col];
        f2t[kc][i] = P[OFF_W2 + col * NH + kc * 32 + k];
        f3[kc][i] = wv == 0 && c < NO ? P[OFF_W3 + (kc * 32 + k) * NO + c] : 0.0f;
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      w1[i] = (bf16)f1[i];
      w3t[i] = (bf16)f3t[i];
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) { w2[kc][i] = (bf16)f2[kc][i]; w2t[kc][i] = (bf16)f2t[kc][i]; w3[kc][i] = (bf16)f3[kc][i]; }
    }
  }
  const float b1 = P[OFF_B1 + col], b2 = P[OFF_B2 + col], b3 = c < NO ? P[OFF_B3 + c] : 0.0f;
  // columns that no sample writes: K padding of the inputs and of dL/dy
  for (int t = threadIdx.x; t < ROWS * 16; t += 256) {
    a.xr[(t >> 4) * LDT + 16 + (t & 15)] = (bf16)0.0f;
    a.dyr[(t >> 4) * LDT + 16 + (t & 15)] = (bf16)0.0f;
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 g1 = zero, g2[4] = {zero, zero, zero, zero}, g3 = zero;
  float gb1 = 0.0f, gb2 = 0.0f, gb3 = 0.0f, ls = 0.0f;
  for (int64_t b = blockIdx.x; b < nblk; b += gridDim.x) {
    {
      const bool in = src >= 0 && xc < NI;
      const bf16 v0 = (bf16)(in ? (x0 - nm.xm[xc]) * nm.xr[xc] : 0.0f);
      const bf16 v1 = (bf16)(in ? (x1 - nm.xm[xc + 1]) * nm.xr[xc + 1] : 0.0f);
      a.xr[xrow * LDT + xc] = v0; a.xr[xrow * LDT + xc + 1] = v1;
      a.xt[xc * LDT + xrow] = v0; a.xt[(xc + 1) * LDT + xrow] = v1;
      if (xc == 0) a.row[xrow] = src;
    }
    __syncthreads();
    float tv[2][4];
    if (wv == 0) {   // targets, in flight until the last layer
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t s = a.row[rt * 16 + g * 4 + i];
          tv[rt][i] = s >= 0 && c < NO ? Tg[s * NO + c] : 0.0f;
        }
    }
    if (b + gridDim.x < nblk) { src = sample(b + gridDim.x); load_x(); }
    float h1[2][4], h2[2][4];   // this lane's activations, as rounded
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const f32x4 acc = mfma(frag(a.xr, LDT, rt * 16, 0, l), w1, zero);
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) { h[i] = (bf16)fast_tanh(acc[i] + b1); h1[rt][i] = (float)h[i]; }
      store_r(a.h1r, LDR, rt * 16, n0, l, h);
      store_t(a.h1t, rt * 16, n0, l, h);
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) acc = mfma(frag(a.h1r, LDR, rt * 16, kc * 32, l), w2[kc], acc);
      bf16x4 h;
#pragma unroll
      for (int i = 0; i < 4; ++i) { h[i] = (bf16)fast_tanh(acc[i] + b2); h2[rt][i] = (float)h[i]; }
      store_r(a.h2r, LDR, rt * 16, n0, l, h);
      store_t(a.h2t, rt * 16, n0, l, h);
    }
    __syncthreads();
    if (wv == 0) {   // y, and dL/dy = (y - t) / B in normalised units
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        f32x4 y = zero;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) y = mfma(frag(a.h2r, LDR, rt * 16, kc * 32, l), w3[kc], y);
        bf16x4 dv;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          y[i] += b3;
          float d = 0.0f;
          if (c < NO && a.row[rt * 16 + g * 4 + i] >= 0) {
            const float t = (tv[rt][i] - nm.ym[c]) / nm.ys[c];
            d = y[i] - t;
            ls += d * d;
          }
          d *= invB;
          gb3 += d;
          dv[i] = (bf16)d;
        }
        store_r(a.dyr, LDT, rt * 16, 0, l, dv);
        store_t(a.dyt, rt * 16, 0, l, dv);
      }
    }
    __syncthreads();
    // gW3 rows of this wave: H2^T dY
    g3 = mfma(frag(a.h2t, LDT, n0, 0, l), frag(a.dyt, LDT, 0, 0, l), g3);
    // dA2 = (dY W3^T) * (1 - h2^2)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const f32x4 acc = mfma(frag(a.dyr, LDT, rt * 16, 0, l), w3t, zero);
      bf16x4 dv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = acc[i] * (1.0f - h2[rt][i] * h2[rt][i]);
        gb2 += d;
        dv[i] = (bf16)d;
      }
      store_r(a.d2r, LDR, rt * 16, n0, l, dv);
      store_t(a.d2t, rt * 16, n0, l, dv);
    }
    __syncthreads();
    // gW2 columns of this wave: H1^T dA2
    const bf16x8 d2 = frag(a.d2t, LDT, n0, 0, l);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) g2[mt] = mfma(frag(a.h1t, LDT, mt * 16, 0, l), d2, g2[mt]);
    // dA1 = (dA2 W2^T) * (1 - h1^2)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      f32x4 acc = zero;
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) acc = mfma(frag(a.d2r, LDR, rt * 16, kc * 32, l), w2t[kc], acc);
      bf16x4 dv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = acc[i] * (1.0f - h1[rt][i] * h1[rt][i]);
        gb1 += d;
        dv[i] = (bf16)d;
      }
      store_t(a.d1t, rt * 16, n0, l, dv);
    }
    __syncthreads();
    // gW1 columns of this wave: X^T dA1 (rows 12.. unused)
    g1 = mfma(frag(a.xt, LDT, 0, 0, l), frag(a.d1t, LDT, n0, 0, l), g1);
    if (b + gridDim.x < nblk) __syncthreads();
  }
  // bias sums: lanes with the same l % 16 hold the same column
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    gb3 += __shfl_xor(gb3, o, 64);
    gb1 += __shfl_xor(gb1, o, 64);
    gb2 += __shfl_xor(gb2, o, 64);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) ls += __shfl_xor(ls, o, 64);
  float* out = partial + (size_t)blockIdx.x * (NPARAM + 1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = 4 * g + i;
    if (k < NI) out[OFF_W1 + k * NH + col] = g1[i];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) out[OFF_W2 + (mt * 16 + k) * NH + col] = g2[mt][i];
    if (c < NO) out[OFF_W3 + (n0 + k) * NO + c] = g3[i];
  }
  if (l < 16) {
    out[OFF_B1 + col] = gb1;
    out[OFF_B2 + col] = gb2;
    if (wv == 0 && l < NO) out[OFF_B3 + l] = gb3;
  }
  if (wv == 0 && l == 0) out[NPARAM] = 0.5f * ls * invB;
}

// grads[p] = sum over workgroups of partial[w][p] in their order, the loss at
// [NPARAM] likewise; with ADAM, then one Adam step on the FP32 master weights.
// The order is a chain of additions, but not of loads: a workgroup takes 64
// parameters, its four waves load 32 rows each ahead of the first addition. At
// 128 rows 4.4 us with the Adam step; a thread per parameter that loaded and added
// in turn took 37 us and another launch of 5 us.
struct AdamStep { float *P, *m, *v; float lr, b1, b2, eps, c1, c2; };
constexpr int RED_ROWS = 32;   // rows a wave loads at a time
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ partial, int nw, float* grads, AdamStep A) {
  __shared__ float sh[4 * RED_ROWS][64];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + l;
  const bool in = p <= NPARAM;
  float pp = 0.0f, pm = 0.0f, pv = 0.0f;
  if (ADAM && wv == 0 && p < NPARAM) { pp = A.P[p]; pm = A.m[p]; pv = A.v[p]; }
  float s = 0.0f;
  for (int w0 = 0; w0 < nw; w0 += 4 * RED_ROWS) {
    const int r0 = w0 + wv * RED_ROWS;
    float v[RED_ROWS];
#pragma unroll
    for (int j = 0; j < RED_ROWS; ++j) v[j] = in && r0 + j < nw ? partial[(size_t)(r0 + j) * (NPARAM + 1) + p] : 0.0f;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RED_ROWS; ++j) sh[wv * RED_ROWS + j][l] = v[j];
    __syncthreads();
    if (wv == 0) {
      const int n = min(4 * RED_ROWS, nw - w0);
#pragma unroll 8
      for (int j = 0; j < n; ++j) s += sh[j][l];
    }
  }
  if (wv != 0 || !in) return;
  grads[p] = s;
  if (ADAM && p < NPARAM) {
    const float mm = A.b1 * pm + (1.0f - A.b1) * s;
    const float vv = A.b2 * pv + (1.0f - A.b2) * s * s;
    A.m[p] = mm;
    A.v[p] = vv;
    A.P[p] = pp - A.lr * (mm / A.c1) / (sqrtf(vv / A.c2) + A.eps);
  }
}

// Column means and standard deviations of X (n x NI) and T (n x NO) in FP64,
// two fixed-order passes (one block per column).
__global__ __launch_bounds__(256) void k_mlp_stats(const float* X, const float* T, int64_t n, double* out) {
  const int c = blockIdx.x;  // 0..NI-1 features, NI..NI+NO-1 targets
  const float* A = c < NI ? X : T;
  const int ld = c < NI ? NI : NO, cc = c < NI ? c : c - NI;
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)A[i * ld + cc];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) { if (threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d]; __syncthreads(); }
  const double mean = sh[0] / (double)n;
  __syncthreads();
  double q = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) { const double d = (double)A[i * ld + cc] - mean; q += d * d; }
  sh[threadIdx.x] = q;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) { if (threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d]; __syncthreads(); }
  if (threadIdx.x == 0) { out[2 * c] = mean; out[2 * c + 1] = sqrt(sh[0] / (double)n); }
}

// ---------------------------------------------------------------- launchers
int mlp_nparam() { return NPARAM; }
int mlp_norm_slots() { return NORM_SLOTS; }
// Partial sums of a batch: their grouping fixes the bits of a gradient and of a
// trained network, so it stays as it is though nothing asks for an even number.
int mlp_backward_parts(int64_t B) {
  const int64_t nblk = (B + ROWS - 1) / ROWS;
  return (int)std::min<int64_t>(std::max<int64_t>(nblk, 2), 1024) / 2 * 2;
}

void launch_mlp_forward(const float* P, const float* norm, const float* X, int64_t n, float* Y, unsigned* maxnorm,
                        unsigned* clear, int nclear, hipStream_t s) {
  MlpNorm nm;
  for (int i = 0; i < NI; ++i) { nm.xm[i] = norm[i]; nm.xs[i] = norm[NI + i]; nm.xr[i] = 1.0f / norm[NI + i]; }
  for (int i = 0; i < NO; ++i) { nm.ym[i] = norm[2 * NI + i]; nm.ys[i] = norm[2 * NI + NO + i]; }
  const int64_t nblk = (n + 31) / 32;  // pairs of 16-sample blocks
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nblk + 3) / 4, 1024));
  if (((uintptr_t)X & 15u) == 0)
    hipLaunchKernelGGL(k_mlp_forward<true>, dim3(grid), dim3(256), 0, s, P, nm, X, n, Y, maxnorm, clear, nclear);
  else
    hipLaunchKernelGGL(k_mlp_forward<false>, dim3(grid), dim3(256), 0, s, P, nm, X, n, Y, maxnorm, clear, nclear);
}

void launch_mlp_backward(const float* P, const float* norm, const float* X, const float* T, int64_t first, int64_t n,
                         int64_t stride, int64_t offset, int64_t B, float* partial, int parts, hipStream_t s) {
  MlpNorm nm;
  for (int i = 0; i < NI; ++i) { nm.xm[i] = norm[i]; nm.xs[i] = norm[NI + i]; nm.xr[i] = 1.0f / norm[NI + i]; }
  for (int i = 0; i < NO; ++i) { nm.ym[i] = norm[2 * NI + i]; nm.ys[i] = norm[2 * NI + NO + i]; }
  const BatchRows rows = {first, n, stride, offset, 1.0 / (double)n};
  hipLaunchKernelGGL(k_mlp_backward, dim3(parts), dim3(256), 0, s, P, nm, X, T, rows, B, partial);
}

void launch_mlp_reduce(const float* partial, int parts, float* grads, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(NPARAM / 64 + 1), dim3(256), 0, s, partial, parts, grads, AdamStep{});
}

void launch_mlp_reduce_adam(const float* partial, int parts, float* grads, float* P, float* m, float* v, float lr,
                            int t, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(NPARAM / 64 + 1), dim3(256), 0, s, partial, parts, grads,
                     AdamStep{P, m, v, lr, b1, b2, 1e-8f, c1, c2});
}

void launch_mlp_stats(const float* X, const float* T, int64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_stats, dim3(NI + NO), dim3(256), 0, s, X, T, n, out);
}

}  // namespace nem
