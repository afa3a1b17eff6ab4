// fd_mlp.hip -- direction-proposal network on gfx950 matrix cores.
//
// 112 -> 256 -> 256 -> 256 -> 3, GELU (tanh form, Hendrycks & Gimpel 2016)
// after the hidden layers, output normalised to a unit direction.  Weights
// have a float master copy (Adam state beside it) and bfloat16 copies laid
// out for v_mfma_f32_16x16x32_bf16; activations are bfloat16, accumulation
// float.
//
// MFMA 16x16x32 operand layout used here (lane l of 64, g = l / 16):
//   A (16 x 32, row-major source): lane holds A[l % 16][8g .. 8g + 7]
//   B (32 x 16):                   lane holds B[8g .. 8g + 7][l % 16]
//   D (16 x 16 float):             lane holds D[4g + r][l % 16], r = 0..3
// A and B use the same k assignment, so the sum over k is the full product.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <cstdio>
#include <cstring>
#include <cmath>
#include <new>

#include "../../include/fusedir.h"
#include "fd_api_internal.hpp"
#include "fd_kernels.hpp"

using namespace fd;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D0 = 112, D0P = 128, DH = 256, DO = 3, DOP = 16;
// flat parameter offsets (W[k][n] row-major, then bias)
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + D0 * DH;
constexpr int OFF_W2 = OFF_B1 + DH, OFF_B2 = OFF_W2 + DH * DH;
constexpr int OFF_W3 = OFF_B2 + DH, OFF_B3 = OFF_W3 + DH * DH;
constexpr int OFF_W4 = OFF_B3 + DH, OFF_B4 = OFF_W4 + DH * DO;
constexpr int N_PARAMS = OFF_B4 + DO;
static_assert(N_PARAMS == FD_MLP_N_PARAMS, "parameter count");

__device__ __forceinline__ uint16_t f2bf(float x) {
  return __bfloat16_as_ushort(__float2bfloat16(x));  // round to nearest even
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// two floats -> bfloat16 pair (round to nearest even), a in the low half;
// a vector conversion, which gfx950 does in one instruction
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  const bf16x2_t v = __builtin_convertvector((f32x2_t){a, b}, bf16x2_t);
  return __builtin_bit_cast(uint32_t, v);
}

// tanh-form GELU: 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)),
// u = sqrt(2/pi) (x + 0.044715 x^3)
__device__ __forceinline__ float gelu(float x) {
  const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
  return x / (1.0f + __expf(-2.0f * u));
}
__device__ __forceinline__ float gelu_grad(float x) {
  const float c = 0.7978845608028654f;
  const float u = c * (x + 0.044715f * x * x * x);
  const float th = tanhf(u);
  const float du = c * (1.0f + 3.0f * 0.044715f * x * x);
  return 0.5f * (1.0f + th) + 0.5f * x * (1.0f - th * th) * du;
}

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---- packing: float master -> bfloat16 matrix-core layouts ------------------------
// Wt[n][k] (k contiguous) for every layer; k of layer 1 padded to 128 and n of
// layer 4 padded to 16 with zeros; biases copied to float arrays (b4 padded).
// W2 and W3 also as they are, [k][n] (n contiguous: the k index of the
// input-gradient products).
struct Packed {
  uint16_t* w1t;  // DH x D0P
  uint16_t* w2t;  // DH x DH
  uint16_t* w3t;  // DH x DH
  uint16_t* w2n;  // DH x DH
  uint16_t* w3n;  // DH x DH
  uint16_t* w4t;  // DOP x DH
  float* bias;    // b1 | b2 | b3 | b4(16)
};

__global__ void k_mlp_pack(const float* __restrict__ m, Packed p) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < DH * D0P) {  // layer 1
    const int n = i / D0P, k = i % D0P;
    p.w1t[i] = k < D0 ? f2bf(m[OFF_W1 + k * DH + n]) : 0;
  }
  if (i < DH * DH) {
    const int n = i / DH, k = i % DH;
    p.w2t[i] = f2bf(m[OFF_W2 + k * DH + n]);
    p.w3t[i] = f2bf(m[OFF_W3 + k * DH + n]);
    p.w2n[i] = f2bf(m[OFF_W2 + i]);
    p.w3n[i] = f2bf(m[OFF_W3 + i]);
  }
  if (i < DOP * DH) {
    const int n = i / DH, k = i % DH;
    p.w4t[i] = n < DO ? f2bf(m[OFF_W4 + k * DO + n]) : 0;
  }
  if (i < DH) {
    p.bias[i] = m[OFF_B1 + i];
    p.bias[DH + i] = m[OFF_B2 + i];
    p.bias[2 * DH + i] = m[OFF_B3 + i];
  }
  if (i < DOP) p.bias[3 * DH + i] = i < DO ? m[OFF_B4 + i] : 0.0f;
}

// ---- inference: fused four-layer forward ----------------------------------------------
// One workgroup = 128 rows.  Activations stay in LDS (128 x 256 bfloat16,
// rows padded by 16 bytes); wave w produces output columns
// [kCols w, kCols (w + 1)) of every hidden layer for all 128 rows.  The product is
// issued as Z^T = W^T X^T (weights as the A operand, activations as B), so
// that each lane ends up holding four consecutive output columns of one row
// and writes them to LDS with one 8-byte store.  Weight fragments come
// straight from the L2-resident packed weights, one k-step ahead.
constexpr int FWD_ROWS = 128;
constexpr int ACT_LD = DH + 8;
// FD_MLP_FWD_WAVES waves per workgroup, each producing kCols output columns
// of every hidden layer (kNt 16-column MFMA tiles) for all 128 rows; the
// output layer gives each wave 128 / (16 kFwdWaves) 16-row tiles.  Eight
// waves (two column tiles each) measure faster than four (four each, half
// the LDS reads per product): 0.49 against 0.53 ms per 1M rows.  The weight
// fragment loads, not the LDS reads, set the pace: splitting the rows
// between two wave groups (half the LDS reads, twice the weight loads per
// product) measured 1.65 against 0.97 ms per 2M rows, loading the weights
// two k-steps ahead instead of one 1.16 against 1.05 ms, and 256-row
// workgroups (half the weight loads per row, one workgroup per CU) 1.19;
// the GELU epilogue costs about 0.15 ms of the 1.05.
#ifndef FD_MLP_FWD_WAVES
#define FD_MLP_FWD_WAVES 8
#endif
constexpr int kFwdWaves = FD_MLP_FWD_WAVES;
constexpr int kFwdThreads = 64 * kFwdWaves;
constexpr int kCols = DH / kFwdWaves;
constexpr int kNt = kCols / 16;
constexpr int kOutTiles = FWD_ROWS / (16 * kFwdWaves);
static_assert(FWD_ROWS % (16 * kFwdWaves) == 0, "whole output-layer row tiles per wave");

// GELU (tanh form) for the inference forward: 0.5 x (1 + tanh(u)) = x / (1 +
// e^(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3), with e^(-2u) = 2^(x (A + B x^2))
// so the constants fold into one multiply-add; hardware exp2 and reciprocal
// (about 1 ulp each, below the bfloat16 rounding that follows).
__device__ __forceinline__ float gelu_fast(float x) {
  constexpr float kA = -2.0f * 0.7978845608028654f * 1.4426950408889634f;
  constexpr float kB = kA * 0.044715f;
  const float t = x * __builtin_fmaf(kB, x * x, kA);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

__global__ __launch_bounds__(kFwdThreads, 2) void k_mlp_fwd(const uint16_t* __restrict__ x,
                                                          int64_t n, Packed p,
                                                          float* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint16_t act[FWD_ROWS * ACT_LD];
  __shared__ float yout[FWD_ROWS][4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, g = lane >> 4, c16 = lane & 15;
  const int64_t row0 = (int64_t)blockIdx.x * FWD_ROWS;

  // input rows -> act[:, 0:128) (k >= 112 and rows >= n zero)
  for (int e = t; e < FWD_ROWS * (D0P / 8); e += kFwdThreads) {
    const int r = e / (D0P / 8), kb = (e % (D0P / 8)) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row0 + r < n && kb < D0) v = *(const uint4*)(x + (row0 + r) * D0 + kb);
    *(uint4*)(act + r * ACT_LD + kb) = v;
  }
  __syncthreads();

#pragma unroll 1
  for (int layer = 0; layer < 3; ++layer) {
    const int K = layer == 0 ? D0P : DH;
    const uint16_t* wt = layer == 0 ? p.w1t : (layer == 1 ? p.w2t : p.w3t);
    // acc[mt][nt]: rows (output columns) kCols w + 16nt + 4g + r, column
    // (batch row) 16mt + c16
    f32x4 acc[8][kNt];
#pragma unroll
    for (int mt = 0; mt < 8; ++mt)
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) acc[mt][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 wa[kNt], wn[kNt];
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt)
      wa[nt] = *(const bf16x8*)(wt + (size_t)(kCols * w + 16 * nt + c16) * K + 8 * g);
#pragma unroll 1
    for (int kc = 0; kc < K; kc += 32) {
      const int kn = kc + 32 < K ? kc + 32 : kc;
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt)
        wn[nt] = *(const bf16x8*)(wt + (size_t)(kCols * w + 16 * nt + c16) * K + kn + 8 * g);
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) {
        const bf16x8 xb = *(const bf16x8*)(act + (16 * mt + c16) * ACT_LD + kc + 8 * g);
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt) acc[mt][nt] = mfma(wa[nt], xb, acc[mt][nt]);
      }
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) wa[nt] = wn[nt];
    }
    __syncthreads();  // every wave has read this layer's input
    const float* bias = p.bias + layer * DH;
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) {
      const int col = kCols * w + 16 * nt + 4 * g;
      const float4 bb = *(const float4*)(bias + col);
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) {
        const int row = 16 * mt + c16;
        const uint32_t lo = pack_bf16x2(gelu_fast(acc[mt][nt][0] + bb.x),
                                        gelu_fast(acc[mt][nt][1] + bb.y));
        const uint32_t hi = pack_bf16x2(gelu_fast(acc[mt][nt][2] + bb.z),
                                        gelu_fast(acc[mt][nt][3] + bb.w));
        *(uint2*)(act + row * ACT_LD + col) = make_uint2(lo, hi);
      }
    }
    __syncthreads();
  }
  // output layer: 256 -> 16 (3 real); wave w takes batch-row tiles
  // w, w + kFwdWaves, ...
#pragma unroll
  for (int ot = 0; ot < kOutTiles; ++ot) {
    const int rt = w + ot * kFwdWaves;
    f32x4 o = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int kc = 0; kc < DH; kc += 32) {
      const bf16x8 b = *(const bf16x8*)(p.w4t + (size_t)c16 * DH + kc + 8 * g);
      const bf16x8 a = *(const bf16x8*)(act + (16 * rt + c16) * ACT_LD + kc + 8 * g);
      o = mfma(a, b, o);
    }
    if (c16 < 3) {
#pragma unroll
      for (int r = 0; r < 4; ++r) yout[16 * rt + 4 * g + r][c16] = o[r] + p.bias[3 * DH + c16];
    }
  }
  __syncthreads();
  if (t < FWD_ROWS && row0 + t < n) {
    const float y0 = yout[t][0], y1 = yout[t][1], y2 = yout[t][2];
    const float inv = 1.0f / sqrtf(y0 * y0 + y1 * y1 + y2 * y2);
    float* o3 = out + 3 * (row0 + t);
    o3[0] = y0 * inv;
    o3[1] = y1 * inv;
    o3[2] = y2 * inv;
  }
}

// ---- training ------------------------------------------------------------------------
// A step is three launches.  At batches of a few thousand rows the products
// are microseconds of matrix-core work, so what bounds a step is how often
// the chain of dependent stages goes through memory and a launch: as one
// kernel per product and per reduction it was 23 launches, 163 us for batch
// 4096; now 50 us (k_train_rows 30, k_train_wgrad 10, k_train_finish 10), and
// 107 -> 35 us for batch 64, 1149 -> 493 us for 65536.
//   k_train_rows    a workgroup owns 16 or 32 rows and takes them
//                   through the forward pass, the loss and the backward
//                   pass; everything on the way stays in LDS and registers.
//                   It writes what sums over the batch need, transposed
//                   (batch index contiguous): activations and gradients in
//                   bfloat16 for the weight-gradient products, gradients in
//                   float for the bias sums.
//   k_train_wgrad   the three weight-gradient products, split over the batch.
//   k_train_finish  every parameter's sum over the batch in a fixed order,
//                   then the Adam update and the bfloat16 copies.
// The shape and order of every sum depend on the batch size only (not on the
// rows a workgroup takes): a step is deterministic.

constexpr int kRowTile = 64;   // rows of a bias sum's partial (b1, b2); batches are padded to it
constexpr int kRowChunk = 32;  // rows of a partial sum (output layer, b3)
constexpr int kMaxSplit = 16;  // batch slices of a weight-gradient product
constexpr int kOutGrad = DH * DO + DO;  // dW4 then db4, contiguous in the parameters
constexpr int kOutLanes = 8;   // lanes per row of the output layer

struct TrainDev {
  const uint16_t* feats;  // B x D0
  const float* tgt;       // B x 3
  int B, Bp;              // rows; rounded up to kRowTile
  Packed pk;
  uint16_t* xT;           // D0P x Bp
  uint16_t* hT[3];        // DH x Bp: activations
  uint16_t* dT[3];        // DH x Bp: gradients of the pre-activations
  float* dzT[3];          // DH x Bp: the same in float
  float* dyT;             // DO x Bp: gradient of the output
  float* lrow;            // B: loss of each row
};

// The workgroup's eight waves take 32 columns each of a (16 MT) x 256
// product: acc[mt][nt] holds D[4 g + r][c16] of rows 16 mt + ..., columns
// 32 w + 16 nt + c16.
constexpr int kTrainThreads = 512;

// All of a wave's weight fragments of one layer (K / 32 steps), loaded at
// once: one wait per layer instead of one per step.  wt: [column][k], k
// contiguous.
template <int K>
__device__ __forceinline__ void load_wfrag(const uint16_t* __restrict__ wt, int w, int c16, int g,
                                           bf16x8 (&b)[K / 32][2]) {
#pragma unroll
  for (int q = 0; q < K / 32; ++q)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
      b[q][nt] = *(const bf16x8*)(wt + (size_t)(32 * w + 16 * nt + c16) * K + 32 * q + 8 * g);
}

template <int K, int MT>
__device__ __forceinline__ void row_gemm(const uint16_t* act, int c16, int g,
                                         const bf16x8 (&b)[K / 32][2], f32x4 (&acc)[MT][2]) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < K / 32; ++q)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const bf16x8 a = *(const bf16x8*)(act + (16 * mt + c16) * ACT_LD + 32 * q + 8 * g);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc[mt][nt] = mfma(a, b[q][nt], acc[mt][nt]);
    }
}

// Four rows' values of one column, as bfloat16, to LDS (row-major) and to
// the transposed copy.
__device__ __forceinline__ void put_rows4(uint16_t* act, uint16_t* tT, int64_t ldt, int row, int col,
                                          const float (&v)[4]) {
  const uint32_t lo = pack_bf16x2(v[0], v[1]), hi = pack_bf16x2(v[2], v[3]);
  act[row * ACT_LD + col] = (uint16_t)lo;
  act[(row + 1) * ACT_LD + col] = (uint16_t)(lo >> 16);
  act[(row + 2) * ACT_LD + col] = (uint16_t)hi;
  act[(row + 3) * ACT_LD + col] = (uint16_t)(hi >> 16);
  *(uint2*)(tT + (int64_t)col * ldt + row) = make_uint2(lo, hi);
}

// z = acc + bias, h = gelu(z) to LDS and transposed; z kept.
template <int MT>
__device__ __forceinline__ void row_forward(uint16_t* act, uint16_t* hT, int64_t ldt,
                                            const float* __restrict__ bias, int w, int c16, int g,
                                            const f32x4 (&acc)[MT][2], f32x4 (&z)[MT][2]) {
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int col = 32 * w + 16 * nt + c16;
    const float bb = bias[col];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float h[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[mt][nt][r] = acc[mt][nt][r] + bb;
        h[r] = gelu(z[mt][nt][r]);
      }
      put_rows4(act, hT, ldt, 16 * mt + 4 * g, col, h);
    }
  }
}

// d = v gelu'(z) (rows >= rows: 0) to LDS and transposed, in bfloat16 and
// float; v(mt, nt, r) is the gradient of the activation.
template <int MT, typename V>
__device__ __forceinline__ void row_backward(uint16_t* act, uint16_t* dT, float* dzT, int64_t ldt,
                                             int rows, int w, int c16, int g, const V& v,
                                             const f32x4 (&z)[MT][2]) {
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int col = 32 * w + 16 * nt + c16;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = 16 * mt + 4 * g;
      float d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r] = v(mt, nt, r) * gelu_grad(z[mt][nt][r]);
        if (row + r >= rows) d[r] = 0.0f;
      }
      put_rows4(act, dT, ldt, row, col, d);
      *(float4*)(dzT + (int64_t)col * ldt + row) = make_float4(d[0], d[1], d[2], d[3]);
    }
  }
}

template <int RT>
__global__ __launch_bounds__(kTrainThreads, 2) void k_train_rows(TrainDev a) {
  constexpr int MT = RT / 16;
  __shared__ __attribute__((aligned(16))) uint16_t act[RT * ACT_LD];
  __shared__ float sdy[RT][4];
  const int t = threadIdx.x, lane = t & 63, g = lane >> 4, c16 = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * RT;
  const int rows = max(0, min(RT, a.B - (int)row0));  // 0: only the padding's zeros are written
  const int64_t ldt = a.Bp;
  f32x4 acc[MT][2], z1[MT][2], z2[MT][2], z3[MT][2];
  bf16x8 wf1[D0P / 32][2], wf[DH / 32][2];

  // input rows -> act[:, 0:128) (k >= 112 and rows >= B zero), and transposed
  load_wfrag<D0P>(a.pk.w1t, w, c16, g, wf1);
  for (int e = t; e < RT * (D0P / 8); e += kTrainThreads) {
    const int r = e / (D0P / 8), kb = (e % (D0P / 8)) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < rows && kb < D0) v = *(const uint4*)(a.feats + (row0 + r) * D0 + kb);
    *(uint4*)(act + r * ACT_LD + kb) = v;
  }
  __syncthreads();
  for (int e = t; e < D0P * (RT / 8); e += kTrainThreads) {
    const int k = e & (D0P - 1), r0 = 8 * (e / D0P);
    uint32_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = (uint32_t)act[(r0 + 2 * q) * ACT_LD + k] |
             ((uint32_t)act[(r0 + 2 * q + 1) * ACT_LD + k] << 16);
    *(uint4*)(a.xT + (int64_t)k * ldt + row0 + r0) = make_uint4(v[0], v[1], v[2], v[3]);
  }

  // forward
  row_gemm<D0P, MT>(act, c16, g, wf1, acc);
  load_wfrag<DH>(a.pk.w2t, w, c16, g, wf);
  __syncthreads();  // every wave has read this layer's input
  row_forward<MT>(act, a.hT[0] + row0, ldt, a.pk.bias, w, c16, g, acc, z1);
  __syncthreads();
  row_gemm<DH, MT>(act, c16, g, wf, acc);
  load_wfrag<DH>(a.pk.w3t, w, c16, g, wf);
  __syncthreads();
  row_forward<MT>(act, a.hT[1] + row0, ldt, a.pk.bias + DH, w, c16, g, acc, z2);
  __syncthreads();
  row_gemm<DH, MT>(act, c16, g, wf, acc);
  load_wfrag<DH>(a.pk.w3n, w, c16, g, wf);
  __syncthreads();
  row_forward<MT>(act, a.hT[2] + row0, ldt, a.pk.bias + 2 * DH, w, c16, g, acc, z3);
  __syncthreads();

  // Output layer, loss and its gradient, eight lanes per row (lane j takes k
  // in [32 j, 32 j + 32) in order; the eight partial sums are added by a
  // fixed shuffle tree): y = h3 W4 + b4 (float, W4 as bfloat16 values),
  // u = y/|y|, loss_b = 1 - (u.t)^2, dL/dy = (gr - u (u.gr)) / |y| with
  // gr = -2 (u.t) t / B.
  static_assert(RT * kOutLanes <= kTrainThreads, "one row per eight threads");
  if (t < RT * kOutLanes) {  // whole waves
    const int b = t / kOutLanes, j = t % kOutLanes;
    float part[3] = {0.0f, 0.0f, 0.0f};
    const int k0 = j * (DH / kOutLanes);
#pragma unroll
    for (int q = 0; q < DH / kOutLanes; q += 8) {
      const uint4 hv = *(const uint4*)(act + b * ACT_LD + k0 + q);
      const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w};
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        const uint4 wv = *(const uint4*)(a.pk.w4t + n * DH + k0 + q);
        const uint32_t ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint16_t he = (uint16_t)(hw[e >> 1] >> (16 * (e & 1)));
          const uint16_t we = (uint16_t)(ww[e >> 1] >> (16 * (e & 1)));
          part[n] += bf2f(he) * bf2f(we);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < 3; ++n)
#pragma unroll
      for (int off = 1; off < kOutLanes; off <<= 1) part[n] += __shfl_xor(part[n], off, 64);
    if (j == 0) {
      float dy[3] = {0.0f, 0.0f, 0.0f};
      if (b < rows) {
        float y[3];
#pragma unroll
        for (int n = 0; n < 3; ++n) y[n] = part[n] + a.pk.bias[3 * DH + n];
        const float nrm = sqrtf(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]);
        float u[3], tt[3], ut = 0.0f;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
          u[n] = y[n] / nrm;
          tt[n] = a.tgt[3 * (row0 + b) + n];
          ut += u[n] * tt[n];
        }
        a.lrow[row0 + b] = 1.0f - ut * ut;
        float gg[3], ug = 0.0f;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
          gg[n] = -2.0f * ut * tt[n] / (float)a.B;
          ug += u[n] * gg[n];
        }
#pragma unroll
        for (int n = 0; n < 3; ++n) dy[n] = (gg[n] - u[n] * ug) / nrm;
      }
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        sdy[b][n] = dy[n];
        a.dyT[n * ldt + row0 + b] = dy[n];
      }
    }
  }
  __syncthreads();

  // dz3 = (dy W4^T) gelu'(z3) (W4 as bfloat16 values), then the input
  // gradients of layers 3 and 2
  {
    float w4[2][3];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int n = 0; n < 3; ++n) w4[nt][n] = bf2f(a.pk.w4t[n * DH + 32 * w + 16 * nt + c16]);
    row_backward<MT>(
        act, a.dT[2] + row0, a.dzT[2] + row0, ldt, rows, w, c16, g,
        [&](int mt, int nt, int r) {
          float s = 0.0f;
#pragma unroll
          for (int n = 0; n < 3; ++n) s += sdy[16 * mt + 4 * g + r][n] * w4[nt][n];
          return s;
        },
        z3);
  }
  __syncthreads();
  const auto from_acc = [&](int mt, int nt, int r) { return acc[mt][nt][r]; };
  row_gemm<DH, MT>(act, c16, g, wf, acc);
  load_wfrag<DH>(a.pk.w2n, w, c16, g, wf);
  __syncthreads();
  row_backward<MT>(act, a.dT[1] + row0, a.dzT[1] + row0, ldt, rows, w, c16, g, from_acc, z2);
  __syncthreads();
  row_gemm<DH, MT>(act, c16, g, wf, acc);
  __syncthreads();
  row_backward<MT>(act, a.dT[0] + row0, a.dzT[0] + row0, ldt, rows, w, c16, g, from_acc, z1);
}

// Weight gradients: dW_l[k][n] = sum_b h_{l-1}[b][k] d_l[b][n], as 64 x 64
// tiles over K slices of the batch; both operands are contiguous along the
// batch.  Every load of a stage (up to kGemmKS rows of the batch) is issued
// first, then stored to LDS (rows padded by 8 elements), and after one
// barrier the products of the stage run from LDS, k ascending.
constexpr int kGemmT = 64, kGemmK = 32, kGemmKS = 128, kGemmLd = kGemmKS + 8;

// Operand staging registers as a native vector type (the uint4 struct
// copied between an array and LDS made the compiler keep the array in
// private memory).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTilesN = DH / kGemmT;                     // 4
constexpr int kTiles1 = D0P / kGemmT * kTilesN;          // layer 1: 8
constexpr int kTilesH = DH / kGemmT * kTilesN;           // layers 2, 3: 16
constexpr int kWgradTiles = kTiles1 + 2 * kTilesH;       // 40
// first float of each layer's partial products (slice-major within a layer)
constexpr int64_t split_off(int l, int S) {
  return l == 0 ? 0 : (int64_t)S * (D0P * DH + (l - 1) * DH * DH);
}

__global__ __launch_bounds__(256) void k_train_wgrad(TrainDev a, int S, float* __restrict__ split) {
  __shared__ __attribute__((aligned(16))) uint16_t As[kGemmT][kGemmLd];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[kGemmT][kGemmLd];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, gr = lane >> 4, c16 = lane & 15;
  int tile = blockIdx.x;
  const int l = tile < kTiles1 ? 0 : (tile < kTiles1 + kTilesH ? 1 : 2);
  tile -= l == 0 ? 0 : (l == 1 ? kTiles1 : kTiles1 + kTilesH);
  const int m0 = tile / kTilesN * kGemmT, n0 = tile % kTilesN * kGemmT;
  const int M = l == 0 ? D0P : DH;
  const uint16_t* A = l == 0 ? a.xT : a.hT[l - 1];
  const uint16_t* Bm = a.dT[l];
  f32x4 acc[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) acc[mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int kslice = a.B / S;
  const int kz0 = blockIdx.y * kslice, kz1 = kz0 + kslice;
  const int lr = t >> 2, lk = (t & 3) * 8;  // thread t: row t / 4, k 8 (t % 4) .. + 7
  const uint16_t* ap = A + (int64_t)(m0 + lr) * a.Bp + lk;
  const uint16_t* bp = Bm + (int64_t)(n0 + lr) * a.Bp + lk;
  for (int ks = kz0; ks < kz1; ks += kGemmKS) {
    const int kn = min(kGemmKS, kz1 - ks);  // a multiple of 32
    u32x4 va[kGemmKS / kGemmK], vb[kGemmKS / kGemmK];
#pragma unroll
    for (int q = 0; q < kGemmKS / kGemmK; ++q)
      if (q * kGemmK < kn) {
        va[q] = *(const u32x4*)(ap + ks + q * kGemmK);
        vb[q] = *(const u32x4*)(bp + ks + q * kGemmK);
      }
    if (ks > kz0) __syncthreads();  // the previous stage's products are done
#pragma unroll
    for (int q = 0; q < kGemmKS / kGemmK; ++q)
      if (q * kGemmK < kn) {
        *(u32x4*)&As[lr][q * kGemmK + lk] = va[q];
        *(u32x4*)&Bs[lr][q * kGemmK + lk] = vb[q];
      }
    __syncthreads();
    for (int kk = 0; kk < kn; kk += kGemmK) {
      const bf16x8 b = *(const bf16x8*)&Bs[16 * w + c16][kk + 8 * gr];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const bf16x8 x = *(const bf16x8*)&As[16 * mt + c16][kk + 8 * gr];
        acc[mt] = mfma(x, b, acc[mt]);
      }
    }
  }
  float* out = split + split_off(l, S) + (int64_t)blockIdx.y * M * DH;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      out[(int64_t)(m0 + 16 * mt + 4 * gr + r) * DH + n0 + 16 * w + c16] = acc[mt][r];
}

// Parameter i's gradient, and with it the Adam update (Kingma & Ba 2015) of
// the float master weights; returns the parameter's new value.
struct AdamDev {
  float* w;
  float* m;
  float* v;
  float* grad;  // gradient out (no update), or NULL: update
  float lr, b1, b2, eps, bc1, bc2;
};

__device__ __forceinline__ float adam_step(const AdamDev& o, int i, float gi) {
  if (o.grad) {
    o.grad[i] = gi;
    return 0.0f;
  }
  const float mi = o.b1 * o.m[i] + (1.0f - o.b1) * gi;
  const float vi = o.b2 * o.v[i] + (1.0f - o.b2) * gi * gi;
  o.m[i] = mi;
  o.v[i] = vi;
  const float x = o.w[i] - o.lr * (mi / o.bc1) / (sqrtf(vi / o.bc2) + o.eps);
  o.w[i] = x;
  return x;
}

// The workgroups of k_train_finish: 16 x 64 tiles of the hidden layers'
// weights (their K slices summed in slice order), then one wave per entry of
// the output layer and of the biases (partial sums over kRowChunk or
// kRowTile rows; lane l adds the partials l, l + 64, ... in order, then a
// fixed shuffle tree), then one workgroup for the loss.
constexpr int kFinTiles1 = D0 / 16 * kTilesN, kFinTilesH = DH / 16 * kTilesN;
constexpr int kFinTiles = kFinTiles1 + 2 * kFinTilesH;
constexpr int kFinEntries = kOutGrad + 3 * DH;
constexpr int kFinWaves = (kFinEntries + 3) / 4;
static_assert(D0 % 16 == 0, "whole tiles");

__global__ __launch_bounds__(256) void k_train_finish(TrainDev a, int S,
                                                      const float* __restrict__ split, AdamDev o,
                                                      float* __restrict__ loss) {
  const int t = threadIdx.x;
  int blk = blockIdx.x;
  if (blk < kFinTiles) {
    __shared__ __attribute__((aligned(16))) uint16_t tr[64][16];  // read 8 bytes at a time
    const int l = blk < kFinTiles1 ? 0 : (blk < kFinTiles1 + kFinTilesH ? 1 : 2);
    blk -= l == 0 ? 0 : (l == 1 ? kFinTiles1 : kFinTiles1 + kFinTilesH);
    const int k0 = blk / kTilesN * 16, n = blk % kTilesN * 64 + (t & 63);
    const int M = l == 0 ? D0P : DH;
    const float* part = split + split_off(l, S);
    const int off = l == 0 ? OFF_W1 : (l == 1 ? OFF_W2 : OFF_W3);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + (t >> 6) + 4 * e;
      float v = 0.0f;
      if (S == kMaxSplit) {
        float x[kMaxSplit];
#pragma unroll
        for (int z = 0; z < kMaxSplit; ++z) x[z] = part[((int64_t)z * M + k) * DH + n];
#pragma unroll
        for (int z = 0; z < kMaxSplit; ++z) v += x[z];
      } else if (S > 1) {
        for (int z = 0; z < S; ++z) v += part[((int64_t)z * M + k) * DH + n];
      } else {
        v = part[(int64_t)k * DH + n];
      }
      const float x = adam_step(o, off + k * DH + n, v);
      if (!o.grad) {
        const uint16_t h = f2bf(x);
        tr[t & 63][k - k0] = h;
        if (l > 0) (l == 1 ? a.pk.w2n : a.pk.w3n)[k * DH + n] = h;
      }
    }
    if (o.grad) return;  // uniform
    __syncthreads();
    uint16_t* wt = l == 0 ? a.pk.w1t : (l == 1 ? a.pk.w2t : a.pk.w3t);
    const int nn = t >> 2, kq = (t & 3) * 4;
    *(uint2*)(wt + (int64_t)(blk % kTilesN * 64 + nn) * M + k0 + kq) = *(const uint2*)&tr[nn][kq];
    return;
  }
  blk -= kFinTiles;
  if (blk < kFinWaves) {
    const int e = 4 * blk + (t >> 6), lane = t & 63;
    if (e >= kFinEntries) return;  // wave-uniform
    const bool outw = e < kOutGrad;
    const int l = outw ? 3 : (e - kOutGrad) / DH, n = outw ? e : (e - kOutGrad) % DH;
    float s = 0.0f;
    if (outw) {
      // dW4[k][m] = sum_b h3[b][k] dy[b][m], db4[m] = sum_b dy[b][m]: chunks
      // of kRowChunk rows, rows in order (B is a multiple of kRowChunk)
      const bool bias = n >= DH * DO;
      const int k = bias ? 0 : n / DO, m = bias ? n - DH * DO : n % DO;
      const uint16_t* h = a.hT[2] + (int64_t)k * a.Bp;
      const float* dy = a.dyT + (int64_t)m * a.Bp;
      for (int b0 = lane * kRowChunk; b0 < a.B; b0 += 64 * kRowChunk) {
        float4 y[kRowChunk / 4];
        uint4 hv[kRowChunk / 8];
#pragma unroll
        for (int q = 0; q < kRowChunk / 4; ++q) y[q] = *(const float4*)(dy + b0 + 4 * q);
#pragma unroll
        for (int q = 0; q < kRowChunk / 8; ++q) hv[q] = *(const uint4*)(h + b0 + 8 * q);
        float c = 0.0f;
#pragma unroll
        for (int q = 0; q < kRowChunk / 4; ++q) {
          const float v[4] = {y[q].x, y[q].y, y[q].z, y[q].w};
          const uint32_t hw[2] = {q & 1 ? hv[q / 2].z : hv[q / 2].x, q & 1 ? hv[q / 2].w : hv[q / 2].y};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x = bf2f((uint16_t)(hw[r >> 1] >> (16 * (r & 1))));
            c += bias ? v[r] : x * v[r];
          }
        }
        s += c;
      }
    } else if (l == 2) {  // b3: chunks of kRowChunk rows, rows in order
      const float* d = a.dzT[2] + (int64_t)n * a.Bp;
      for (int b0 = lane * kRowChunk; b0 < a.B; b0 += 64 * kRowChunk) {
        float4 y[kRowChunk / 4];
#pragma unroll
        for (int q = 0; q < kRowChunk / 4; ++q) y[q] = *(const float4*)(d + b0 + 4 * q);
        float c = 0.0f;
#pragma unroll
        for (int q = 0; q < kRowChunk / 4; ++q) c = (((c + y[q].x) + y[q].y) + y[q].z) + y[q].w;
        s += c;
      }
    } else {
      // b1, b2: tiles of kRowTile rows, as four sums over the rows
      // 16 mt + 4 q + r (q = 0..3) in order, added in the order of q
      const float* d = a.dzT[l] + (int64_t)n * a.Bp;
      for (int b0 = lane * kRowTile; b0 < a.Bp; b0 += 64 * kRowTile) {
        float c[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          c[q] = 0.0f;
#pragma unroll
          for (int mt = 0; mt < kRowTile / 16; ++mt) {
            const float4 y = *(const float4*)(d + b0 + 16 * mt + 4 * q);
            c[q] = (((c[q] + y.x) + y.y) + y.z) + y.w;
          }
        }
        s += ((c[0] + c[1]) + c[2]) + c[3];
      }
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane != 0) return;
    const int i = outw ? OFF_W4 + n : (l == 0 ? OFF_B1 : (l == 1 ? OFF_B2 : OFF_B3)) + n;
    const float x = adam_step(o, i, s);
    if (o.grad) return;
    if (!outw)
      a.pk.bias[l * DH + n] = x;
    else if (n < DH * DO)
      a.pk.w4t[n % DO * DH + n / DO] = f2bf(x);
    else
      a.pk.bias[3 * DH + n - DH * DO] = x;
    return;
  }
  // mean loss: thread t sums rows t, t + 256, ... in order, then a fixed tree
  if (!loss) return;
  __shared__ float red[256];
  float s = 0.0f;
  for (int i = t; i < a.B; i += 256) s += a.lrow[i];
  red[t] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (t < off) red[t] += red[t + off];
    __syncthreads();
  }
  if (t == 0) loss[0] = red[0] / (float)a.B;
}

__global__ void k_init_params(float* __restrict__ w, uint64_t seed) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N_PARAMS) return;
  // counter-based uniform in [-1, 1): splitmix64 of (seed, i)
  uint64_t z = seed + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const float u = (float)(z >> 40) * (1.0f / 8388608.0f) - 1.0f;
  int fan_in;
  bool bias;
  if (i < OFF_B1) { fan_in = D0; bias = false; }
  else if (i < OFF_W2) { fan_in = D0; bias = true; }
  else if (i < OFF_B2) { fan_in = DH; bias = false; }
  else if (i < OFF_W3) { fan_in = DH; bias = true; }
  else if (i < OFF_B3) { fan_in = DH; bias = false; }
  else if (i < OFF_W4) { fan_in = DH; bias = true; }
  else if (i < OFF_B4) { fan_in = DH; bias = false; }
  else { fan_in = DH; bias = true; }
  // uniform with variance 2 / fan_in (He) for weights, zero biases
  w[i] = bias ? 0.0f : u * sqrtf(6.0f / (float)fan_in);
}

}  // namespace

// ---- host object ----------------------------------------------------------------------

struct fd_mlp {
  int device = 0;
  float* master = nullptr;
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  int64_t step = 0;
  Packed pk{};
  float learned_step0 = 0.0f;
  float fallback_cost = INFINITY;
  // training workspace, sized for cap_batch rows
  int cap_batch = 0;
  uint16_t* acts = nullptr;  // transposed activations and gradients, bfloat16
  float* grads = nullptr;    // transposed gradients in float, row losses
  float* split = nullptr;    // partial weight-gradient products
};

namespace {

int mlp_pack(fd_mlp* m, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((DH * DH + 255) / 256), dim3(256), 0, st, m->master, m->pk);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "mlp pack");
}

constexpr int kActCols = D0P + 6 * DH;     // xT, hT[3], dT[3]
constexpr int kGradCols = 3 * DH + DO + 1;  // dzT[3], dyT, lrow

int ensure_train_ws(fd_mlp* m, int B) {
  if (m->cap_batch >= B) return FD_OK;
  void* old[] = {m->acts, m->grads, m->split};
  for (void* q : old)
    if (q) (void)hipFree(q);
  m->acts = nullptr;
  m->grads = m->split = nullptr;
  m->cap_batch = 0;
  const size_t Bp = (size_t)(B + kRowTile - 1) / kRowTile * kRowTile;
  hipError_t e = hipMalloc(&m->acts, Bp * kActCols * 2);
  if (e == hipSuccess) e = hipMalloc(&m->grads, Bp * kGradCols * 4);
  if (e == hipSuccess)
    e = hipMalloc(&m->split, (size_t)kMaxSplit * (D0P + 2 * DH) * DH * 4);
  if (e != hipSuccess) return hip_error(e, "mlp training workspace");
  m->cap_batch = B;
  return FD_OK;
}

// Batch slices of the weight-gradient products over B rows: up to
// kMaxSplit, each at least 256 rows and a whole number of 32-row steps.
int wgrad_split(int B) {
  int S = 1;
  while (S < kMaxSplit && B % (64 * S) == 0 && B / (2 * S) >= 256) S *= 2;
  return S;
}

// Loss (may be NULL) and, by o, the full gradient or the Adam update.
int train_pass(fd_mlp* m, const uint16_t* feats, const float* tgt, int B, const AdamDev& o,
               float* loss, hipStream_t st) {
  int r;
  if ((r = ensure_train_ws(m, B))) return r;
  TrainDev a;
  a.feats = feats;
  a.tgt = tgt;
  a.B = B;
  a.Bp = (B + kRowTile - 1) / kRowTile * kRowTile;
  a.pk = m->pk;
  uint16_t* p = m->acts;
  a.xT = p;
  p += (size_t)D0P * a.Bp;
  for (int l = 0; l < 3; ++l, p += (size_t)DH * a.Bp) a.hT[l] = p;
  for (int l = 0; l < 3; ++l, p += (size_t)DH * a.Bp) a.dT[l] = p;
  float* f = m->grads;
  for (int l = 0; l < 3; ++l, f += (size_t)DH * a.Bp) a.dzT[l] = f;
  a.dyT = f;
  a.lrow = f + (size_t)DO * a.Bp;
  const int S = wgrad_split(B);
  // Rows per workgroup.  Its time is mostly its chain of layers, and each
  // workgroup reads all weights: 16 rows while every compute unit (256) then
  // has at most one workgroup, 32 from there on.  A step of batch 4096: 50
  // (16 rows) / 59 us (32); 6144: 78 / 63; 8192: 84 / 68; 65536: 645 / 493.
  // 64 rows (registers spill): 112 us at 4096, 146 against 120 at 16384.
  if (a.Bp <= 16 * 256)
    hipLaunchKernelGGL(k_train_rows<16>, dim3(a.Bp / 16), dim3(kTrainThreads), 0, st, a);
  else
    hipLaunchKernelGGL(k_train_rows<32>, dim3(a.Bp / 32), dim3(kTrainThreads), 0, st, a);
  hipLaunchKernelGGL(k_train_wgrad, dim3(kWgradTiles, S), dim3(256), 0, st, a, S, m->split);
  hipLaunchKernelGGL(k_train_finish, dim3(kFinTiles + kFinWaves + 1), dim3(256), 0, st, a, S,
                     m->split, o, loss);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "mlp training");
}

}  // namespace

namespace fd {
int mlp_forward_dev(const fd_mlp* m, const uint16_t* feats, int64_t n, float* out, hipStream_t st) {
  if (n <= 0) return FD_OK;
  const int64_t nb = (n + FWD_ROWS - 1) / FWD_ROWS;
  hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)nb), dim3(kFwdThreads), 0, st, feats, n, m->pk,
                     out);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "mlp forward");
}
}  // namespace fd

extern "C" int fd_mlp_create(fd_mlp** out, uint64_t seed) {
  if (!out) return set_error(FD_E_INVAL, "fd_mlp_create: out is NULL");
  int dev, r;
  if ((r = check_device(&dev))) return r;
  fd_mlp* m = new (std::nothrow) fd_mlp();
  if (!m) return set_error(FD_E_NOMEM, "fd_mlp_create: host allocation failed");
  m->device = dev;
  bump_workspace_generation();  // a captured batched graph holds weight pointers
  hipError_t e = hipMalloc(&m->master, N_PARAMS * 4);
  if (e == hipSuccess) e = hipMalloc(&m->adam_m, N_PARAMS * 4);
  if (e == hipSuccess) e = hipMalloc(&m->adam_v, N_PARAMS * 4);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w1t, DH * D0P * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w2t, DH * DH * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w3t, DH * DH * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w2n, DH * DH * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w3n, DH * DH * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.w4t, DOP * DH * 2);
  if (e == hipSuccess) e = hipMalloc(&m->pk.bias, (3 * DH + DOP) * 4);
  if (e != hipSuccess) {
    fd_mlp_destroy(m);
    return hip_error(e, "fd_mlp_create");
  }
  hipLaunchKernelGGL(k_init_params, dim3((N_PARAMS + 255) / 256), dim3(256), 0, 0, m->master,
                     seed);
  (void)hipMemset(m->adam_m, 0, N_PARAMS * 4);
  (void)hipMemset(m->adam_v, 0, N_PARAMS * 4);
  if ((r = mlp_pack(m, 0))) {
    fd_mlp_destroy(m);
    return r;
  }
  e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    fd_mlp_destroy(m);
    return hip_error(e, "fd_mlp_create");
  }
  *out = m;
  return FD_OK;
}

extern "C" void fd_mlp_destroy(fd_mlp* m) {
  if (!m) return;
  (void)hipDeviceSynchronize();
  void* bufs[] = {m->master, m->adam_m, m->adam_v, m->pk.w1t, m->pk.w2t, m->pk.w3t, m->pk.w2n,
                  m->pk.w3n, m->pk.w4t, m->pk.bias, m->acts, m->grads, m->split};
  for (void* p : bufs)
    if (p) (void)hipFree(p);
  delete m;
}

extern "C" int fd_mlp_set_params(fd_mlp* m, const float* host) {
  if (!m || !host) return set_error(FD_E_INVAL, "fd_mlp_set_params: null argument");
  hipError_t e = hipMemcpy(m->master, host, N_PARAMS * 4, hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_error(e, "fd_mlp_set_params");
  (void)hipMemset(m->adam_m, 0, N_PARAMS * 4);
  (void)hipMemset(m->adam_v, 0, N_PARAMS * 4);
  m->step = 0;
  int r = mlp_pack(m, 0);
  if (r) return r;
  e = hipDeviceSynchronize();
  return e == hipSuccess ? FD_OK : hip_error(e, "fd_mlp_set_params");
}

extern "C" int fd_mlp_get_params(const fd_mlp* m, float* host) {
  if (!m || !host) return set_error(FD_E_INVAL, "fd_mlp_get_params: null argument");
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(host, m->master, N_PARAMS * 4, hipMemcpyDeviceToHost);
  return e == hipSuccess ? FD_OK : hip_error(e, "fd_mlp_get_params");
}

extern "C" int fd_mlp_set_calibration(fd_mlp* m, float step0, float tau) {
  if (!m) return set_error(FD_E_INVAL, "fd_mlp_set_calibration: mlp is NULL");
  m->learned_step0 = step0;
  m->fallback_cost = tau;
  return FD_OK;
}

extern "C" int fd_mlp_get_calibration(const fd_mlp* m, float* step0, float* tau) {
  if (!m || !step0 || !tau) return set_error(FD_E_INVAL, "fd_mlp_get_calibration: null argument");
  *step0 = m->learned_step0;
  *tau = m->fallback_cost;
  return FD_OK;
}

// Checkpoint file: "FDMLP001", int32 version, int32 dims[5], int64 step,
// float learned_step0, float fallback_cost, float master[N], m[N], v[N].
extern "C" int fd_mlp_save(const fd_mlp* m, const char* path) {
  if (!m || !path) return set_error(FD_E_INVAL, "fd_mlp_save: null argument");
  float* buf = new (std::nothrow) float[3 * (size_t)N_PARAMS];
  if (!buf) return set_error(FD_E_NOMEM, "fd_mlp_save: host allocation failed");
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(buf, m->master, N_PARAMS * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(buf + N_PARAMS, m->adam_m, N_PARAMS * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(buf + 2 * N_PARAMS, m->adam_v, N_PARAMS * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) {
    delete[] buf;
    return hip_error(e, "fd_mlp_save");
  }
  FILE* f = fopen(path, "wb");
  if (!f) {
    delete[] buf;
    return set_error(FD_E_INVAL, "fd_mlp_save: cannot open %s", path);
  }
  const char magic[8] = {'F', 'D', 'M', 'L', 'P', '0', '0', '1'};
  const int32_t ver = 1, dims[5] = {D0, DH, DH, DH, DO};
  bool ok = fwrite(magic, 1, 8, f) == 8 && fwrite(&ver, 4, 1, f) == 1 &&
            fwrite(dims, 4, 5, f) == 5 && fwrite(&m->step, 8, 1, f) == 1 &&
            fwrite(&m->learned_step0, 4, 1, f) == 1 && fwrite(&m->fallback_cost, 4, 1, f) == 1 &&
            fwrite(buf, 4, 3 * (size_t)N_PARAMS, f) == 3 * (size_t)N_PARAMS;
  ok = (fclose(f) == 0) && ok;
  delete[] buf;
  return ok ? FD_OK : set_error(FD_E_INVAL, "fd_mlp_save: write to %s failed", path);
}

extern "C" int fd_mlp_load(fd_mlp* m, const char* path) {
  if (!m || !path) return set_error(FD_E_INVAL, "fd_mlp_load: null argument");
  FILE* f = fopen(path, "rb");
  if (!f) return set_error(FD_E_INVAL, "fd_mlp_load: cannot open %s", path);
  char magic[8];
  int32_t ver = 0, dims[5] = {0, 0, 0, 0, 0};
  int64_t step = 0;
  float s0 = 0, tau = 0;
  float* buf = new (std::nothrow) float[3 * (size_t)N_PARAMS];
  bool ok = buf && fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "FDMLP001", 8) == 0 &&
            fread(&ver, 4, 1, f) == 1 && ver == 1 && fread(dims, 4, 5, f) == 5 &&
            dims[0] == D0 && dims[1] == DH && dims[2] == DH && dims[3] == DH && dims[4] == DO &&
            fread(&step, 8, 1, f) == 1 && fread(&s0, 4, 1, f) == 1 && fread(&tau, 4, 1, f) == 1 &&
            fread(buf, 4, 3 * (size_t)N_PARAMS, f) == 3 * (size_t)N_PARAMS;
  fclose(f);
  if (!ok) {
    delete[] buf;
    return set_error(FD_E_INVAL, "fd_mlp_load: %s is not a valid checkpoint", path);
  }
  hipError_t e = hipMemcpy(m->master, buf, N_PARAMS * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->adam_m, buf + N_PARAMS, N_PARAMS * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->adam_v, buf + 2 * N_PARAMS, N_PARAMS * 4, hipMemcpyHostToDevice);
  delete[] buf;
  if (e != hipSuccess) return hip_error(e, "fd_mlp_load");
  m->step = step;
  m->learned_step0 = s0;
  m->fallback_cost = tau;
  int r = mlp_pack(m, 0);
  if (r) return r;
  e = hipDeviceSynchronize();
  return e == hipSuccess ? FD_OK : hip_error(e, "fd_mlp_load");
}

static int check_mlp_batch(const fd_mlp* m, const void* feats, int64_t batch, const char* fn) {
  if (!m) return set_error(FD_E_INVAL, "%s: mlp is NULL", fn);
  if (batch < 0) return set_error(FD_E_INVAL, "%s: batch < 0", fn);
  if (batch > 0 && !feats) return set_error(FD_E_INVAL, "%s: feats is NULL", fn);
  if (((uintptr_t)feats & 15) != 0)
    return set_error(FD_E_INVAL, "%s: feats must be 16-byte aligned", fn);
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (dev != m->device)
    return set_error(FD_E_INVAL, "%s: network lives on device %d, current is %d", fn, m->device,
                     dev);
  return FD_OK;
}

extern "C" int fd_mlp_forward(const fd_mlp* m, const void* feats, int64_t batch, float* out,
                              void* stream) {
  int r;
  if ((r = check_mlp_batch(m, feats, batch, "fd_mlp_forward"))) return r;
  if (batch > 0 && !out) return set_error(FD_E_INVAL, "fd_mlp_forward: out is NULL");
  return mlp_forward_dev(m, (const uint16_t*)feats, batch, out, (hipStream_t)stream);
}

static int check_train(fd_mlp* m, const void* feats, const float* tgt, int32_t batch,
                       const char* fn) {
  int r;
  if ((r = check_mlp_batch(m, feats, batch, fn))) return r;
  if (batch < 16 || batch > 65536 || batch % 32 != 0)
    return set_error(FD_E_INVAL, "%s: batch must be a multiple of 32 in [32, 65536], got %d", fn,
                     batch);
  if (!tgt) return set_error(FD_E_INVAL, "%s: targets is NULL", fn);
  return FD_OK;
}

extern "C" int fd_mlp_loss_grad(fd_mlp* m, const void* feats, const float* tgt, int32_t batch,
                                float* grad, float* loss, void* stream) {
  int r;
  if ((r = check_train(m, feats, tgt, batch, "fd_mlp_loss_grad"))) return r;
  if (!grad) return set_error(FD_E_INVAL, "fd_mlp_loss_grad: grad is NULL");
  AdamDev o{};
  o.grad = grad;
  return train_pass(m, (const uint16_t*)feats, tgt, batch, o, loss, (hipStream_t)stream);
}

extern "C" int fd_mlp_train_step(fd_mlp* m, const void* feats, const float* tgt, int32_t batch,
                                 const fd_adam* opt, float* loss, void* stream) {
  int r;
  if ((r = check_train(m, feats, tgt, batch, "fd_mlp_train_step"))) return r;
  if (!opt) return set_error(FD_E_INVAL, "fd_mlp_train_step: opt is NULL");
  const int64_t step = m->step + 1;
  const double bc1 = 1.0 - std::pow((double)opt->beta1, (double)step);
  const double bc2 = 1.0 - std::pow((double)opt->beta2, (double)step);
  const AdamDev o{m->master,  m->adam_m,  m->adam_v, nullptr,    opt->lr,
                  opt->beta1, opt->beta2, opt->eps,  (float)bc1, (float)bc2};
  if ((r = train_pass(m, (const uint16_t*)feats, tgt, batch, o, loss, (hipStream_t)stream))) return r;
  m->step = step;
  return FD_OK;
}
