// fd_gabor.hip -- orientation and confidence maps from grey-level frames on
// gfx950 (the Gabor-filter extraction the paper names at the start of Sec. 3.1;
// its reading is documented with fd_orientation_maps in fusedir.h).
//
// The filter bank is a dense contraction over the taps, run on the matrix
// cores.  The choice of an orientation is defined by one sum, binary32 over
// the taps in order.  Tiles of 16 x 64 pixels where that choice is clear take
// the faster binary16 operations with both factors split in two
// (k_gabor_split), the others the binary32 ones (k_gabor_f32); k_gabor_sort
// looks at 16 pixels of each tile and says which.  Either stages a tile in LDS
// with its radius-R halo and takes the argmax orientation and the raw
// confidence, and a workgroup's largest raw confidence goes to the frame
// maximum (an integer atomic on the bits of a non-negative float).
// k_gabor_norm divides by that maximum.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "../../include/fusedir.h"
#include "fd_api_internal.hpp"
#include "fd_kernels.hpp"

using namespace fd;

namespace {

constexpr int kTile = 16;
constexpr int kMaxRadius = 12;
constexpr float kPi = 3.14159265358979323846f;

template <typename TO>
__device__ __forceinline__ void store_map(void* out, size_t i, float v) {
  if constexpr (sizeof(TO) == 2)
    ((__half*)out)[i] = __float2half(v);
  else
    ((float*)out)[i] = v;
}

// One frame per grid row (its maximum read once), 8 pixels per thread in
// 16-byte loads and stores where the plane and the output allow it.
template <typename TO>
__global__ __launch_bounds__(256) void k_gabor_norm(const float* __restrict__ raw,
                                                    const uint32_t* __restrict__ frame_max,
                                                    int64_t plane, int vec,
                                                    void* __restrict__ conf_out) {
  const int64_t f = blockIdx.y;
  const float m = __uint_as_float(frame_max[f]);
  const float* r = raw + plane * f;
  TO* out = (TO*)conf_out + plane * f;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (vec) {
    const int64_t n8 = plane >> 3;
    for (int64_t i = t0; i < n8; i += stride) {
      const float4 a = ((const float4*)r)[2 * i], b = ((const float4*)r)[2 * i + 1];
      const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      float o[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) o[k] = m > 0.0f ? v[k] / m : 0.0f;
      if constexpr (sizeof(TO) == 2) {
        uint32_t h[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = __half_as_ushort(__float2half(o[k]));
        ((uint4*)out)[i] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16),
                                      h[4] | (h[5] << 16), h[6] | (h[7] << 16));
      } else {
        ((float4*)out)[2 * i] = make_float4(o[0], o[1], o[2], o[3]);
        ((float4*)out)[2 * i + 1] = make_float4(o[4], o[5], o[6], o[7]);
      }
    }
  } else {
    for (int64_t i = t0; i < plane; i += stride)
      store_map<TO>(out, (size_t)i, m > 0.0f ? r[i] / m : 0.0f);
  }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowsPerWave = 8;
constexpr int kTileRows = 64;

constexpr int kRound = 32;        // taps of a round of sum_in_order
constexpr int kBankPad = kRound;  // a last round's taps past the window are 0
__host__ __device__ inline int round_taps(int taps) { return (taps + kRound - 1) / kRound * kRound; }

// What every kernel reads.  tid counts the 16 x 64 tiles, frame by frame; the
// tiles of successive tile rows and frames are shifted against each other, so
// that no workgroup that strides over them gets nothing but tiles of a frame's
// edge.
struct GaborDev {
  const float* frames;
  int W, H, R, NO;
  const float* bank;  // [tap][orientation], kBankPad taps of 0, each orientation's sum
  const uint32_t* split;  // its halves as k_gabor_split reads them (k_gabor_halves)
  int n_tiles, tiles_x, tiles_y;
  size_t plane;

  __device__ __forceinline__ void place(int tid, int* f, int* x0, int* y0) const {
    place_of(tid, tiles_y, kTileRows, f, x0, y0);
  }
  // the same for tiles of `high` rows, n_y in a column
  __device__ __forceinline__ void place_of(int tid, int n_y, int high, int* f, int* x0,
                                           int* y0) const {
    const int per_frame = tiles_x * n_y;
    *f = tid / per_frame;
    const int rem = tid - *f * per_frame, r = rem / tiles_x;
    *y0 = (r + *f) % n_y * high;
    *x0 = (rem - r * tiles_x + r + *f) % tiles_x * kTile;
  }
};
struct GaborOut {
  void* theta;
  float* raw;
  uint32_t* frame_max;
};

// d2tab[NO + k] = squared line distance of two bins k apart (|k| < NO), 64
// entries by the workgroup's first 64 threads.
__device__ __forceinline__ void fill_d2(float* d2tab, int NO) {
  if (threadIdx.x < 64) {
    const int k = abs((int)threadIdx.x - NO);
    float v = 0.0f;
    if (k < NO) {
      const float dd = (float)min(k, NO - k) * (kPi / NO);
      v = dd * dd;
    }
    d2tab[threadIdx.x] = v;
  }
}

// The bank in binary32 for the 16 x 16 x 4 operation, n taps (a multiple of 4,
// past the window's 0), zero-padded to 16-orientation tiles and laid out
// [tap / 4][orientation tile][tap % 4][16], so that a wave's A operand is 64
// consecutive words.
__host__ __device__ inline int padded_taps(int taps) { return (taps + 3) & ~3; }
template <int NT>
__device__ __forceinline__ void fill_bank(float* sbank, const GaborDev& d, int n) {
  constexpr int NJ = 16 * NT;
  constexpr int kAhead = 4;  // loads in flight together
  for (int e0 = threadIdx.x; e0 < n * NJ; e0 += kAhead * (int)blockDim.x) {
    float v[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int e = min(e0 + u * (int)blockDim.x, n * NJ - 1), t = e / NJ, j = e - t * NJ;
      v[u] = d.bank[t * d.NO + min(j, d.NO - 1)];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int e = e0 + u * (int)blockDim.x, t = e / NJ, j = e - t * NJ;
      const int dst = (t >> 2) * 4 * NJ + (j >> 4) * 64 + (t & 3) * 16 + (j & 15);
      if (e < n * NJ) sbank[dst] = j < d.NO ? v[u] : 0.0f;
    }
  }
}

// The distance in the frame of each tap from the window's first, whole rounds
// (past the window: the first).
__device__ __forceinline__ void fill_offsets(uint32_t* offs, int W, int w2) {
  for (int t = threadIdx.x; t < round_taps(w2 * w2); t += blockDim.x)
    offs[t] = t < w2 * w2 ? (uint32_t)(t / w2 * W + t % w2) : 0u;
}

// The largest and the second largest response of one pixel, which 2 or 4 lanes
// (first_xor 32 or 16) hold: a lane orientations p0 + step * (k / 4) + k % 4.
// Responses past the last orientation become -1 (FULL: there are none).
template <bool FULL, int K>
__device__ __forceinline__ void top_two(float (&fv)[K], int p0, int step, int first_xor, int NO,
                                        float& fb, float& f2) {
  fb = f2 = -1.0f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (!FULL && p0 + step * (k / 4) + k % 4 >= NO) fv[k] = -1.0f;
    f2 = __builtin_amdgcn_fmed3f(fv[k], fb, f2);
    fb = fmaxf(fb, fv[k]);
  }
  for (int off = first_xor; off < 64; off <<= 1) {
    const float o1 = __shfl_xor(fb, off, 64), o2 = __shfl_xor(f2, off, 64);
    f2 = fmaxf(fminf(fb, o1), fmaxf(f2, o2));
    fb = fmaxf(fb, o1);
  }
}

// The first orientation with the largest response fb, and the spread of the
// responses around it.
template <bool FULL, int K>
__device__ __forceinline__ void choose(const float (&fv)[K], float fb, int p0, int step,
                                       int first_xor, int NO, const float* d2tab, int& jb,
                                       float& conf) {
  jb = 1 << 30;
#pragma unroll
  for (int k = K - 1; k >= 0; --k) jb = fv[k] == fb ? p0 + step * (k / 4) + k % 4 : jb;
  for (int off = first_xor; off < 64; off <<= 1) jb = min(jb, __shfl_xor(jb, off, 64));
  jb = jb < NO ? jb : 0;  // (no response equals a NaN)
  float s = 0.0f;
  const float* d2 = d2tab + (NO + p0 - jb);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int o = step * (k / 4) + k % 4;
    const float e = FULL || p0 + o < NO ? fv[k] - fb : 0.0f;
    s = __builtin_fmaf(d2[o], e * e, s);
  }
  for (int off = first_xor; off < 64; off <<= 1) s += __shfl_xor(s, off, 64);
  conf = sqrtf(s);
}

// ---- the sum in order --------------------------------------------------------
// Binary32 fused multiply-adds over all taps, row by row, as the 16 x 16 x 4
// operation evaluates them (v_mfma_f32_16x16x4_f32, 4 taps a step).  In its
// result lane (g, c) = (lane / 16, lane % 16) holds orientations 16 nt + 4 g + r
// (r < 4) of pixel c.

// For 16 pixels a wave, lane (g, c) has pixel c's place (px, py) and frame img:
// read from the frame itself.  tap(k, nt) gives the lane's bank value of taps k
// .. k + 3, 0 past the last one.  lo, hi: the range of the lane's taps (0 outside
// the frame).  Bound by the vector instructions around a step's one load: with
// the window's place kept and checked step by step a wave took 9 us alone.
template <int NT, typename F>
__device__ __forceinline__ void sum_in_order(const GaborDev& d, const F& tap, const uint32_t* offs,
                                             const float* img, int px, int py, int g,
                                             f32x4 (&acc)[NT], float& lo, float& hi) {
  const int R = d.R, W = d.W, H = d.H, w2 = 2 * R + 1, taps = w2 * w2;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  lo = INFINITY;
  hi = -INFINITY;
  const int x0 = px - R, y0 = py - R;
  const float* win = img + ((int64_t)y0 * W + x0);  // (not read outside the frame)
  // uniform: no window of the wave leaves the frame
  const bool inner = __all(x0 >= 0 && px + R < W && y0 >= 0 && py + R < H);
  offs += g;
  constexpr int kAhead = kRound / 4;  // steps whose loads are in flight together
  for (int k0 = 0; k0 < taps; k0 += kRound) {
    float v[kAhead], a[kAhead][NT];
    if (inner) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) v[u] = win[offs[k0 + 4 * u]];
    } else {
      bool in[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int t = k0 + 4 * u + g, dy = t / w2, dx = t - dy * w2;
        in[u] = t < taps && (unsigned)(x0 + dx) < (unsigned)W && (unsigned)(y0 + dy) < (unsigned)H;
        v[u] = *(in[u] ? win + offs[k0 + 4 * u] : img);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) v[u] = in[u] ? v[u] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) a[u][nt] = tap(k0 + 4 * u, nt);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      lo = fminf(lo, v[u]);
      hi = fmaxf(hi, v[u]);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][nt], v[u], acc[nt], 0, 0, 0);
    }
  }
}

// All pixels of the listed tiles (from the list's end), or of all n_half half
// tiles, half_y in a column (two for every tile would leave workgroups without
// work where the last tiles are less than half full: 15 frames of 253 x 81 96 us
// in place of 74).  Persistent workgroups of four waves keep the bank in LDS and walk half tiles
// of 16 x 32, wave w owning rows 8w .. 8w + 7, so each bank read feeds 8 matrix
// operations.  The tile rows are kTw
// words apart for every radius: the 8 row reads of a step take immediate
// offsets and pair up.  The matrix cores only reach their peak when little
// else is issued beside them, so the per-step bookkeeping is kept small: the
// position of the step's first tap is wave-uniform (scalar registers) and a
// lane's tap is at most one row further.
// FULL: n_orient fills the NT orientation tiles (no per-lane validity
// tests).  Three waves per SIMD is what the LDS allows (three workgroups per
// CU at radius 8); the register bound keeps the compiler to it.
constexpr int kF32Rows = 4 * kRowsPerWave;   // rows of a half tile: four waves
constexpr int kTw = kTile + 2 * kMaxRadius;  // LDS tile row stride for every radius

template <typename TO, int NT, bool FULL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_gabor_f32(
    GaborDev d, int half_y, int n_half, const uint32_t* __restrict__ n_listed,
    const uint32_t* __restrict__ list, GaborOut o) {
  extern __shared__ float lds_f32[];
  __shared__ float wmax[256 / 64];
  if (list) n_half = 2 * (int)*n_listed;
  if ((int)blockIdx.x >= n_half) return;
  constexpr int NJ = 16 * NT;
  const int W = d.W, H = d.H, R = d.R, NO = d.NO;
  const int w2 = 2 * R + 1, taps = w2 * w2, kpad = padded_taps(taps), tw = kTile + 2 * R;
  const int th = kF32Rows + 2 * R;  // tile rows with the halo
  float* sbank = lds_f32;           // kpad x NJ
  float* tile = lds_f32 + kpad * NJ;  // th x kTw
  fill_bank<NT>(sbank, d, kpad);
  float* d2tab = tile + kTw * th;  // 64
  fill_d2(d2tab, NO);
  const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  for (int i = blockIdx.x; i < n_half; i += gridDim.x) {
    int f, x0, y0;
    if (list) {
      d.place((int)list[d.n_tiles - 1 - (i >> 1)], &f, &x0, &y0);
      y0 += kF32Rows * (i & 1);
      if (y0 >= H) continue;  // uniform
    } else {
      d.place_of(i, half_y, kF32Rows, &f, &x0, &y0);
    }
    const float* img = d.frames + d.plane * f;
    __syncthreads();  // the bank is in place; the previous tile is no longer read
    for (int e = threadIdx.x; e < kTw * th; e += blockDim.x) {
      const int yy = e / kTw, xx = e - yy * kTw;
      const int x = x0 + xx - R, y = y0 + yy - R;
      tile[e] = (xx < tw && x >= 0 && x < W && y >= 0 && y < H) ? img[(size_t)y * W + x] : 0.0f;
    }
    __syncthreads();
    f32x4 acc[kRowsPerWave][NT];
#pragma unroll
    for (int p = 0; p < kRowsPerWave; ++p)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[p][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float* base = tile + kRowsPerWave * w * kTw + c16 + g;
    const float* bk = sbank + lane;
    // wave-uniform (row offset, column) of tap k0; a lane's tap k0 + g is at
    // most one row further (g < 4 <= w2 + 1 and the column stays < w2)
    int s_off = 0, s_dx = 0;
    for (int k0 = 0; k0 < kpad; k0 += 4) {
      const int wrap = g >= w2 - s_dx ? kTw - w2 : 0;
      const int off = k0 + g < taps ? s_off + wrap : -g;
      float a[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) a[nt] = bk[k0 * NJ + 64 * nt];
      const float* src = base + off;
#pragma unroll
      for (int p = 0; p < kRowsPerWave; ++p) {
        const float v = src[p * kTw];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[p][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[nt], v, acc[p][nt], 0, 0, 0);
      }
      // issue order: the step's LDS reads (the bank, then the row pairs),
      // then its matrix operations
      __builtin_amdgcn_sched_group_barrier(0x100, 5, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, kRowsPerWave * NT, 0);
      s_dx += 4;
      s_off += 4;
      if (s_dx >= w2) { s_dx -= w2; s_off += kTw - w2; }
      if (s_dx >= w2) { s_dx -= w2; s_off += kTw - w2; }
    }
    float m = 0.0f;
#pragma unroll
    for (int p = 0; p < kRowsPerWave; ++p) {
      float fv[4 * NT], fb, wv;
      int jb;
#pragma unroll
      for (int k = 0; k < 4 * NT; ++k)
        fv[k] = FULL || 16 * (k / 4) + 4 * g + k % 4 < NO ? fabsf(acc[p][k / 4][k % 4]) : -1.0f;
      fb = -1.0f;
#pragma unroll
      for (int k = 0; k < 4 * NT; ++k) fb = fmaxf(fb, fv[k]);
      fb = fmaxf(fb, __shfl_xor(fb, 16, 64));
      fb = fmaxf(fb, __shfl_xor(fb, 32, 64));
      choose<FULL>(fv, fb, 4 * g, 16, 16, NO, d2tab, jb, wv);
      const int x = x0 + c16, y = y0 + kRowsPerWave * w + p;
      if (g == 0 && x < W && y < H) {
        const size_t at = d.plane * f + (size_t)y * W + x;
        store_map<TO>(o.theta, at, (float)jb * (kPi / NO));
        o.raw[at] = wv;
        m = fmaxf(m, wv);
      }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if (lane == 0) wmax[w] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      float bm = wmax[0];
      for (int k = 1; k < (int)(blockDim.x >> 6); ++k) bm = fmaxf(bm, wmax[k]);
      atomicMax(&o.frame_max[f], __float_as_uint(bm));  // bm >= 0: bits order as values
    }
  }
}

// Per bank, in units of 2^-24: the rounding bounds of both sums for a window
// whose pixels lie within `half` of `mid`, per unit of mid and half.
struct GaborMargin {
  float mid, half;
};

// ---- which sum a tile takes --------------------------------------------------
// A pixel of a split tile whose two best responses are within the rounding of
// the sums is summed again in order, one by one.  That costs about twice what
// the pixel costs in k_gabor_f32, and the split sum half of it, so a tile many
// of whose pixels would wait is better off there.  A wave sums 8 pixels of two
// tiles in order, or 16 of one where the binary32 sum has half the operations
// (NT = 1: it pays from half the share on); a tile of which two or more would
// wait takes that sum.  What a tile takes depends on its own pixels only.
constexpr int kSortWaves = 16, kSortMost = 8;  // tiles a wave, at most

template <int NT, bool FULL>
__global__ __launch_bounds__(64 * kSortWaves) void k_gabor_sort(GaborDev d, GaborMargin margin,
                                                                int per,
                                                                unsigned long long* cursor,
                                                                uint32_t* __restrict__ list) {
  extern __shared__ float lds_sort[];
  __shared__ uint32_t bits[kSortWaves];
  __shared__ uint64_t base;
  constexpr int NJ = 16 * NT;
  const int w2 = 2 * d.R + 1, n = round_taps(w2 * w2);
  fill_bank<NT>(lds_sort, d, n);
  uint32_t* const offs = (uint32_t*)(lds_sort + n * NJ);
  fill_offsets(offs, d.W, w2);
  __syncthreads();
  const int lane = (int)(threadIdx.x & 63u), g = lane >> 4, c16 = lane & 15;
  const int second = NT == 2 ? c16 >> 3 : 0;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int waves = (int)(blockDim.x >> 6), first = (int)blockIdx.x * (waves * per);
  const int t0 = first + w * per;
  const auto tap = [&](int k, int nt) { return lds_sort[k * NJ + 64 * nt + lane]; };
  uint32_t f32s = 0;  // bit k: tile t0 + k takes the binary32 sum
  for (int k = 0; k < per && t0 + k < d.n_tiles; k += NT) {
    int f, x0, y0, f1, x1, y1;
    const bool two = NT == 2 && t0 + k + 1 < d.n_tiles;
    d.place(t0 + k, &f, &x0, &y0);
    d.place(t0 + k + two, &f1, &x1, &y1);
    // four or eight pixels of each of two rows
    const int row = c16 >> (NT == 2 ? 2 : 3) & 1;
    const int col = NT == 2 ? 4 * (c16 & 3) + 2 * row + 1 : 2 * (c16 & 7) + row;
    const int px = (second ? x1 : x0) + col, py = (second ? y1 : y0) + 15 + 33 * row;
    const bool on = px < d.W && py < d.H;
    f32x4 acc[NT];
    float lo, hi, fb, f2, fv[4 * NT];
    sum_in_order<NT>(d, tap, offs, d.frames + d.plane * (size_t)(second ? f1 : f), px, py, g, acc, lo,
                     hi);
    for (int off = 16; off < 64; off <<= 1) {
      lo = fminf(lo, __shfl_xor(lo, off, 64));
      hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
#pragma unroll
    for (int j = 0; j < 4 * NT; ++j) fv[j] = fabsf(acc[j / 4][j % 4]);
    top_two<FULL>(fv, 4 * g, 16, 16, d.NO, fb, f2);
    const float mg = margin.mid * fabsf(0.5f * (hi + lo)) + margin.half * (0.5f * (hi - lo));
    const uint64_t near = __ballot(on && !(fb >= 0.0f && fb - f2 >= mg));
    if (__popcll(near & (NT == 2 ? 0xffull : 0xffffull)) >= 2) f32s |= 1u << k;
    if (two && __popcll(near & 0xff00ull) >= 2) f32s |= 2u << k;
  }
  if (lane == 0) bits[w] = f32s;
  __syncthreads();
  // places in the list: split tiles from its start, the others from its end
  const int n_here = min(max(d.n_tiles - first, 0), waves * per);
  int n_f32 = 0, before = 0;
  for (int k = 0; k < waves; ++k) {
    n_f32 += __popc(bits[k]);
    before += k < w ? __popc(bits[k]) : 0;
  }
  if (threadIdx.x == 0)
    base = atomicAdd(cursor, (unsigned long long)n_f32 << 32 | (unsigned)(n_here - n_f32));
  __syncthreads();
  if (lane < per && t0 + lane < d.n_tiles) {
    before += __popc(f32s & ((1u << lane) - 1u));
    const int at = f32s >> lane & 1u
                       ? d.n_tiles - 1 - ((int)(base >> 32) + before)
                       : (int)(uint32_t)base + w * per + lane - before;
    list[at] = (uint32_t)(t0 + lane);
  }
}

// ---- the split sum -----------------------------------------------------------
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
static_assert(kTileRows == kWaves * kRowsPerWave, "a wave's rows");
constexpr float kBankScale = 16384.0f;  // 2^14: |g| <= 2 stays below 2^15

// The taps of the (2R + 1)^2 window in groups of 8, two groups per matrix
// operation: 8 columns of a row (columns 8c .. 8c + 7, rows 0 .. 2R and one
// of padding, so that an operation takes two rows of one c), then the columns
// that are left over: in groups of 8 rows of one column where that is fewer
// groups than another (padded) c takes.
struct Taps {
  int w;        // window edge
  int cols;     // column groups c
  int steps;    // matrix steps (16 taps)
  int rows8;    // groups of 8 rows in a column
  int left;     // leftover columns in groups of rows

  __host__ __device__ explicit Taps(int R) {
    w = 2 * R + 1;
    rows8 = (w + 7) / 8;
    left = w % 8;
    if (left * rows8 >= w) left = 0;
    cols = (w - left + 7) / 8;
    steps = (cols * (w + 1) + left * rows8 + 1) / 2;
  }
  // tap i (0..7) of group q: its row and column, false if it is padding
  __host__ __device__ bool tap(int q, int i, int* dy, int* dx) const {
    const int v = q - cols * (w + 1);
    if (v < 0) {
      *dy = q % (w + 1);
      *dx = 8 * (q / (w + 1)) + i;
    } else {
      *dy = 8 * (v % rows8) + i;
      *dx = 8 * cols + v / rows8;
    }
    return *dy < w && *dx < w;
  }
};

// LDS of a workgroup, in 4-byte words.  The tile is 64 pixel rows of 16
// with the window's halo (and the rows that padded taps touch), RS pixels a
// row, split in two binary16 halves (high and low), each in an even and an
// odd copy (the odd one a pixel further) so that 8 pixels from any column
// start on a word.  The even and odd copies lie 8 banks apart and rows 16 or
// 20, so that the 64 lanes of a read (two pixel rows, 8 words each from
// either copy, and the same a tap row further) touch no bank twice.
struct GaborLds {
  int RS, th, plane, bank, planes, d2, total;
  __host__ __device__ GaborLds(int R, bool pair) {
    const Taps t(R);
    RS = R <= 8 ? 32 : 40;
    th = kTileRows + 8 * t.rows8;
    plane = ((th * RS / 2 + 63) & ~63) + 8;
    bank = 0;
    planes = t.steps * (pair ? 1 : 2) * 64 * 4;
    d2 = planes + 4 * plane;
    total = d2 + 64 + 32 + round_taps(t.w * t.w);
  }
};

// The split bank, [step][high, low][lane] 8 taps of orientation lane % 32; pair:
// [step][lane], the high halves of 16 orientations, then the low ones.  Once per
// bank.
__global__ __launch_bounds__(64) void k_gabor_halves(const float* __restrict__ bank, int NO,
                                                     bool pair, Taps taps8,
                                                     uint32_t* __restrict__ split) {
  const int st = (int)blockIdx.x, l = (int)threadIdx.x, m = l & (pair ? 15 : 31);
  f16x8 hi, lo;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int dy, dx;
    const bool on = taps8.tap(2 * st + (l >> 5), i, &dy, &dx) && m < NO;
    const float v = on ? bank[(size_t)(dy * taps8.w + dx) * NO + m] * kBankScale : 0.0f;
    hi[i] = (_Float16)v;
    lo[i] = (_Float16)(v - (float)hi[i]);
  }
  f16x8* out = (f16x8*)split;
  if (pair) {
    out[st * 64 + l] = l & 16 ? lo : hi;
  } else {
    out[st * 2 * 64 + l] = hi;
    out[(st * 2 + 1) * 64 + l] = lo;
  }
}

// The filter bank as a matrix product on the matrix cores,
// F[orientation][pixel] = sum_tap G[orientation][tap] I[pixel + tap]: 32
// orientations x 16 taps times 16 taps x 32 pixels per operation
// (v_mfma_f32_32x32x16_f16, accumulated in float).  Both factors are split
// into a high and a low binary16 half (v = h + l + r, |r| <= 2^-23 |v| and
// mostly 0; the tile scaled by a power of two so that its largest pixel is near
// 2^14, the bank by 2^14), and the four products of the halves stand for one.
// Those with a low half are summed first, over all taps, while the sum is
// small; the high halves' come after, with two roundings per 16 taps (each half
// of its taps, as measured) where the binary32 operation rounds once per tap.
// A tile of one sign whose largest pixel is at most three times its smallest
// is taken less its middle (nearer to each pixel than 0 is), and the middle's
// response, from the exact sum of the rounded taps, is added at the end.
// Errors of the confidences against binary64, rms, in-order binary32 sum and
// this: rendered hair, radius 8, 32 orientations 1.8e-6 and 0.7e-6, radius 12
// 2.1e-6 and 1.0e-6; relative to the confidence on 0.15 with noise of 0.02
// 9.7e-7 and 4.8e-7 (16 orientations 9.6e-7 and 5.6e-7), on bare scalp between
// hair at radius 5 5.0e-7 and 5.0e-7.  Below radius 5 such windows would be
// worse off: 5.5e-7 and 6.5e-7 at 4, 4.9e-7 and 6.9e-7 at 3 (kSplitRadius).
//
// Persistent workgroups of eight waves keep the split bank in LDS and walk
// the listed tiles, wave w owning rows 8w .. 8w + 7 as four
// groups of 32 pixels (two rows).  A step takes two tap rows, so what group q
// reads at one step group q - 1 reads at the next: the image operands stay in
// registers and move down by one group, and only the last group's is loaded
// (reading all four made the LDS the bound).  In the result lane (h, n) = (lane / 32, lane % 32)
// holds orientations 8 q + 4 h + r (q, r < 4) of pixel n: the argmax (first
// of equals) and the confidence sum run over those 16 values in the lane,
// then across the two halves; the squared bin distances come from a small
// LDS table.  With at most 16 orientations (PAIR) the operation's 32 rows are
// the bank's high halves and its low ones, two products in one, and a lane's
// values 8 apart belong to one orientation.
//
// A pixel whose best response leads by less than the two sums can differ
// (their rounding bounds: choice_margin) is summed again in order; its
// confidence is then taken from that sum.  Those pixels wait in LDS until
// there are 16 for each wave.  Which sum a pixel's confidence comes from
// depends on its tile alone, so a frame's maps do not depend on the other
// frames of a call.
//
// Four waves per SIMD (two workgroups per CU) hold the registers to 128, which
// it just fits: a tile loaded ahead, and thread indexes kept through the
// products, spilled 42 registers (1511 against 1364 us below; the start with
// the second sum of whole tiles in the same kernel 56 to 71).  Radii above 8
// with 32 orientations have one workgroup per CU and twice the registers.
// 16 frames of 1024 x 1024 of rendered hair, all tiles in k_gabor_f32 and so
// (with k_gabor_sort and what it leaves to k_gabor_f32), us: 32 orientations
// 1253 and 768 at radius 5, 2625 and 1313 at 8, 6418 and 2858 at 12; 16
// orientations 817 and 519, 1570 and 826, 3172 and 1653.
// FULL: 32 orientations (no validity tests).
constexpr int kFixRound = 16 * kWaves;
constexpr int kFixCap = kFixRound + kTile * kTileRows;  // a round less one, plus a tile's

// The thread index as a value that the compiler knows nothing of: what follows
// from it is formed again where it is used, and not held in registers through
// the products.
__device__ __forceinline__ int fresh_thread() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <typename TO, int RS, int NT, bool FULL>
__global__ __launch_bounds__(kThreads, RS == 32 || NT == 1 ? 4 : 2) void k_gabor_split(
    GaborDev d, GaborMargin margin, Taps taps8, GaborLds L, const uint32_t* __restrict__ n_listed,
    const uint32_t* __restrict__ list, GaborOut o) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ float2 wred[kWaves];
  __shared__ int wlost[kWaves];  // the wave staged a non-zero pixel as 0
  __shared__ int2 fix[kFixCap];  // (frame, pixel) to be summed again
  __shared__ int n_fix;
  const int n_tiles = (int)*n_listed;
  if ((int)blockIdx.x >= n_tiles) return;
  const int W = d.W, H = d.H, R = d.R, NO = d.NO;
  constexpr bool PAIR = NT == 1;
  constexpr int kLoads = (kTileRows + 32) * RS / kThreads + 1;
  const int w2 = 2 * R + 1, tw = kTile + 2 * R;
  float* d2tab = (float*)(lds + L.d2);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int e = threadIdx.x; e < (L.planes - L.bank) / 4; e += kThreads)
    ((uint4*)(lds + L.bank))[e] = ((const uint4*)d.split)[e];
  fill_d2(d2tab, NO);
  float* sums = d2tab + 64;  // of each orientation's taps
  if (threadIdx.x < 32)
    sums[threadIdx.x] =
        (int)threadIdx.x < NO ? d.bank[(size_t)(w2 * w2 + kBankPad) * NO + threadIdx.x] : 0.0f;
  uint32_t* const offs = (uint32_t*)sums + 32;
  fill_offsets(offs, W, w2);
  if (threadIdx.x == 0) n_fix = 0;

  // The waiting pixels fix[first .. first + count), 16 per wave.
  auto fix_round = [&](int first, int count) {
    if (16 * w >= count) return;  // wave-uniform
    const int lane = fresh_thread() & 63, g = lane >> 4, c16 = lane & 15;
    const bool on = 16 * w + c16 < count;
    const int2 q = fix[first + (on ? 16 * w + c16 : 0)];
    f32x4 acc[NT];
    float lo, hi, fb, f2, wv, fv[4 * NT];
    int jb;
    // orientations past the last read it; such responses are not looked at
    const uint32_t b0 = (uint32_t)(g * NO + (FULL ? c16 : min(c16, NO - 1)));
    const auto tap = [&](int k, int nt) { return (d.bank + (size_t)k * NO + 16 * nt)[b0]; };
    sum_in_order<NT>(d, tap, offs, d.frames + d.plane * (size_t)q.x, q.y % W, q.y / W, g, acc, lo, hi);
#pragma unroll
    for (int k = 0; k < 4 * NT; ++k) fv[k] = fabsf(acc[k / 4][k % 4]);
    top_two<FULL>(fv, 4 * g, 16, 16, NO, fb, f2);
    choose<FULL>(fv, fb, 4 * g, 16, 16, NO, d2tab, jb, wv);
    if (g == 0 && on) {
      const size_t i = d.plane * (size_t)q.x + q.y;
      store_map<TO>(o.theta, i, (float)jb * (kPi / NO));
      o.raw[i] = wv;
      // few of these pixels raise their frame's maximum (a NaN none)
      const uint32_t top = __float_as_uint(fmaxf(wv, 0.0f));
      if (top > __atomic_load_n(&o.frame_max[q.x], __ATOMIC_RELAXED))
        atomicMax(&o.frame_max[q.x], top);
    }
  };

  // A tile's pixels, kLoads a thread; the loads are unconditional (outside
  // the frame at its first pixel, then dropped), so that they go out together.
  uint32_t keep = 0;   // bit u: tv[u] is a pixel of the frame
  bool edge = false;  // the thread's part of the windows leaves the frame
  auto load_tile = [&](int f, int x0, int y0, float (&tv)[kLoads]) {
    const float* img = d.frames + d.plane * (size_t)f;
    edge = false;
    const int t = fresh_thread(), lx = t % RS, ly = t / RS;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = t + u * kThreads;
      const int xx = RS == 32 ? lx : e % RS, yy = RS == 32 ? ly + u * (kThreads / 32) : e / RS;
      const int x = x0 + xx - R, y = y0 + yy - R;
      const bool read = xx < tw && yy < kTileRows + 2 * R;
      const bool in = read && (unsigned)x < (unsigned)W && (unsigned)y < (unsigned)H;
      uint32_t at = in ? (uint32_t)(y * W + x) : 0u;
      asm volatile("" : "+v"(at));  // keeps the load out of a branch
      const float v = img[at];
      tv[u] = v;
      keep = (keep & ~(1u << u)) | (in ? 1u << u : 0u);
      edge |= read && !in;
    }
  };
  for (int i = blockIdx.x; i < n_tiles; i += gridDim.x) {
    int cf, cx0, cy0;
    float tv[kLoads];
    d.place((int)list[i], &cf, &cx0, &cy0);
    load_tile(cf, cx0, cy0, tv);
    const int t0 = fresh_thread(), lane = t0 & 63;
    float tlo = edge ? 0.0f : INFINITY, thi = edge ? 0.0f : -INFINITY;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const bool in = keep >> u & 1u;
      tlo = in ? fminf(tlo, tv[u]) : tlo;
      thi = in ? fmaxf(thi, tv[u]) : thi;
    }
    for (int off = 32; off > 0; off >>= 1) {
      tlo = fminf(tlo, __shfl_xor(tlo, off, 64));
      thi = fmaxf(thi, __shfl_xor(thi, off, 64));
    }
    __syncthreads();  // the bank is in place; the previous tile is no longer read
    if (lane == 0) wred[w] = make_float2(tlo, thi);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      tlo = fminf(tlo, wred[k].x);
      thi = fmaxf(thi, wred[k].y);
    }
    // a tile of one sign and low contrast: less its middle, which then is
    // nearer to every pixel than 0 is
    const float mid = thi - tlo <= 2.0f * fmaxf(tlo, -thi) ? 0.5f * tlo + 0.5f * thi : 0.0f;
    const float mx = fmaxf(fabsf(thi - mid), fabsf(tlo - mid));
    // the power of two that takes mx to [2^13, 2^14) (within the normal range)
    const int ex = min(max((int)(__float_as_uint(mx) >> 23) - 127, -99), 127);
    const float scale = __uint_as_float((uint32_t)(13 - ex + 127) << 23);
    const float unscale = __uint_as_float((uint32_t)(ex - 13 - 14 + 127) << 23);
    bool lost = false;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = t0 + u * kThreads;
      if (e < L.th * RS) {
        const float c = keep >> u & 1u ? tv[u] - mid : 0.0f;
        const float v = c * scale;
        const _Float16 h = (_Float16)v;
        const _Float16 l = (_Float16)(v - (float)h);
        lost |= c != 0.0f && h == (_Float16)0.0f;
        _Float16* pl = (_Float16*)(lds + L.planes);
        pl[e] = h;
        pl[4 * L.plane + e] = l;
        if (e > 0) {  // the odd copies: word k holds pixels 2k + 1, 2k + 2
          pl[2 * L.plane + e - 1] = h;
          pl[6 * L.plane + e - 1] = l;
        }
      }
    }
    lost = __ballot(lost) != 0;
    if (lane == 0) wlost[w] = lost;
    __syncthreads();
    // The range of the pixels that the wave's rows read, from the high
    // halves (which are within 2^-11 of them).
    f16x2 lo2 = {(_Float16)INFINITY, (_Float16)INFINITY}, hi2 = -lo2;
    for (int e = lane; e < (kRowsPerWave + 2 * R) * (RS / 2); e += 64) {
      const bool on = e % (RS / 2) < tw / 2;
      const f16x2 v = __builtin_bit_cast(f16x2, lds[L.planes + kRowsPerWave * w * (RS / 2) + e]);
      lo2 = on ? __builtin_elementwise_min(lo2, v) : lo2;
      hi2 = on ? __builtin_elementwise_max(hi2, v) : hi2;
    }
    float lo = fminf((float)lo2[0], (float)lo2[1]), hi = fmaxf((float)hi2[0], (float)hi2[1]);
    for (int off = 32; off > 0; off >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, off, 64));
      hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
    lo = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(lo)));
    hi = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(hi)));
    // in units of the scaled responses
    const float level = mid * scale;
    float mg = kBankScale * (margin.mid * fabsf(level + 0.5f * (hi + lo)) +
                                   margin.half * (0.5f * (hi - lo) +
                                                  0x1p-10f * fmaxf(fabsf(hi), fabsf(lo))));
    // A window far below the tile's largest pixel has lost bits to the split's
    // smallest step (2^-24, as 2^-22 of a pixel of 1/4): summed again.
    const float top = fmaxf(fabsf(hi), fabsf(lo));
    if (top < 1.0f) {  // uniform
      int any = top > 0.0f;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) any |= wlost[k];
      if (any) mg = INFINITY;
    }
    float m = 0.0f;
    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;
    // LOW: the products with a low half; else the high halves'.  PAIR: those
    // of the low or the high halves of the pixels, with both of the bank.
    auto products = [&](auto low) {
      constexpr bool LOW = decltype(low)::value, BL = LOW, BH = !PAIR || !LOW;
      const int lane = fresh_thread() & 63, c16 = lane & 15, hf = lane >> 5;
      const uint32_t* ab = lds + L.bank + lane * 4;
      // this lane's pixel of group 0, a tap row further in the upper half, in
      // the copy of its column's parity
      const int row = kRowsPerWave * w + ((lane >> 4) & 1);
      const uint32_t* pb =
          lds + L.planes + (c16 & 1) * L.plane + ((row + hf) * RS + c16 - (c16 & 1)) / 2;
      const int n2 = (w2 + 1) / 2;  // steps of a column group
      f16x8 bh[4], bl[4];           // group q's operands at step s: slot (q + s) % 4
      f16x8 ah, al;
      auto load_a = [&]() {
        ah = *(const f16x8*)ab;
        if (LOW && !PAIR) al = *(const f16x8*)(ab + 256);
        ab += PAIR ? 256 : 512;
      };
      auto load_b = [&](int slot, const uint32_t* sh) {
        const uint32_t* sl = sh + 2 * L.plane;
        if (BH) bh[slot] = __builtin_bit_cast(f16x8, (u32x4){sh[0], sh[1], sh[2], sh[3]});
        if (BL) bl[slot] = __builtin_bit_cast(f16x8, (u32x4){sl[0], sl[1], sl[2], sl[3]});
      };
      auto step = [&](int u) {
        auto mul = [&](const f16x8& x, const f16x8 (&y)[4]) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y[(q + u) & 3], acc[q], 0, 0, 0);
        };
        if constexpr (LOW && !PAIR) {
          mul(al, bl);
          mul(al, bh);
        }
        if constexpr (LOW)
          mul(ah, bl);
        else
          mul(ah, bh);
      };
      for (int c = 0; c < taps8.cols; ++c) {
        const uint32_t* src = pb + 4 * c;
#pragma unroll
        for (int q = 0; q < 3; ++q) load_b(q, src + q * RS);
        for (int s0 = 0; s0 < n2; s0 += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (s0 + u >= n2) break;  // uniform
            load_b((u + 3) & 3, src + (s0 + u + 3) * RS);
            load_a();
            step(u);
          }
        }
      }
      // groups of 8 rows of one column
      const _Float16* vb = (const _Float16*)(lds + L.planes) + row * RS + c16 + 8 * taps8.cols;
      for (int v0 = 0; v0 < taps8.left * taps8.rows8; v0 += 2) {
        load_a();
        // a padding group past the last one reads the last one
        const int v = min(v0 + hf, taps8.left * taps8.rows8 - 1);
        const _Float16* src = vb + v / taps8.rows8 + 8 * (v % taps8.rows8) * RS;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            if (BH) bh[q][i] = src[(2 * q + i) * RS];
            if (BL) bl[q][i] = src[4 * L.plane + (2 * q + i) * RS];
          }
        step(0);
      }
    };
    products(std::true_type{});
    products(std::false_type{});
    const int el = fresh_thread() & 63, hf = el >> 5;
    if (mid != 0.0f) {  // uniform: the middle's responses
#pragma unroll
      for (int k = 0; k < 8 * NT; ++k) {
        const float part = level * kBankScale * sums[8 * (k / 4) + 4 * hf + k % 4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q][k] += part;
      }
    }
    const int prow = cy0 + kRowsPerWave * w + ((el >> 4) & 1), pcol = cx0 + (el & 15);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float fv[8 * NT], fb, f2, wv;
      int jb;
#pragma unroll
      for (int k = 0; k < 8 * NT; ++k)  // in scaled units
        fv[k] = fabsf(PAIR ? acc[q][k] + acc[q][k + 8] : acc[q][k]);
      top_two<FULL>(fv, 4 * hf, 8, 32, NO, fb, f2);
      choose<FULL>(fv, fb, 4 * hf, 8, 32, NO, d2tab, jb, wv);
      wv *= unscale;
      const bool near = !(fb >= 0.0f && fb - f2 >= mg);  // also where every response is a NaN
      const int y = prow + 2 * q;
      if (el < 32 && pcol < W && y < H) {
        if (near) {
          fix[atomicAdd(&n_fix, 1)] = make_int2(cf, y * W + pcol);
        } else {
          const size_t at = d.plane * (size_t)cf + (size_t)y * W + pcol;
          store_map<TO>(o.theta, at, (float)jb * (kPi / NO));
          o.raw[at] = wv;
          m = fmaxf(m, wv);
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    __syncthreads();  // wred and the waiting pixels
    if (el == 0) wred[w].x = m;
    int waiting = n_fix;
    __syncthreads();
    if (threadIdx.x == 0) {
      float bm = wred[0].x;
      for (int k = 1; k < kWaves; ++k) bm = fmaxf(bm, wred[k].x);
      atomicMax(&o.frame_max[cf], __float_as_uint(bm));  // bm >= 0: bits order as values
    }
    if (waiting >= kFixRound) {  // uniform: whole rounds, from the end of the list
      for (; waiting >= kFixRound; waiting -= kFixRound)
        fix_round(waiting - kFixRound, kFixRound);
      if (threadIdx.x == 0) n_fix = waiting;  // read again after the next barriers
    }
  }
  __syncthreads();
  if (n_fix > 0) fix_round(0, n_fix);
}

uint64_t fnv1(uint64_t h, const void* p, size_t n) {
  const unsigned char* c = (const unsigned char*)p;
  for (size_t i = 0; i < n; ++i) h = (h ^ c[i]) * 1099511628211ull;
  return h;
}

// floats of the bank, and where its halves start (whole 16 bytes)
size_t bank_size(int N, int w) { return (size_t)N * (w * w + kBankPad + 1); }
size_t split_offset(size_t bank) { return (bank + 3) / 4 * 4; }

// The bank in binary64 from its definition, rounded to binary32, tap-major;
// then taps of 0 and the sum of each orientation's rounded taps.
std::vector<float> make_bank(const fd_gabor_params* p) {
  const int N = p->n_orient, R = p->radius, w = 2 * R + 1;
  std::vector<double> g((size_t)N * w * w);
  for (int i = 0; i < N; ++i) {
    const double t = 3.14159265358979323846 * i / N, ct = std::cos(t), st = std::sin(t);
    double mean = 0.0;
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) {
        const double a = dx * ct + dy * st, b = -dx * st + dy * ct;
        const double sa = p->sigma_along, sb = p->sigma_across;
        const double v = std::exp(-a * a / (2 * sa * sa) - b * b / (2 * sb * sb)) *
                         std::cos(2 * 3.14159265358979323846 * b / p->wavelength);
        g[((size_t)i * w + (dy + R)) * w + (dx + R)] = v;
        mean += v;
      }
    mean /= (double)(w * w);
    for (int k = 0; k < w * w; ++k) g[(size_t)i * w * w + k] -= mean;
  }
  std::vector<float> out(bank_size(N, w));
  for (int i = 0; i < N; ++i) {
    double sum = 0.0;
    for (int k = 0; k < w * w; ++k)
      sum += out[(size_t)k * N + i] = (float)g[(size_t)i * w * w + k];
    out[(size_t)(w * w + kBankPad) * N + i] = (float)sum;
  }
  return out;
}

// Twice the most by which the two sums of one response can differ, for a
// window of pixels I = mid + v, |v| <= half, per unit of |mid| and of half.
// A rounding is at most 2^-24 of the running sum, which is bounded by
// |mid| |sum of the taps so far| + half (sum of their magnitudes so far).
// Sum in order: one rounding per tap (the bound is taken at the start of a
// 4-tap step, the step's own magnitudes on top).
// Split sum: the products with a low half first, whose sum stays below 2^-10 of
// the magnitudes and takes three roundings and cuts of that for each of the
// others', then the high halves', two roundings per 16 taps and as much cut off
// again where the operation aligns its products.  What the splits do not hold
// is within 2^-23 of either factor (and, for pixels or taps far below the
// largest, 2^-36 of the largest, which is within 2^14 of the window's: else the
// pixel is summed again without a look at the margin).  First order, one percent
// on top for the rest.
GaborMargin choice_margin(const std::vector<float>& bank, int N, int R) {
  const Taps tp(R);
  const int w = tp.w, taps = w * w;
  double most_p = 0.0, most_g = 0.0;
  for (int j = 0; j < N; ++j) {
    double P = 0.0, G = 0.0, sp = 0.0, sg = 0.0;
    for (int k = 0; k < taps; ++k) {
      if (k % 4 == 0) {
        sp += 4.0 * std::fabs(P);
        sg += 4.0 * G;
      }
      P += bank[(size_t)k * N + j];
      G += std::fabs((double)bank[(size_t)k * N + j]);
    }
    const double all = G;
    P = G = 0.0;
    for (int st = 0; st < tp.steps; ++st) {
      sp += 4.0 * std::fabs(P);
      sg += 4.0 * G;
      for (int q = 2 * st; q < 2 * st + 2; ++q)
        for (int i = 0; i < 8; ++i) {
          int dy, dx;
          if (!tp.tap(q, i, &dy, &dx)) continue;
          P += bank[(size_t)(dy * w + dx) * N + j];
          G += std::fabs((double)bank[(size_t)(dy * w + dx) * N + j]);
        }
    }
    // each sum's own steps, the splits, the middle's subtraction, the low
    // halves' roundings
    const double rest = all * (4 + 4 + 4 + 1 + 12.0 * tp.steps / 1024.0 + 4) + taps;
    most_p = std::max(most_p, sp + rest);
    most_g = std::max(most_g, sg + rest);
  }
  const double u = 2.0 * 1.01 / 16777216.0;
  return GaborMargin{(float)(u * most_p), (float)(u * most_g)};
}

// Split sums from radius 5 on: below it a sum in order over so few taps is
// nearer to the exact one on low-contrast windows (figures with k_gabor_split),
// and there is less to gain: 16 frames of rendered hair, 32 orientations, 716
// and 524 us at radius 3, 456 and 472 at 1.  And for frames that are large
// enough for one of them alone to take no longer, sorted first, than in the
// binary32 kernel (a frame's maps do not depend on how many there are); noise,
// binary32 and split, us, waited for after each call:
//   32 orientations   radius 8                    radius 12
//     64 tiles        57 and 78                   88 and 119
//     256             79 and 83                   138 and 182
//     1024            198 and 166                 442 and 297
//   16 orientations   radius 8                    radius 11
//     256             59 and 69                   78 and 125
//     1024            127 and 98                  196 and 146
constexpr int kSplitRadius = 5;
bool split_sums(const GaborDev& d) {
  return d.R >= kSplitRadius && d.tiles_x * d.tiles_y >= (d.NO > 16 ? 320 : 640);
}

template <typename TO, int NT, bool FULL>
hipError_t launch_gabor(GaborDev d, const float* margin, uint32_t* cursor, uint32_t* list,
                        const GaborOut& o, hipStream_t st) {
  hipError_t e;
  const bool split = split_sums(d);
  const int taps = (2 * d.R + 1) * (2 * d.R + 1);
  if (split) {
    const GaborMargin mg{margin[0], margin[1]};
    // one wave per SIMD and a tile or a pair for each wave while that is all
    // the work there is (256 tiles: 21 us, 38 with 16 waves), else 16 waves and
    // as many tiles for each as leave two workgroups for a compute unit
    const int waves = d.n_tiles <= 4 * 256 * NT ? 4 : kSortWaves;
    int per = std::min(kSortMost, std::max(1, d.n_tiles / (512 * kSortWaves)));
    per = (per + NT - 1) / NT * NT;
    const int here = per * waves;
    const size_t sort_lds = sizeof(float) * (size_t)round_taps(taps) * (16 * NT + 1);
    const auto sort = k_gabor_sort<NT, FULL>;
    e = hipFuncSetAttribute((const void*)sort, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)sort_lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sort, dim3((unsigned)((d.n_tiles + here - 1) / here)), dim3(64 * waves),
                       sort_lds, st, d, mg, per, (unsigned long long*)cursor, list);
    const GaborLds L(d.R, NT == 1);
    const size_t lds = 4 * (size_t)L.total;
    const auto kern = d.R <= 8 ? k_gabor_split<TO, 32, NT, FULL> : k_gabor_split<TO, 40, NT, FULL>;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e != hipSuccess) return e;
    // persistent: each workgroup splits the bank once; two resident per CU
    // where the LDS allows it
    const int per_cu = 2 * (lds + 8 * kFixCap + 512) <= 160 * 1024 ? 2 : 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(d.n_tiles, 256 * per_cu)), dim3(kThreads), lds,
                       st, d, mg, Taps(d.R), L, cursor, list, o);
  }
  const size_t lds = sizeof(float) * ((size_t)padded_taps(taps) * 16 * NT +
                                      (size_t)kTw * (kF32Rows + 2 * d.R) + 64);
  e = hipFuncSetAttribute((const void*)k_gabor_f32<TO, NT, FULL>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // persistent: each workgroup loads the bank once; several resident per CU
  const int per_cu = (int)std::max<size_t>(1, (160 * 1024) / (lds + 1024));
  const int half_y = (d.H + kF32Rows - 1) / kF32Rows;
  const int n_half = split ? 2 * d.n_tiles : d.n_tiles / d.tiles_y * half_y;
  hipLaunchKernelGGL((k_gabor_f32<TO, NT, FULL>),
                     dim3((unsigned)std::min(n_half, 256 * std::min(per_cu, 4))), dim3(256), lds,
                     st, d, half_y, n_half, split ? cursor + 1 : nullptr, split ? list : nullptr, o);
  return hipGetLastError();
}

}  // namespace

extern "C" void fd_gabor_params_init(fd_gabor_params* p) {
  if (!p) return;
  std::memset(p, 0, sizeof *p);
  p->n_orient = 32;
  p->radius = 8;
  p->sigma_along = 2.4f;
  p->sigma_across = 1.8f;
  p->wavelength = 4.0f;
  p->out_dtype = FD_F16;
  p->stream = nullptr;
  p->ctx = nullptr;
}

extern "C" int fd_orientation_maps(const float* frames, int32_t n_frames, int32_t width,
                                   int32_t height, const fd_gabor_params* p, void* theta_out,
                                   void* conf_out) {
  const char* fn = "fd_orientation_maps";
  int r;
  if (!p) return set_error(FD_E_INVAL, "%s: params is NULL", fn);
  if (p->n_orient != 8 && p->n_orient != 16 && p->n_orient != 32)
    return set_error(FD_E_INVAL, "%s: n_orient must be 8, 16 or 32, got %d", fn, p->n_orient);
  if (p->radius < 1 || p->radius > kMaxRadius)
    return set_error(FD_E_INVAL, "%s: radius must be in [1, %d], got %d", fn, kMaxRadius,
                     p->radius);
  if (!(p->sigma_along > 0.0f) || !(p->sigma_across > 0.0f) || !(p->wavelength > 0.0f) ||
      !std::isfinite(p->sigma_along) || !std::isfinite(p->sigma_across) ||
      !std::isfinite(p->wavelength))
    return set_error(FD_E_INVAL, "%s: sigmas and wavelength must be finite and > 0", fn);
  if (p->out_dtype != FD_F32 && p->out_dtype != FD_F16)
    return set_error(FD_E_INVAL, "%s: unknown out_dtype %d", fn, p->out_dtype);
  if (n_frames < 0 || n_frames > FD_MAX_VIEWS)
    return set_error(FD_E_INVAL, "%s: n_frames must be in [0, %d]", fn, FD_MAX_VIEWS);
  if (width < 1 || height < 1 || width > 32768 || height > 32768)
    return set_error(FD_E_INVAL, "%s: frame size out of range", fn);
  if (n_frames > 0 && (!frames || !theta_out || !conf_out))
    return set_error(FD_E_INVAL, "%s: null pointer argument", fn);
  int dev = 0;
  if ((r = check_device(&dev))) return r;
  if (n_frames == 0) return FD_OK;
  fd_context* c = p->ctx;
  if (c) {
    if (c->device != dev)
      return set_error(FD_E_INVAL, "%s: context belongs to device %d", fn, c->device);
  } else {
    c = default_context(dev, 0, &r);
    if (!c) return r;
  }
  hipStream_t st = (hipStream_t)p->stream;
  // the filter bank, rebuilt when its parameters change
  uint64_t sig = 1469598103934665603ull;
  sig = fnv1(sig, &p->n_orient, sizeof p->n_orient);
  sig = fnv1(sig, &p->radius, sizeof p->radius);
  sig = fnv1(sig, &p->sigma_along, sizeof p->sigma_along);
  sig = fnv1(sig, &p->sigma_across, sizeof p->sigma_across);
  sig = fnv1(sig, &p->wavelength, sizeof p->wavelength);
  hipError_t e;
  if (c->gabor_sig != sig || !c->gabor_bank) {
    const std::vector<float> bank = make_bank(p);
    // a previous call on this stream may still read the old bank
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return hip_error(e, "filter bank");
    const GaborLds L(p->radius, p->n_orient <= 16);
    if ((r = ctx_buffer((void**)&c->gabor_bank, &c->cap_gabor_bank,
                        split_offset(bank.size()) * sizeof(float) + 4 * (size_t)(L.planes - L.bank),
                        "filter bank")))
      return r;
    e = hipMemcpy(c->gabor_bank, bank.data(), bank.size() * sizeof(float),
                  hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_error(e, "filter bank upload");
    const Taps t(p->radius);
    hipLaunchKernelGGL(k_gabor_halves, dim3((unsigned)t.steps), dim3(64), 0, st, c->gabor_bank,
                       p->n_orient, p->n_orient <= 16, t,
                       (uint32_t*)(c->gabor_bank + split_offset(bank.size())));
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess)
      return hip_error(e, "filter bank halves");
    const GaborMargin mg = choice_margin(bank, p->n_orient, p->radius);
    c->gabor_margin[0] = mg.mid;
    c->gabor_margin[1] = mg.half;
    c->gabor_sig = sig;
  }
  const size_t plane = (size_t)width * height, total = plane * (size_t)n_frames;
  if (total > ((size_t)1 << 34))
    return set_error(FD_E_INVAL, "%s: more than 2^34 pixels in one call", fn);
  if ((r = ctx_buffer((void**)&c->gabor_raw, &c->cap_gabor_raw, total * sizeof(float),
                      "raw confidence")))
    return r;
  // the maxima after the cursor of the tile list
  if ((r = ctx_buffer((void**)&c->gabor_max, &c->cap_gabor_max,
                      (2 + (size_t)n_frames) * sizeof(uint32_t), "frame maxima")))
    return r;
  uint32_t* const fmax = c->gabor_max + 2;
  const int w2 = 2 * p->radius + 1;
  const uint32_t* const split =
      (const uint32_t*)(c->gabor_bank + split_offset(bank_size(p->n_orient, w2)));
  GaborDev d{frames, width, height, p->radius, p->n_orient, c->gabor_bank, split, 0, 0, 0, plane};
  d.tiles_x = (width + kTile - 1) / kTile;
  d.tiles_y = (height + kTileRows - 1) / kTileRows;
  // n_frames <= FD_MAX_VIEWS, at most 2^34 pixels: below 2^30
  d.n_tiles = d.tiles_x * d.tiles_y * n_frames;
  if (split_sums(d) &&
      (r = ctx_buffer((void**)&c->gabor_list, &c->cap_gabor_list,
                      (size_t)d.n_tiles * sizeof(uint32_t), "tile list")))
    return r;
  if ((e = launch_fill_u32(c->gabor_max, 2 + (int64_t)n_frames, 0u, st)) != hipSuccess)
    return hip_error(e, "frame maxima reset");
  const GaborOut o{theta_out, c->gabor_raw, fmax};
  StageTimer tg(c, FD_STAGE_GABOR, st);
#define FD_GABOR(TO)                                                                               \
  (p->n_orient == 32   ? launch_gabor<TO, 2, true>(d, c->gabor_margin, c->gabor_max, c->gabor_list, o, st) \
   : p->n_orient == 16 ? launch_gabor<TO, 1, true>(d, c->gabor_margin, c->gabor_max, c->gabor_list, o, st) \
                       : launch_gabor<TO, 1, false>(d, c->gabor_margin, c->gabor_max, c->gabor_list, o, st))
  e = p->out_dtype == FD_F16 ? FD_GABOR(__half) : FD_GABOR(float);
#undef FD_GABOR
  if (e != hipSuccess) return hip_error(e, "orientation kernel");
  tg.stop();
  StageTimer tn(c, FD_STAGE_GABOR_NORM, st);
  // raw is a workspace allocation, so only the plane and the caller's output
  // decide whether whole 16-byte groups line up
  const int vec = plane % 8 == 0 && (uintptr_t)conf_out % 16 == 0;
  const int64_t work = vec ? (int64_t)plane / 8 : (int64_t)plane;
  const dim3 ng((unsigned)std::min<int64_t>((work + 255) / 256, 1 << 20), (unsigned)n_frames);
  if (p->out_dtype == FD_F16)
    hipLaunchKernelGGL(k_gabor_norm<__half>, ng, dim3(256), 0, st, c->gabor_raw, fmax,
                       (int64_t)plane, vec, conf_out);
  else
    hipLaunchKernelGGL(k_gabor_norm<float>, ng, dim3(256), 0, st, c->gabor_raw, fmax,
                       (int64_t)plane, vec, conf_out);
  if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "confidence kernel");
  tn.stop();
  return FD_OK;
}
