// fd_volume.hip -- occupancy and orientation volume from oriented points on
// gfx950 (the fused volume of Sec. 3.2, opening paragraph; the rule is
// documented with fd_fuse_volume in fusedir.h).
//
// A counting sort of the points by voxel, then one thread per busy voxel:
//   k_vol_key       one thread per point: binary32 voxel index and one u32
//                   atomic on the voxel's count, whose old value is the
//                   point's rank within its voxel (the counts are the
//                   occupancy output itself);
//   k_vol_alloc     one pass over the counts: every busy voxel gets its slots
//                   and its place in the list of busy voxels, a block of
//                   voxels at a time from one counter (empty voxels get their
//                   outputs);
//   k_vol_place     each point's direction and weight to slot offset[v] +
//                   rank (16 B per point);
//   k_vol_reduce    one thread per busy voxel: the structure-tensor terms
//                   w d d^T of its slots, each formed in binary64 and rounded
//                   to a multiple of 2^-32, summed as 64-bit integers in
//                   registers, then cyclic Jacobi rotations to the top
//                   eigenvector and the coherence (l1 - l2) / l1.
// Integer sums do not depend on the order of the points within a voxel, nor
// any output on where a voxel's slots lie, so the volume is deterministic.
// Device-scope atomics on memory shared by all XCDs are performed past the L2
// (each one a 32-byte transaction), so this form issues one per point where
// summing in place would issue seven.
//
// Bound by random transactions: 2M points in 7.7M voxels, 0.87M of them busy:
// k_vol_key 86 us (23 G atomics/s), k_vol_place 65 us, k_vol_reduce 54 us,
// k_vol_alloc 29 us, the call 364 -> 244 us (four scan passes with their
// helpers in place of k_vol_alloc took 95 us, 48-byte records 102 + 73 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "../../include/fusedir.h"
#include "fd_api_internal.hpp"
#include "fd_kernels.hpp"
#include "fd_voxel.hpp"

using namespace fd;

namespace {

constexpr double kFix = 4294967296.0;        // 2^32 units per 1.0
constexpr double kUnfix = 1.0 / 4294967296.0;
constexpr uint32_t kOutside = 0xffffffffu;
// k_vol_reduce takes kGroup lanes a voxel where the busy ones hold more than
// kFew points on average, else one.  Whole calls with one and eight lanes, us:
// 250 and 469 at 2.3 points, 187 and 215 at 15, 215 and 188 at 34, 157 and 114
// at 38, 555 and 363 at 143.
constexpr int kGroup = 8, kFew = 24;
// A voxel with more than this many points for each of its lanes takes the whole
// wave: few voxels far above the average would otherwise be all that runs (half
// of 1M points in 100 voxels, the call: 3.0 ms -> 247 us, 1.3 ms with 48-byte
// records; points per voxel by a power law of 1.2 up to 3000: 862 -> 130 us).
constexpr int kHeavy = 128;
constexpr int kRun = 1024;       // threads of k_vol_alloc
constexpr int kRunVoxels = 4096;  // voxels of one of its blocks

__device__ __forceinline__ unsigned long long fix(double t) {
  t = fmin(fmax(t, -1.0), 1.0);
  return (unsigned long long)__double2ll_rn(t * kFix);
}

__global__ __launch_bounds__(256) void k_vol_key(const float* __restrict__ points, int64_t n,
                                                 GridDev g, uint32_t* __restrict__ cnt,
                                                 uint32_t* __restrict__ key_rank,
                                                 uint32_t* __restrict__ cursor) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 2) cursor[i] = 0u;  // k_vol_alloc's
  if (i >= n) return;
  const int64_t v = voxel_index(g, points[3 * i], points[3 * i + 1], points[3 * i + 2]);
  if (v < 0) {
    key_rank[2 * i] = kOutside;
    return;
  }
  key_rank[2 * i] = (uint32_t)v;
  key_rank[2 * i + 1] = atomicAdd(&cnt[v], 1u);
}

// inclusive scan of one value per thread over a block of kRun threads
__device__ __forceinline__ uint64_t run_incl_scan(uint64_t x, uint64_t* wsum) {
  const int lane = (int)(threadIdx.x & 63u), w = (int)(threadIdx.x >> 6);
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t o = __shfl_up((unsigned long long)x, off, 64);
    if (lane >= off) x += o;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  if (w == 0) {
    uint64_t t = lane < kRun / 64 ? wsum[lane] : 0u;
    for (int off = 1; off < kRun / 64; off <<= 1) {
      const uint64_t o = __shfl_up((unsigned long long)t, off, 64);
      if (lane >= off) t += o;
    }
    if (lane < kRun / 64) wsum[lane] = t;
  }
  __syncthreads();
  return x + (w > 0 ? wsum[w - 1] : 0u);
}

// Slots and list places for a block of kRunVoxels voxels, four a thread: a
// scan within the block, one atomic for its range.  The cursor holds the
// slots given out in its high half (at most n < 2^31) and the busy voxels in
// its low half (at most 2^30), so one never carries into the other.  All the
// block's outputs are cleared in whole lines; the busy voxels' are written
// again later.
__global__ __launch_bounds__(kRun) void k_vol_alloc(const uint32_t* __restrict__ cnt, int64_t nv,
                                                    unsigned long long* __restrict__ cursor,
                                                    uint32_t* __restrict__ off,
                                                    uint32_t* __restrict__ list,
                                                    float* __restrict__ dir_out,
                                                    float* __restrict__ coh_out,
                                                    double* __restrict__ tensor_out) {
  __shared__ uint64_t wsum[kRun / 64];
  __shared__ uint64_t base;
  const int64_t b0 = (int64_t)blockIdx.x * kRunVoxels;
  const int nb = (int)(nv - b0 < kRunVoxels ? nv - b0 : kRunVoxels);
  uint32_t c[4];
  uint64_t x = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int u = 4 * (int)threadIdx.x + k;
    c[k] = u < nb ? cnt[b0 + u] : 0u;
    x += (uint64_t)c[k] << 32 | (c[k] != 0u ? 1u : 0u);
  }
  for (int u = threadIdx.x; u < 3 * nb; u += kRun) dir_out[3 * b0 + u] = 0.0f;
  for (int u = threadIdx.x; u < nb; u += kRun) coh_out[b0 + u] = 0.0f;
  if (tensor_out)
    for (int u = threadIdx.x; u < 6 * nb; u += kRun) tensor_out[6 * b0 + u] = 0.0;
  const uint64_t incl = run_incl_scan(x, wsum);
  if (threadIdx.x == kRun - 1) base = incl ? atomicAdd(cursor, (unsigned long long)incl) : 0u;
  __syncthreads();
  uint64_t at = base + incl - x;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int u = 4 * (int)threadIdx.x + k;
    if (c[k] != 0u) {
      off[b0 + u] = (uint32_t)(at >> 32);
      list[(uint32_t)at] = (uint32_t)(b0 + u);
      at += (uint64_t)c[k] << 32 | 1u;
    }
  }
}

// Each point to slot offset[v] + rank, so the per-voxel sums read contiguous,
// independent records.
__global__ __launch_bounds__(256) void k_vol_place(const uint32_t* __restrict__ key_rank,
                                                   const float* __restrict__ dirs,
                                                   const float* __restrict__ weights, int64_t n,
                                                   const uint32_t* __restrict__ off,
                                                   float4* __restrict__ rec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t v = key_rank[2 * i];
  if (v == kOutside) return;
  const uint64_t slot = (uint64_t)off[v] + key_rank[2 * i + 1];
  if (slot >= (uint64_t)n) return;
  float w = weights ? weights[i] : 1.0f;
  w = w > 0.0f ? fminf(w, 1.0f) : 0.0f;  // NaN and negatives count as 0
  rec[slot] = make_float4(dirs[3 * i], dirs[3 * i + 1], dirs[3 * i + 2], w);
}

// 1 / x and 1 / sqrt(x) in binary64, x normal: the hardware's estimate and one
// step that takes its relative error e to e^3 (to the last bit or two).
__device__ __forceinline__ double recip(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, y, 1.0);
  return __builtin_fma(y, __builtin_fma(e, e, e), y);
}
__device__ __forceinline__ double recip_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// One Jacobi rotation in the (P, Q) plane of the symmetric A, accumulated
// into the columns of V (Golub and Van Loan, symmetric Schur step): t = tan
// of the smaller angle, from a = A[Q][Q] - A[P][P] and b = 2 A[P][Q] as
// sign(a) b / (|a| + sqrt(a^2 + b^2)).  An element below 1e-150 is as good as
// 0 (the non-zero tensors are multiples of 2^-32).
template <int P, int Q>
__device__ __forceinline__ void jacobi_rotate(double (&A)[3][3], double (&V)[3][3]) {
  constexpr int K = 3 - P - Q;
  const double apq = A[P][Q];
  if (fabs(apq) < 1e-150) return;
  const double a = A[Q][Q] - A[P][P], b = 2.0 * apq, r2 = __builtin_fma(a, a, b * b);
  const double den = fabs(a) + r2 * recip_sqrt(r2);
  const double t = (a > 0.0 ? b : (a < 0.0 ? -b : fabs(b))) * recip(den);
  const double c = recip_sqrt(__builtin_fma(t, t, 1.0)), s = t * c;
  A[P][P] -= t * apq;
  A[Q][Q] += t * apq;
  A[P][Q] = A[Q][P] = 0.0;
  const double x = A[K][P], y = A[K][Q];
  A[K][P] = A[P][K] = c * x - s * y;
  A[K][Q] = A[Q][K] = s * x + c * y;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double u = V[k][P], v = V[k][Q];
    V[k][P] = c * u - s * v;
    V[k][Q] = s * u + c * v;
  }
}

__global__ __launch_bounds__(256) void k_vol_reduce(const float4* __restrict__ rec, int64_t n,
                                                    const uint32_t* __restrict__ cnt,
                                                    const uint32_t* __restrict__ off, int64_t nv,
                                                    const uint32_t* __restrict__ list,
                                                    const uint32_t* __restrict__ cursor,
                                                    float* __restrict__ dir_out,
                                                    float* __restrict__ coh_out,
                                                    double* __restrict__ tensor_out) {
  const int64_t n_busy = cursor[0];
  // uniform: lanes per voxel
  const bool many = (uint64_t)cursor[1] > (uint64_t)kFew * (uint64_t)n_busy;
  const int group = many ? kGroup : 1, part = (int)threadIdx.x & (group - 1);
  const int64_t e = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / group;
  const int64_t v = e < n_busy ? list[e] : nv;
  unsigned long long S[6] = {0ull, 0ull, 0ull, 0ull, 0ull, 0ull};
  auto add = [&](float4 q) {
    if (q.w != 0.0f && !(q.x == 0.0f && q.y == 0.0f && q.z == 0.0f)) {
      const double wd = q.w, dx = q.x, dy = q.y, dz = q.z;
      S[0] += fix(wd * dx * dx);
      S[1] += fix(wd * dy * dy);
      S[2] += fix(wd * dz * dz);
      S[3] += fix(wd * dx * dy);
      S[4] += fix(wd * dx * dz);
      S[5] += fix(wd * dy * dz);
    }
  };
  uint32_t c = 0, s0 = 0;
  if (v < nv) {
    s0 = off[v];
    c = cnt[v];
    if ((int64_t)s0 + c > n) c = (int64_t)s0 < n ? (uint32_t)(n - s0) : 0u;
  }
  // the slots [s, s + m), every step-th from the at-th on
  auto add_slots = [&](uint32_t s, uint32_t m, uint32_t at, uint32_t step) {
    for (uint32_t j = at; j < m; j += 4 * step) {
      float4 q[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) q[k] = rec[s + min(j + k * step, m - 1)];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        if (j + k * step >= m) q[k].w = 0.0f;
        add(q[k]);
      }
    }
  };
  const bool heavy = c > (uint32_t)(kHeavy * group);
  add_slots(s0, heavy ? 0u : c, part, group);
  if (many) {
#pragma unroll
    for (int k = 0; k < 6; ++k)
      for (int o = kGroup / 2; o > 0; o >>= 1) S[k] += __shfl_xor(S[k], o, 64);
  }
  // the wave's heavy voxels, one by one with all its lanes
  const int lane = (int)(threadIdx.x & 63u);
  for (uint64_t b = __ballot(heavy && part == 0); b; b &= b - 1) {
    const int l = __ffsll((unsigned long long)b) - 1;
    unsigned long long own[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      own[k] = S[k];
      S[k] = 0ull;
    }
    add_slots((uint32_t)__shfl((int)s0, l, 64), (uint32_t)__shfl((int)c, l, 64), lane, 64);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      for (int o = 32; o > 0; o >>= 1) S[k] += __shfl_xor(S[k], o, 64);
      S[k] = lane == l ? S[k] : own[k];
    }
  }
  if (v >= nv || part != 0) return;
  double T[6];
  bool any = false;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    any |= S[k] != 0ull;
    T[k] = (double)(long long)S[k] * kUnfix;
  }
  if (tensor_out) {
#pragma unroll
    for (int k = 0; k < 6; ++k) tensor_out[6 * v + k] = T[k];
  }
  float d0 = 0.0f, d1 = 0.0f, d2 = 0.0f, coh = 0.0f;
  if (any) {
    double A[3][3] = {{T[0], T[3], T[4]}, {T[3], T[1], T[5]}, {T[4], T[5], T[2]}};
    double V[3][3] = {{1.0, 0.0, 0.0}, {0.0, 1.0, 0.0}, {0.0, 0.0, 1.0}};
    for (int sweep = 0; sweep < 32; ++sweep) {
      const double od = A[0][1] * A[0][1] + A[0][2] * A[0][2] + A[1][2] * A[1][2];
      const double dg = A[0][0] * A[0][0] + A[1][1] * A[1][1] + A[2][2] * A[2][2];
      if (od == 0.0 || od <= 1e-36 * dg) break;
      jacobi_rotate<0, 1>(A, V);
      jacobi_rotate<0, 2>(A, V);
      jacobi_rotate<1, 2>(A, V);
    }
    // largest, then second largest eigenvalue (first index wins ties)
    const double l0 = A[0][0], l1 = A[1][1], l2 = A[2][2];
    int top = 0;
    double lt = l0;
    if (l1 > lt) { top = 1; lt = l1; }
    if (l2 > lt) { top = 2; lt = l2; }
    const double lo = top == 0 ? fmax(l1, l2) : (top == 1 ? fmax(l0, l2) : fmax(l0, l1));
    double e0 = V[0][top], e1 = V[1][top], e2 = V[2][top];
    const double nr = recip_sqrt(e0 * e0 + e1 * e1 + e2 * e2);
    e0 *= nr;
    e1 *= nr;
    e2 *= nr;
    const double key = e2 != 0.0 ? e2 : (e1 != 0.0 ? e1 : e0);
    if (key < 0.0) {
      e0 = -e0;
      e1 = -e1;
      e2 = -e2;
    }
    d0 = (float)e0;
    d1 = (float)e1;
    d2 = (float)e2;
    coh = lt > 0.0 ? (float)((lt - lo) / lt) : 0.0f;
  }
  dir_out[3 * v] = d0;
  dir_out[3 * v + 1] = d1;
  dir_out[3 * v + 2] = d2;
  coh_out[v] = coh;
}

}  // namespace

extern "C" int fd_fuse_volume(const float* points, const float* dirs, const float* weights,
                              int64_t n_points, const fd_volume_grid* grid, void* stream,
                              fd_context* ctx, uint32_t* occ_out, float* dir_out,
                              float* coherence_out, double* tensor_out) {
  const char* fn = "fd_fuse_volume";
  int r;
  if (!grid) return set_error(FD_E_INVAL, "%s: grid is NULL", fn);
  if (!(grid->voxel > 0.0f) || !std::isfinite(grid->voxel))
    return set_error(FD_E_INVAL, "%s: voxel edge must be finite and > 0", fn);
  for (int a = 0; a < 3; ++a) {
    if (!std::isfinite(grid->origin[a]))
      return set_error(FD_E_INVAL, "%s: grid origin must be finite", fn);
    if (grid->dims[a] < 1 || grid->dims[a] > FD_MAX_VOLUME_DIM)
      return set_error(FD_E_INVAL, "%s: dims must be in [1, %d]", fn, FD_MAX_VOLUME_DIM);
  }
  const int64_t nv = (int64_t)grid->dims[0] * grid->dims[1] * grid->dims[2];
  if (nv > FD_MAX_VOLUME_VOXELS)
    return set_error(FD_E_INVAL, "%s: %lld voxels, at most %lld", fn, (long long)nv,
                     (long long)FD_MAX_VOLUME_VOXELS);
  if (n_points < 0 || n_points > FD_MAX_VOLUME_POINTS)
    return set_error(FD_E_INVAL, "%s: n_points must be in [0, %lld]", fn,
                     (long long)FD_MAX_VOLUME_POINTS);
  if (n_points > 0 && (!points || !dirs))
    return set_error(FD_E_INVAL, "%s: points and dirs are required", fn);
  if (!occ_out || !dir_out || !coherence_out)
    return set_error(FD_E_INVAL, "%s: null output pointer", fn);
  int dev = 0;
  if ((r = check_device(&dev))) return r;
  fd_context* c = ctx;
  if (c) {
    if (c->device != dev)
      return set_error(FD_E_INVAL, "%s: context belongs to device %d", fn, c->device);
  } else {
    c = default_context(dev, 0, &r);
    if (!c) return r;
  }
  const int64_t nb = (nv + kRunVoxels - 1) / kRunVoxels;
  const size_t un = (size_t)(n_points > 0 ? n_points : 1);
  const int64_t max_busy = nv < n_points ? nv : n_points;
  if ((r = ctx_buffer((void**)&c->vol_key, &c->cap_vol_key, 8 * un, "volume keys")) ||
      (r = ctx_buffer((void**)&c->vol_perm, &c->cap_vol_perm, 16 * un, "volume records")) ||
      (r = ctx_buffer((void**)&c->vol_off, &c->cap_vol_off, 4 * (size_t)nv, "volume offsets")) ||
      (r = ctx_buffer((void**)&c->vol_list, &c->cap_vol_list, 4 * (size_t)(2 + max_busy),
                      "volume busy list")))
    return r;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  GridDev g;
  for (int a = 0; a < 3; ++a) {
    g.o[a] = grid->origin[a];
    g.dims[a] = grid->dims[a];
  }
  g.h = grid->voxel;
  {
    StageTimer t(c, FD_STAGE_VOLUME_CLEAR, st);
    if ((e = launch_fill_u32(occ_out, nv, 0u, st)) != hipSuccess)
      return hip_error(e, "volume clear");
    t.stop();
  }
  uint32_t* list = c->vol_list + 2;  // after the cursor
  const dim3 pg((unsigned)((un + 255) / 256));
  {
    StageTimer t(c, FD_STAGE_VOLUME_SCATTER, st);
    hipLaunchKernelGGL(k_vol_key, pg, dim3(256), 0, st, points, n_points, g, occ_out, c->vol_key,
                       c->vol_list);
    hipLaunchKernelGGL(k_vol_alloc, dim3((unsigned)nb), dim3(kRun), 0, st, occ_out, nv,
                       (unsigned long long*)c->vol_list, c->vol_off, list, dir_out, coherence_out,
                       tensor_out);
    if (n_points > 0)
      hipLaunchKernelGGL(k_vol_place, pg, dim3(256), 0, st, c->vol_key, dirs, weights, n_points,
                         c->vol_off, (float4*)c->vol_perm);
    if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "volume sort");
    t.stop();
  }
  {
    StageTimer t(c, FD_STAGE_VOLUME_FINAL, st);
    // enough for either number of lanes a voxel (kGroup: at most n / kFew voxels)
    const int64_t lanes = std::max(max_busy, kGroup * std::min(nv, n_points / kFew));
    if (max_busy > 0)
      hipLaunchKernelGGL(k_vol_reduce, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st,
                         (const float4*)c->vol_perm, n_points, occ_out, c->vol_off, nv, list,
                         c->vol_list, dir_out, coherence_out, tensor_out);
    if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "volume reduce");
    t.stop();
  }
  return FD_OK;
}
