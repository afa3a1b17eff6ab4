// fd_tile.hip -- spatial tiling of the points (gfx950).
//
// Points are grouped by a Morton-ordered cell of a 64^3 grid over their
// bounding box, so that the points one wavefront fuses together project to
// neighbouring pixels and their patch gathers share cache lines.  Cell order
// is a counting sort (histogram, exclusive scan, scatter).  The order of
// points inside one cell depends on atomic timing; nothing downstream
// depends on it, because every point is fused independently of the others.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fd_device.hpp"
#include "fd_kernels.hpp"

namespace fd {

constexpr int kCellBits = 6;  // per axis
constexpr int kCells = 1 << (3 * kCellBits);

__device__ __forceinline__ int float_to_ordered(float f) {
  int i = __float_as_int(f);
  return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ __forceinline__ float ordered_to_float(int i) {
  return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// The smallest (v[0..2]) and largest (v[3..5]) ordered value over the
// workgroup's 256 threads, in every thread.
__device__ __forceinline__ void block_box(int (&v)[6]) {
  __shared__ int red[4][6];
  for (int a = 0; a < 3; ++a) {
    for (int off = 32; off > 0; off >>= 1) {
      v[a] = min(v[a], __shfl_xor(v[a], off, 64));
      v[3 + a] = max(v[3 + a], __shfl_xor(v[3 + a], off, 64));
    }
  }
  if ((threadIdx.x & 63) == 0)
    for (int a = 0; a < 6; ++a) red[threadIdx.x >> 6][a] = v[a];
  __syncthreads();
  for (int a = 0; a < 3; ++a) {
    v[a] = min(min(red[0][a], red[1][a]), min(red[2][a], red[3][a]));
    v[3 + a] = max(max(red[0][3 + a], red[1][3 + a]), max(red[2][3 + a], red[3][3 + a]));
  }
}

// All that a call starts with, in one launch (five before, 2 to 4 us each):
// the cell counts and (unless NULL) the fallback counters cleared, the search
// constants, the camera table, and every workgroup's part of the points' bounding box
// (boxes[6 b ..]; the next kernel folds the parts, so that none of them
// needs a value to start from).
constexpr int kSetupBlocks = 256;
__global__ __launch_bounds__(256) void k_setup(const float* __restrict__ pts, int64_t n,
                                               int* __restrict__ boxes,
                                               uint32_t* __restrict__ counts,
                                               uint32_t* __restrict__ fb_count, ConstsDev c,
                                               int n_candidates, double step0, double lstep0,
                                               const float* __restrict__ cams, int V,
                                               double* __restrict__ cam64) {
  const int first = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  constexpr int kStride = kSetupBlocks * 256;
  int v[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
  for (int64_t i = first; i < n; i += kStride) {
    for (int a = 0; a < 3; ++a) {
      const float f = pts[3 * i + a];
      if (f == f) {  // skip NaN
        const int o = float_to_ordered(f);
        v[a] = min(v[a], o);
        v[3 + a] = max(v[3 + a], o);
      }
    }
  }
  for (int k = first; k < kCells; k += kStride) counts[k] = 0u;
  if (fb_count && first < 2) fb_count[first] = 0u;
  // from the last thread down: the first workgroups may have more points
  const int last = kStride - 1 - first;
  for (int k = last; k < n_constants(n_candidates); k += kStride)
    search_constants(c, n_candidates, step0, lstep0, k);
  for (int k = last; k < V; k += kStride) camera_record(cams, k, cam64);
  block_box(v);
  if (threadIdx.x == 0)
    for (int a = 0; a < 6; ++a) boxes[6 * blockIdx.x + a] = v[a];
}

__device__ __forceinline__ uint32_t spread3(uint32_t x) {
  // 6-bit x -> bits at positions 0, 3, 6, ...
  uint32_t r = 0;
  for (int b = 0; b < kCellBits; ++b) r |= ((x >> b) & 1u) << (3 * b);
  return r;
}

// The count's old value is the point's rank within its cell, so that the
// scatter is a plain write (with a second atomic there: count and scatter 30 +
// 34 us for 500,000 points, now 31 + 8).
__global__ __launch_bounds__(256) void k_cell_count(const float* __restrict__ pts,
                                                    int64_t n, const int* __restrict__ boxes,
                                                    uint32_t* __restrict__ key,
                                                    uint32_t* __restrict__ rank,
                                                    uint32_t* __restrict__ counts) {
  static_assert(kSetupBlocks == 256, "one part of the box per thread");
  int box[6];
  for (int a = 0; a < 6; ++a) box[a] = boxes[6 * threadIdx.x + a];
  block_box(box);
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t q[3];
  for (int a = 0; a < 3; ++a) {
    float lo = ordered_to_float(box[a]), hi = ordered_to_float(box[3 + a]);
    float f = pts[3 * i + a];
    float ext = hi - lo;
    float s = ext > 0.0f ? (f - lo) / ext : 0.0f;
    int c = (int)(s * (float)(1 << kCellBits));
    c = (f == f) ? c : 0;
    q[a] = (uint32_t)min(max(c, 0), (1 << kCellBits) - 1);
  }
  uint32_t k = spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
  key[i] = k;
  rank[i] = atomicAdd(&counts[k], 1u);
}

// Exclusive scan of the kCells counts in two passes: k_cell_block_sums
// reduces each run of 1024 cells; k_cell_scan scans those sums and then its
// own run, writing the cell start offsets into `cursor`.  Both read coalesced.
constexpr int kScanRun = 1024;
constexpr int kScanRuns = kCells / kScanRun;  // 256

__device__ __forceinline__ uint32_t block_incl_scan(uint32_t v, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  if (w == 0) {
    uint32_t s = lane < nw ? wsum[lane] : 0u;
    for (int off = 1; off < 16; off <<= 1) {
      uint32_t o = __shfl_up(s, off, 64);
      if (lane >= off) s += o;
    }
    if (lane < nw) wsum[lane] = s;
  }
  __syncthreads();
  return v + (w > 0 ? wsum[w - 1] : 0u);
}

__global__ __launch_bounds__(1024) void k_cell_block_sums(const uint32_t* __restrict__ counts,
                                                          uint32_t* __restrict__ sums) {
  __shared__ uint32_t wsum[16];
  uint32_t v = counts[blockIdx.x * kScanRun + threadIdx.x];
  uint32_t incl = block_incl_scan(v, wsum);
  if (threadIdx.x == kScanRun - 1) sums[blockIdx.x] = incl;
}

__global__ __launch_bounds__(1024) void k_cell_scan(const uint32_t* __restrict__ counts,
                                                    const uint32_t* __restrict__ sums,
                                                    uint32_t* __restrict__ cursor) {
  __shared__ uint32_t wsum[16];
  __shared__ uint32_t base;
  // prefix of the run sums before this block (kScanRuns <= 1024)
  uint32_t s = threadIdx.x < (unsigned)blockIdx.x ? sums[threadIdx.x] : 0u;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) b += wsum[k];
    base = b;
  }
  __syncthreads();
  const uint32_t b = base;
  __syncthreads();
  uint32_t v = counts[blockIdx.x * kScanRun + threadIdx.x];
  uint32_t incl = block_incl_scan(v, wsum);
  cursor[blockIdx.x * kScanRun + threadIdx.x] = b + incl - v;
}

__global__ __launch_bounds__(256) void k_cell_scatter(const uint32_t* __restrict__ key,
                                                      const uint32_t* __restrict__ rank,
                                                      int64_t n,
                                                      const uint32_t* __restrict__ cursor,
                                                      uint32_t* __restrict__ perm) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  perm[cursor[key[i]] + rank[i]] = (uint32_t)i;
}

hipError_t launch_setup(const float* pts, int64_t n, TileWork w, uint32_t* fb_count,
                        const ConstsDev& c, int n_candidates, double step0, double lstep0,
                        const float* cams, int V, double* cam64, hipStream_t st) {
  // the parts of the box in the cursors' place: they are read before the scan
  static_assert(6 * kSetupBlocks <= kCells, "");
  hipLaunchKernelGGL(k_setup, dim3(kSetupBlocks), dim3(256), 0, st, pts, n, (int*)w.cursor,
                     w.counts, fb_count, c, n_candidates, step0, lstep0, cams, V, cam64);
  return hipGetLastError();
}

// After launch_setup.
hipError_t launch_tiling(const float* pts, int64_t n, TileWork w, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int bs = 256;
  const int64_t nb = (n + bs - 1) / bs;
  hipLaunchKernelGGL(k_cell_count, dim3((unsigned)nb), dim3(bs), 0, st, pts, n,
                     (const int*)w.cursor, w.key, w.rank, w.counts);
  hipLaunchKernelGGL(k_cell_block_sums, dim3(kScanRuns), dim3(kScanRun), 0, st, w.counts,
                     w.sums);
  hipLaunchKernelGGL(k_cell_scan, dim3(kScanRuns), dim3(kScanRun), 0, st, w.counts, w.sums,
                     w.cursor);
  hipLaunchKernelGGL(k_cell_scatter, dim3((unsigned)nb), dim3(bs), 0, st, w.key, w.rank, n,
                     w.cursor, w.perm);
  return hipGetLastError();
}

// Exclusive scan in place of the n run sums (one block; each thread scans
// a chunk of at most kMaxRunsPerThread consecutive sums).
constexpr int kMaxRunsPerThread = 16;
__global__ __launch_bounds__(1024) void k_run_scan(uint32_t* __restrict__ sums, int n) {
  __shared__ uint32_t wsum[16];
  const int per = (n + kScanRun - 1) / kScanRun;
  const int r0 = threadIdx.x * per;
  uint32_t loc = 0;
  for (int k = 0; k < per; ++k)
    if (r0 + k < n) loc += sums[r0 + k];
  uint32_t run = block_incl_scan(loc, wsum) - loc;
  for (int k = 0; k < per; ++k)
    if (r0 + k < n) {
      const uint32_t v = sums[r0 + k];
      sums[r0 + k] = run;
      run += v;
    }
}

// Run r's cell starts: its exclusive prefix (sums[r]) plus the scan within
// the run.
__global__ __launch_bounds__(1024) void k_cell_scan_from(const uint32_t* __restrict__ counts,
                                                         const uint32_t* __restrict__ sums,
                                                         uint32_t* __restrict__ cursor) {
  __shared__ uint32_t wsum[16];
  const uint32_t b = sums[blockIdx.x];
  const uint32_t v = counts[(size_t)blockIdx.x * kScanRun + threadIdx.x];
  const uint32_t incl = block_incl_scan(v, wsum);
  cursor[(size_t)blockIdx.x * kScanRun + threadIdx.x] = b + incl - v;
}

// Exclusive scan of n_runs x 1024 counts (n_runs <= 16384) into cursor, in
// three passes: run sums, their scan, the runs; `sums` (n_runs entries)
// ends up holding each run's exclusive prefix.
hipError_t launch_scan_runs(const uint32_t* counts, int n_runs, uint32_t* sums, uint32_t* cursor,
                            hipStream_t st) {
  if (n_runs < 1 || n_runs > kScanRun * kMaxRunsPerThread) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cell_block_sums, dim3(n_runs), dim3(kScanRun), 0, st, counts, sums);
  hipLaunchKernelGGL(k_run_scan, dim3(1), dim3(kScanRun), 0, st, sums, n_runs);
  hipLaunchKernelGGL(k_cell_scan_from, dim3(n_runs), dim3(kScanRun), 0, st, counts, sums,
                     cursor);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t nb = (n + 255) / 256;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256), 0, st, p,
                     n, v);
  return hipGetLastError();
}

int tile_cells() { return kCells; }

}  // namespace fd
