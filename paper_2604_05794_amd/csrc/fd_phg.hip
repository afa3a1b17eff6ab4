// fd_phg.hip -- parallel hair growing on gfx950: guide strands and segments
// traced through the occupancy / orientation volume with deferred occupancy
// (Sec. 3.2.1), and segment connection by the test of Eq. 13 (Sec. 3.2.2).
// The rules are documented with fd_grow_strands and fd_link_segments in
// fusedir.h.
//
// Growing: a batch of strands reads the crossing counts as the earlier batches
// left them, one wave per strand (k_grow) or, in large batches, one lane for the
// first steps and either for the rest (k_grow_first, k_grow_rest); the end of
// its launches is the batch barrier, after which k_cross adds every step of the
// batch to the count of the voxel it read (integer atomics, so the counts do
// not depend on the order of the additions).  Each step is a
// voxel lookup (count, coherence, crossings, orientation) and binary32
// arithmetic written as fused multiply-adds in a fixed order: a trace is a
// deterministic function of its inputs.
//
// Linking: the pieces that accept a predecessor are bucketed by the cell of
// their start point (cells a little larger than d_max, hashed into 2^20
// buckets, counting sort with the library's two-level scan); each piece end
// scans the 27 cells around its own and proposes its nearest compatible
// start (then the lowest index); each start keeps its nearest proposer
// through a 64-bit atomic minimum of (squared distance bits, proposer).
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

constexpr int kBucketBits = 20;
constexpr uint32_t kBuckets = 1u << kBucketBits;
constexpr uint32_t kNoBucket = 0xffffffffu;

struct GrowDev {
  GridDev g;
  const uint32_t* occ;
  const float* dir;
  const float* coh;
  float step;
  int32_t max_steps;
  float min_coh;
  float bend_cos;
  uint32_t cap;  // 0: none
  int32_t mode;
  float centre[3];
};

__device__ __forceinline__ float dot3(const float* a, const float* b) {
  return __builtin_fmaf(a[2], b[2], __builtin_fmaf(a[1], b[1], a[0] * b[0]));
}

// ---- growing, one lane per strand ------------------------------------------------
// Each step is four loads issued together, whose latency the other strands of
// the SIMD hide, where there are enough of them.
//
// A batch of many seeds is traced in two launches, the first kFirstSteps steps
// and the rest (k_grow_rest).  Between them, and until k_cross has counted it, a
// trace that goes on after the first has -n in n_verts; its state is its last
// vertex and last_dir.
constexpr int kFirstSteps = 32;

__device__ __forceinline__ void grow_resume(const GrowDev& d, int32_t i, const float* out,
                                            const float* last_dir, float* x, float* r) {
  const float sg = d.mode == FD_SEED_TOWARDS ? -1.0f : 1.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x[a] = out[3 * kFirstSteps + a];
    r[a] = sg * last_dir[3 * (size_t)i + a];
  }
}

// Strand i by a lane: steps up to `last`, from the seed or from the first
// launch's end.
__device__ __forceinline__ void grow_lane(
    const GrowDev& d, int32_t i, bool rest, int last, const float* __restrict__ seeds,
    const float* __restrict__ seed_dirs, const uint32_t* __restrict__ crossings,
    float* __restrict__ verts, int32_t* __restrict__ n_verts, float* __restrict__ last_dir) {
  float* out = verts + (size_t)i * (size_t)(d.max_steps + 1) * 3;
  float x[3], r[3];
  int n = 1;
  if (rest) {
    n = 1 + kFirstSteps;
    grow_resume(d, i, out, last_dir, x, r);
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = out[a] = seeds[3 * (size_t)i + a];
      r[a] = 0.0f;
    }
    if (d.mode == FD_SEED_GIVEN) {
#pragma unroll
      for (int a = 0; a < 3; ++a) r[a] = seed_dirs[3 * (size_t)i + a];
    } else {
      const int64_t v = voxel_index(d.g, x[0], x[1], x[2]);
      if (v >= 0) {
        const float t[3] = {d.dir[3 * v], d.dir[3 * v + 1], d.dir[3 * v + 2]};
        const float off[3] = {x[0] - d.centre[0], x[1] - d.centre[1], x[2] - d.centre[2]};
        const bool away = !(dot3(t, off) < 0.0f);
        const float sg = (away == (d.mode == FD_SEED_AWAY)) ? 1.0f : -1.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) r[a] = sg * t[a];
      }
    }
  }
  int k = n;
  for (; k <= last; ++k) {
    const int64_t v = voxel_index(d.g, x[0], x[1], x[2]);
    if (v < 0) break;
    const uint32_t o = d.occ[v];
    const float c0 = d.coh[v];
    const uint32_t cr = crossings[v];
    float t[3] = {d.dir[3 * v], d.dir[3 * v + 1], d.dir[3 * v + 2]};
    if (o == 0u || !(c0 >= d.min_coh)) break;
    if (d.cap > 0u && cr >= d.cap) break;
    if (t[0] == 0.0f && t[1] == 0.0f && t[2] == 0.0f) break;
    float c = dot3(t, r);
    if (c < 0.0f) {
      t[0] = -t[0];
      t[1] = -t[1];
      t[2] = -t[2];
      c = -c;
    }
    if (k > 1 && c < d.bend_cos) break;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = __builtin_fmaf(d.step, t[a], x[a]);
      r[a] = t[a];
      out[3 * n + a] = x[a];
    }
    ++n;
  }
  n_verts[i] = rest || (k > last && last < d.max_steps) ? -n : n;
  const float sg = d.mode == FD_SEED_TOWARDS ? -1.0f : 1.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) last_dir[3 * (size_t)i + a] = n > 1 ? sg * r[a] : 0.0f;
}

// ---- growing, one wave per strand ------------------------------------------------
// What bounds a trace is its chain of dependent lookups: a step reads the
// voxel of the point that the previous step produced, close to a microsecond
// from memory, up to max_steps times.  A wave takes one strand: its lanes
// all compute the same steps, so every branch is a scalar one, and together
// they load a block of 4 x 4 x 4 voxels ahead of the point at once, one
// each.  The steps inside the block read LDS, and the block that the strand
// would enter next if it went on straight is loaded meanwhile, so that
// memory is waited for only where the strand turned away from it.  A voxel
// is kept as its orientation, or 0 where a trace stops (empty, incoherent,
// at the cap, no orientation).  Steps that stay inside a voxel keep its
// orientation and need no lookup.  The voxel rule's division is replaced by
// a multiplication unless the quotient is so close to a whole number that
// the two could differ.  The seed's own voxel is read by itself first: most
// interior seeds stop there.  Vertices are kept one per lane and stored 64
// at a time.  4096 guide strands through a 3 mm volume (mean 22 steps, longest
// 200) take 76 us, 243 us with one lane per strand (1.15 us a step).  Measured
// between the two: 16 lanes a strand with 4 x 2 x 2 blocks 92 us, 64 lanes under
// divergent branches 88 us.  What is left is the wait where a
// strand leaves its block sideways and, early in a batch, the cache lines
// that its blocks touch.

// floor(s / h) per axis by the rule of voxel_index (binary32, IEEE division),
// false outside.  inv_h = 1 / h, or 0 where that is not a normal number: the
// product then always takes the exact path.  s * inv_h is within 3 x 2^-24 of
// the rounded quotient relatively, so away from whole numbers both have the
// same floor and lie on the same side of 0 and dims.
__device__ __forceinline__ bool voxel_near(const GridDev& g, float inv_h, const float* x,
                                           int32_t* ix) {
  float q[3];
  bool sure = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    q[a] = (x[a] - g.o[a]) * inv_h;
    sure = sure && fabsf(q[a] - rintf(q[a])) > __builtin_fmaf(5e-7f, fabsf(q[a]), 1e-30f);
  }
  if (!sure) {
#pragma unroll
    for (int a = 0; a < 3; ++a) q[a] = (x[a] - g.o[a]) / g.h;
  }
  bool in = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    in = in && q[a] >= 0.0f && q[a] < (float)g.dims[a];
    ix[a] = (int32_t)q[a];
  }
  return in;
}

// What a trace reads of a voxel, and its orientation as the trace sees it:
// 0 where it stops.
struct GrowVoxel {
  uint32_t occ, cross;
  float coh, dx, dy, dz;
};

__device__ __forceinline__ GrowVoxel grow_load(const GrowDev& d, const uint32_t* crossings,
                                               int32_t ix, int32_t iy, int32_t iz) {
  const int64_t v = ((int64_t)iz * d.g.dims[1] + iy) * d.g.dims[0] + ix;
  GrowVoxel g;
  g.occ = d.occ[v];
  g.coh = d.coh[v];
  g.cross = d.cap > 0u ? crossings[v] : 0u;
  g.dx = d.dir[3 * v];
  g.dy = d.dir[3 * v + 1];
  g.dz = d.dir[3 * v + 2];
  return g;
}

__device__ __forceinline__ float4 grow_dir(const GrowDev& d, const GrowVoxel& g) {
  const bool stop = g.occ == 0u || !(g.coh >= d.min_coh) || (d.cap > 0u && g.cross >= d.cap);
  return stop ? make_float4(0.0f, 0.0f, 0.0f, 0.0f) : make_float4(g.dx, g.dy, g.dz, 0.0f);
}

// A block of 4 x 4 x 4 voxels by its low corner, placed so that it holds
// the voxel ix and reaches ahead of it along r.
struct GrowBlock {
  int32_t org[3];

  __device__ __forceinline__ bool holds(const int32_t* ix) const {
    return (uint32_t)(ix[0] - org[0]) < 4u && (uint32_t)(ix[1] - org[1]) < 4u &&
           (uint32_t)(ix[2] - org[2]) < 4u;
  }
  __device__ __forceinline__ void place(const int32_t* ix, const float* r) {
#pragma unroll
    for (int a = 0; a < 3; ++a) org[a] = ix[a] - (r[a] > 0.3f ? 0 : (r[a] < -0.3f ? 3 : 1));
  }
  // the lane's voxel; beyond the grid's faces the nearest one inside (never
  // looked up)
  __device__ __forceinline__ GrowVoxel load(const GrowDev& d, const uint32_t* crossings,
                                            int lane) const {
    return grow_load(d, crossings, min(max(org[0] + (lane & 3), 0), d.g.dims[0] - 1),
                     min(max(org[1] + ((lane >> 2) & 3), 0), d.g.dims[1] - 1),
                     min(max(org[2] + (lane >> 4), 0), d.g.dims[2] - 1));
  }
  __device__ __forceinline__ int slot(const int32_t* ix) const {
    return ((((ix[2] - org[2]) << 2) + (ix[1] - org[1])) << 2) + (ix[0] - org[0]);
  }
};

// A condition that is the same in every lane of the wave, as a scalar.
__device__ __forceinline__ bool wave_cond(bool c) { return __ballot(c) != 0ull; }

// Strand i by the wave, from the seed or from the first launch's end; blk: its
// 64 places in LDS.
__device__ __forceinline__ void grow_wave(
    const GrowDev& d, float inv_h, int32_t i, bool rest, int lane, float4* blk,
    const float* __restrict__ seeds, const float* __restrict__ seed_dirs, const uint32_t* __restrict__ crossings,
    float* __restrict__ verts, int32_t* __restrict__ n_verts, float* __restrict__ last_dir) {
  float* out = verts + (size_t)i * (size_t)(d.max_steps + 1) * 3;
  float x[3], r[3] = {0.0f, 0.0f, 0.0f};
  float keep[3];  // the lane's vertex n with n % 64 == lane
  int n = 1;
  if (rest) {
    n = 1 + kFirstSteps;
    grow_resume(d, i, out, last_dir, x, r);
#pragma unroll
    for (int a = 0; a < 3; ++a) keep[a] = out[3 * min(lane, kFirstSteps) + a];
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a) keep[a] = x[a] = seeds[3 * (size_t)i + a];
  }
  GrowBlock here, next;                // the block in LDS, the one being loaded into pre
  GrowVoxel pre{};
  bool pending = false;
  int32_t ix[3];
  float tv[3] = {0.0f, 0.0f, 0.0f};
  if (wave_cond(voxel_near(d.g, inv_h, x, ix))) {
    const GrowVoxel g = grow_load(d, crossings, ix[0], ix[1], ix[2]);
    const float4 t4 = grow_dir(d, g);
    tv[0] = t4.x;
    tv[1] = t4.y;
    tv[2] = t4.z;
    if (!rest && d.mode != FD_SEED_GIVEN) {
      const float t[3] = {g.dx, g.dy, g.dz};
      const float off[3] = {x[0] - d.centre[0], x[1] - d.centre[1], x[2] - d.centre[2]};
      const bool away = !(dot3(t, off) < 0.0f);
      const float sg = (away == (d.mode == FD_SEED_AWAY)) ? 1.0f : -1.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a) r[a] = sg * t[a];
    }
  }
  if (!rest && d.mode == FD_SEED_GIVEN) {
#pragma unroll
    for (int a = 0; a < 3; ++a) r[a] = seed_dirs[3 * (size_t)i + a];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) here.org[a] = next.org[a] = INT32_MIN / 2;  // holds nothing

  // the vertex that r leads to from x
  auto push = [&]() {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      x[a] = __builtin_fmaf(d.step, r[a], x[a]);
      keep[a] = (n & 63) == lane ? x[a] : keep[a];
    }
    ++n;
    if ((n & 63) == 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) out[3 * (n - 64 + lane) + a] = keep[a];
    }
  };
  // tv: the orientation of x's voxel ix (0: the trace stops)
  while (wave_cond(tv[0] != 0.0f || tv[1] != 0.0f || tv[2] != 0.0f)) {
    const float c = dot3(tv, r);
    const float sg = c < 0.0f ? -1.0f : 1.0f;
    if (n > 1 && wave_cond(fabsf(c) < d.bend_cos)) break;
#pragma unroll
    for (int a = 0; a < 3; ++a) r[a] = sg * tv[a];
    push();
    // The steps that stay well inside this voxel: its orientation agrees
    // with itself, so the direction does not change and the bend test is the
    // same for all of them.  "Well inside" leaves out the rounding of the
    // voxel rule (three roundings of numbers up to (ix + 1) h, under 2e-7 of
    // them).
    const float rr = dot3(r, r);  // 0: underflow, where the agreement has no sign
    float mid[3], half[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      mid[a] = ((float)ix[a] + 0.5f) * d.g.h;
      half[a] = inv_h > 0.0f && rr > 0.0f ? (0.5f - 1e-6f * (float)(ix[a] + 1)) * d.g.h : -1.0f;
    }
    const bool bent = wave_cond(rr < d.bend_cos);
    bool stop = false;
    while (n <= d.max_steps && wave_cond(fabsf((x[0] - d.g.o[0]) - mid[0]) < half[0] &&
                                         fabsf((x[1] - d.g.o[1]) - mid[1]) < half[1] &&
                                         fabsf((x[2] - d.g.o[2]) - mid[2]) < half[2])) {
      stop = bent;
      if (bent) break;
      push();
    }
    if (stop || n > d.max_steps) break;
    if (!wave_cond(voxel_near(d.g, inv_h, x, ix))) break;
    if (!wave_cond(here.holds(ix))) {
      if (!(pending && wave_cond(next.holds(ix)))) {
        next.place(ix, r);
        pre = next.load(d, crossings, lane);
      }
      here = next;
      blk[lane] = grow_dir(d, pre);
      // written and read by the lanes of one wave, whose LDS operations
      // complete in order: only the compiler has to keep them in order
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // the voxel where the straight line along r leaves this block
      float far = INFINITY;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float face = d.g.o[a] + d.g.h * (float)(here.org[a] + (r[a] < 0.0f ? 0 : 4));
        const float t = (face - x[a]) * __builtin_amdgcn_rcpf(r[a]);
        far = r[a] != 0.0f ? fminf(far, t) : far;
      }
      far = fmaxf(far, 0.0f) + 0.25f * d.g.h;
      int32_t px[3];
      bool in = true;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float q = (__builtin_fmaf(far, r[a], x[a]) - d.g.o[a]) * inv_h;
        in = in && q >= 0.0f && q < (float)d.g.dims[a];
        px[a] = (int32_t)q;
      }
      pending = wave_cond(in);
      if (pending) {
        next.place(px, r);
        pre = next.load(d, crossings, lane);
      }
    }
    const float4 t4 = blk[here.slot(ix)];
    tv[0] = t4.x;
    tv[1] = t4.y;
    tv[2] = t4.z;
  }
  if (lane < (n & 63)) {
#pragma unroll
    for (int a = 0; a < 3; ++a) out[3 * (n - (n & 63) + lane) + a] = keep[a];
  }
  if (lane == 0) {
    n_verts[i] = rest ? -n : n;
    const float sg = d.mode == FD_SEED_TOWARDS ? -1.0f : 1.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) last_dir[3 * (size_t)i + a] = n > 1 ? sg * r[a] : 0.0f;
  }
}

__global__ __launch_bounds__(256) void k_grow(
    GrowDev d, float inv_h, const float* __restrict__ seeds, const float* __restrict__ seed_dirs,
    int32_t b0, int32_t b1, const uint32_t* __restrict__ crossings, float* __restrict__ verts,
    int32_t* __restrict__ n_verts, float* __restrict__ last_dir) {
  __shared__ float4 blocks[4][64];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int32_t i = b0 + (int32_t)(blockIdx.x * 4u) + w;
  if (i >= b1) return;  // wave-uniform
  grow_wave(d, inv_h, i, false, (int)(threadIdx.x & 63u), blocks[w], seeds, seed_dirs, crossings,
            verts, n_verts, last_dir);
}

// Batches above kFewSeeds, as many waves as the card holds at once (256 compute
// units of 32).  A wave per strand shortens the chain of steps but does 64
// lanes' work for it; in a large batch it pays only for the strands that go far,
// if they are few, and how many do only the volume says: most interior seeds
// stop in their own voxel.  So a lane each takes the first steps of all, and
// k_grow_rest the rest in the form that their number asks for.  A batch, us, a
// lane for all / a wave for all / this:
//   68,000 interior seeds of a hairstyle, 12,000 of which grow  254 / 137 / 132
//   65,536 in a smooth field, 103 steps   448 / 672 / 472; 21 steps  100 / 169 / 100
//   65,536 in a noisy field, bend 45 deg   58 / 126 / 56
//   65,536 in a field a sixth occupied     22 /  33 / 24 (two launches)
//   131,072 in a noisy field, no bend limit, 176 steps  1802 / 4600 / 1804
// First steps of 16: 134 for the interior seeds, and short traces longer (52
// for 30 at 20 steps); 8: 244; 48: 131.
constexpr int32_t kFewSeeds = 8192;
// Above kFewSeeds, so that a sample of 256 does not take 8000 for more: 7354 of
// 80,000 seeds, as waves 100 us, as lanes 160.  12,000 that take 176 steps each
// would be 430 and 330.
constexpr int32_t kFewFar = 12288;
constexpr int kRestBlocks = kFewSeeds / 4;

__global__ __launch_bounds__(256) void k_grow_first(
    GrowDev d, int last, const float* __restrict__ seeds, const float* __restrict__ seed_dirs,
    int32_t b0, int32_t b1, const uint32_t* __restrict__ crossings, float* __restrict__ verts,
    int32_t* __restrict__ n_verts, float* __restrict__ last_dir) {
  const int64_t i = b0 + (int64_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < b1)
    grow_lane(d, (int32_t)i, false, last, seeds, seed_dirs, crossings, verts, n_verts, last_dir);
}

// The traces that go on: a wave each where they are few, a lane each where there
// are enough to hide their latency.  Every workgroup looks at the same places of
// n_verts, spread over the batch, and so takes the same form (the signs do not
// change in here).  The seeds of a workgroup lie far apart, since those that grow
// lie together; its waves take their traces in turn.
__global__ __launch_bounds__(256, 8) void k_grow_rest(
    GrowDev d, float inv_h, const float* __restrict__ seeds, const float* __restrict__ seed_dirs,
    int32_t b0, int32_t b1, const uint32_t* __restrict__ crossings, float* __restrict__ verts,
    int32_t* __restrict__ n_verts, float* __restrict__ last_dir) {
  __shared__ float4 blocks[4][64];
  __shared__ uint32_t part[4], list[256], listed;
  const int lane = (int)(threadIdx.x & 63u);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t n = (uint32_t)(b1 - b0);
  // multiples of the golden ratio, modulo 1, are spread evenly
  const uint32_t at = (uint32_t)(((uint64_t)(threadIdx.x * 0x9e3779b9u) * n) >> 32);
  const uint32_t c = (uint32_t)__builtin_popcountll(__ballot(n_verts[b0 + (int32_t)at] < 0));
  if (lane == 0) part[w] = c;
  __syncthreads();
  const uint32_t on = part[0] + part[1] + part[2] + part[3];  // of 256
  if ((uint64_t)on * n > (uint64_t)kFewFar * 256u) {
    for (uint32_t k = blockIdx.x * 256u + threadIdx.x; k < n; k += gridDim.x * 256u)
      if (n_verts[b0 + (int32_t)k] < 0)
        grow_lane(d, b0 + (int32_t)k, true, d.max_steps, seeds, seed_dirs, crossings, verts,
                  n_verts, last_dir);
    return;
  }
  for (uint32_t r = 0; r * gridDim.x < n; r += 256u) {  // the same for the whole workgroup
    __syncthreads();
    if (threadIdx.x == 0) listed = 0u;
    __syncthreads();
    const uint32_t k = blockIdx.x + (r + threadIdx.x) * gridDim.x;
    if (k < n && n_verts[b0 + (int32_t)k] < 0) list[atomicAdd(&listed, 1u)] = k;
    __syncthreads();
    const int m = __builtin_amdgcn_readfirstlane((int)listed);
    // In turn, by a scalar counter.  Not from a queue that lane 0 takes from: the
    // compiler joins that condition with the one at the end of grow_wave, and
    // the other lanes then go round without lane 0, for ever.
    for (int j = w; j < m; j += 4) {
      const int32_t i = b0 + __builtin_amdgcn_readfirstlane((int)list[j]);
      grow_wave(d, inv_h, i, true, lane, blocks[w], seeds, seed_dirs, crossings, verts, n_verts,
                last_dir);
    }
  }
}

// The deferred occupancy update of one batch: every step counts once in the
// voxel it read (the voxel of the vertex it started from).  One wave per
// strand, its lanes over the steps: the vertex reads coalesce and the
// atomics of a strand issue together.
__global__ __launch_bounds__(256) void k_cross(GridDev g, const float* __restrict__ verts,
                                               int32_t* __restrict__ n_verts, int32_t b0,
                                               int32_t b1, int32_t stride,
                                               uint32_t* __restrict__ crossings) {
  const int lane = (int)(threadIdx.x & 63u);
  const int32_t i = b0 + (int32_t)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (i >= b1) return;  // wave-uniform
  const float* p = verts + (size_t)i * (size_t)stride * 3;
  int32_t n = n_verts[i];
  if (n < 0) {  // traced in two launches
    n = -n;
    if (lane == 0) n_verts[i] = n;
  }
  for (int k = lane; k + 1 < n; k += 64) {
    const int64_t v = voxel_index(g, p[3 * k], p[3 * k + 1], p[3 * k + 2]);
    if (v >= 0) atomicAdd(&crossings[v], 1u);
  }
}

// ---- linking -----------------------------------------------------------------

__device__ __forceinline__ int32_t cell_of(float x, float cell) {
  const float q = floorf(x / cell);
  return (int32_t)fminf(fmaxf(q, -1073741824.0f), 1073741824.0f);
}

__device__ __forceinline__ uint32_t bucket_of(int32_t cx, int32_t cy, int32_t cz) {
  return (((uint32_t)cx * 73856093u) ^ ((uint32_t)cy * 19349663u) ^ ((uint32_t)cz * 83492791u)) &
         (kBuckets - 1u);
}

__global__ __launch_bounds__(256) void k_link_hash(const float* __restrict__ starts,
                                                   const uint8_t* __restrict__ flags, int32_t n,
                                                   float cell, uint32_t* __restrict__ counts,
                                                   uint32_t* __restrict__ bucket_rank) {
  const int32_t j = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (j >= n) return;
  if ((flags[j] & 3u) != 3u) {
    bucket_rank[2 * (size_t)j] = kNoBucket;
    return;
  }
  const uint32_t b = bucket_of(cell_of(starts[3 * (size_t)j], cell),
                               cell_of(starts[3 * (size_t)j + 1], cell),
                               cell_of(starts[3 * (size_t)j + 2], cell));
  bucket_rank[2 * (size_t)j] = b;
  bucket_rank[2 * (size_t)j + 1] = atomicAdd(&counts[b], 1u);
}

__global__ __launch_bounds__(256) void k_link_place(const uint32_t* __restrict__ bucket_rank,
                                                    int32_t n, const uint32_t* __restrict__ cursor,
                                                    uint32_t* __restrict__ perm) {
  const int32_t j = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (j >= n) return;
  const uint32_t b = bucket_rank[2 * (size_t)j];
  if (b == kNoBucket) return;
  perm[cursor[b] + bucket_rank[2 * (size_t)j + 1]] = (uint32_t)j;
}

__global__ __launch_bounds__(256) void k_link_propose(
    const float* __restrict__ starts, const float* __restrict__ start_dirs,
    const float* __restrict__ ends, const float* __restrict__ end_dirs,
    const uint8_t* __restrict__ flags, int32_t n, float d2max, float min_cos, float cell,
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ cursor,
    const uint32_t* __restrict__ perm, int32_t* __restrict__ succ,
    unsigned long long* __restrict__ key, unsigned long long* __restrict__ best) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= n) return;
  succ[i] = -1;
  key[i] = ~0ull;
  if (!(flags[i] & 1u)) return;
  const float e[3] = {ends[3 * (size_t)i], ends[3 * (size_t)i + 1], ends[3 * (size_t)i + 2]};
  const float u[3] = {end_dirs[3 * (size_t)i], end_dirs[3 * (size_t)i + 1],
                      end_dirs[3 * (size_t)i + 2]};
  const int32_t cx = cell_of(e[0], cell), cy = cell_of(e[1], cell), cz = cell_of(e[2], cell);
  int32_t bj = -1;
  float bd = 0.0f;
  for (int dz = -1; dz <= 1; ++dz)
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        const uint32_t b = bucket_of(cx + dx, cy + dy, cz + dz);
        const uint32_t s0 = cursor[b], s1 = s0 + counts[b];
        for (uint32_t s = s0; s < s1; ++s) {
          const int32_t j = (int32_t)perm[s];
          if (j == i) continue;
          const float* sj = starts + 3 * (size_t)j;
          const float ddx = e[0] - sj[0], ddy = e[1] - sj[1], ddz = e[2] - sj[2];
          const float d2 = __builtin_fmaf(ddz, ddz, __builtin_fmaf(ddy, ddy, ddx * ddx));
          if (!(d2 < d2max)) continue;
          if (!(dot3(u, start_dirs + 3 * (size_t)j) > min_cos)) continue;
          if (bj < 0 || d2 < bd || (d2 == bd && j < bj)) {
            bj = j;
            bd = d2;
          }
        }
      }
  if (bj < 0) return;
  const unsigned long long k = ((unsigned long long)__float_as_uint(bd) << 32) | (uint32_t)i;
  succ[i] = bj;
  key[i] = k;
  atomicMin(&best[bj], k);
}

__global__ __launch_bounds__(256) void k_link_accept(int32_t n,
                                                     const unsigned long long* __restrict__ key,
                                                     const unsigned long long* __restrict__ best,
                                                     int32_t* __restrict__ succ) {
  const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= n) return;
  const int32_t j = succ[i];
  if (j >= 0 && best[j] != key[i]) succ[i] = -1;
}


// ---- strands from linked pieces ------------------------------------------------
// Piece g < n_guide is guide trace g; piece n_guide + s is segment s (its
// backward trace reversed without the seed, then its forward trace).  A
// chain ends at -1, at a guide piece, or after n_guide + n_seg hops.

struct PiecesDev {
  const int32_t* gn;
  const int32_t* fn;
  const int32_t* bn;
  const int32_t* succ;
  int32_t n_guide, n_seg;
};

__global__ __launch_bounds__(256) void k_strand_len(PiecesDev P, int64_t* __restrict__ len,
                                                    int32_t* __restrict__ pieces) {
  const int32_t g = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (g >= P.n_guide) return;
  int64_t L = P.gn[g];
  int32_t np = 1;
  int32_t j = P.succ[g];
  for (int32_t hop = 0; j >= P.n_guide && j < P.n_guide + P.n_seg && hop < P.n_guide + P.n_seg;
       ++hop) {
    const int32_t sg = j - P.n_guide;
    L += (int64_t)(P.bn[sg] - 1) + P.fn[sg];
    ++np;
    j = P.succ[j];
  }
  len[g] = L;
  if (pieces) pieces[g] = np;
}

// Inclusive scan of one value per thread across a block of 1024 threads:
// within each wave by shuffles, then over the 16 wave totals.  Every thread
// of the block calls it once.
__device__ __forceinline__ int64_t block_incl_scan(int64_t x, int64_t* wsum) {
  const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  if (wv == 0) {
    int64_t y = lane < 1024 / 64 ? wsum[lane] : 0;
    for (int o = 1; o < 1024 / 64; o <<= 1) {
      const int64_t z = __shfl_up(y, o, 64);
      if (lane >= o) y += z;
    }
    if (lane < 1024 / 64) wsum[lane] = y;
  }
  __syncthreads();
  return x + (wv > 0 ? wsum[wv - 1] : 0);
}

// Exclusive scan of n entries into off (n + 1 entries, off[n] = the total)
// in one block: thread t owns a contiguous run, summed in order, and writes
// it after the block scan of the run sums.  Used on the per-block sums of
// the lengths (and on an empty list).
__global__ __launch_bounds__(1024) void k_len_scan(const int64_t* __restrict__ len, int32_t n,
                                                   int64_t* __restrict__ off) {
  __shared__ int64_t wsum[1024 / 64];
  const int t = (int)threadIdx.x;
  const int32_t per = (n + 1023) / 1024;
  const int32_t a = t * per, b = min(n, a + per);
  int64_t s = 0;
  for (int32_t i = a; i < b; ++i) s += len[i];
  const int64_t incl = block_incl_scan(s, wsum);
  if (t == 1023) off[n] = incl;
  int64_t acc = incl - s;
  for (int32_t i = a; i < b; ++i) {
    off[i] = acc;
    acc += len[i];
  }
}

// The lengths in blocks of 1024 (coalesced): each block's sum, then, once
// those are scanned, each entry's offset.
__global__ __launch_bounds__(1024) void k_len_bsum(const int64_t* __restrict__ len, int32_t n,
                                                   int64_t* __restrict__ bsum) {
  __shared__ int64_t wsum[1024 / 64];
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  const int64_t incl = block_incl_scan(i < n ? len[i] : 0, wsum);
  if (threadIdx.x == 1023) bsum[blockIdx.x] = incl;
}

__global__ __launch_bounds__(1024) void k_len_apply(const int64_t* __restrict__ len, int32_t n,
                                                    const int64_t* __restrict__ boff,
                                                    int64_t* __restrict__ off) {
  __shared__ int64_t wsum[1024 / 64];
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  const int64_t v = i < n ? len[i] : 0;
  const int64_t incl = block_incl_scan(v, wsum);
  if (i < n) off[i] = boff[blockIdx.x] + incl - v;
  if (blockIdx.x == 0 && threadIdx.x == 0) off[n] = boff[gridDim.x];
}

__global__ __launch_bounds__(256) void k_assemble(PiecesDev P, const float* __restrict__ gv,
                                                  int32_t gs, const float* __restrict__ fv,
                                                  int32_t fs, const float* __restrict__ bv,
                                                  int32_t bs, const int64_t* __restrict__ off,
                                                  int64_t cap, float* __restrict__ out) {
  const int lane = (int)(threadIdx.x & 63u);
  const int32_t g = (int32_t)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (g >= P.n_guide) return;  // wave-uniform
  int64_t pos = off[g];
  auto put = [&](int64_t at, const float* src) {
    if (at < cap) {
      out[3 * at] = src[0];
      out[3 * at + 1] = src[1];
      out[3 * at + 2] = src[2];
    }
  };
  {
    const float* src = gv + (size_t)g * gs * 3;
    const int32_t n = min(max(P.gn[g], 0), gs);  // reads stay inside the trace
    for (int32_t k = lane; k < n; k += 64) put(pos + k, src + 3 * k);
    pos += n;
  }
  int32_t j = P.succ[g];
  for (int32_t hop = 0; j >= P.n_guide && j < P.n_guide + P.n_seg && hop < P.n_guide + P.n_seg;
       ++hop) {
    const int32_t sg = j - P.n_guide;
    const int32_t nb = min(max(P.bn[sg], 1), bs), nf = min(max(P.fn[sg], 0), fs);
    const float* b = bv + (size_t)sg * bs * 3;
    const float* f = fv + (size_t)sg * fs * 3;
    for (int32_t k = lane; k < nb - 1; k += 64) put(pos + k, b + 3 * (nb - 1 - k));
    pos += nb - 1;
    for (int32_t k = lane; k < nf; k += 64) put(pos + k, f + 3 * k);
    pos += nf;
    j = P.succ[j];
  }
}

int check_grid(const fd_volume_grid* grid, const char* fn, GridDev* g) {
  if (!grid) return set_error(FD_E_INVAL, "%s: grid is NULL", fn);
  if (!(grid->voxel > 0.0f) || !std::isfinite(grid->voxel))
    return set_error(FD_E_INVAL, "%s: voxel edge must be finite and > 0", fn);
  for (int a = 0; a < 3; ++a) {
    if (!std::isfinite(grid->origin[a]))
      return set_error(FD_E_INVAL, "%s: grid origin must be finite", fn);
    if (grid->dims[a] < 1 || grid->dims[a] > FD_MAX_VOLUME_DIM)
      return set_error(FD_E_INVAL, "%s: dims must be in [1, %d]", fn, FD_MAX_VOLUME_DIM);
    g->o[a] = grid->origin[a];
    g->dims[a] = grid->dims[a];
  }
  if ((int64_t)grid->dims[0] * grid->dims[1] * grid->dims[2] > FD_MAX_VOLUME_VOXELS)
    return set_error(FD_E_INVAL, "%s: too many voxels", fn);
  g->h = grid->voxel;
  return FD_OK;
}

fd_context* context_for(fd_context* ctx, const char* fn, int* err) {
  int dev = 0;
  if ((*err = check_device(&dev))) return nullptr;
  if (ctx) {
    if (ctx->device != dev) {
      *err = set_error(FD_E_INVAL, "%s: context belongs to device %d", fn, ctx->device);
      return nullptr;
    }
    return ctx;
  }
  return default_context(dev, 0, err);
}

}  // namespace

extern "C" void fd_grow_params_init(fd_grow_params* p) {
  if (!p) return;
  p->step = 1e-3f;
  p->max_steps = 200;
  p->min_coherence = 0.2f;
  p->max_bend_cos = 0.8660254f;  // 30 degrees
  p->voxel_cap = 8;
  p->batch = 4096;
  p->seed_mode = FD_SEED_GIVEN;
  p->centre[0] = p->centre[1] = p->centre[2] = 0.0f;
  p->stream = nullptr;
  p->ctx = nullptr;
}

extern "C" int fd_grow_strands(const fd_volume_grid* grid, const uint32_t* occ, const float* dir,
                               const float* coherence, const float* seeds,
                               const float* seed_dirs, int32_t n_seeds,
                               const fd_grow_params* p, uint32_t* crossings, float* verts,
                               int32_t* n_verts, float* last_dir) {
  const char* fn = "fd_grow_strands";
  int r;
  GrowDev d;
  if ((r = check_grid(grid, fn, &d.g))) return r;
  if (!p) return set_error(FD_E_INVAL, "%s: params is NULL", fn);
  if (!(p->step > 0.0f) || !std::isfinite(p->step))
    return set_error(FD_E_INVAL, "%s: step must be finite and > 0", fn);
  if (p->max_steps < 1 || p->max_steps > FD_MAX_GROW_STEPS)
    return set_error(FD_E_INVAL, "%s: max_steps must be in [1, %d]", fn, FD_MAX_GROW_STEPS);
  if (!std::isfinite(p->min_coherence) || !std::isfinite(p->max_bend_cos))
    return set_error(FD_E_INVAL, "%s: thresholds must be finite", fn);
  if (p->voxel_cap < 0 || p->batch < 1)
    return set_error(FD_E_INVAL, "%s: voxel_cap must be >= 0 and batch >= 1", fn);
  if (p->seed_mode != FD_SEED_GIVEN && p->seed_mode != FD_SEED_AWAY &&
      p->seed_mode != FD_SEED_TOWARDS)
    return set_error(FD_E_INVAL, "%s: unknown seed_mode %d", fn, p->seed_mode);
  for (int a = 0; a < 3; ++a)
    if (!std::isfinite(p->centre[a]))
      return set_error(FD_E_INVAL, "%s: centre must be finite", fn);
  if (n_seeds < 0 || n_seeds > FD_MAX_GROW_SEEDS)
    return set_error(FD_E_INVAL, "%s: n_seeds must be in [0, %d]", fn, FD_MAX_GROW_SEEDS);
  if (!occ || !dir || !coherence || !crossings)
    return set_error(FD_E_INVAL, "%s: null volume or crossings pointer", fn);
  if (n_seeds > 0 && (!seeds || !verts || !n_verts || !last_dir))
    return set_error(FD_E_INVAL, "%s: null seed or output pointer", fn);
  if (n_seeds > 0 && p->seed_mode == FD_SEED_GIVEN && !seed_dirs)
    return set_error(FD_E_INVAL, "%s: FD_SEED_GIVEN needs seed_dirs", fn);
  fd_context* c = context_for(p->ctx, fn, &r);
  if (!c) return r;
  if (n_seeds == 0) return FD_OK;
  d.occ = occ;
  d.dir = dir;
  d.coh = coherence;
  d.step = p->step;
  d.max_steps = p->max_steps;
  d.min_coh = p->min_coherence;
  d.bend_cos = p->max_bend_cos;
  d.cap = (uint32_t)p->voxel_cap;
  d.mode = p->seed_mode;
  for (int a = 0; a < 3; ++a) d.centre[a] = p->centre[a];
  hipStream_t st = (hipStream_t)p->stream;
  hipError_t e;
  float inv_h = 1.0f / d.g.h;
  if (!std::isnormal(inv_h) || !std::isnormal(d.g.h)) inv_h = 0.0f;
  for (int32_t b0 = 0; b0 < n_seeds; b0 += p->batch) {
    const int32_t b1 = n_seeds - b0 > p->batch ? b0 + p->batch : n_seeds;
    {
      StageTimer t(c, FD_STAGE_GROW, st);
      const int64_t m = b1 - b0;
      if (m > kFewSeeds) {
        hipLaunchKernelGGL(k_grow_first, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, d,
                           std::min(kFirstSteps, d.max_steps), seeds, seed_dirs, b0, b1, crossings,
                           verts, n_verts, last_dir);
        if ((e = hipGetLastError()) == hipSuccess && d.max_steps > kFirstSteps)
          hipLaunchKernelGGL(k_grow_rest, dim3((unsigned)std::min<int64_t>(kRestBlocks, (m + 15) / 16)),
                             dim3(256), 0, st, d, inv_h, seeds, seed_dirs, b0, b1, crossings, verts,
                             n_verts, last_dir);
        if (e != hipSuccess) return hip_error(e, "grow");
      } else {
        hipLaunchKernelGGL(k_grow, dim3((unsigned)((b1 - b0 + 3) / 4)), dim3(256), 0, st, d, inv_h,
                           seeds, seed_dirs, b0, b1, crossings, verts, n_verts, last_dir);
      }
      if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "grow");
      t.stop();
    }
    {
      StageTimer t(c, FD_STAGE_GROW_CROSS, st);
      const unsigned nbw = (unsigned)(((int64_t)(b1 - b0) * 64 + 255) / 256);
      hipLaunchKernelGGL(k_cross, dim3(nbw), dim3(256), 0, st, d.g, verts, n_verts, b0, b1,
                         p->max_steps + 1, crossings);
      if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "crossing update");
      t.stop();
    }
  }
  return FD_OK;
}

extern "C" int fd_link_segments(const float* starts, const float* start_dirs, const float* ends,
                                const float* end_dirs, const uint8_t* flags, int32_t n,
                                float max_dist, float min_cos, void* stream, fd_context* ctx,
                                int32_t* succ) {
  const char* fn = "fd_link_segments";
  int r;
  if (n < 0 || n > FD_MAX_LINK_PIECES)
    return set_error(FD_E_INVAL, "%s: n must be in [0, %d]", fn, FD_MAX_LINK_PIECES);
  if (!(max_dist > 0.0f) || !std::isfinite(max_dist) || !std::isfinite(min_cos))
    return set_error(FD_E_INVAL, "%s: max_dist must be finite and > 0, min_cos finite", fn);
  if (n > 0 && (!starts || !start_dirs || !ends || !end_dirs || !flags || !succ))
    return set_error(FD_E_INVAL, "%s: null pointer argument", fn);
  fd_context* c = context_for(ctx, fn, &r);
  if (!c) return r;
  if (n == 0) return FD_OK;
  const size_t un = (size_t)n;
  if ((r = ctx_buffer((void**)&c->link_counts, &c->cap_link_counts, 4 * (size_t)kBuckets,
                      "link buckets")) ||
      (r = ctx_buffer((void**)&c->link_cursor, &c->cap_link_cursor, 4 * (size_t)kBuckets,
                      "link offsets")) ||
      (r = ctx_buffer((void**)&c->link_sums, &c->cap_link_sums, 4 * 1024, "link run sums")) ||
      (r = ctx_buffer((void**)&c->link_bucket, &c->cap_link_bucket, 8 * un, "link slots")) ||
      (r = ctx_buffer((void**)&c->link_perm, &c->cap_link_perm, 4 * un, "link order")) ||
      (r = ctx_buffer((void**)&c->link_key, &c->cap_link_key, 8 * un, "link proposals")) ||
      (r = ctx_buffer((void**)&c->link_best, &c->cap_link_best, 8 * un, "link winners")))
    return r;
  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  // cells a little wider than max_dist: every start within max_dist of an
  // end lies in the 27 cells around the end's cell despite the rounding of
  // the cell division
  const float cell = max_dist * 1.001f;
  const float d2max = max_dist * max_dist;
  const unsigned nb = (unsigned)((n + 255) / 256);
  StageTimer t(c, FD_STAGE_LINK, st);
  if ((e = launch_fill_u32(c->link_counts, kBuckets, 0u, st)) != hipSuccess ||
      (e = launch_fill_u32((uint32_t*)c->link_best, 2 * (int64_t)n, 0xffffffffu, st)) !=
          hipSuccess)
    return hip_error(e, "link reset");
  hipLaunchKernelGGL(k_link_hash, dim3(nb), dim3(256), 0, st, starts, flags, n, cell,
                     c->link_counts, c->link_bucket);
  if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "link hash");
  if ((e = launch_scan_runs(c->link_counts, (int)(kBuckets / 1024), c->link_sums,
                            c->link_cursor, st)) != hipSuccess)
    return hip_error(e, "link scan");
  hipLaunchKernelGGL(k_link_place, dim3(nb), dim3(256), 0, st, c->link_bucket, n,
                     c->link_cursor, c->link_perm);
  hipLaunchKernelGGL(k_link_propose, dim3(nb), dim3(256), 0, st, starts, start_dirs, ends,
                     end_dirs, flags, n, d2max, min_cos, cell, c->link_counts, c->link_cursor,
                     c->link_perm, succ, c->link_key, c->link_best);
  hipLaunchKernelGGL(k_link_accept, dim3(nb), dim3(256), 0, st, n, c->link_key, c->link_best,
                     succ);
  if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "link kernels");
  t.stop();
  return FD_OK;
}

static int check_pieces(const int32_t* gn, int32_t n_guide, const int32_t* fn,
                        const int32_t* bn, int32_t n_seg, const int32_t* succ, const char* name) {
  if (n_guide < 0 || n_seg < 0 || n_guide > FD_MAX_GROW_SEEDS || n_seg > FD_MAX_GROW_SEEDS)
    return set_error(FD_E_INVAL, "%s: piece counts out of range", name);
  if (n_guide > 0 && (!gn || !succ))
    return set_error(FD_E_INVAL, "%s: null guide lengths or links", name);
  if (n_seg > 0 && (!fn || !bn))
    return set_error(FD_E_INVAL, "%s: null segment lengths", name);
  return FD_OK;
}

extern "C" int fd_strand_offsets(const int32_t* guide_n, int32_t n_guide, const int32_t* fwd_n,
                                 const int32_t* bwd_n, int32_t n_seg, const int32_t* succ,
                                 void* stream, fd_context* ctx, int64_t* offsets,
                                 int32_t* pieces) {
  const char* fn = "fd_strand_offsets";
  int r;
  if ((r = check_pieces(guide_n, n_guide, fwd_n, bwd_n, n_seg, succ, fn))) return r;
  if (!offsets) return set_error(FD_E_INVAL, "%s: offsets is NULL", fn);
  fd_context* c = context_for(ctx, fn, &r);
  if (!c) return r;
  hipStream_t st = (hipStream_t)stream;
  // lengths (n_guide), then the block sums (nb) and their offsets (nb + 1)
  const int32_t nb = (n_guide + 1023) / 1024;
  if ((r = ctx_buffer((void**)&c->strand_len, &c->cap_strand_len,
                      8 * ((size_t)n_guide + 2 * (size_t)nb + 1), "strand lengths")))
    return r;
  PiecesDev P{guide_n, fwd_n, bwd_n, succ, n_guide, n_seg};
  if (n_guide > 0) {
    int64_t* bsum = c->strand_len + n_guide;
    int64_t* boff = bsum + nb;
    hipLaunchKernelGGL(k_strand_len, dim3((unsigned)((n_guide + 255) / 256)), dim3(256), 0, st,
                       P, c->strand_len, pieces);
    hipLaunchKernelGGL(k_len_bsum, dim3((unsigned)nb), dim3(1024), 0, st, c->strand_len,
                       n_guide, bsum);
    hipLaunchKernelGGL(k_len_scan, dim3(1), dim3(1024), 0, st, bsum, nb, boff);
    hipLaunchKernelGGL(k_len_apply, dim3((unsigned)nb), dim3(1024), 0, st, c->strand_len,
                       n_guide, boff, offsets);
  } else {
    hipLaunchKernelGGL(k_len_scan, dim3(1), dim3(1024), 0, st, c->strand_len, 0, offsets);
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "strand offsets");
}

extern "C" int fd_assemble_strands(const float* guide_v, const int32_t* guide_n, int32_t n_guide,
                                   int32_t g_stride, const float* fwd_v, const int32_t* fwd_n,
                                   int32_t f_stride, const float* bwd_v, const int32_t* bwd_n,
                                   int32_t b_stride, int32_t n_seg, const int32_t* succ,
                                   const int64_t* offsets, int64_t capacity, void* stream,
                                   fd_context* ctx, float* out) {
  const char* fn = "fd_assemble_strands";
  int r;
  if ((r = check_pieces(guide_n, n_guide, fwd_n, bwd_n, n_seg, succ, fn))) return r;
  if (g_stride < 1 || f_stride < 1 || b_stride < 1)
    return set_error(FD_E_INVAL, "%s: strides must be >= 1", fn);
  if (capacity < 0) return set_error(FD_E_INVAL, "%s: capacity must be >= 0", fn);
  if (n_guide > 0 && (!guide_v || !offsets || (capacity > 0 && !out)))
    return set_error(FD_E_INVAL, "%s: null pointer argument", fn);
  if (n_seg > 0 && (!fwd_v || !bwd_v))
    return set_error(FD_E_INVAL, "%s: null segment traces", fn);
  fd_context* c = context_for(ctx, fn, &r);
  if (!c) return r;
  if (n_guide == 0) return FD_OK;
  hipStream_t st = (hipStream_t)stream;
  PiecesDev P{guide_n, fwd_n, bwd_n, succ, n_guide, n_seg};
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)(((int64_t)n_guide * 64 + 255) / 256)), dim3(256),
                     0, st, P, guide_v, g_stride, fwd_v, f_stride, bwd_v, b_stride, offsets,
                     capacity, out);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "strand assembly");
}

