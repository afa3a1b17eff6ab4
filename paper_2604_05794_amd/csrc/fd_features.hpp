// fd_features.hpp -- per-point device code of the proposal-network input
// (the most frontal views of a point and what each of them observes).
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/fusedir.h"
#include "fd_device.hpp"
#include "fd_kernels.hpp"
#include "fd_search.hpp"

namespace fd {

constexpr int kSlots = FD_FEATURE_SLOTS;
// Scenes with at most this many views select their views in two passes
// (vis_topk_masked, then frontal_masked), the visibility bits passed between
// the two through the feature row.
constexpr int kMaskViews = 128;
constexpr float kInvPi = 0.318309886183790671538f;

typedef float feat_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 feat_bf16x2_t __attribute__((ext_vector_type(2)));

// (a, b) rounded to bfloat16 (nearest even; the packed conversion
// instruction), a in the low half.
__device__ __forceinline__ uint32_t feat_bf16x2(float a, float b) {
  const feat_bf16x2_t v = __builtin_convertvector((feat_f32x2){a, b}, feat_bf16x2_t);
  return __builtin_bit_cast(uint32_t, v);
}

// Frontal ranking key of a view (the "most frontal" views of the proposal
// features), in binary64 (the ranking is a discrete decision): with the
// camera centre c = -R^T t from the binary64 table, a = c - p and
// b = p - o (o the head centre, b formed once per point),
//   key = (a . b) / |a|,
// the cosine between the point->camera direction and the outward direction
// p - o, times |p - o| (common to every view of the point); the reciprocal
// square root is the refined hardware estimate.
__device__ __forceinline__ double frontal_key(const double* __restrict__ c64, double px,
                                              double py, double pz, double bx, double by,
                                              double bz) {
  const double ax = c64[12] - px, ay = c64[13] - py, az = c64[14] - pz;
  const double dot = __builtin_fma(ax, bx, __builtin_fma(ay, by, az * bz));
  const double la2 = __builtin_fma(ax, ax, __builtin_fma(ay, ay, az * az));
  return dot * rsq64(la2);
}

// Whether two views' frontal keys are equal for every point: their centres are
// the same bits.
__device__ __forceinline__ bool same_centre(const double* __restrict__ tab, int v, int w) {
  const double *a = tab + kCam64 * v + 12, *b = tab + kCam64 * w + 12;
  return a[0] == b[0] && a[1] == b[1] && a[2] == b[2];
}

// Stable insertion of view v with frontal score cs into the descending list
// (sc, id) of kSlots entries (empty entries hold -inf): equal scores keep the
// lower view index first; a view that does not beat the last entry is
// skipped.  The score of an eligible view is finite (the point lies more
// than z_near in front of the camera, so its distance to the centre is not
// zero for any z_near > 0), so it always beats an empty entry.
__device__ __forceinline__ void frontal_insert(double (&sc)[kSlots], int (&id)[kSlots],
                                               double cs, int cv) {
  if (!(cs > sc[kSlots - 1])) return;
  bool ins = false;
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    const bool take = ins || (cs > sc[k]);
    const double ts = sc[k];
    const int tv = id[k];
    sc[k] = take ? cs : ts;
    id[k] = take ? cv : tv;
    cs = take ? ts : cs;
    cv = take ? tv : cv;
    ins = ins || take;
  }
}

// The same list with the view's index in the low kBits bits of its key, so
// that an entry is one binary64 value and a step of the insertion a maximum
// and a minimum (8 cycles a wave, where comparing and moving a key and an
// index apart takes 28).  Keys that differ above those bits are ordered as
// the whole keys are, equal ones by the index (which counts down where the key
// is positive).  Keys that agree there are equal if the views' centres are;
// `top` keeps the largest entry that left the list, and `odd` notes one that
// agreed with it from another centre.  settled() forms the whole keys of
// neighbouring entries that agree (the last one with `top`) and tells whether
// their order stands; where it does not, or after an odd one, the caller makes
// the list again with frontal_insert (keys within 2^-45 or 2^-36 of each other
// from different places).  60,000 points of 64 views: the features call with
// all cameras different 97 us, in pairs at the same place 108, all at one 115;
// with every list that had keys agree made again 94, 216, 161; with keys and
// indexes apart 118, 116, 85.
// kBits: 7 for scenes of at most 128 views, else 16.
template <int kBits>
struct FrontalList {
  static constexpr uint32_t kMask = (1u << kBits) - 1u;
  static constexpr double kEmpty = -1e300;  // below every key that is taken
  double e[kSlots], top;
  bool odd;  // a key that the packing does not hold, or see above

  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < kSlots; ++k) e[k] = kEmpty;
    top = kEmpty;
    odd = false;
  }
  static __device__ __forceinline__ bool agree(double a, double b) {
    return ((__builtin_bit_cast(uint64_t, a) ^ __builtin_bit_cast(uint64_t, b)) >> kBits) == 0;
  }
  static __device__ __forceinline__ int view(double a) {
    const uint64_t b = __builtin_bit_cast(uint64_t, a);
    return (int)(((int64_t)b < 0 ? (uint32_t)b : ~(uint32_t)b) & kMask);
  }
  // (an empty entry agrees with nothing)
  static __device__ __forceinline__ bool may_agree(double a, double b) {
    return __double2hiint(a) == __double2hiint(b) && __double2hiint(a) != __double2hiint(kEmpty);
  }
  // same(v, w): the views' centres are equal
  template <typename F>
  __device__ __forceinline__ void insert(double key, int v, const F& same) {
    odd |= !(fabs(key) < 1e299);
    const uint64_t b = __builtin_bit_cast(uint64_t, key + 0.0);  // -0 as 0
    const uint32_t low = ((int64_t)b < 0 ? (uint32_t)v : ~(uint32_t)v) & kMask;
    double x = __builtin_bit_cast(double, (b & ~(uint64_t)kMask) | low);
    if (x > e[kSlots - 1]) {
#pragma unroll
      for (int k = 0; k < kSlots; ++k) {
        double hi, lo;  // (no operand is a NaN: nothing to quiet)
        asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(e[k]), "v"(x));
        asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(e[k]), "v"(x));
        e[k] = hi;
        x = lo;
      }
    }
    if (may_agree(x, top)) odd |= agree(x, top) && !same(view(x), view(top));
    top = __builtin_fmax(top, x);
  }
  // key(v): the whole key of view v
  template <typename F>
  __device__ __forceinline__ bool settled(const F& key) const {
    bool ok = !odd, any = false;
    auto after = [&](int k) { return k + 1 < kSlots ? e[k + 1 < kSlots ? k + 1 : k] : top; };
#pragma unroll
    for (int k = 0; k < kSlots; ++k) any |= may_agree(e[k], after(k));
    if (!__ballot(any)) return ok;
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
      const double n = after(k);
      if (may_agree(e[k], n) && agree(e[k], n)) {
        const int v = view(e[k]), w = view(n);
        const double a = key(v), b = key(w);
        ok = ok && (a > b || (a == b && v < w));
      }
    }
    return ok;
  }
  __device__ __forceinline__ void views(int (&id)[kSlots]) const {
#pragma unroll
    for (int k = 0; k < kSlots; ++k) id[k] = e[k] == kEmpty ? -1 : view(e[k]);
  }
};

// The list with whole keys: each_view(take) calls take(key, view) for the
// views in increasing order.
template <typename F>
__device__ __forceinline__ void list_whole_keys(const F& each_view, int (&id)[kSlots]) {
  double sc[kSlots];
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    sc[k] = -INFINITY;
    id[k] = -1;
  }
  each_view([&](double key, int v) { frontal_insert(sc, id, key, v); });
}

// A slot of a feature row, without branches (a slot that is empty passes
// valid = false, reads view 0 and yields zeros).  tab is the scene's camera
// table (kCam64 slots per view).  PAIRS: the scene allows texel-pair loads
// (binary16).
template <typename T, bool PAIRS>
__device__ __forceinline__ void feature_slot(const SceneDev& s, const double* __restrict__ tab,
                                             double px, double py, double pz, int v, bool valid,
                                             float (&f)[7]) {
  const T* th = (const T*)s.theta;
  const T* cf = (const T*)s.conf;
  const size_t plane = (size_t)s.W * s.H;
  // the binary32 record, two values per binary64 slot (read as the slots'
  // own type and split by value, so the accesses match how it was stored)
  const double* rec = tab + kCam64 * v + kCam32Off;
  float cr[16];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float2 pr2 = __builtin_bit_cast(float2, rec[e]);
    cr[2 * e] = pr2.x;
    cr[2 * e + 1] = pr2.y;
  }
  const float4 q0 = make_float4(cr[0], cr[1], cr[2], cr[3]);
  const float4 q1 = make_float4(cr[4], cr[5], cr[6], cr[7]);
  const float4 q2 = make_float4(cr[8], cr[9], cr[10], cr[11]);
  const float4 q3 = make_float4(cr[12], cr[13], cr[14], cr[15]);
  // fx fy cx cy | R0 R1 R2 R3 | R4 R5 R6 R7 | R8 t0 t1 t2
  // the sample position in binary64 from the same record (binary32 would
  // move the bilinear weights by ~5e-5 and flip the bfloat16 rounding of
  // many more values)
  const double dX = __builtin_fma((double)q1.x, px, __builtin_fma((double)q1.y, py,
                                  __builtin_fma((double)q1.z, pz, (double)q3.y)));
  const double dY = __builtin_fma((double)q1.w, px, __builtin_fma((double)q2.x, py,
                                  __builtin_fma((double)q2.y, pz, (double)q3.z)));
  const double dZ = __builtin_fma((double)q2.z, px, __builtin_fma((double)q2.w, py,
                                  __builtin_fma((double)q3.x, pz, (double)q3.w)));
  // a slot's view sees the point: dZ > z_near > 0
  const double idz = rcp64(valid ? dZ : 1.0);
  const double su = valid ? __builtin_fma((double)q0.x, dX * idz, (double)q0.z) : 0.0;
  const double sv = valid ? __builtin_fma((double)q0.y, dY * idz, (double)q0.w) : 0.0;
  const float pX = (float)dX, pY = (float)dY, pZ = (float)dZ;
  // the visible projection lies in [0, W-1] x [0, H-1] (up to the last bit
  // of this binary64 evaluation; the clamp keeps the weights continuous)
  const int ix = min(max((int)floor(su), 0), s.W - 1), iy = min(max((int)floor(sv), 0), s.H - 1);
  const float fx = (float)(su - (double)ix), fy = (float)(sv - (double)iy);
  const bool yin = iy + 1 < s.H;
  // the 2 x 2 texels (zero outside the image)
  float tq[2][2], cq[2][2];
  if constexpr (PAIRS) {
    // one 8-byte load per row and map: the texel pair at a = min(ix & ~1,
    // W - 4) and the next pair (W even, W >= 4, rows 4-byte aligned)
    const uint32_t a = min((uint32_t)ix & ~1u, (uint32_t)s.W - 4u);
    const uint32_t d = (uint32_t)ix - a;  // 0..3
    const uint32_t r0 = (uint32_t)iy * (uint32_t)s.W;
    const uint32_t r1 = r0 + (yin ? (uint32_t)s.W : 0u);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t off = ((b ? r1 : r0) + a) * 2u;
      const uint2 wt = *(const uint2*)((const char*)(th + plane * v) + off);
      const uint2 wc = *(const uint2*)((const char*)(cf + plane * v) + off);
      const uint64_t pt = ((uint64_t)wt.y << 32) | wt.x, pc = ((uint64_t)wc.y << 32) | wc.x;
      const bool row_in = b == 0 || yin;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t k = d + (uint32_t)e;  // 4: texel W, outside
        const bool in = row_in && k < 4u;
        const uint32_t sh = 16u * (k & 3u);
        tq[b][e] = in ? __half2float(__ushort_as_half((unsigned short)(pt >> sh))) : 0.0f;
        cq[b][e] = in ? __half2float(__ushort_as_half((unsigned short)(pc >> sh))) : 0.0f;
      }
    }
  } else {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        tq[b][e] = tex_load_nb<T>(th + plane * v, s.W, s.H, ix + e, iy + b);
        cq[b][e] = tex_load_nb<T>(cf + plane * v, s.W, s.H, ix + e, iy + b);
      }
  }
  float cb = 0.0f, mx = 0.0f, my = 0.0f;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float w = (e ? fx : 1.0f - fx) * (b ? fy : 1.0f - fy);
      const float wc = w * cq[b][e];
      cb += wc;
      mx = __builtin_fmaf(wc, __builtin_amdgcn_cosf(tq[b][e] * kInvPi), mx);
      my = __builtin_fmaf(wc, __builtin_amdgcn_sinf(tq[b][e] * kInvPi), my);
    }
  // unit point -> camera direction vd: centre c = -R^T t
  const float qx0 = (float)px, qy0 = (float)py, qz0 = (float)pz;
  const float ccx = -__builtin_fmaf(q1.x, q3.y, __builtin_fmaf(q1.w, q3.z, q2.z * q3.w));
  const float ccy = -__builtin_fmaf(q1.y, q3.y, __builtin_fmaf(q2.x, q3.z, q2.w * q3.w));
  const float ccz = -__builtin_fmaf(q1.z, q3.y, __builtin_fmaf(q2.y, q3.z, q3.x * q3.w));
  float vd[3] = {ccx - qx0, ccy - qy0, ccz - qz0};
  {
    const float il = __builtin_amdgcn_rsqf(
        __builtin_fmaf(vd[0], vd[0], __builtin_fmaf(vd[1], vd[1], vd[2] * vd[2])));
    vd[0] *= il;
    vd[1] *= il;
    vd[2] *= il;
  }
  // The observed image line back-projects to a plane through the camera
  // centre containing the line of sight vd; its direction across vd,
  // tt = n x vd, is given by the angle psi in the frame
  // e1 = normalize(z x vd), e2 = vd x e1, carried as |m| (cos 2psi, sin 2psi).
  float qx = 0.0f, qy = 0.0f;
  const float m2 = __builtin_fmaf(mx, mx, my * my);
  if (m2 > 0.0f) {
    const float imag = __builtin_amdgcn_rsqf(m2);
    const float mag = m2 * imag;
    const float ch = mx * imag, sh = my * imag;  // cos, sin of 2 theta
    const float ox = __builtin_amdgcn_sqrtf(fmaxf(0.5f * (1.0f + ch), 0.0f));
    const float oy = copysignf(__builtin_amdgcn_sqrtf(fmaxf(0.5f * (1.0f - ch), 0.0f)), sh);
    const float dlx = ox * __builtin_amdgcn_rcpf(q0.x), dly = oy * __builtin_amdgcn_rcpf(q0.y);
    const float ncx = -pZ * dly, ncy = pZ * dlx, ncz = pX * dly - pY * dlx;
    const float nwx = __builtin_fmaf(q1.x, ncx, __builtin_fmaf(q1.w, ncy, q2.z * ncz));
    const float nwy = __builtin_fmaf(q1.y, ncx, __builtin_fmaf(q2.x, ncy, q2.w * ncz));
    const float nwz = __builtin_fmaf(q1.z, ncx, __builtin_fmaf(q2.y, ncy, q3.x * ncz));
    const float tx = nwy * vd[2] - nwz * vd[1];
    const float ty = nwz * vd[0] - nwx * vd[2];
    const float tz = nwx * vd[1] - nwy * vd[0];
    const bool vert = fabsf(vd[2]) > 1.0f - 1e-6f;
    const float ux = vert ? 1.0f : 0.0f, uz = vert ? 0.0f : 1.0f;
    // e1 = up x vd, up = (ux, 0, uz)
    float e1x = -uz * vd[1], e1y = uz * vd[0] - ux * vd[2], e1z = ux * vd[1];
    const float il = __builtin_amdgcn_rsqf(
        __builtin_fmaf(e1x, e1x, __builtin_fmaf(e1y, e1y, e1z * e1z)));
    e1x *= il;
    e1y *= il;
    e1z *= il;
    const float e2x = vd[1] * e1z - vd[2] * e1y;
    const float e2y = vd[2] * e1x - vd[0] * e1z;
    const float e2z = vd[0] * e1y - vd[1] * e1x;
    const float t1 = __builtin_fmaf(tx, e1x, __builtin_fmaf(ty, e1y, tz * e1z));
    const float t2 = __builtin_fmaf(tx, e2x, __builtin_fmaf(ty, e2y, tz * e2z));
    const float tn = __builtin_fmaf(t1, t1, t2 * t2);
    if (tn > 0.0f) {
      const float r = mag * __builtin_amdgcn_rcpf(tn);
      qx = r * __builtin_fmaf(t1, t1, -t2 * t2);
      qy = r * 2.0f * t1 * t2;
    }
  }
  f[0] = valid ? qx : 0.0f;
  f[1] = valid ? qy : 0.0f;
  f[2] = valid ? cb : 0.0f;
  f[3] = valid ? vd[0] : 0.0f;
  f[4] = valid ? vd[1] : 0.0f;
  f[5] = valid ? vd[2] : 0.0f;
  f[6] = valid ? 1.0f : 0.0f;
}

// The frontal lists of a wave's points on their way to the lanes that form the
// slots: in LDS, 16 bits a slot (0xffff: empty), nine words a point (every
// lane's list starts at another bank).
constexpr int kFeatureBlock = 256;  // threads of the kernels that write rows
constexpr int kListWords = kSlots / 2 + 1;
struct FrontalLists {
  uint32_t w[kFeatureBlock / kWave][kWave * kListWords];
};

// Per slot of the frontal list: the observed orientation as
// (q_x, q_y) = |m| (cos 2psi, sin 2psi) (m the bilinear confidence-weighted
// doubled-angle vector, psi the angle of the plane it back-projects to, in a
// frame tied to the line of sight), the bilinear confidence C, the unit
// point->camera direction and 1; empty slots are 0.  Written as 112
// bfloat16 to the point's row.  These are values,
// not decisions (the slot views are chosen in binary64 beforehand), and they
// are rounded to bfloat16 (relative step 2^-8), so apart from the sample
// position (binary64) they are formed in binary32 with the hardware
// reciprocal, square root and sine / cosine (errors ~1e-6 relative).
//
// Called by whole waves: lane l < PW has the list id of point j0 + l (if that
// is below n), the points' rows follow one another from row0.  One lane per
// slot, the 16 of a point side by side, four points at a time.  A slot's
// texels and camera record are gathers; a lane that took a point's slots in
// turn held another view than most of its 64 neighbours, where four
// neighbouring points share most of theirs.  Two lanes' 14 values make seven
// words, four of them stored by the even one (rows are 224 bytes, so every
// pair starts on a 4-byte boundary).
// 60,000 points of 64 views, binary32 maps: the call 171 -> 128 us, with the
// list and the grouped depth texels; 2M points of up to 128 views: list and
// rows 1344 -> 1020 us (a kernel of the list alone 330, of the rows alone
// 760: the loads of the rows).  Going through a wave's views one by one, the
// lanes that have it together, measured 620 where this measures 160 (a
// serial chain of scalar and vector loads per view).
template <typename T, int PW = kWave>
__device__ __forceinline__ void wave_feature_rows(const SceneDev& s, FrontalLists& lists,
                                                  const int (&id)[kSlots], int64_t j0, int64_t n,
                                                  int64_t row0, uint16_t* __restrict__ feats) {
  const int lane = (int)(threadIdx.x & (kWave - 1));
  uint32_t* const w = lists.w[threadIdx.x / kWave];
#pragma unroll
  for (int k = 0; k < kSlots; k += 2)
    w[lane * kListWords + k / 2] = ((uint32_t)id[k] & 0xffffu) | ((uint32_t)id[k + 1] << 16);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int slot = lane % kSlots;
  const bool odd = slot & 1;
#pragma unroll 1
  for (int p = lane / kSlots; p < PW; p += kWave / kSlots) {
    if (j0 + p >= n) break;  // the same for a point's lanes
    const uint32_t i = s.perm ? s.perm[j0 + p] : (uint32_t)(j0 + p);
    const double px = s.pts[3 * (size_t)i], py = s.pts[3 * (size_t)i + 1],
                 pz = s.pts[3 * (size_t)i + 2];
    const uint32_t v = (w[p * kListWords + slot / 2] >> (odd ? 16 : 0)) & 0xffffu;
    const bool valid = v != 0xffffu;
    float f[7];
    if (sizeof(T) == 2 && s.pairs)
      feature_slot<T, true>(s, s.cam64, px, py, pz, valid ? (int)v : 0, valid, f);
    else
      feature_slot<T, false>(s, s.cam64, px, py, pz, valid ? (int)v : 0, valid, f);
    const float f7 = __shfl_xor(f[0], 1, kWave);  // the odd slot's first, in the even lane
    uint32_t* const dst = (uint32_t*)(feats + (size_t)(row0 + p) * (7 * kSlots)) +
                          7 * (slot >> 1) + (odd ? 4 : 0);
    dst[0] = feat_bf16x2(odd ? f[1] : f[0], odd ? f[2] : f[1]);
    dst[1] = feat_bf16x2(odd ? f[3] : f[2], odd ? f[4] : f[3]);
    dst[2] = feat_bf16x2(odd ? f[5] : f[4], odd ? f[6] : f[5]);
    if (!odd) dst[3] = feat_bf16x2(f[6], f7);
  }
}

// One lane per point: the kSlots most frontal eligible views.
template <typename T>
__device__ __forceinline__ void features_point(const SceneDev& s, double z_near, int64_t j,
                                               int (&id)[kSlots]) {
  const uint32_t i = s.perm ? s.perm[j] : (uint32_t)j;
  const double px = s.pts[3 * (size_t)i], py = s.pts[3 * (size_t)i + 1],
               pz = s.pts[3 * (size_t)i + 2];
  const size_t plane = (size_t)s.W * s.H;
  const T* depth = (const T*)s.depth;
  const double bx = px - (double)s.hc[0], by = py - (double)s.hc[1], bz = pz - (double)s.hc[2];
  // views in groups, the depth texels of a group issued together
  constexpr int kGroup = 4;
  auto each_view = [&](auto&& take) {
    for (int v0 = 0; v0 < s.V; v0 += kGroup) {
      bool seen[kGroup];
#pragma unroll
      for (int u = 0; u < kGroup; ++u) {
        const int v = min(v0 + u, s.V - 1);
        ProjT pr;
        const bool ok = project_tab(s.cam64 + kCam64 * v, px, py, pz, s.W, s.H, z_near, pr);
        seen[u] = visible_at<T>(depth ? depth + plane * v : nullptr, s.W, ok, pr,
                                (double)s.vis_tau) && v0 + u < s.V;
      }
#pragma unroll
      for (int u = 0; u < kGroup; ++u)
        if (seen[u])
          take(frontal_key(s.cam64 + kCam64 * (v0 + u), px, py, pz, bx, by, bz), v0 + u);
    }
  };
  FrontalList<16> list;
  list.clear();
  const auto same = [&](int v, int w) { return same_centre(s.cam64, v, w); };
  each_view([&](double key, int v) { list.insert(key, v, same); });
  list.views(id);
  const auto key = [&](int v) {
    return frontal_key(s.cam64 + kCam64 * v, px, py, pz, bx, by, bz);
  };
  if (__ballot(!list.settled(key))) list_whole_keys(each_view, id);
}

// Eq. (4) view selection and the frontal list in one pass over the views (one
// projection per view): writes views / kcount like topk_point and leaves the
// list in id.
template <typename T, int KS>
__device__ __forceinline__ void topk_features_point(const SceneDev& s, const SearchDev& q,
                                                    int64_t j, int (&id)[kSlots]) {
  const uint32_t i = s.perm[j];
  const double px = s.pts[3 * (size_t)i], py = s.pts[3 * (size_t)i + 1],
               pz = s.pts[3 * (size_t)i + 2];
  double ck[KS];
  int vk[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    ck[k] = -1.0;
    vk[k] = 0;
  }
  double sc[kSlots];
#pragma unroll
  for (int k = 0; k < kSlots; ++k) {
    sc[k] = -INFINITY;
    id[k] = -1;
  }
  const T* conf = (const T*)s.conf;
  const T* depth = (const T*)s.depth;
  const size_t plane = (size_t)s.W * s.H;
  const double tau = (double)s.vis_tau;
  const double bx = px - (double)s.hc[0], by = py - (double)s.hc[1], bz = pz - (double)s.hc[2];
  // views in groups of two (four as in topk_point would hold more registers
  // next to the frontal list): a view no lane of the wave sees skips its
  // confidence texels and both insertions
  constexpr int kGroup = 2;
  for (int v0 = 0; v0 < s.V; v0 += kGroup) {
    ProjT pr[kGroup];
    bool seen[kGroup];
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int v = min(v0 + u, s.V - 1);
      const bool ok = project_tab(s.cam64 + kCam64 * v, px, py, pz, s.W, s.H, q.z_near, pr[u]);
      seen[u] = visible_at<T>(depth ? depth + plane * v : nullptr, s.W, ok, pr[u], tau) &&
                v0 + u < s.V;
    }
    ConfTexels tx[kGroup];
    bool any[kGroup];
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      any[u] = __ballot(seen[u]) != 0;  // wave-uniform
      if (any[u]) tx[u] = conf_texels<T>(conf + plane * (v0 + u), s.W, s.H, seen[u], pr[u], s.pairs);
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      if (!any[u]) continue;
      const int v = v0 + u;
      const double c = seen[u] ? conf_combine(tx[u]) : 0.0;
      if (c > 0.0) topk_insert<KS>(ck, vk, c, v);
      // frontal slots: eligible and visible views, whatever their confidence
      if (seen[u])
        frontal_insert(sc, id, frontal_key(s.cam64 + kCam64 * v, px, py, pz, bx, by, bz), v);
    }
  }
  int keff = 0;
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    if (k < q.K && ck[k] > 0.0) keff = k + 1;
    s.views[FD_TOPK_SLOTS * j + k] = (uint16_t)vk[k];
  }
  s.kcount[j] = (uint8_t)keff;
}

// Bitwise OR of m over the wave, in a scalar register.
__device__ __forceinline__ uint32_t wave_or32(uint32_t m) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) m |= (uint32_t)__shfl_xor((int)m, off, kWave);
  return __builtin_amdgcn_readfirstlane(m);
}

// For scenes of at most 32 MW views the view selection and the frontal list
// run as two kernels, each holding less state.  The first
// (vis_topk_masked) makes the Eq. (4) selection (four views at a time, as
// topk_point) and keeps each view's visibility as a bit in MW registers,
// which it leaves in the first 4 MW bytes of the point's feature row; the
// second (frontal_masked) takes the bits back, ranks the visible views
// by frontality (projections and depth texels are not read again; the
// views are taken in increasing order, so the list is the same as the
// one-pass form's) and returns the list.  The gather loop of the
// first then runs at the occupancy its own registers allow.  ctab is the
// scene's camera table, read at wave-uniform addresses only (the caller may
// pass the global table, whose records then come through the scalar cache
// without taking vector registers, or a copy in LDS).
template <typename T, int KS, int MW>
__device__ __forceinline__ void vis_topk_masked(const SceneDev& s, const SearchDev& q,
                                                const double* __restrict__ ctab, int64_t j,
                                                int64_t row, uint16_t* __restrict__ feats) {
  static_assert(4 * MW <= 14 * kSlots, "the bits fit in the row");
  const uint32_t i = s.perm[j];
  const double px = s.pts[3 * (size_t)i], py = s.pts[3 * (size_t)i + 1],
               pz = s.pts[3 * (size_t)i + 2];
  const T* conf = (const T*)s.conf;
  const T* depth = (const T*)s.depth;
  const size_t plane = (size_t)s.W * s.H;
  const double tau = (double)s.vis_tau;
  uint32_t mask[MW];
  {
    double ck[KS];
    int vk[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      ck[k] = -1.0;
      vk[k] = 0;
    }
    constexpr int kGroup = 4;
#pragma unroll
    for (int w = 0; w < MW; ++w) {
      uint32_t bits = 0;
      const int vend = min(s.V, 32 * (w + 1));
      for (int v0 = 32 * w; v0 < vend; v0 += kGroup) {
        ProjT pr[kGroup];
        bool seen[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
          const int v = min(v0 + u, s.V - 1);
          const bool ok =
              project_tab(ctab + kCam64 * v, px, py, pz, s.W, s.H, q.z_near, pr[u]);
          seen[u] = visible_at<T>(depth ? depth + plane * v : nullptr, s.W, ok, pr[u], tau) &&
                    v0 + u < s.V;
          bits |= (seen[u] ? 1u : 0u) << (v0 + u - 32 * w);
        }
        ConfTexels tx[kGroup];
        bool any[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
          any[u] = __ballot(seen[u]) != 0;  // wave-uniform
          if (any[u]) tx[u] = conf_texels<T>(conf + plane * (v0 + u), s.W, s.H, seen[u], pr[u], s.pairs);
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
          if (!any[u]) continue;
          const double c = seen[u] ? conf_combine(tx[u]) : 0.0;
          if (c > 0.0) topk_insert<KS>(ck, vk, c, v0 + u);
        }
      }
      mask[w] = bits;
    }
    int keff = 0;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      if (k < q.K && ck[k] > 0.0) keff = k + 1;
      s.views[FD_TOPK_SLOTS * j + k] = (uint16_t)vk[k];
    }
    s.kcount[j] = (uint8_t)keff;
  }
  uint32_t* bits_out = (uint32_t*)(feats + (size_t)row * (7 * kSlots));
#pragma unroll
  for (int w = 0; w < MW; ++w) bits_out[w] = mask[w];
}

template <int MW>
__device__ __forceinline__ void frontal_masked(const SceneDev& s,
                                               const double* __restrict__ ctab, int64_t j,
                                               int64_t row, const uint16_t* feats,
                                               int (&id)[kSlots]) {
  const uint32_t i = s.perm[j];
  const double px = s.pts[3 * (size_t)i], py = s.pts[3 * (size_t)i + 1],
               pz = s.pts[3 * (size_t)i + 2];
  uint32_t mask[MW];
  const uint32_t* bits_in = (const uint32_t*)(feats + (size_t)row * (7 * kSlots));
#pragma unroll
  for (int w = 0; w < MW; ++w) mask[w] = bits_in[w];
  const double bx = px - (double)s.hc[0], by = py - (double)s.hc[1], bz = pz - (double)s.hc[2];
  auto each_view = [&](auto&& take) {
#pragma unroll
    for (int w = 0; w < MW; ++w) {
      uint32_t um = wave_or32(mask[w]);  // views some lane of the wave sees
      while (um) {
        const int b = __builtin_ctz(um);
        um &= um - 1u;
        const int v = 32 * w + b;
        if ((mask[w] >> b) & 1u)
          take(frontal_key(ctab + kCam64 * v, px, py, pz, bx, by, bz), v);
      }
    }
  };
  static_assert(32 * MW <= 128, "seven bits of view index");
  FrontalList<7> list;
  list.clear();
  const auto same = [&](int v, int w) { return same_centre(ctab, v, w); };
  each_view([&](double key, int v) { list.insert(key, v, same); });
  list.views(id);
  const auto key = [&](int v) {
    return frontal_key(ctab + kCam64 * v, px, py, pz, bx, by, bz);
  };
  if (__ballot(!list.settled(key))) list_whole_keys(each_view, id);
}

}  // namespace fd
