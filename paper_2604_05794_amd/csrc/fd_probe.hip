// fd_probe.hip -- probes: read bandwidth for the roofline of the search (the L2
// ceiling, which has no published figure), and the search's own normalisation
// on operands of the caller's.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/fusedir.h"
#include "fd_api_internal.hpp"
#include "fd_device.hpp"

using namespace fd;

namespace {

// Every workgroup walks the whole buffer with 16-byte loads; lane values
// are folded so that no load is dead.
__global__ __launch_bounds__(256) void k_probe_read(const uint4* __restrict__ buf, int64_t n16,
                                                    int reps, uint32_t* __restrict__ sink) {
  uint32_t acc = 0;
  for (int r = 0; r < reps; ++r) {
    for (int64_t i = threadIdx.x; i < n16; i += 4 * 256) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t k = i + u * 256;
        v[u] = k < n16 ? buf[k] : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    acc = (acc << 1) | (acc >> 31);
  }
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

__global__ __launch_bounds__(256) void k_probe_norm(const float* __restrict__ n2,
                                                    const float* __restrict__ al,
                                                    const float* __restrict__ p,
                                                    const float* __restrict__ q, int64_t n,
                                                    float* __restrict__ pr,
                                                    float* __restrict__ qr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float a, b;
  over_norm(n2[i], al[i], p[i], q[i], n2[i] > 0.0f, a, b);
  pr[i] = a;
  qr[i] = b;
}

}  // namespace

extern "C" int fd_probe_norm(const float* n2, const float* al, const float* p, const float* q,
                             int64_t n, float* pr, float* qr, void* stream) {
  if (n < 0 || n > ((int64_t)1 << 31))
    return set_error(FD_E_INVAL, "fd_probe_norm: n must be in [0, 2^31]");
  if (n > 0 && (!n2 || !al || !p || !q || !pr || !qr))
    return set_error(FD_E_INVAL, "fd_probe_norm: null pointer");
  int r;
  if ((r = check_device(nullptr))) return r;
  if (n == 0) return FD_OK;
  hipLaunchKernelGGL(k_probe_norm, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, n2, al, p, q, n, pr, qr);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "fd_probe_norm");
}

extern "C" int fd_probe_read(const void* buf, int64_t bytes, int32_t reps, int32_t blocks,
                             uint32_t* sink, void* stream) {
  if (!buf || !sink) return set_error(FD_E_INVAL, "fd_probe_read: null pointer");
  if (bytes <= 0 || (bytes & 15) || bytes > ((int64_t)1 << 31))
    return set_error(FD_E_INVAL, "fd_probe_read: bytes must be a positive multiple of 16, "
                     "at most 2^31");
  if (reps < 1 || blocks < 1) return set_error(FD_E_INVAL, "fd_probe_read: reps and blocks >= 1");
  int r;
  if ((r = check_device(nullptr))) return r;
  hipLaunchKernelGGL(k_probe_read, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                     (const uint4*)buf, bytes / 16, reps, sink);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? FD_OK : hip_error(e, "fd_probe_read");
}
