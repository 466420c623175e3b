// Copy of part of an expert blob by some workgroups of a launch (a fault's W2 and scales, host -> slot).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace wisp {

// Workgroup q of n copies its share of [off, off + bytes) from src to dst, four 16-byte loads in flight per
// thread (256 threads); the last one also the bytes after the last whole 16.
__device__ __forceinline__ void copy_share(const uint8_t* src_blob, uint8_t* dst_blob, size_t off, size_t bytes, int q,
                                           int n) {
  const size_t n16 = bytes / 16;
  const size_t per = (n16 + n - 1) / n;
  const size_t c0 = static_cast<size_t>(q) * per;
  const size_t c1 = c0 + per < n16 ? c0 + per : n16;
  const uint4* src = reinterpret_cast<const uint4*>(src_blob + off);
  uint4* dst = reinterpret_cast<uint4*>(dst_blob + off);
  size_t i = c0 + threadIdx.x;
  for (; i + 768 < c1; i += 1024) {
    const uint4 a = src[i], b = src[i + 256], c = src[i + 512], e = src[i + 768];
    dst[i] = a; dst[i + 256] = b; dst[i + 512] = c; dst[i + 768] = e;
  }
  for (; i < c1; i += 256) dst[i] = src[i];
  if (q == n - 1) {
    for (size_t b = n16 * 16 + threadIdx.x; b < bytes; b += 256) dst_blob[off + b] = src_blob[off + b];
  }
}

}  // namespace wisp
