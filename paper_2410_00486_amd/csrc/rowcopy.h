// Copies of rows from scattered places into a contiguous range: the pool's
// reordering and its densification.
#pragma once

#include "gs_internal.h"

namespace gs {

constexpr int kCopyThreads = 256;
constexpr int64_t kRowZero = -1;  // the row is set to zero
constexpr int64_t kRowSkip = -2;  // the row is written by someone else

template <int W, typename V, typename Map>
__device__ __forceinline__ void copy_rows_as(const V* __restrict__ src, V* __restrict__ dst,
                                             int nrow, Map map) {
  constexpr int U = 4;  // loads in flight per thread
  const int total = nrow * W;
  for (int e0 = (int)threadIdx.x; e0 < total; e0 += U * kCopyThreads) {
    V x[U];
    int64_t from[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kCopyThreads;
      from[u] = kRowSkip;
      x[u] = V{};
      if (e < total) {
        const int row = e / W;
        from[u] = map(row);
        if (from[u] >= 0) x[u] = src[from[u] * W + (e - row * W)];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (from[u] != kRowSkip) dst[e0 + u * kCopyThreads] = x[u];
  }
}

// Writes rows 0..nrow of W floats at dst; row r comes from row map(r) of src,
// or is one of the marks above.  One workgroup of kCopyThreads; consecutive
// threads take consecutive elements of the output, 16 bytes each where the
// width and both addresses allow it.
template <int W, typename Map>
__device__ __forceinline__ void copy_rows(const float* src, float* dst, int nrow, Map map) {
  if (W % 4 == 0 &&
      ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15u) == 0)
    copy_rows_as<W < 4 ? 1 : W / 4>(reinterpret_cast<const float4*>(src),
                                  reinterpret_cast<float4*>(dst), nrow, map);
  else
    copy_rows_as<W>(src, dst, nrow, map);
}

}  // namespace gs
