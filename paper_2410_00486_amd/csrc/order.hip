// Spatial order of a Gaussian pool: a data-layout step, not part of an
// iteration.  Neighbouring Gaussians of a view then sit in the same
// wavefronts of the per-Gaussian kernels (projection, binning counts,
// projection backward), whose per-view branches and tile atomics stop
// diverging over the whole pool.  The mapping loop re-orders the pool
// whenever it re-plans after densification.
//
// Order: the Morton code of each mean in the pool's bounding box (10 bits
// per axis), sorted stably (ties keep the index order), so the permutation
// is deterministic.
#include <cfloat>

#include "rowcopy.h"
#include "sort.h"

namespace gs {
namespace {

constexpr int kBoxThreads = 256;
constexpr int kBoxBlocks = 256;
constexpr int kMortonBits = 10;

// Per-block bounding boxes of the means (min x y z, max x y z).
__global__ void __launch_bounds__(kBoxThreads) k_box_part(const float* __restrict__ means,
                                                          int64_t n, float* __restrict__ part) {
  __shared__ float s[6][kBoxThreads];
  float lo[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, hi[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
  for (int64_t i = (int64_t)blockIdx.x * kBoxThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBoxThreads)
    for (int d = 0; d < 3; ++d) {
      const float x = means[3 * i + d];
      if (x == x) {  // a NaN mean takes no part in the box
        lo[d] = fminf(lo[d], x);
        hi[d] = fmaxf(hi[d], x);
      }
    }
  for (int d = 0; d < 3; ++d) {
    s[d][threadIdx.x] = lo[d];
    s[3 + d][threadIdx.x] = hi[d];
  }
  __syncthreads();
  for (int w = kBoxThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int d = 0; d < 3; ++d) {
        s[d][threadIdx.x] = fminf(s[d][threadIdx.x], s[d][threadIdx.x + w]);
        s[3 + d][threadIdx.x] = fmaxf(s[3 + d][threadIdx.x], s[3 + d][threadIdx.x + w]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = s[threadIdx.x][0];
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  // bit b of v to bit 3b
  uint64_t x = v & 0x3FFu;
  x = (x | (x << 16)) & 0x30000FFull;
  x = (x | (x << 8)) & 0x300F00Full;
  x = (x | (x << 4)) & 0x30C30C3ull;
  x = (x | (x << 2)) & 0x9249249ull;
  return x;
}

// Morton code of every mean in the box of the block partials; values are
// the indices 0..n-1.
__global__ void __launch_bounds__(256) k_morton(const float* __restrict__ means, int64_t n,
                                                const float* __restrict__ part, int n_part,
                                                uint64_t* __restrict__ keys,
                                                uint32_t* __restrict__ vals) {
  // the box: thread t takes partial t (at most one each), then wave
  // butterflies and the four wavefronts' results
  static_assert(kBoxBlocks <= 256, "one partial per thread");
  __shared__ float wbox[256 / kWave][6], box[6];
  const int t = (int)threadIdx.x;
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    float v = t < n_part ? part[t * 6 + d] : (d < 3 ? FLT_MAX : -FLT_MAX);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const float x = __shfl_xor(v, o, kWave);
      v = d < 3 ? fminf(v, x) : fmaxf(v, x);
    }
    if (lane_id() == 0) wbox[t / kWave][d] = v;
  }
  __syncthreads();
  if (t < 6) {
    float v = wbox[0][t];
    for (int k = 1; k < 256 / kWave; ++k) v = t < 3 ? fminf(v, wbox[k][t]) : fmaxf(v, wbox[k][t]);
    box[t] = v;
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  constexpr float kCells = (float)((1 << kMortonBits) - 1);
  uint32_t q[3];
  for (int d = 0; d < 3; ++d) {
    const float ext = box[3 + d] - box[d];
    const float x = means[3 * i + d];
    float t = ext > 0.0f ? (x - box[d]) / ext : 0.0f;
    t = (t == t) ? fminf(1.0f, fmaxf(0.0f, t)) : 1.0f;  // NaN last
    q[d] = (uint32_t)(t * kCells);
  }
  keys[i] = spread3(q[0]) | (spread3(q[1]) << 1) | (spread3(q[2]) << 2);
  vals[i] = (uint32_t)i;
}

// Row j of every array of dst = row perm[j] of src.  A workgroup takes 128
// rows of all five arrays: one launch for a set, the order read once.  Bound
// by HBM; one launch per array, with a 64-bit division per element, took
// 92 us for 300k Gaussians of degree 3 (146 MB, and as much again because a
// random row of 4 to 16 bytes costs a whole cache line), now 47 us.  Rows per
// workgroup (32 to 256) and loads in flight (2 to 8) change nothing.
constexpr int kPermRows = 128;

template <int K3>
__global__ void __launch_bounds__(kCopyThreads) k_permute(gs_gaussians src,
                                                          const int32_t* __restrict__ perm,
                                                          gs_gaussian_grads dst) {
  __shared__ int32_t from[kPermRows];
  const int64_t j0 = (int64_t)blockIdx.x * kPermRows;
  const int nrow = (int)min((int64_t)kPermRows, src.n - j0);
  if ((int)threadIdx.x < nrow) from[threadIdx.x] = perm[j0 + threadIdx.x];
  __syncthreads();
  const auto row = [&](int r) -> int64_t { return from[r]; };
  copy_rows<K3>(src.sh, dst.sh + j0 * K3, nrow, row);
  copy_rows<4>(src.quats, dst.quats + j0 * 4, nrow, row);
  copy_rows<3>(src.means, dst.means + j0 * 3, nrow, row);
  copy_rows<3>(src.log_scales, dst.log_scales + j0 * 3, nrow, row);
  copy_rows<1>(src.opacity_logits, dst.opacity_logits + j0, nrow, row);
}

struct OrderTmp {
  size_t keys, part, sort, bytes;
};
OrderTmp order_layout(int64_t n) {
  OrderTmp t{};
  t.keys = 0;
  t.part = sort_align(t.keys + (size_t)n * 8 + 8);
  t.sort = sort_align(t.part + (size_t)kBoxBlocks * 6 * 4);
  t.bytes = t.sort + sort_scratch(n).bytes;
  return t;
}

}  // namespace

size_t spatial_order_tmp_bytes(int64_t n) { return n < 0 ? 0 : order_layout(n).bytes; }

// perm: [n] int32 output (the Gaussian at new position j is the old perm[j]).
hipError_t launch_spatial_order(const float* means, int64_t n, int32_t* perm, void* tmp,
                                hipStream_t s) {
  const OrderTmp L = order_layout(n);
  char* b = static_cast<char*>(tmp);
  uint64_t* keys = reinterpret_cast<uint64_t*>(b + L.keys);
  float* part = reinterpret_cast<float*>(b + L.part);
  const int nbox = (int)std::min<int64_t>(kBoxBlocks, (n + kBoxThreads - 1) / kBoxThreads);
  hipLaunchKernelGGL(k_box_part, dim3(nbox), dim3(kBoxThreads), 0, s, means, n, part);
  // the permutation doubles as the sort's values
  uint32_t* vals = reinterpret_cast<uint32_t*>(perm);
  hipLaunchKernelGGL(k_morton, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, means, n,
                     part, nbox, keys, vals);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? launch_sort_pairs(keys, vals, n, 3 * kMortonBits, b + L.sort, s) : e;
}

hipError_t launch_permute(const gs_gaussians& src, const int32_t* perm,
                          const gs_gaussian_grads& dst, hipStream_t s) {
  if (src.n == 0) return hipSuccess;
  const dim3 grid((unsigned)((src.n + kPermRows - 1) / kPermRows));
  const auto kernel = src.sh_degree == 0   ? k_permute<3>
                      : src.sh_degree == 1 ? k_permute<12>
                      : src.sh_degree == 2 ? k_permute<27>
                                           : k_permute<48>;
  hipLaunchKernelGGL(kernel, grid, dim3(kCopyThreads), 0, s, src, perm, dst);
  return hipGetLastError();
}

}  // namespace gs
