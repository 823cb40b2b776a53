// Adaptive densification and opacity pruning (CaRtGS Sec. IV-A: densify every
// 500 iterations with a positional-gradient threshold, remove Gaussians with
// opacity below a threshold; clone / split as in 3DGS).
//
// gs_grad_stats: per Gaussian and view, the 2D mean gradient is the fixed-
// order sum of its pair partials (the same slots the projection backward
// reads); its norm in normalised device coordinates is added to `accum` and
// the visibility to `denom`.
//
// gs_densify_prune: per Gaussian an output count (0 pruned, 1 kept, 2 cloned
// or split), an exclusive scan of the counts, and a scatter that writes the
// new parameters and Adam moments in input order.  Split children use the
// caller's standard normal draws.  The new count is written to the device;
// nothing is written past the output capacity.
#include "rowcopy.h"

namespace gs {
namespace {

constexpr int kDThreads = 256;
constexpr int kDItems = 8;
constexpr int kDTile = kDThreads * kDItems;

__global__ void __launch_bounds__(256) k_grad_stats(
    const uint32_t* __restrict__ tt, const uint32_t* __restrict__ poff,
    const float* __restrict__ grad_pair, const int32_t* __restrict__ fl, int64_t n, ViewTable vt,
    float* __restrict__ accum, float* __restrict__ denom) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || fl[F_OVERFLOW]) return;
  float a = 0.0f, d = 0.0f;
  for (int v = 0; v < vt.n_views; ++v) {
    const int64_t ri = (int64_t)v * n + i;
    const uint32_t c = tt[ri];
    if (c == 0) continue;
    const float* gp = grad_pair + (int64_t)poff[ri] * kPairGrad;
    double gx = 0.0, gy = 0.0;
    uint32_t k = 0;
    for (; k + 8 <= c; k += 8) {  // eight loads in flight, additions in order
      float2 m[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        m[u] = *reinterpret_cast<const float2*>(gp + (int64_t)(k + u) * kPairGrad + 8);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        gx += m[u].x;
        gy += m[u].y;
      }
    }
    for (; k < c; ++k) {
      gx += gp[(int64_t)k * kPairGrad + 8];
      gy += gp[(int64_t)k * kPairGrad + 9];
    }
    const double nx = gx * 0.5 * vt.v[v].W, ny = gy * 0.5 * vt.v[v].H;
    a += (float)sqrt(nx * nx + ny * ny);
    d += 1.0f;
  }
  accum[i] += a;
  denom[i] += d;
}

struct DensifyCfg {
  float tau_p, eps_alpha, percent_dense, extent;
};

__device__ __forceinline__ int out_count(const float* logits, const float* log_scales,
                                         const float* accum, const float* denom, int64_t i,
                                         const DensifyCfg& c, bool* split) {
  const float o = 1.0f / (1.0f + expf(-logits[i]));
  *split = false;
  if (!(o >= c.eps_alpha)) return 0;
  const float dn = denom[i];
  const bool sel = dn > 0.0f && accum[i] / dn >= c.tau_p;
  if (!sel) return 1;
  const float smax = expf(fmaxf(log_scales[3 * i], fmaxf(log_scales[3 * i + 1], log_scales[3 * i + 2])));
  *split = smax > c.percent_dense * c.extent;
  return 2;
}

__global__ void __launch_bounds__(kDThreads) k_densify_count(
    const float* __restrict__ logits, const float* __restrict__ log_scales,
    const float* __restrict__ accum, const float* __restrict__ denom, int64_t n, DensifyCfg cfg,
    uint32_t* __restrict__ offs, uint64_t* __restrict__ btot) {
  __shared__ uint32_t wsum[kDThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kDTile + (int64_t)threadIdx.x * kDItems;
  uint32_t c[kDItems];
  uint32_t s = 0;
  for (int k = 0; k < kDItems; ++k) {
    const int64_t i = base + k;
    bool sp;
    c[k] = i < n ? (uint32_t)out_count(logits, log_scales, accum, denom, i, cfg, &sp) : 0u;
    s += c[k];
  }
  const int lane = lane_id(), w = threadIdx.x / kWave;
  uint32_t incl = s;
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  if (lane == kWave - 1) wsum[w] = incl;
  __syncthreads();
  uint32_t woff = 0;
  for (int k = 0; k < w; ++k) woff += wsum[k];
  uint32_t run = woff + incl - s;
  for (int k = 0; k < kDItems; ++k) {
    const int64_t i = base + k;
    if (i < n) offs[i] = run;
    run += c[k];
  }
  if (threadIdx.x == kDThreads - 1) btot[blockIdx.x] = run;
}

__global__ void __launch_bounds__(1024) k_densify_totals(uint64_t* __restrict__ btot,
                                                         int64_t nblocks,
                                                         int32_t* __restrict__ n_out) {
  __shared__ uint64_t wsum[1024 / kWave];
  __shared__ uint64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int lane = lane_id(), w = threadIdx.x / kWave;
  for (int64_t base = 0; base < nblocks; base += 1024) {
    const int64_t idx = base + threadIdx.x;
    const uint64_t x = idx < nblocks ? btot[idx] : 0ull;
    uint64_t incl = x;
    for (int o = 1; o < kWave; o <<= 1) {
      const uint64_t y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    uint64_t woff = carry;
    for (int k = 0; k < w; ++k) woff += wsum[k];
    if (idx < nblocks) btot[idx] = woff + incl - x;
    __syncthreads();
    if (threadIdx.x == 1023) carry = woff + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) *n_out = (int32_t)carry;
}

// The five arrays of one set (parameters, first or second moments).
struct GaussianSet {
  const float *mean, *ls, *q, *op, *sh;
  float *o_mean, *o_ls, *o_q, *o_op, *o_sh;
};
struct DensifyIO {
  GaussianSet set[3];
};

// A workgroup takes 256 Gaussians of one set.  Their outputs are one range of
// rows, so each thread notes its rows' source in LDS and the workgroup then
// copies array after array in output order, coalesced and with four loads in
// flight; the moments of new Gaussians are zero.  Bound by HBM.  Before, one
// thread wrote all 15 arrays' rows of its Gaussian, 4 bytes at a time and up
// to 192 bytes from its neighbour's: 1197 us for 300k Gaussians of degree 3
// (430 MB), now 97 us (4.4 TB/s).
template <int K3>
__global__ void __launch_bounds__(kCopyThreads) k_densify_write(
    DensifyIO io, const float* __restrict__ accum, const float* __restrict__ denom,
    const float* __restrict__ normals, int64_t n, DensifyCfg cfg,
    const uint32_t* __restrict__ offs, const uint64_t* __restrict__ bpre, int64_t cap) {
  // source of each output row: bit 31 a split child, bit 30 a new Gaussian
  constexpr uint32_t kSplit = 1u << 31, kNew = 1u << 30, kIdx = kNew - 1u;
  static_assert(kDTile % kCopyThreads == 0, "a workgroup's Gaussians share one block offset");
  __shared__ uint32_t from[2 * kCopyThreads];
  __shared__ int rows;
  const float *p_mean = io.set[0].mean, *p_ls = io.set[0].ls, *p_q = io.set[0].q;
  const int64_t i0 = (int64_t)blockIdx.x * kCopyThreads, i = i0 + threadIdx.x;
  const bool params = blockIdx.y == 0;
  const int64_t o0 = (int64_t)offs[i0] + (int64_t)bpre[i0 / kDTile];
  if (threadIdx.x == 0) rows = 0;
  __syncthreads();
  if (i < n) {
    bool split;
    const int c = out_count(io.set[0].op, p_ls, accum, denom, i, cfg, &split);
    const int64_t o = (int64_t)offs[i] + (int64_t)bpre[i0 / kDTile];
    if (c > 0 && o + c <= cap) {
      const int r = (int)(o - o0);
      const uint32_t mark = threadIdx.x | (split ? kSplit | kNew : 0u);
      from[r] = mark;
      if (c == 2) from[r + 1] = mark | kNew;
      atomicMax(&rows, r + c);
      if (split && params) {
        // two children with means p + R (s * n_k) and scales s / 1.6
        double q[4] = {p_q[4 * i], p_q[4 * i + 1], p_q[4 * i + 2], p_q[4 * i + 3]};
        const double qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
        for (int k = 0; k < 4; ++k) q[k] /= qn;
        const double w = q[0], x = q[1], y = q[2], z = q[3];
        const double R[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                             2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                             2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)};
        const double s[3] = {exp((double)p_ls[3 * i]), exp((double)p_ls[3 * i + 1]),
                             exp((double)p_ls[3 * i + 2])};
        for (int ch = 0; ch < 2; ++ch) {
          const int64_t oc = o + ch;
          const float* nk = normals + 6 * i + 3 * ch;
          const double d[3] = {s[0] * nk[0], s[1] * nk[1], s[2] * nk[2]};
          for (int k = 0; k < 3; ++k) {
            io.set[0].o_mean[3 * oc + k] =
                (float)((double)p_mean[3 * i + k] + R[3 * k] * d[0] + R[3 * k + 1] * d[1] +
                        R[3 * k + 2] * d[2]);
            io.set[0].o_ls[3 * oc + k] = (float)((double)p_ls[3 * i + k] - log(1.6));
          }
        }
      }
    }
  }
  __syncthreads();
  const int nrow = rows;
  const GaussianSet g = io.set[blockIdx.y];
  const auto row = [&](int r) -> int64_t {
    const uint32_t f = from[r];
    return !params && (f & kNew) ? kRowZero : i0 + (int64_t)(f & kIdx);
  };
  const auto row_unsplit = [&](int r) -> int64_t {
    return params && (from[r] & kSplit) ? kRowSkip : row(r);
  };
  copy_rows<K3>(g.sh, g.o_sh + o0 * K3, nrow, row);
  copy_rows<4>(g.q, g.o_q + o0 * 4, nrow, row);
  copy_rows<3>(g.mean, g.o_mean + o0 * 3, nrow, row_unsplit);
  copy_rows<3>(g.ls, g.o_ls + o0 * 3, nrow, row_unsplit);
  copy_rows<1>(g.op, g.o_op + o0, nrow, row);
}

template <int K3>
void write_launch(const DensifyIO& io, const float* accum, const float* denom,
                  const float* normals, int64_t n, const DensifyCfg& cfg, const uint32_t* offs,
                  const uint64_t* bpre, int64_t cap, hipStream_t s) {
  const dim3 grid((unsigned)((n + kCopyThreads - 1) / kCopyThreads), 3);
  hipLaunchKernelGGL(k_densify_write<K3>, grid, dim3(kCopyThreads), 0, s, io, accum, denom,
                     normals, n, cfg, offs, bpre, cap);
}

}  // namespace

size_t densify_tmp_bytes(int64_t n) {
  const int64_t nb = (n + kDTile - 1) / kDTile;
  return (size_t)(n + 64) * 4 + (size_t)(nb + 8) * 8 + 256;
}

hipError_t launch_grad_stats(const Plan& P, void* ws, float* accum, float* denom, hipStream_t s) {
  if (P.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_grad_stats, dim3((unsigned)((P.n + 255) / 256)), dim3(256), 0, s,
                     ws_at<uint32_t>(ws, P.off_tt), ws_at<uint32_t>(ws, P.off_poff),
                     ws_at<float>(ws, P.off_grad_pair), ws_at<int32_t>(ws, P.off_flags), P.n,
                     P.vt, accum, denom);
  return hipGetLastError();
}

hipError_t launch_densify(const gs_gaussians& g, const gs_gaussian_grads& m,
                          const gs_gaussian_grads& v, const float* accum, const float* denom,
                          const float* normals, float tau_p, float eps_alpha, float percent_dense,
                          float extent, const gs_gaussian_grads& out, const gs_gaussian_grads& out_m,
                          const gs_gaussian_grads& out_v, int64_t cap, int32_t* n_out, void* tmp,
                          hipStream_t s) {
  const int64_t n = g.n;
  const int64_t nb = (n + kDTile - 1) / kDTile;
  uint32_t* offs = static_cast<uint32_t*>(tmp);
  uint64_t* btot = reinterpret_cast<uint64_t*>(static_cast<char*>(tmp) + (((size_t)(n + 64) * 4 + 255) / 256) * 256);
  const DensifyCfg cfg{tau_p, eps_alpha, percent_dense, extent};
  if (nb > 0)
    hipLaunchKernelGGL(k_densify_count, dim3((unsigned)nb), dim3(kDThreads), 0, s, g.opacity_logits,
                       g.log_scales, accum, denom, n, cfg, offs, btot);
  hipLaunchKernelGGL(k_densify_totals, dim3(1), dim3(1024), 0, s, btot, nb, n_out);
  if (n > 0) {
    const auto set = [](const auto& in, const gs_gaussian_grads& o) {
      return GaussianSet{in.means, in.log_scales, in.quats, in.opacity_logits, in.sh,
                         o.means,  o.log_scales,  o.quats,  o.opacity_logits,  o.sh};
    };
    const DensifyIO io{{set(g, out), set(m, out_m), set(v, out_v)}};
    const auto launch = g.sh_degree == 0   ? write_launch<3>
                        : g.sh_degree == 1 ? write_launch<12>
                        : g.sh_degree == 2 ? write_launch<27>
                                           : write_launch<48>;
    launch(io, accum, denom, normals, n, cfg, offs, btot, cap, s);
  }
  return hipGetLastError();
}

}  // namespace gs
