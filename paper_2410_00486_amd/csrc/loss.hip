// Rendered loss of Eq. (9) with a depth term:
//   L = (1 - ls) mean|C - C*| + ls (1 - SSIM(C, C*)) + ld mean|D - D*|
// and its image gradients dL/dC, dL/dD, which then drive the raster
// backward as explicit upstream gradients.  SSIM follows the 3DGS pipeline
// the paper retains (Sec. IV-A): per channel, 11x11 Gaussian window with
// sigma 1.5, zero padding, C1 = 0.01^2, C2 = 0.03^2.
//
// Stencil work on 32x32 output tiles: the 42x42 halo of the image (and the
// target) is staged in LDS, filtered along rows then columns, a thread forming
// eight (four) neighbouring outputs from the inputs it reads once.  On 16x16
// tiles, with an LDS read per tap and the halo fetched one element after
// another, 1200x680 took 47 and 35 us, now 32 and 25 (45 and 33 before the
// loads of the halo were issued together).  Bound by VALU issue (16 us of the
// first) and the phases' latencies; 59 and 49 MB move.  Pass 1 forms
// the five windowed moments, the SSIM value and its derivatives with respect
// to the moments of C (three maps); pass 2 filters those maps with the
// (symmetric) window -- the adjoint of the forward filtering -- and
// assembles dL/dC.  Per-tile sums are reduced per view in a fixed order.
#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kT = 32;            // output tile edge
constexpr int kR = 5;             // window radius
constexpr int kH = kT + 2 * kR;   // halo edge, 42
constexpr int kRowOut = 8;        // outputs per thread, row filter
constexpr int kColOut = 4;        // and column filter
static_assert(kH * (kT / kRowOut) <= 256 && kT * (kT / kColOut) == 256, "one pass of 256 threads");
constexpr float kC1 = 1e-4f;      // 0.01^2
constexpr float kC2 = 9e-4f;      // 0.03^2

__constant__ float c_win[11] = {
    0.0010284048259f, 0.0075987582919f, 0.0360007721186f, 0.1093606895208f,
    0.2130055377627f, 0.2660117248603f, 0.2130055377627f, 0.1093606895208f,
    0.0360007721186f, 0.0075987582919f, 0.0010284048259f};

struct SsimView {
  int32_t W, H, tiles_x, tile_off, pix_off;
};
struct SsimTable {
  int32_t n_views, total_tiles;
  SsimView v[kMaxViews];
};

__device__ __forceinline__ int ssim_view(const SsimTable& t, int tile) {
  int v = 0;
  while (v + 1 < t.n_views && tile >= t.v[v + 1].tile_off) ++v;
  return v;
}

// The pixel (index in its plane) of the halo element that this thread loads
// in round u, -1 outside the image.  The loads of all rounds are issued
// unconditionally (from the plane's first pixel instead), so that they are in
// flight together.
constexpr int kLoads = (kH * kH + 255) / 256;
__device__ __forceinline__ int64_t halo_pixel(int u, int x0, int y0, const SsimView& vi) {
  const int k = (int)threadIdx.x + 256 * u;
  const int gx = x0 + k % kH, gy = y0 + k / kH;
  const bool in = k < kH * kH && gx >= 0 && gy >= 0 && gx < vi.W && gy < vi.H;
  return in ? (int64_t)gy * vi.W + gx : -1;
}

// Pass 1: grid (tiles over all views, 3 channels), 256 threads.
__global__ void __launch_bounds__(256) k_ssim_fwd(const float* __restrict__ color,
                                                  const float* __restrict__ target,
                                                  SsimTable tb, float* __restrict__ dmaps,
                                                  int64_t plane, float* __restrict__ part) {
  __shared__ float sx[kH][kH + 1], sy[kH][kH + 1];
  __shared__ float hm[5][kH][kT + 1];
  __shared__ float red[2][256 / kWave];
  const int tile = blockIdx.x, ch = blockIdx.y;
  const int v = ssim_view(tb, tile);
  const SsimView vi = tb.v[v];
  const int lt = tile - vi.tile_off;
  const int x0 = (lt % vi.tiles_x) * kT - kR, y0 = (lt / vi.tiles_x) * kT - kR;
  const int64_t npx = (int64_t)vi.W * vi.H;
  const float* X = color + 3 * (int64_t)vi.pix_off + ch * npx;
  const float* Y = target + 3 * (int64_t)vi.pix_off + ch * npx;
  {
    float x[kLoads], y[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int64_t at = halo_pixel(u, x0, y0, vi);
      x[u] = X[at < 0 ? 0 : at];
      y[u] = Y[at < 0 ? 0 : at];
      if (at < 0) x[u] = y[u] = 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int k = (int)threadIdx.x + 256 * u;
      if (k < kH * kH) {
        sx[k / kH][k % kH] = x[u];
        sy[k / kH][k % kH] = y[u];
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < kH * (kT / kRowOut)) {
    const int r = threadIdx.x / (kT / kRowOut), c = threadIdx.x % (kT / kRowOut) * kRowOut;
    float a[kRowOut][5];
#pragma unroll
    for (int o = 0; o < kRowOut; ++o)
#pragma unroll
      for (int q = 0; q < 5; ++q) a[o][q] = 0.0f;
#pragma unroll
    for (int j = 0; j < kRowOut + 2 * kR; ++j) {
      const float x = sx[r][c + j], y = sy[r][c + j];
      const float in5[5] = {x, y, x * x, y * y, x * y};
#pragma unroll
      for (int o = 0; o < kRowOut; ++o)
        if (j - o >= 0 && j - o < 11) {
#pragma unroll
          for (int q = 0; q < 5; ++q) a[o][q] = fmaf(c_win[j - o], in5[q], a[o][q]);
        }
    }
#pragma unroll
    for (int o = 0; o < kRowOut; ++o)
#pragma unroll
      for (int q = 0; q < 5; ++q) hm[q][r][c + o] = a[o][q];
  }
  __syncthreads();
  const int c = threadIdx.x % kT, r0 = threadIdx.x / kT * kColOut;
  float m[kColOut][5];
#pragma unroll
  for (int o = 0; o < kColOut; ++o)
#pragma unroll
    for (int q = 0; q < 5; ++q) m[o][q] = 0.0f;
#pragma unroll
  for (int j = 0; j < kColOut + 2 * kR; ++j) {
    float h[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) h[q] = hm[q][r0 + j][c];
#pragma unroll
    for (int o = 0; o < kColOut; ++o)
      if (j - o >= 0 && j - o < 11) {
#pragma unroll
        for (int q = 0; q < 5; ++q) m[o][q] = fmaf(c_win[j - o], h[q], m[o][q]);
      }
  }
  const int gx = x0 + kR + c;
  float s_val = 0.0f, l1 = 0.0f;
#pragma unroll
  for (int o = 0; o < kColOut; ++o) {
    const int r = r0 + o, gy = y0 + kR + r;
    if (gx >= vi.W || gy >= vi.H) continue;
    const float m1 = m[o][0], my = m[o][1], m2 = m[o][2], myy = m[o][3], m3 = m[o][4];
    const float A1 = 2.0f * m1 * my + kC1;
    const float A2 = 2.0f * (m3 - m1 * my) + kC2;
    const float B1 = m1 * m1 + my * my + kC1;
    const float B2 = (m2 - m1 * m1) + (myy - my * my) + kC2;
    const float S = (A1 * A2) / (B1 * B2);
    const float d1 = S * (2.0f * my / A1 - 2.0f * my / A2 - 2.0f * m1 / B1 + 2.0f * m1 / B2);
    const float d2 = -S / B2;
    const float d3 = 2.0f * S / A2;
    const int64_t p = (int64_t)vi.pix_off * 3 + ch * npx + (int64_t)gy * vi.W + gx;
    dmaps[p] = d1;
    dmaps[p + plane] = d2;
    dmaps[p + 2 * plane] = d3;
    s_val += S;
    l1 += fabsf(sx[r + kR][c + kR] - sy[r + kR][c + kR]);
  }
  s_val = wave_sum(s_val);
  l1 = wave_sum(l1);
  if (lane_id() == 0) {
    red[0][threadIdx.x / kWave] = s_val;
    red[1][threadIdx.x / kWave] = l1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float a = 0, b = 0;
    for (int k = 0; k < 256 / kWave; ++k) {
      a += red[0][k];
      b += red[1][k];
    }
    part[4 * ((int64_t)tile * 3 + ch)] = a;
    part[4 * ((int64_t)tile * 3 + ch) + 1] = b;
  }
}

// Pass 2: adjoint filtering of the derivative maps, dL/dC and dL/dD.
__global__ void __launch_bounds__(256) k_ssim_bwd(
    const float* __restrict__ color, const float* __restrict__ target,
    const float* __restrict__ depth, const float* __restrict__ target_depth, SsimTable tb,
    const float* __restrict__ dmaps, int64_t plane, float lambda_ssim, float lambda_depth,
    float* __restrict__ dL_dcolor, float* __restrict__ dL_ddepth, float* __restrict__ part) {
  __shared__ float sd[3][kH][kH + 1];
  __shared__ float hm[3][kH][kT + 1];
  __shared__ float red[256 / kWave];
  const int tile = blockIdx.x, ch = blockIdx.y;
  const int v = ssim_view(tb, tile);
  const SsimView vi = tb.v[v];
  const int lt = tile - vi.tile_off;
  const int x0 = (lt % vi.tiles_x) * kT - kR, y0 = (lt / vi.tiles_x) * kT - kR;
  const int64_t npx = (int64_t)vi.W * vi.H;
  const int64_t cbase = 3 * (int64_t)vi.pix_off + ch * npx;
  {
    float d[kLoads][3];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int64_t at = halo_pixel(u, x0, y0, vi);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        d[u][q] = dmaps[cbase + (at < 0 ? 0 : at) + q * plane];
        if (at < 0) d[u][q] = 0.0f;
      }
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int k = (int)threadIdx.x + 256 * u;
      if (k < kH * kH) {
#pragma unroll
        for (int q = 0; q < 3; ++q) sd[q][k / kH][k % kH] = d[u][q];
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < kH * (kT / kRowOut)) {
    const int r = threadIdx.x / (kT / kRowOut), c = threadIdx.x % (kT / kRowOut) * kRowOut;
    float a[kRowOut][3];
#pragma unroll
    for (int o = 0; o < kRowOut; ++o) a[o][0] = a[o][1] = a[o][2] = 0.0f;
#pragma unroll
    for (int j = 0; j < kRowOut + 2 * kR; ++j) {
      const float d[3] = {sd[0][r][c + j], sd[1][r][c + j], sd[2][r][c + j]};
#pragma unroll
      for (int o = 0; o < kRowOut; ++o)
        if (j - o >= 0 && j - o < 11) {
#pragma unroll
          for (int q = 0; q < 3; ++q) a[o][q] = fmaf(c_win[j - o], d[q], a[o][q]);
        }
    }
#pragma unroll
    for (int o = 0; o < kRowOut; ++o)
#pragma unroll
      for (int q = 0; q < 3; ++q) hm[q][r][c + o] = a[o][q];
  }
  __syncthreads();
  const int c = threadIdx.x % kT, r0 = threadIdx.x / kT * kColOut;
  float g[kColOut][3];
#pragma unroll
  for (int o = 0; o < kColOut; ++o) g[o][0] = g[o][1] = g[o][2] = 0.0f;
#pragma unroll
  for (int j = 0; j < kColOut + 2 * kR; ++j) {
    const float h[3] = {hm[0][r0 + j][c], hm[1][r0 + j][c], hm[2][r0 + j][c]};
#pragma unroll
    for (int o = 0; o < kColOut; ++o)
      if (j - o >= 0 && j - o < 11) {
#pragma unroll
        for (int q = 0; q < 3; ++q) g[o][q] = fmaf(c_win[j - o], h[q], g[o][q]);
      }
  }
  const int gx = x0 + kR + c;
  float ld = 0.0f;
#pragma unroll
  for (int o = 0; o < kColOut; ++o) {
    const int gy = y0 + kR + r0 + o;
    if (gx >= vi.W || gy >= vi.H) continue;
    const float g1 = g[o][0], g2 = g[o][1], g3 = g[o][2];
    const int64_t p = cbase + (int64_t)gy * vi.W + gx;
    const float x = color[p], y = target[p];
    const float inv_n = 1.0f / (3.0f * (float)npx);
    const float dssim = (g1 + 2.0f * x * g2 + y * g3) * inv_n;
    const float dx = x - y;
    const float sgn = dx > 0.0f ? 1.0f : (dx < 0.0f ? -1.0f : 0.0f);
    dL_dcolor[p] = (1.0f - lambda_ssim) * sgn * inv_n - lambda_ssim * dssim;
    if (ch == 0) {
      const int64_t q = (int64_t)vi.pix_off + (int64_t)gy * vi.W + gx;
      float gd = 0.0f;
      if (target_depth) {
        const float dd = depth[q] - target_depth[q];
        gd = dd > 0.0f ? lambda_depth / (float)npx : (dd < 0.0f ? -lambda_depth / (float)npx : 0.0f);
        ld += fabsf(dd);
      }
      dL_ddepth[q] = gd;
    }
  }
  if (ch == 0) {
    ld = wave_sum(ld);
    if (lane_id() == 0) red[threadIdx.x / kWave] = ld;
    __syncthreads();
    if (threadIdx.x == 0) {
      float a = 0;
      for (int k = 0; k < 256 / kWave; ++k) a += red[k];
      part[4 * ((int64_t)tile * 3) + 2] = a;
    }
  }
}

// Per-view loss from the per-tile sums, fixed order.
__global__ void __launch_bounds__(256) k_ssim_loss(const float* __restrict__ part, SsimTable tb,
                                                   float lambda_ssim, float lambda_depth,
                                                   int has_depth, float* __restrict__ loss) {
  const int v = blockIdx.x;
  const SsimView vi = tb.v[v];
  const int nt = (v + 1 < tb.n_views ? tb.v[v + 1].tile_off : tb.total_tiles) - vi.tile_off;
  double s = 0, l1 = 0, ld = 0;
  for (int k = threadIdx.x; k < nt; k += 256) {
    const int64_t t = vi.tile_off + k;
    for (int ch = 0; ch < 3; ++ch) {
      s += part[4 * (t * 3 + ch)];
      l1 += part[4 * (t * 3 + ch) + 1];
    }
    ld += part[4 * (t * 3) + 2];
  }
  __shared__ double red[3][256 / kWave];
  s = wave_sum(s);
  l1 = wave_sum(l1);
  ld = wave_sum(ld);
  if (lane_id() == 0) {
    red[0][threadIdx.x / kWave] = s;
    red[1][threadIdx.x / kWave] = l1;
    red[2][threadIdx.x / kWave] = ld;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0, b = 0, c = 0;
    for (int k = 0; k < 256 / kWave; ++k) {
      a += red[0][k];
      b += red[1][k];
      c += red[2][k];
    }
    const double n3 = 3.0 * (double)vi.W * vi.H;
    double L = (1.0 - lambda_ssim) * b / n3 + lambda_ssim * (1.0 - a / n3);
    if (has_depth) L += lambda_depth * c / ((double)vi.W * vi.H);
    loss[v] = (float)L;
  }
}

}  // namespace

int64_t ssim_tiles(const Plan& P) {
  int64_t t = 0;
  for (int v = 0; v < P.vt.n_views; ++v)
    t += (int64_t)((P.vt.v[v].W + kT - 1) / kT) * ((P.vt.v[v].H + kT - 1) / kT);
  return t;
}

hipError_t launch_render_loss(const Plan& P, void* ws, const float* color, const float* depth,
                              const float* target_rgb, const float* target_depth,
                              double lambda_ssim, float* dL_dcolor, float* dL_ddepth,
                              float* loss_per_view, hipStream_t s) {
  SsimTable tb{};
  tb.n_views = P.vt.n_views;
  int32_t t = 0;
  for (int v = 0; v < P.vt.n_views; ++v) {
    const ViewInfo& vi = P.vt.v[v];
    SsimView& sv = tb.v[v];
    sv.W = vi.W;
    sv.H = vi.H;
    sv.tiles_x = (vi.W + kT - 1) / kT;
    sv.tile_off = t;
    sv.pix_off = vi.pix_off;
    t += sv.tiles_x * ((vi.H + kT - 1) / kT);
  }
  tb.total_tiles = t;
  if (t == 0) return hipSuccess;
  float* dmaps = ws_at<float>(ws, P.off_ssim_maps);
  float* part = ws_at<float>(ws, P.off_ssim_part);
  const int64_t plane = 3 * ((int64_t)P.vt.v[P.vt.n_views - 1].pix_off +
                             (int64_t)P.vt.v[P.vt.n_views - 1].W * P.vt.v[P.vt.n_views - 1].H);
  hipLaunchKernelGGL(k_ssim_fwd, dim3(t, 3), dim3(256), 0, s, color, target_rgb, tb, dmaps, plane,
                     part);
  hipLaunchKernelGGL(k_ssim_bwd, dim3(t, 3), dim3(256), 0, s, color, target_rgb, depth,
                     target_depth, tb, dmaps, plane, (float)lambda_ssim, P.cfg.lambda_depth,
                     dL_dcolor, dL_ddepth, part);
  if (loss_per_view)
    hipLaunchKernelGGL(k_ssim_loss, dim3(P.vt.n_views), dim3(256), 0, s, part, tb,
                       (float)lambda_ssim, P.cfg.lambda_depth, target_depth ? 1 : 0,
                       loss_per_view);
  return hipGetLastError();
}

}  // namespace gs
