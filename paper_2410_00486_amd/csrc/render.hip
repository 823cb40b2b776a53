// a3-a5: per-tile compositing (Eq. (1)), its pixel-wise backward
// (Eqs. (2)-(4)) and the splat-wise backward (Sec. III-C-1, below).
//
// Forward: one wave64 per 8x8 block of pixels, one pixel per lane.  The
// tile's depth-sorted list is taken in batches of 64: a lane holds one
// record, forms its offsets from the block's columns and rows of sample
// points, and drops it when it is below alpha 1/255 over the whole block (a
// tile box is the axis-aligned box of an ellipse: 18-22 % of the pairs of
// 8x8 tiles reach no pixel of theirs, 55 % of the blocks of a 16x16 tile's
// pairs).  What is left goes to LDS in list order and every lane walks it
// front to back.  The wavefront leaves when every pixel has stopped.
//
// Measured (forward kernel, before -> after): 1200x680 view in 16x16 tiles,
// 627k pairs: 398 -> 69 us (before: one wavefront per 16x16 tile, four
// pixels per lane); four such views, 2.7M pairs: 778 -> 188 us; 8x8 tiles:
// 16 views, 25M pairs: 1443 -> 859 us; 8 mixed views, 6.0M pairs: 579 ->
// 332 us (the longest list, 4562 pairs, is one wavefront's serial work).
// Bound by VALU issue (about 80 instructions for four splats of 64 pixels)
// and, for the longest lists, by the latency of one wavefront.  Neighbouring
// tiles on one XCD (xcd_item): 901 -> 850 us on the 16-view batch.
//
// Backward (pixel-wise): a workgroup per tile, again a wavefront per 8x8
// block, back to front from the tile's last used position.  Each lane
// recomputes alpha with the forward's code (so every skip decision is the
// forward's), undoes the transmittance by division from T_final and keeps
// the loss-weighted sum of what lies behind.  The ten per-pair partial
// gradients of a Gaussian are summed over the wavefront with DPP, over the
// tile's blocks in LDS in a fixed order, and written to the pair's own slot:
// no atomics, deterministic.
#include <type_traits>

#include "tilesort.h"

namespace gs {
namespace {

constexpr float kAlphaMax = 0.99f;
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kTMin = 1e-4f;
// Pixel gradients and splat colours below this cannot overflow the raster
// backward's sums of their products.
constexpr float kTame = 1e15f;

// DPP move with zero fill where the lane has no source or its row is masked.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xF, true));
}

// Sum over the wavefront, result in lane 63: xor 1 and xor 2 within quads,
// half-row and row mirrors (sums of 8 and 16), then row broadcasts of lanes
// 15 and 31 into the upper rows.  Every lane must be active.
__device__ __forceinline__ float wave_sum_to_last(float x) {
  x += dpp<0xB1>(x);        // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);        // quad_perm [2,3,0,1]
  x += dpp<0x141>(x);       // row_half_mirror
  x += dpp<0x140>(x);       // row_mirror
  x += dpp<0x142, 0xA>(x);  // row_bcast:15 -> rows 1 and 3
  x += dpp<0x143, 0xC>(x);  // row_bcast:31 -> rows 2 and 3
  return x;
}

// Sums of ten values over the wavefront, scattered: afterwards lane l of
// the first row holds the total of value rs_index(l) (lanes whose index is
// -1 hold nothing).  Four in-row halving steps -- each lane keeps half of
// its values and adds the partner's copy of that half: row mirror (partner
// differs in bit 3), half-row mirror (bit 2), quad reversal (bit 1), quad
// swap (bit 0) -- then the row pairs (bit 4) and half-waves (bit 5) are
// added with the gfx950 lane swaps.  In the first two steps the halves are
// whole banks of four lanes, so the lanes that keep the other value are
// written by a second DPP add with a bank mask and nothing is selected (two
// instructions for two values instead of three).  28 VALU operations instead
// of the 60 of ten separate reductions.  Every lane must be active.  (A DPP
// read needs two wait states after the VALU write of its register.)
__device__ __forceinline__ float sel(bool c, float a, float b) { return c ? a : b; }

#define GS_ADD_MIRROR(D, X, CTRL, BANKS) \
  "v_add_f32_dpp " D ", " X ", " X " " CTRL " row_mask:0xf bank_mask:" BANKS "\n\t"
__device__ __forceinline__ float reduce_scatter10(const float* g) {
  const int l = threadIdx.x & 15;
  const bool b1 = l & 2, b0 = l & 1;
  float h0, h1, h2, h3, h4, u0, u1, u2;
  asm("s_nop 1\n\t"
      GS_ADD_MIRROR("%0", "%5", "row_mirror", "0xf") GS_ADD_MIRROR("%1", "%6", "row_mirror", "0xf")
      GS_ADD_MIRROR("%2", "%7", "row_mirror", "0xf") GS_ADD_MIRROR("%3", "%8", "row_mirror", "0xf")
      GS_ADD_MIRROR("%4", "%9", "row_mirror", "0xf") GS_ADD_MIRROR("%0", "%10", "row_mirror", "0xc")
      GS_ADD_MIRROR("%1", "%11", "row_mirror", "0xc") GS_ADD_MIRROR("%2", "%12", "row_mirror", "0xc")
      GS_ADD_MIRROR("%3", "%13", "row_mirror", "0xc") GS_ADD_MIRROR("%4", "%14", "row_mirror", "0xc")
      : "=&v"(h0), "=&v"(h1), "=&v"(h2), "=&v"(h3), "=&v"(h4)
      : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(g[4]), "v"(g[5]), "v"(g[6]), "v"(g[7]),
        "v"(g[8]), "v"(g[9]));
  asm("s_nop 1\n\t"
      GS_ADD_MIRROR("%0", "%3", "row_half_mirror", "0xf") GS_ADD_MIRROR("%1", "%4", "row_half_mirror", "0xf")
      GS_ADD_MIRROR("%2", "%5", "row_half_mirror", "0xf") GS_ADD_MIRROR("%0", "%6", "row_half_mirror", "0xa")
      GS_ADD_MIRROR("%1", "%7", "row_half_mirror", "0xa")
      : "=&v"(u0), "=&v"(u1), "=&v"(u2)
      : "v"(h0), "v"(h1), "v"(h2), "v"(h3), "v"(h4));
  const float w0 = sel(b1, u2, u0) + dpp<0x1B>(sel(b1, u0, u2));  // quad [3,2,1,0]
  const float w1 = u1 + dpp<0x1B>(u1);                            // (lanes with b1: unused)
  float z = sel(b0, w1, w0) + dpp<0xB1>(sel(b0, w0, w1));         // quad [1,0,3,2]
  const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(z),
                                                    false, false);
  z = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
  const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z),
                                                    false, false);
  return __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
}
#undef GS_ADD_MIRROR

// Which of the ten values reduce_scatter10 leaves in lane l (first 16 lanes
// meaningful), -1 for none.
__device__ __forceinline__ int rs_index(int lane) {
  const int l = lane & 15;
  const int j = ((l & 2) ? 2 : 0) + (l & 1);       // index among u
  if (j >= 3) return -1;
  const int hidx = ((l & 4) ? 3 : 0) + j;          // index among h
  if (hidx >= 5) return -1;
  return ((l & 8) ? 5 : 0) + hidx;
}

__device__ __forceinline__ int find_view(const ViewTable& vt, int gtile) {
  int v = 0;
  while (v + 1 < vt.n_views && gtile >= vt.v[v + 1].tile_off) ++v;
  return v;
}

// ------------------------------------------------------------------ forward
// A wavefront composites one 8x8 block of pixels ("sub-tile", one pixel per
// lane): the whole tile of 8x8 plans, one of the two or four blocks of 16x8
// and 16x16 tiles (a wavefront per tile there left 3225 wavefronts for a
// 1200x680 view, three per SIMD, and the longest list set the time).
constexpr int kSub = 8;
template <int TW, int TH>
constexpr int sub_tiles() {
  return TW * TH / (kSub * kSub);
}

// The largest last position over a tile's sub-tiles.
template <int NS>
__device__ __forceinline__ uint32_t tile_last_of(const uint32_t* __restrict__ tile_last,
                                                 int gtile) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < NS; ++k) m = max(m, tile_last[(int64_t)gtile * NS + k]);
  return m;
}

// What the compositing reads of a record.
struct FwdRec {
  double mx, my;
  float t, s1, s2, lo, z, r, g, b;
};
static_assert(sizeof(FwdRec) == 48 && offsetof(Rec, b) == 44, "first 48 bytes of a record");

// Highest exponent (base 2) at which a splat may still be skipped as a
// whole: alpha < 1/255 is an exponent below -7.9944, so what lies under -8
// is skipped at every pixel by the alpha test as well.  Both start from the
// same FP32 offsets and form p and q with one rounding each, so they differ
// by a few ulp of terms of at most 8 (1e-6 measured), and by the bound's own
// error far from the mean (max_exponent).
constexpr float kCullExp = -8.0f;
// Above this log2(opacity) the clamp at 0.99 can act (log2(0.99) = -0.0145).
constexpr float kClampLo = -0.0146f;

// Upper bound of the splat's exponent over the sample points of a block of
// pixels whose offsets (mean - sample point) span [xl, xh] x [yl, yh].  The
// quadratic's minimum over the rectangle is 0 when it holds the origin, and
// otherwise lies on an edge that faces the origin: the nearest x (y) of the
// rectangle with the best y (x) on it.  Both candidates lie in the
// rectangle.  The best y (x) is off by up to 8 half ulp (of cb, the edge's x,
// cc, its reciprocal and their products), 4.8e-7 of the largest offset d, and
// the quadratic there rises by at most cc (4.8e-7 d)^2, cc < 2.41 with the
// dilation of 0.3 px^2: (1e-6 d)^2 is added to the bound.  That is below the
// margin of kCullExp up to 7e4 pixels; splats close to the camera's plane
// reach the image from further away.
__device__ __forceinline__ float max_exponent(const FwdRec& r, float xl, float xh, float yl,
                                              float yh) {
  const float tt = r.t * r.t;
  const float ca = fmaf(r.s2, tt, r.s1), cb = r.t * (r.s1 - r.s2), cc = fmaf(r.s1, tt, r.s2);
  const float x0 = fminf(fmaxf(0.0f, xl), xh), y0 = fminf(fmaxf(0.0f, yl), yh);
  const float y1 = fminf(fmaxf(-cb * x0 * __builtin_amdgcn_rcpf(cc), yl), yh);
  const float x1 = fminf(fmaxf(-cb * y0 * __builtin_amdgcn_rcpf(ca), xl), xh);
  auto quad = [&](float dx, float dy) {
    const float p = fmaf(r.t, dy, dx), q = fmaf(-r.t, dx, dy);
    return fmaf(r.s1 * p, p, r.s2 * q * q);
  };
  // (the block's other offsets are within 8 pixels of the nearest one)
  const float d = fmaf(1e-6f, fmaxf(fabsf(x0), fabsf(y0)), 8e-6f);
  return fmaf(d, d, r.lo - fminf(quad(x0, y1), quad(x1, y0)));
}

// LDS of one forward wavefront: the batch's splats that can reach the
// sub-tile, in list order.  The offsets of a splat from the block's eight
// columns and eight rows of sample points are formed once per splat, in
// FP64, and rounded to FP32 -- the values each evaluation used to form for
// itself (two FP64 differences and two conversions, 20 of its about 92
// issue cycles).  A lane reads the offsets of four splats from its own
// column and row at once; rows of 68 floats keep the eight columns' 16-byte
// reads on different banks.
constexpr int kFwdSplats = 4;  // splats per step of the compositing loop
constexpr int kOffStride = kWave + 4;
struct FwdLds {
  float dx[kSub][kOffStride], dy[kSub][kOffStride];
  float4 shape[kWave];   // t, s1, s2, lo
  float4 colour[kWave];  // r, g, b, z
  uint32_t pos[kWave];   // 1 + position in the tile's list
};

// What the forward leaves for the splat-wise backward.  The slots of its
// steps, batch after batch, are the backward's lanes: a bucket is 64 slots.
// Stored: the state of every pixel before each bucket but a tile's first
// (bucket boff + k), the list position of every slot (kNoSplat in the few
// that only fill up a step), which of each 64 list positions were kept (one
// word per bucket entry of the list), and per tile the number of slots and of
// list positions looked at.
constexpr uint32_t kNoSplat = 0xFFFFFFFFu;
struct FwdSplat {
  const uint32_t* boff;
  float* ckpt;
  uint32_t* cand;
  uint64_t* kept;
  uint2* seen;
};

template <int TW, int TH, bool CKPT>
__device__ __forceinline__ void fwd_tile(int gtile, int sub, RecSrc lrec,
                                         const uint32_t* __restrict__ ranges,
                                         const float* __restrict__ cams, const ViewTable& vt,
                                         float* __restrict__ color,
                                         float* __restrict__ depth, float* __restrict__ T_final,
                                         uint32_t* __restrict__ last,
                                         uint32_t* __restrict__ tile_last,
                                         const float* __restrict__ target_rgb,
                                         const float* __restrict__ target_depth,
                                         float* __restrict__ tile_loss,
                                         const FwdSplat& K, FwdLds& S) {
  constexpr int NS = sub_tiles<TW, TH>();
  const int v = find_view(vt, gtile);
  const ViewInfo vi = vt.v[v];
  const int lt = gtile - vi.tile_off;
  const int lane = threadIdx.x;
  const int sx0 = NS == 1 ? 0 : kSub * (sub % (TW / kSub)), sy0 = NS == 1 ? 0 : kSub * (sub / (TW / kSub));
  const int bx0 = (lt % vi.tiles_x) * TW + sx0, by0 = (lt / vi.tiles_x) * TH + sy0;
  const int col = lane & (kSub - 1), row = lane / kSub;
  const int px = bx0 + col, py = by0 + row;
  const uint32_t s = ranges[2 * (int64_t)gtile], e = ranges[2 * (int64_t)gtile + 1];
  // the longest lists start first (work order) and end last: their
  // wavefronts take precedence at instruction issue over the shorter ones
  // sharing a SIMD
  if (e - s > 512) __builtin_amdgcn_s_setprio(3);
  else if (e - s > 128) __builtin_amdgcn_s_setprio(2);
  else if (e - s > 48) __builtin_amdgcn_s_setprio(1);

  const bool inside = (px < vi.W) && (py < vi.H);
  float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, D = 0.0f;
  uint32_t lastpos = 0;
  // pixels that have not stopped; the least alpha that is blended (none once
  // the pixel has stopped)
  uint64_t live = ballot64(inside);
  bool clamps = false;  // some splat so far can exceed the 0.99 clamp
  float amin = inside ? kAlphaMin : INFINITY;
  const double cx0 = (double)bx0 + 0.5, cy0 = (double)by0 + 0.5;
  // the next batch's records are fetched while this one is composited, and
  // the record ids of the batch after that one
  const uint32_t lane_u = (uint32_t)lane;
  auto fetch = [&](FwdRec& r, uint32_t id) {
    const float4* src = reinterpret_cast<const float4*>(lrec.base + id);
    float4* d4 = reinterpret_cast<float4*>(&r);
    d4[0] = src[0]; d4[1] = src[1]; d4[2] = src[2];
  };
  FwdRec r{};
  uint32_t id = 0;
  if (s + lane_u < e) fetch(r, lrec.id(s + lane_u));
  if (s + kWave + lane_u < e) id = lrec.id(s + kWave + lane_u);
  uint32_t slots = 0;  // steps' slots of the batches before this one
  // the tile's first bucket
  const uint32_t bucket0 = CKPT ? (uint32_t)__builtin_amdgcn_readfirstlane((int)K.boff[gtile]) : 0u;
  uint32_t b = s;
  for (; live != 0 && b < e; b += (uint32_t)kWave) {
    const bool has = b + lane_u < e;
    // (the sample points' coordinates are counted up from the block's corner
    // in each batch: kept over the batches they would take 32 registers)
    float ox[kSub], oy[kSub];
    double ax = cx0, ay = cy0;
    asm volatile("" : "+v"(ax), "+v"(ay));
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
      ox[k] = (float)(r.mx - ax);
      oy[k] = (float)(r.my - ay);
      ax += 1.0;
      ay += 1.0;
    }
    const bool keep = has && !(max_exponent(r, ox[kSub - 1], ox[0], oy[kSub - 1], oy[0]) < kCullExp);
    const uint64_t kept = ballot64(keep);
    // whole steps: the batch is filled up with splats of alpha 2^-inf = 0
    // (carrying up to three splats over to the next batch instead cost more
    // than the 3 % of slots that this leaves empty: 970 against 945 us on the
    // 16-view batch)
    const int total = (int)__popcll(kept);
    const int n = (total + kFwdSplats - 1) & ~(kFwdSplats - 1);
    clamps = clamps || ballot64(keep && r.lo > kClampLo) != 0;
    __syncthreads();  // (one wavefront: orders the LDS reads before its writes)
    if (keep) {
      const int at = (int)__popcll(kept & lanemask_lt());
#pragma unroll
      for (int k = 0; k < kSub; ++k) {
        S.dx[k][at] = ox[k];
        S.dy[k][at] = oy[k];
      }
      S.shape[at] = make_float4(r.t, r.s1, r.s2, r.lo);
      S.colour[at] = make_float4(r.r, r.g, r.b, r.z);
      S.pos[at] = b - s + lane_u + 1u;
      if constexpr (CKPT) K.cand[(int64_t)bucket0 * kBucket + slots + (uint32_t)at] = b - s + lane_u;
    }
    if (CKPT && lane == 0) K.kept[bucket0 + (b - s) / kWave] = kept;
    if (total + lane < n) {
#pragma unroll
      for (int k = 0; k < kSub; ++k) S.dx[k][total + lane] = S.dy[k][total + lane] = 0.0f;
      S.shape[total + lane] = make_float4(0.0f, 0.0f, 0.0f, -INFINITY);
      S.colour[total + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      S.pos[total + lane] = 0u;
      if constexpr (CKPT) K.cand[(int64_t)bucket0 * kBucket + slots + (uint32_t)(total + lane)] = kNoSplat;
    }
    __syncthreads();
    if (b + kWave + lane_u < e) fetch(r, id);
    if (b + 2 * kWave + lane_u < e) id = lrec.id(b + 2 * kWave + lane_u);
    // One step = kFwdSplats splats: their alphas first (independent), then
    // the blends in order.  All of a step's LDS reads are requested ahead of
    // its arithmetic (left to itself, the compiler saves registers by reading
    // each colour just before its use, an LDS latency per splat).  The
    // transmittance runs through the step as if no pixel stopped: it never
    // rises, so the splats that the stop rule leaves out are those whose
    // transmittance ends below the limit, and a step at whose end no lane is
    // below it (no pixel stops) needs no further test.  CLAMP: some splat
    // can exceed the 0.99 clamp.
    uint32_t lastslot = 0;  // 1 + slot of the last blended splat of the batch
    auto composite = [&](auto clamp_c, int j0, int j1) {
      constexpr bool CLAMP = decltype(clamp_c)::value;
      constexpr int NU = kFwdSplats;
      for (int j = j0; j < j1; j += NU) {
        const float4 dx4 = *reinterpret_cast<const float4*>(&S.dx[col][j]);
        const float4 dy4 = *reinterpret_cast<const float4*>(&S.dy[row][j]);
        float4 sh[NU], cl[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) sh[u] = S.shape[j + u];
#pragma unroll
        for (int u = 0; u < NU; ++u) cl[u] = S.colour[j + u];
        __builtin_amdgcn_sched_barrier(0);
        const float dx[NU] = {dx4.x, dx4.y, dx4.z, dx4.w};
        const float dy[NU] = {dy4.x, dy4.y, dy4.z, dy4.w};
        float w[NU], Tu[NU];
        bool hit[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          w[u] = __builtin_amdgcn_exp2f(exponent(sh[u].x, sh[u].y, sh[u].z, sh[u].w, dx[u], dy[u]));
          if (CLAMP) w[u] = fminf(kAlphaMax, w[u]);
          hit[u] = w[u] >= amin;
          w[u] = hit[u] ? w[u] : 0.0f;  // a splat that is not blended weighs 0
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const float Tb = u == 0 ? T : Tu[u - 1];
          w[u] *= Tb;
          Tu[u] = Tb - w[u];  // T (1 - alpha)
        }
        const uint64_t low = ballot64(Tu[NU - 1] < kTMin);
        // (The step without a stop is the straight path and a stop corrects
        // it: with an arm for each, every value that both write costs a copy
        // at the join, 14 of about 95 instructions per step.  8 mixed views
        // 359 -> 332 us, 4 views of 0.5M Gaussians 201 -> 190 us, one view of
        // 0.3M 69.7 -> 64.6 us.)
        float Tn = Tu[NU - 1];
        uint32_t in_step = 0;  // 1 + place in the step of the last blended splat
#pragma unroll
        for (int u = 0; u < NU; ++u) in_step = hit[u] ? (uint32_t)(u + 1) : in_step;
        if (__builtin_expect(low != 0, 0)) {
          Tn = T;
          in_step = 0;
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const bool go = Tu[u] >= kTMin;
            w[u] = go ? w[u] : 0.0f;
            Tn = go ? Tu[u] : Tn;
            in_step = (hit[u] & go) ? (uint32_t)(u + 1) : in_step;
          }
          amin = Tu[NU - 1] < kTMin ? INFINITY : amin;
          live &= ~low;
        }
        T = Tn;
        lastslot = in_step ? (uint32_t)j + in_step : lastslot;
        // (colour and depth are non-negative and finite, so fma(x, 0, acc)
        // leaves acc as it is)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          c0 = fmaf(cl[u].x, w[u], c0);
          c1 = fmaf(cl[u].y, w[u], c1);
          c2 = fmaf(cl[u].z, w[u], c2);
          D = fmaf(cl[u].w, w[u], D);
        }
        if (live == 0) break;
      }
    };
    if constexpr (CKPT) {
      // in segments between the 64-splat bucket boundaries (multiples of a
      // step), the pixel states stored before each bucket but the first
      for (int j = 0; live != 0 && j < n;) {
        const uint32_t q = slots + (uint32_t)j;
        if (q != 0 && q % kBucket == 0) {
          float* cp = K.ckpt + (int64_t)(bucket0 + q / kBucket) * (kStateFloats * kWave) + lane;
          cp[0] = T;
          cp[kWave] = c0;
          cp[2 * kWave] = c1;
          cp[3 * kWave] = c2;
          cp[4 * kWave] = D;
        }
        const int jend = min(n, j + (int)(kBucket - q % kBucket));
        if (clamps) composite(std::true_type{}, j, jend);
        else composite(std::false_type{}, j, jend);
        j = jend;
      }
    } else {
      if (clamps) composite(std::true_type{}, 0, n);
      else composite(std::false_type{}, 0, n);
    }
    if (lastslot) lastpos = S.pos[lastslot - 1];
    slots += (uint32_t)n;
  }
  if constexpr (CKPT) {
    if (lane == 0) K.seen[gtile] = make_uint2(slots, min(b, e) - s);
  }
  const float* cam = cams + (int64_t)v * GS_CAMERA_FLOATS;
  const float bg0 = cam[17], bg1 = cam[18], bg2 = cam[19];
  const int64_t npx = (int64_t)vi.W * vi.H;
  float lrgb = 0.0f, ld = 0.0f;
  if (inside) {
    const int64_t pl = (int64_t)py * vi.W + px;
    const int64_t pix = (int64_t)vi.pix_off + pl;
    const int64_t cbase = 3 * (int64_t)vi.pix_off + pl;
    const float o0 = fmaf(T, bg0, c0), o1 = fmaf(T, bg1, c1), o2 = fmaf(T, bg2, c2);
    color[cbase] = o0;
    color[cbase + npx] = o1;
    color[cbase + 2 * npx] = o2;
    depth[pix] = D;
    T_final[pix] = T;
    last[pix] = lastpos;
    if (target_rgb) {
      lrgb += fabsf(o0 - target_rgb[cbase]) + fabsf(o1 - target_rgb[cbase + npx]) +
              fabsf(o2 - target_rgb[cbase + 2 * npx]);
      if (target_depth) ld += fabsf(D - target_depth[pix]);
    }
  }
  const uint32_t m = wave_max(lastpos);
  if (target_rgb) {
    lrgb = wave_sum_to_last(lrgb);
    ld = wave_sum_to_last(ld);
  }
  if (lane == kWave - 1) {
    const int64_t u = (int64_t)gtile * NS + sub;
    tile_last[u] = m;
    if (target_rgb) {
      tile_loss[2 * u] = lrgb;
      tile_loss[2 * u + 1] = ld;
    }
  }
}

struct FwdArgs {
  RecSrc lrec;
  const uint32_t* ranges;
  const float* cams;
  float *color, *depth, *T_final;
  uint32_t *last, *tile_last;
  const float *target_rgb, *target_depth;
  float* tile_loss;
  const uint32_t* order;
  const int32_t* fl;
  FwdSplat splat;
};

// One workgroup per unit, handed out by the hardware in work order: a
// resident grid that walks the units with a static stride (one unit's cost
// varies a hundredfold) left the chip to the unluckiest wavefronts at the
// end (16 views, 25M pairs: 1141 us, this way 878).
template <int TW, int TH, bool CKPT>
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(5))) k_render_fwd(
    FwdArgs A, ViewTable vt) {
  __shared__ __align__(16) FwdLds S;
  constexpr uint32_t NS = sub_tiles<TW, TH>();
  const uint32_t u = xcd_item(blockIdx.x, (uint32_t)vt.total_tiles * NS);
  const int gtile = order_tile(A.order, A.fl, vt.total_tiles, u / NS);
  fwd_tile<TW, TH, CKPT>(gtile, (int)(u % NS), A.lrec, A.ranges, A.cams, vt, A.color, A.depth,
                         A.T_final, A.last, A.tile_last, A.target_rgb, A.target_depth,
                         A.tile_loss, A.splat, S);
}

// Per-view L1 loss from the per-tile sums, in a fixed order.
constexpr int kLossThreads = kLossVirtual;
__global__ void __launch_bounds__(kLossThreads) k_loss_reduce(const float* __restrict__ tile_loss,
                                                              ViewTable vt, float lambda_depth,
                                                              int has_depth, float* __restrict__ loss) {
  const int v = blockIdx.x;
  const ViewInfo vi = vt.v[v];
  const int ns = vt.tw * vt.th / (kSub * kSub);  // partials per tile
  loss_reduce_view<kLossThreads>(reinterpret_cast<const float2*>(tile_loss) + (int64_t)vi.tile_off * ns,
                                 vi.tiles_x * vi.tiles_y * ns, (double)vi.W * vi.H, lambda_depth,
                                 has_depth, loss + v);
}

// ------------------------------------------------------------------ backward
// Loss gradients of a pixel: given, or those of the fused L1 loss.
struct PixelLoss {
  const float *dL_dcolor, *dL_ddepth, *target_rgb, *target_depth;
  int fused;
  float lambda_depth;
  // (r, g, b, depth) gradients at the colour buffers' index cbase and the
  // one-channel buffers' index pix; o0..od: the pixel's outputs
  __device__ __forceinline__ float4 at(int64_t cbase, int64_t npx, int64_t pix, float o0, float o1,
                                       float o2, float od) const {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (fused) {
      const float inv3 = 1.0f / (3.0f * (float)npx);
      const float d0 = o0 - target_rgb[cbase];
      const float d1 = o1 - target_rgb[cbase + npx];
      const float d2 = o2 - target_rgb[cbase + 2 * npx];
      a.x = d0 > 0.0f ? inv3 : (d0 < 0.0f ? -inv3 : 0.0f);
      a.y = d1 > 0.0f ? inv3 : (d1 < 0.0f ? -inv3 : 0.0f);
      a.z = d2 > 0.0f ? inv3 : (d2 < 0.0f ? -inv3 : 0.0f);
      if (target_depth) {
        const float dd = od - target_depth[pix];
        const float sc = lambda_depth / (float)npx;
        a.w = dd > 0.0f ? sc : (dd < 0.0f ? -sc : 0.0f);
      }
    } else {
      a.x = dL_dcolor[cbase];
      a.y = dL_dcolor[cbase + npx];
      a.z = dL_dcolor[cbase + 2 * npx];
      a.w = dL_ddepth ? dL_ddepth[pix] : 0.0f;
    }
    return a;
  }
};

struct BwdArgs {
  RecSrc lrec;
  const uint32_t *sorted_vals, *ranges, *tile_last;
  const float *cams, *color, *depth, *T_final;
  const uint32_t* last;
  PixelLoss loss;
  float* grad_pair;
  const uint32_t* order;
  const int32_t* fl;
};

// LDS of a workgroup of the pixel-wise backward: a batch of 64 list
// positions -- offsets from every column and row of the tile's sample points,
// shapes and colours by position -- the positions each block keeps, and each
// block's sums of the ten partials by position.
template <int TW, int TH>
struct BwdLds {
  static constexpr int NS = sub_tiles<TW, TH>();
  float dx[TW][kWave + 1], dy[TH][kWave + 1];  // (odd rows: a lane's column is its bank)
  float4 shape[kWave], colour[kWave];
  float o[kWave];
  uint64_t kept[NS];
  float part[NS][kWave][10];
};

// Pixel-wise backward of a tile: a workgroup of one wavefront per 8x8 block,
// one pixel per lane, over the tile's list from its last used position to
// the front, 64 positions a batch.  As in the forward, a wavefront leaves out
// the splats that cannot reach its block, and a splat's offsets are formed
// once; then every wavefront walks its own kept positions and leaves the ten
// sums of each in LDS, which the workgroup adds over its blocks in a fixed
// order and writes to the pairs' slots.
//
// One wavefront per tile with four pixels per lane left 3225 wavefronts (and
// one serial chain per tile) for a 1200x680 view in 16x16 tiles: 1206 us for
// 627k pairs, this form 228 us (a 128x96 view, 48 tiles: 369 -> 53 us).
// Bound by VALU issue (88.6M instructions, 144 us of the 228): about 80 per
// kept splat and block, a third of them the reduction of the ten partials
// over the lanes.  The walk over the kept positions is the scalar unit's,
// which the last positions read into scalar registers see to (227 -> 221 us;
// in 8x8 tiles 171 -> 158; eight mixed views 1504 -> 1436, 16x8 1091 -> 1046).
template <int TW, int TH>
__global__ void __launch_bounds__(TW * TH) k_render_bwd(BwdArgs A, ViewTable vt) {
  constexpr int NS = sub_tiles<TW, TH>(), NT = kWave * NS, BX = TW / kSub;
  __shared__ __align__(16) BwdLds<TW, TH> S;
  const int lane = lane_id(), sub = NS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int gtile =
      order_tile(A.order, A.fl, vt.total_tiles, xcd_item(blockIdx.x, (uint32_t)vt.total_tiles));
  const int v = find_view(vt, gtile);
  const ViewInfo vi = vt.v[v];
  const int lt = gtile - vi.tile_off;
  const int tx0 = (lt % vi.tiles_x) * TW, ty0 = (lt / vi.tiles_x) * TH;
  const int sx = sub % BX, sy = sub / BX;  // the block's place in the tile
  const int col = lane & (kSub - 1), row = lane / kSub;
  const int px = tx0 + kSub * sx + col, py = ty0 + kSub * sy + row;
  const uint32_t s = A.ranges[2 * (int64_t)gtile], e = A.ranges[2 * (int64_t)gtile + 1];
  const uint32_t tl =
      (uint32_t)__builtin_amdgcn_readfirstlane((int)tile_last_of<NS>(A.tile_last, gtile));

  // pairs beyond the last used position get zero gradients
  for (uint32_t k = tl + threadIdx.x; k < e - s; k += NT) {
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    store_pair(A.grad_pair, A.sorted_vals[s + k], z, z, make_float2(0.f, 0.f));
  }

  float T = 1.0f, B = 0.0f;  // transmittance behind; loss-weighted output behind
  float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
  uint32_t L = 0;
  if (px < vi.W && py < vi.H) {
    const float* cam = A.cams + (int64_t)v * GS_CAMERA_FLOATS;
    const int64_t npx = (int64_t)vi.W * vi.H, pl = (int64_t)py * vi.W + px;
    const int64_t pix = (int64_t)vi.pix_off + pl, cbase = 3 * (int64_t)vi.pix_off + pl;
    T = A.T_final[pix];
    L = A.last[pix];
    if (A.loss.fused)
      g = A.loss.at(cbase, npx, pix, A.color[cbase], A.color[cbase + npx], A.color[cbase + 2 * npx],
                    A.depth[pix]);
    else
      g = A.loss.at(cbase, npx, pix, 0.f, 0.f, 0.f, 0.f);
    // behind: the background seen through T_final, nothing in depth
    B = T * (g.x * cam[17] + g.y * cam[18] + g.z * cam[19]);
    if (L == 0) {  // nothing blended: its gradient reaches no splat
      g = make_float4(0.f, 0.f, 0.f, 0.f);
      T = 1.0f;
      B = 0.0f;
    }
  }
  // A gradient that is no number, or so large that a product with it may not
  // be one, must reach the splats blended at its pixel alone: 0 times it is
  // not 0, so such blocks select what a splat adds by its hit.
  const float gmax = fmaxf(fmaxf(fabsf(g.x), fabsf(g.y)), fmaxf(fabsf(g.z), fabsf(g.w)));
  const bool tame_px = g.x == g.x && g.y == g.y && g.z == g.z && g.w == g.w && gmax < kTame &&
                       fabsf(B) < kTame && T <= 1.0f;
  const bool tame_block = ballot64(!tame_px) == 0;
  const uint32_t Lmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max(L));
  const int my_idx = lane < 16 ? rs_index(lane) : -1;
  const double ax0 = (double)(tx0 + kSub * sx) + 0.5, ay0 = (double)(ty0 + kSub * sy) + 0.5;

  // the record of this lane's position in the batch that ends at `end`; the
  // next batch's is fetched while this one is worked on
  FwdRec r{};
  float ro = 0.0f;
  auto fetch = [&](int end) {
    const int start = end > kWave ? end - kWave : 0;
    if (start + lane < end) {
      const Rec* rec = A.lrec.at(s + (uint32_t)(start + lane));
      const float4* src = reinterpret_cast<const float4*>(rec);
      float4* d4 = reinterpret_cast<float4*>(&r);
      d4[0] = src[0]; d4[1] = src[1]; d4[2] = src[2];
      if (sub == 0) ro = rec->o;
    }
  };
  fetch((int)tl);
  for (int bend = (int)tl; bend > 0; bend -= kWave) {
    const int bstart = bend > kWave ? bend - kWave : 0;
    const int nb = bend - bstart;
    const bool has = lane < nb;
    float ox[kSub], oy[kSub];
    double ax = ax0, ay = ay0;
    asm volatile("" : "+v"(ax), "+v"(ay));
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
      ox[k] = (float)(r.mx - ax);
      oy[k] = (float)(r.my - ay);
      ax += 1.0;
      ay += 1.0;
    }
    const bool keep = !(max_exponent(r, ox[kSub - 1], ox[0], oy[kSub - 1], oy[0]) < kCullExp);
    uint64_t kept = ballot64(has & keep);
    // (nothing of this block is used from position Lmax on)
    const int used = (int)Lmax - bstart;
    kept &= used >= kWave ? ~0ull : (used <= 0 ? 0ull : (1ull << used) - 1ull);
    // the first block of a column (row) of blocks writes its offsets
    if (sy == 0) {
#pragma unroll
      for (int k = 0; k < kSub; ++k) S.dx[kSub * sx + k][lane] = ox[k];
    }
    if (sx == 0) {
#pragma unroll
      for (int k = 0; k < kSub; ++k) S.dy[kSub * sy + k][lane] = oy[k];
    }
    if (sub == 0) {
      S.shape[lane] = make_float4(r.t, r.s1, r.s2, r.lo);
      S.colour[lane] = make_float4(r.r, r.g, r.b, r.z);
      S.o[lane] = ro;
    }
    if (lane == 0) S.kept[sub] = kept;
    const bool tame =
        tame_block && ballot64(has && !(fmaxf(fmaxf(r.r, r.g), fmaxf(r.b, r.z)) < kTame)) == 0;
    __syncthreads();
    fetch(bend - kWave);
    // N kept positions j[0] > j[1] .. at once: independent alphas and
    // reductions, only T and B run through them in order.  TAME: a splat that
    // is not blended adds its products with alpha 0.
    auto step = [&](auto n_c, auto tame_c, const int* j) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value;
      constexpr bool TAME = decltype(tame_c)::value;
      float p_ax[N], q_ax[N], oG[N], a[N], front[N];
      bool hit[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const float dx = S.dx[kSub * sx + col][j[k]], dy = S.dy[kSub * sy + row][j[k]];
        const float4 sh = S.shape[j[k]], cl = S.colour[j[k]];
        p_ax[k] = fmaf(sh.x, dy, dx);
        q_ax[k] = fmaf(-sh.x, dx, dy);
        oG[k] = __builtin_amdgcn_exp2f(exponent_pq(sh.y, sh.z, sh.w, p_ax[k], q_ax[k]));
        front[k] = fmaf(g.w, cl.w, fmaf(g.z, cl.z, fmaf(g.y, cl.y, g.x * cl.x)));
        a[k] = fminf(kAlphaMax, oG[k]);
        hit[k] = (a[k] >= kAlphaMin) & ((uint32_t)(bstart + j[k]) < L);
        // alpha of a blended splat, 0 otherwise: then 1 - alpha = 1 and every
        // term below is 0 or leaves its sum as it is
        a[k] = hit[k] ? a[k] : 0.0f;
      }
      float z[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const float inv_om = __builtin_amdgcn_rcpf(1.0f - a[k]);
        T *= inv_om;  // in front of this splat
        const float wgt = a[k] * T;
        const float g_alpha = fmaf(T, front[k], -(B * inv_om));
        const float Bn = fmaf(front[k], wgt, B);
        B = TAME || hit[k] ? Bn : B;
        // unclamped alpha only (no gradient through the 0.99 clamp); the
        // conic and mean partials are moments of gpow = alpha dL/dalpha along
        // the footprint's axes, put together after the sums
        const float gpow = oG[k] <= kAlphaMax ? a[k] * g_alpha : 0.0f;
        const float t = gpow * p_ax[k], u = gpow * q_ax[k];
        float p[10] = {wgt * g.x, wgt * g.y, wgt * g.z, wgt * g.w, gpow,
                       t * p_ax[k], t * q_ax[k], u * q_ax[k], t, u};
        if constexpr (!TAME) {
#pragma unroll
          for (int f = 0; f < 10; ++f) p[f] = hit[k] ? p[f] : 0.0f;
        }
        z[k] = reduce_scatter10(p);
      }
      if (my_idx >= 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) S.part[sub][j[k]][my_idx] = z[k];
        asm volatile("" ::"i"(N));  // (merged with the other form's store, the walk leaves the scalar unit)
      }
    };
    auto walk = [&](auto tame_c) __attribute__((always_inline)) {
      for (uint64_t m = kept; m;) {
        int j[2];
        j[0] = 63 - __builtin_clzll(m);
        m &= ~(1ull << j[0]);
        if (m == 0) {
          step(std::integral_constant<int, 1>{}, tame_c, j);
          break;
        }
        j[1] = 63 - __builtin_clzll(m);
        m &= ~(1ull << j[1]);
        step(std::integral_constant<int, 2>{}, tame_c, j);
      }
    };
    if (__builtin_expect(tame, 1)) walk(std::true_type{});
    else walk(std::false_type{});
    __syncthreads();
    for (int q = (int)threadIdx.x; q < nb; q += NT) {
      float f[10];
#pragma unroll
      for (int k = 0; k < 10; ++k) f[k] = 0.0f;
#pragma unroll
      for (int b = 0; b < NS; ++b)
        if ((S.kept[b] >> q) & 1ull) {
#pragma unroll
          for (int k = 0; k < 10; ++k) f[k] += S.part[b][q][k];
        }
      const float4 sh = S.shape[q];
      const double t = sh.x, n2 = (1.0 + t * t) * (1.0 + t * t);
      const double pp = f[5], pq = f[6], qq = f[7];  // dx = (p - t q) / (1 + t^2), dy = (q + t p) / ..
      const float o = S.o[q];
      store_pair(A.grad_pair, A.sorted_vals[s + (uint32_t)(bstart + q)],
                 make_float4(f[0], f[1], f[2], f[3]),
                 make_float4(o > 0.0f ? f[4] / o : 0.0f,
                             (float)(-0.5 * (pp - 2.0 * t * pq + t * t * qq) / n2),
                             (float)(-((1.0 - t * t) * pq + t * (pp - qq)) / n2),
                             (float)(-0.5 * (qq + 2.0 * t * pq + t * t * pp) / n2)),
                 mean_grad(t, sh.y, sh.z, f[8], f[9]));
    }
    __syncthreads();
  }
}

// ----------------------------------------------------- splat-wise backward
// Sec. III-C-1 / Fig. 4a mapped to wave64, for 8x8 tiles.  The splats that
// the forward kept of a tile's list are cut into buckets of 64; one wavefront
// takes a bucket and lane l owns its l-th splat.  The forward stored each
// pixel's state X = (T, RGB, D) before every 64th kept splat, so a bucket
// starts from stored states and needs nothing from the other buckets of its
// tile: buckets are the unit of parallelism, which also splits long lists
// over many wavefronts.
//
// All lanes of a segment take the same pixel at each step.  Lane l
// evaluates its splat's alpha with the forward's code (the same bits, so
// the same skip decisions; the forward's stop rule is its stored last
// position).  What lies in front of lane l's splat at the pixel is the
// segment's stored state advanced over the blended splats of lanes < l: the
// transmittance is T_in times the product of (1 - alpha) over those lanes
// (the inclusive prefix product divided by the lane's own factor), and the
// front part of the loss-weighted output Q = gC . C + gD . D an inclusive
// prefix sum of alpha T gC . c, both taken across the lanes with DPP.  What
// lies behind the splat is the final pixel minus the front part, P - Q with
// P = gC . (colour output) + gD . (depth output).  A bucket thus costs one
// step per pixel, with no pipeline to fill or drain.  Each lane accumulates
// its own splat's ten partial gradients over the tile's pixels and writes
// them once: no reduction over lanes and no atomics.
//
// A bucket of at most 32 (16) splats runs two (four) segments of 32 (16)
// lanes that hold the same splats and take every second (fourth) row of
// pixels; their sums are added at the end.
//
// Bound by VALU issue.  The steps run over rows of pixels: a lane's offsets
// from the eight columns stay in registers and the row's is formed once per
// row (two FP64 differences and two conversions per step before), and the
// moments of the mean and conic partials are summed over a row without the
// row's offset: with buckets of kept splats only, 1430M -> 1015M VALU
// instructions on the 16-view batch (25M pairs).  One workgroup per bucket, 32
// consecutive ones to an XCD: the buckets of a tile and its neighbours read
// the same pixels and splats from one L2 (a resident grid with a static
// stride: 2100 us; this way 1535 us, the VALU busy throughout; 5 to 7
// wavefronts per SIMD measure the same).  Before these: 2608 us; 8 mixed views
// 530 -> 340 us; one 1200x680 view 70 -> 56 us.

// Inclusive product / sum over segments of SEG (64, 32 or 16) lanes, in
// place, of two independent values at once (two pixels): steps in rows of 16
// (row_shr 1, 2, 4, 8), then for 32 lanes and more the ends of rows 0 and 2
// into rows 1 and 3 (row_bcast:15), and for 64 the end of row 1 into rows 2
// and 3 (row_bcast:31).  Each step is one DPP multiply or add whose lanes
// without a source (or outside the row mask) are not written, i.e. keep
// their value.  A DPP read of a VGPR written by the previous VALU
// instruction needs two wait states: the two scans' steps alternate, so
// one wait state plus the other scan's step covers it (two before the
// first step, whose inputs the compiler's code has just written).
#define GS_DPP2(OP, CTRL) OP " %0, %0, %0 " CTRL " bank_mask:0xf\n\t" OP " %1, %1, %1 " CTRL " bank_mask:0xf\n\t"
#define GS_SEG_SCAN16_2(OP)                             \
  "s_nop 1\n\t" GS_DPP2(OP, "row_shr:1 row_mask:0xf") \
  "s_nop 0\n\t" GS_DPP2(OP, "row_shr:2 row_mask:0xf") \
  "s_nop 0\n\t" GS_DPP2(OP, "row_shr:4 row_mask:0xf") \
  "s_nop 0\n\t" GS_DPP2(OP, "row_shr:8 row_mask:0xf")
#define GS_SEG_SCAN32_2(OP) GS_SEG_SCAN16_2(OP) "s_nop 0\n\t" GS_DPP2(OP, "row_bcast:15 row_mask:0xa")
#define GS_SEG_SCAN64_2(OP) GS_SEG_SCAN32_2(OP) "s_nop 0\n\t" GS_DPP2(OP, "row_bcast:31 row_mask:0xc")
template <int SEG>
__device__ __forceinline__ void seg_scan_mul2(float& x, float& y) {
  if (SEG == 64) asm volatile(GS_SEG_SCAN64_2("v_mul_f32_dpp") : "+v"(x), "+v"(y));
  else if (SEG == 32) asm volatile(GS_SEG_SCAN32_2("v_mul_f32_dpp") : "+v"(x), "+v"(y));
  else asm volatile(GS_SEG_SCAN16_2("v_mul_f32_dpp") : "+v"(x), "+v"(y));
}
template <int SEG>
__device__ __forceinline__ void seg_scan_add2(float& x, float& y) {
  if (SEG == 64) asm volatile(GS_SEG_SCAN64_2("v_add_f32_dpp") : "+v"(x), "+v"(y));
  else if (SEG == 32) asm volatile(GS_SEG_SCAN32_2("v_add_f32_dpp") : "+v"(x), "+v"(y));
  else asm volatile(GS_SEG_SCAN16_2("v_add_f32_dpp") : "+v"(x), "+v"(y));
}
#undef GS_SEG_SCAN64_2
#undef GS_SEG_SCAN32_2
#undef GS_SEG_SCAN16_2
#undef GS_DPP2

// Sum over the segments of SEG lanes of a wavefront, in every lane.
template <int SEG>
__device__ __forceinline__ float sum_segments(float x) {
  if (SEG <= 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if (SEG <= 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return x;
}

struct SplatArgs {
  RecSrc lrec;
  const uint32_t *sorted_vals, *ranges, *cand;
  const uint64_t* kept;
  const uint2* seen;
  const float* ckpt;
  const uint2* bq;
  const int32_t* fl;
  const float *color, *depth;
  const uint32_t* last;
  PixelLoss loss;
  float* grad_pair;
};

// Pixel table of a bucket: (gC, gD) and (P - Q_in, last position, T_in, -).
struct SplatLds {
  float4 g[kWave], x[kWave];
};

// A lane's splat.
struct LaneSplat {
  double my;
  float dx[kSub];
  float t, s1, s2, lo, z, r, g, b;
  uint32_t pos;
};

// The ten sums of the lane's splat over the tile's live pixels (alive: bit
// per pixel).  SEG lanes take one pixel; R = 64 / SEG rows of pixels go
// through at once.  CLAMP: some splat of the bucket can exceed the 0.99 clamp.
template <int SEG, bool CLAMP>
__device__ __forceinline__ void splat_rows(const LaneSplat& r, const SplatLds& S, uint64_t alive,
                                           int ty0, int lane, float (&acc)[10]) {
  constexpr int R = kWave / SEG, NR = kSub * R;
  const int seg = lane / SEG;
#pragma unroll
  for (int f = 0; f < 10; ++f) acc[f] = 0.0f;
  for (int it = 0; it < kSub / R; ++it) {
    uint64_t m = (alive >> (NR * it)) & (NR == 64 ? ~0ull : (1ull << NR) - 1ull);
    if (m == 0) continue;  // (uniform)
    if (R >= 2) m |= m >> kSub;
    if (R >= 4) m |= m >> (2 * kSub);
    const int row = it * R + seg;
    const float dy = (float)(r.my - ((double)(ty0 + row) + 0.5));
    const float4* sx = S.x + row * kSub;
    const float4* sg = S.g + row * kSub;
    // moments over the row of gpow = dL/dpower: 1, p, p^2, p = dx + t dy
    float m0 = 0.0f, m1 = 0.0f, m2 = 0.0f;
    // two pixels per step, their scans interleaved; each lane accumulates
    // the left one first
#pragma unroll
    for (int p = 0; p < kSub; p += 2) {
      if (((m >> p) & 3ull) == 0) continue;  // (uniform)
      float4 x[2], g[2];
      float p_ax[2], oG[2], a[2], inv_om[2], f[2];
      bool hit[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        x[u] = sx[p + u];
        g[u] = sg[p + u];
        // alpha as in the forward (same bits)
        p_ax[u] = fmaf(r.t, dy, r.dx[p + u]);
        oG[u] = __builtin_amdgcn_exp2f(
            exponent_pq(r.s1, r.s2, r.lo, p_ax[u], fmaf(-r.t, r.dx[p + u], dy)));
        a[u] = CLAMP ? fminf(kAlphaMax, oG[u]) : oG[u];
        hit[u] = (r.pos < __float_as_uint(x[u].y)) & (a[u] >= kAlphaMin);
        // alpha of a blended splat, 0 otherwise: its 1 - alpha is the scan's
        // factor and alpha T the blend weight, with no further selects
        a[u] = hit[u] ? a[u] : 0.0f;
        f[u] = 1.0f - a[u];
        inv_om[u] = __builtin_amdgcn_rcpf(f[u]);
      }
      // transmittance in front of the splat: the segment's inclusive product
      // over its blended splats with the lane's own factor taken out again
      // (read by blended lanes only, whose factor 1 - alpha >= 0.01)
      seg_scan_mul2<SEG>(f[0], f[1]);
      float Tl[2], wgt[2], front[2], q[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        Tl[u] = (x[u].z * f[u]) * inv_om[u];
        wgt[u] = a[u] * Tl[u];
        front[u] = fmaf(g[u].w, r.z, fmaf(g[u].z, r.b, fmaf(g[u].y, r.g, g[u].x * r.r)));
        q[u] = wgt[u] * front[u];
      }
      seg_scan_add2<SEG>(q[0], q[1]);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        // behind the splat: P - (Q_in + the front part after the splat)
        const float g_alpha = fmaf(-(x[u].x - q[u]), inv_om[u], Tl[u] * front[u]);
        acc[0] = fmaf(wgt[u], g[u].x, acc[0]);
        acc[1] = fmaf(wgt[u], g[u].y, acc[1]);
        acc[2] = fmaf(wgt[u], g[u].z, acc[2]);
        acc[3] = fmaf(wgt[u], g[u].w, acc[3]);
        // gpow = alpha dL/dalpha of the unclamped splats; the opacity, conic
        // and mean partials are formed from its moments once, after the
        // pixels (dL/do = sum gpow / o)
        const float gpow = !CLAMP || oG[u] <= kAlphaMax ? a[u] * g_alpha : 0.0f;
        const float t = gpow * p_ax[u];
        m0 += gpow;
        m1 += t;
        m2 = fmaf(t, p_ax[u], m2);
      }
    }
    const float my = dy * m0;
    acc[4] += m0;
    acc[5] += m2;
    acc[6] = fmaf(dy, m1, acc[6]);
    acc[7] = fmaf(dy, my, acc[7]);
    acc[8] += m1;
    acc[9] += my;
  }
#pragma unroll
  for (int f = 0; f < 10; ++f) acc[f] = sum_segments<SEG>(acc[f]);
}

// One bucket: entry qi of the queue.
__device__ __forceinline__ void splat_bucket(const SplatArgs& A, const ViewTable& vt, uint32_t qi,
                                             SplatLds& S, int lane) {
  const uint2 ent = A.bq[qi];  // (tile, k)
  const int gtile = __builtin_amdgcn_readfirstlane((int)ent.x);
  const uint32_t q0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.y) * kBucket;
  const uint2 seen = A.seen[gtile];  // (slots, list positions looked at)
  const uint32_t s = A.ranges[2 * (int64_t)gtile], e = A.ranges[2 * (int64_t)gtile + 1];
  // entry k also writes the zero gradients of the pairs that no bucket holds
  // among the list's k-th 64 positions
  {
    const uint32_t p = q0 + (uint32_t)lane;
    const uint64_t kept = q0 < seen.y ? A.kept[qi] : 0ull;
    if (s + p < e && !((kept >> lane) & 1ull)) {
      const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
      store_pair(A.grad_pair, A.sorted_vals[s + p], z, z, make_float2(0.f, 0.f));
    }
  }
  if (q0 >= seen.x) return;  // the tile's list has more entries than its slots have buckets
  const int cnt = (int)min((uint32_t)kBucket, seen.x - q0);
  const int seg_lanes = cnt > 32 ? 64 : cnt > 16 ? 32 : 16;
  // the lane's splat (the same ones in every segment)
  const int ls = lane & (seg_lanes - 1);
  const uint32_t pos = ls < cnt ? A.cand[(int64_t)qi * kBucket + ls] : kNoSplat;
  const bool live = pos != kNoSplat;
  const uint32_t pos0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);

  // pixel table: loss gradients, P, last position, stored state.  A pixel
  // whose last position lies at or before the bucket's first splat has none
  // of its splats blended and adds nothing.
  const int v = find_view(vt, gtile);
  const ViewInfo vi = vt.v[v];
  const int lt = gtile - vi.tile_off;
  const int tx0 = (lt % vi.tiles_x) * kSub, ty0 = (lt / vi.tiles_x) * kSub;
  const int64_t npx = (int64_t)vi.W * vi.H;
  const int px = tx0 + (lane & (kSub - 1)), py = ty0 + lane / kSub;
  float4 g = make_float4(0.f, 0.f, 0.f, 0.f), x = make_float4(0.f, 0.f, 1.f, 0.f);
  bool alive_px = false;
  if (px < vi.W && py < vi.H) {
    const int64_t pl = (int64_t)py * vi.W + px;
    const int64_t pix = (int64_t)vi.pix_off + pl;
    const int64_t cbase = 3 * (int64_t)vi.pix_off + pl;
    const uint32_t lp = A.last[pix];
    alive_px = lp > pos0;
    if (alive_px) {
      const float o0 = A.color[cbase], o1 = A.color[cbase + npx], o2 = A.color[cbase + 2 * npx];
      const float od = A.depth[pix];
      g = A.loss.at(cbase, npx, pix, o0, o1, o2, od);
      float Qin = 0.0f;
      if (q0 > 0) {  // the first bucket starts from T = 1 and nothing accumulated
        const float* cp = A.ckpt + (int64_t)qi * (kStateFloats * kWave) + lane;
        x.z = cp[0];
        Qin = g.x * cp[kWave] + g.y * cp[2 * kWave] + g.z * cp[3 * kWave] + g.w * cp[4 * kWave];
      }
      x.x = (g.x * o0 + g.y * o1 + g.z * o2 + g.w * od) - Qin;
      x.y = __uint_as_float(lp);
    }
  }
  const uint64_t alive = ballot64(alive_px);
  float acc[10];
  float ro = 0.0f, rt = 0.0f, rs1 = 0.0f, rs2 = 0.0f;
  if (alive == 0) {  // (uniform)
#pragma unroll
    for (int f = 0; f < 10; ++f) acc[f] = 0.0f;
  } else {
    S.g[lane] = g;
    S.x[lane] = x;
    LaneSplat r;
    r.t = r.s1 = r.s2 = r.z = r.r = r.g = r.b = 0.0f;
    r.lo = -INFINITY;  // alpha = 0 in a lane without a splat
    r.my = 0.0;
    r.pos = pos;
#pragma unroll
    for (int k = 0; k < kSub; ++k) r.dx[k] = 0.0f;
    if (live) {
      Rec rec;
      const float4* src = reinterpret_cast<const float4*>(A.lrec.at(s + pos));
      float4* dst = reinterpret_cast<float4*>(&rec);
      dst[0] = src[0]; dst[1] = src[1]; dst[2] = src[2]; dst[3] = src[3];
      r.t = rec.t; r.s1 = rec.s1; r.s2 = rec.s2; r.lo = rec.lo;
      r.z = rec.z; r.r = rec.r; r.g = rec.g; r.b = rec.b;
      r.my = rec.my;
      double ax = (double)tx0 + 0.5;
#pragma unroll
      for (int k = 0; k < kSub; ++k) {
        r.dx[k] = (float)(rec.mx - ax);
        ax += 1.0;
      }
      ro = rec.o;
      rt = rec.t; rs1 = rec.s1; rs2 = rec.s2;
    }
    const bool clamps = ballot64(r.lo > kClampLo) != 0;
    __syncthreads();
    auto rows = [&](auto seg_c) {
      constexpr int SEG = decltype(seg_c)::value;
      if (clamps) splat_rows<SEG, true>(r, S, alive, ty0, lane, acc);
      else splat_rows<SEG, false>(r, S, alive, ty0, lane, acc);
    };
    if (seg_lanes == 64) rows(std::integral_constant<int, 64>{});
    else if (seg_lanes == 32) rows(std::integral_constant<int, 32>{});
    else rows(std::integral_constant<int, 16>{});
  }
  if (live && lane < seg_lanes) {
    // acc: sums of gpow times p^2, p dy, dy^2, p, dy; dx = p - t dy and
    // q = (1 + t^2) dy - t p
    const double t = rt, pp = acc[5], pd = acc[6], yy = acc[7], sp = acc[8], sy = acc[9];
    store_pair(A.grad_pair, A.sorted_vals[s + pos], make_float4(acc[0], acc[1], acc[2], acc[3]),
               make_float4(ro > 0.0f ? acc[4] / ro : 0.0f,
                           (float)(-0.5 * (pp - 2.0 * t * pd + t * t * yy)),
                           (float)(-(pd - t * yy)), -0.5f * acc[7]),
               mean_grad(t, rs1, rs2, sp, (1.0 + t * t) * sy - t * sp));
  }
}

// One workgroup (a wavefront) per entry of the bucket queue.  The grid covers
// the plan's checkpoint slots; but an idle workgroup costs 0.11 ns, a thirtieth
// of one with a bucket, so that plans with room for a few hundred times their
// pairs spent more on them than on the buckets.  Where the slots exceed
// kGridBuckets a tile (512 pairs, four times the mean list of the batches
// above) by more than kGridIdle, 7 us, the rest is left to a second, looping
// launch (4 us if nothing is).  640x480, 61k pairs, whole iteration: with room
// for 1.3 times as many 92 us, 256 times 130 without the second launch and
// 100 with it, 1024 times 284 and 100.  As one looping launch the large
// batches lose 4 % (1616 -> 1681 us, 79 registers instead of 69).
constexpr int64_t kGridBuckets = 8, kGridLeast = 1 << 14, kGridIdle = 1 << 16, kGridRest = 1 << 14;
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(6))) k_render_bwd_splat(
    SplatArgs A, ViewTable vt) {
  __shared__ SplatLds S;
  const uint32_t n = (uint32_t)A.fl[F_BUCKETS];
  const uint32_t q = xcd_item(blockIdx.x, gridDim.x);
  if (q < n) splat_bucket(A, vt, q, S, (int)threadIdx.x);
}
__global__ void __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(6))) k_render_bwd_splat_rest(
    SplatArgs A, ViewTable vt, uint32_t first) {
  __shared__ SplatLds S;
  const uint32_t n = (uint32_t)A.fl[F_BUCKETS];
  for (uint32_t q = first + xcd_item(blockIdx.x, gridDim.x); q < n; q += gridDim.x) {
    int lane = (int)threadIdx.x;
    asm volatile("" : "+v"(lane));  // (what hangs on it, kept over the buckets, would spill)
    splat_bucket(A, vt, q, S, lane);
    __syncthreads();  // the pixel table is rewritten by the next bucket
  }
}

// (Until the kernels fetched the records of a batch while they worked on the
// one before, the per-tile binning wrote a 64-byte copy of every pair's
// record in list order.  Without them the render kernels take the same time
// and the tile sort less: 433k pairs 35 -> 22 us, 2.7M pairs 183 -> 128.)
RecSrc rec_src(const Plan& P, void* ws) {
  return RecSrc{ws_at<Rec>(ws, P.off_rec), ws_at<uint32_t>(ws, P.off_sorted_rec)};
}

template <int TW, int TH>
hipError_t fwd_launch(const Plan& P, void* ws, const float* cams, float* color, float* depth,
                      float* T_final, uint32_t* last, const float* target_rgb,
                      const float* target_depth, hipStream_t s) {
  FwdArgs A{rec_src(P, ws), ws_at<uint32_t>(ws, P.off_ranges), cams, color, depth, T_final,
            last, ws_at<uint32_t>(ws, P.off_tile_last), target_rgb, target_depth,
            ws_at<float>(ws, P.off_tile_loss), ws_at<uint32_t>(ws, P.off_order),
            ws_at<int32_t>(ws, P.off_flags), FwdSplat{}};
  const dim3 g((unsigned)P.vt.total_tiles * sub_tiles<TW, TH>()), block(kWave);
  if constexpr (TW * TH == kWave) {
    if (P.splat) {
      A.splat = FwdSplat{ws_at<uint32_t>(ws, P.off_boff), ws_at<float>(ws, P.off_ckpt),
                         ws_at<uint32_t>(ws, P.off_cand), ws_at<uint64_t>(ws, P.off_kept),
                         ws_at<uint2>(ws, P.off_seen)};
      hipLaunchKernelGGL((k_render_fwd<TW, TH, true>), g, block, 0, s, A, P.vt);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_render_fwd<TW, TH, false>), g, block, 0, s, A, P.vt);
  return hipGetLastError();
}

template <int TW, int TH>
hipError_t bwd_launch(const Plan& P, void* ws, const float* cams, const float* color,
                      const float* depth, const float* T_final, const uint32_t* last,
                      const PixelLoss& loss, const uint32_t* sorted_vals, hipStream_t s) {
  const BwdArgs A{rec_src(P, ws), sorted_vals, ws_at<uint32_t>(ws, P.off_ranges),
                  ws_at<uint32_t>(ws, P.off_tile_last), cams, color, depth, T_final, last, loss,
                  ws_at<float>(ws, P.off_grad_pair), ws_at<uint32_t>(ws, P.off_order),
                  ws_at<int32_t>(ws, P.off_flags)};
  hipLaunchKernelGGL((k_render_bwd<TW, TH>), dim3((unsigned)P.vt.total_tiles),
                     dim3(kWave * sub_tiles<TW, TH>()), 0, s, A, P.vt);
  return hipGetLastError();
}

}  // namespace

// 8x8 blocks of pixels per tile: the forward's wavefronts per tile.
int blocks_per_tile(const Plan& P) { return P.cfg.tile_w * P.cfg.tile_h / (kSub * kSub); }

hipError_t launch_render_fwd(const Plan& P, void* ws, const float* cams, float* color,
                             float* depth, float* T_final, uint32_t* last,
                             const float* target_rgb, const float* target_depth,
                             float* loss_per_view, hipStream_t s) {
  if (P.vt.total_tiles == 0) return hipSuccess;
  hipError_t e;
  const int tw = P.cfg.tile_w, th = P.cfg.tile_h;
  if (tw == 16 && th == 16)
    e = fwd_launch<16, 16>(P, ws, cams, color, depth, T_final, last, target_rgb, target_depth, s);
  else if (tw == 16 && th == 8)
    e = fwd_launch<16, 8>(P, ws, cams, color, depth, T_final, last, target_rgb, target_depth, s);
  else
    e = fwd_launch<8, 8>(P, ws, cams, color, depth, T_final, last, target_rgb, target_depth, s);
  if (e != hipSuccess) return e;
  if (target_rgb && loss_per_view) {
    hipLaunchKernelGGL(k_loss_reduce, dim3(P.vt.n_views), dim3(kLossThreads), 0, s,
                       ws_at<float>(ws, P.off_tile_loss), P.vt, P.cfg.lambda_depth,
                       target_depth ? 1 : 0, loss_per_view);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_render_bwd(const Plan& P, void* ws, const float* cams, const float* color,
                             const float* depth, const float* T_final, const uint32_t* last,
                             const float* dL_dcolor, const float* dL_ddepth,
                             const float* target_rgb, const float* target_depth, int fused,
                             const uint32_t* sorted_vals, hipStream_t s) {
  if (P.vt.total_tiles == 0) return hipSuccess;
  const int tw = P.cfg.tile_w, th = P.cfg.tile_h;
  const PixelLoss loss{dL_dcolor, dL_ddepth, target_rgb, target_depth, fused, P.cfg.lambda_depth};
  // GS_SPLAT_BWD with larger tiles takes the pixel-wise form: a bucket's lanes
  // would sit idle on the blocks of the tile that their splats do not reach
  // (55 %).  Forward and backward, before -> after: one 1200x680 view, 16x16
  // tiles 253 -> 91 us, 16x8 159 -> 89 us; 8 mixed views (6.0M pairs in 8x8
  // tiles), 16x16 4.7 -> 2.0 ms, 16x8 2.3 -> 1.4 ms
  if (P.splat) {
    const SplatArgs A{rec_src(P, ws), sorted_vals, ws_at<uint32_t>(ws, P.off_ranges),
                      ws_at<uint32_t>(ws, P.off_cand), ws_at<uint64_t>(ws, P.off_kept),
                      ws_at<uint2>(ws, P.off_seen), ws_at<float>(ws, P.off_ckpt),
                      ws_at<uint2>(ws, P.off_bq), ws_at<int32_t>(ws, P.off_flags), color, depth,
                      last, loss, ws_at<float>(ws, P.off_grad_pair)};
    const int64_t most = std::max(kGridBuckets * P.vt.total_tiles, kGridLeast);
    const int64_t grid = P.ckpt_slots > most + kGridIdle ? most : P.ckpt_slots;
    const int64_t rest = P.ckpt_slots - grid;
    hipLaunchKernelGGL(k_render_bwd_splat, dim3((unsigned)grid), dim3(kWave), 0, s, A, P.vt);
    if (rest > 0)
      hipLaunchKernelGGL(k_render_bwd_splat_rest, dim3((unsigned)std::min(rest, kGridRest)),
                         dim3(kWave), 0, s, A, P.vt, (uint32_t)grid);
    return hipGetLastError();
  }
  if (tw == 16 && th == 16)
    return bwd_launch<16, 16>(P, ws, cams, color, depth, T_final, last, loss, sorted_vals, s);
  if (tw == 16 && th == 8)
    return bwd_launch<16, 8>(P, ws, cams, color, depth, T_final, last, loss, sorted_vals, s);
  return bwd_launch<8, 8>(P, ws, cams, color, depth, T_final, last, loss, sorted_vals, s);
}

}  // namespace gs
