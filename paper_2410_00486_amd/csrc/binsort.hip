// a2: tile binning.  Pairs are the (Gaussian, tile) incidences of the exact
// tile boxes, numbered in generation order (record-major, row-major tiles
// within a box).  The order the renderer needs is (tile, depth, generation
// index): unique, so the result is bit-exact whatever the schedule.
//
// The projection counts pairs per tile and per chunk of 64 Gaussians as it
// computes the boxes.  Then: one block scans the chunk counts (generation
// offsets, visible-list positions) and the tile counts (list starts, bucket
// offsets and queue positions); one scatter puts every pair into its tile's
// list at an atomically taken slot with the key (depth bits << 32 |
// generation index); a per-tile sort orders those keys (one wavefront per
// tile: ranks up to 64 keys, a bitonic network in registers up to 128; longer
// lists take a wavefront, or a 1024-thread block, each).  No spin-waits;
// graph-capturable.
//
// The scan also writes the work order of the render kernels: tiles with long
// lists first.
#include "tilesort.h"
#include "wavescan.h"

namespace gs {
namespace {

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t value, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = value;
}

// Clears a[0, na) and b[0, nb).
__global__ void k_fill2_u32(uint32_t* __restrict__ a, int64_t na, uint32_t* __restrict__ b,
                            int64_t nb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0u;
  if (i < nb) b[i] = 0u;
}

// ---------------------------------------------------------------- scans
// The projection writes, for every chunk of 64 Gaussians of a view (one
// wavefront), its pair count and its number of visible records; and the
// pair count of every tile.  One block scans both: chunks -> generation
// offset and visible-list position of the chunk's first record; tiles ->
// list start and bucket offset (the tile's place in the splat-wise bucket
// queue).  One block needs no inter-block handshake (a grid-wide fence
// costs more than the scan itself at these sizes), and the results are
// absolute, so the consumers add nothing.
//
// Offsets are stored as u32, exact whenever the pair total fits the pair
// capacity (< 2^31); otherwise the overflow flag stops every consumer.  The
// running sums are 64-bit.

constexpr int kScanBlock = 1024;  // threads of the scan block
constexpr int kScanVec = 2;       // uint4 loads per thread and array in a round
// A round: 4 * kScanVec consecutive tiles and 2 * kScanVec consecutive
// chunks per thread, loaded and stored as uint4.
constexpr int64_t kTileRound = (int64_t)kScanBlock * 4 * kScanVec;
constexpr int64_t kChunkRound = (int64_t)kScanBlock * 2 * kScanVec;

struct ScanArgs {
  const uint2* chunk_cnt;  // (pairs, visible records) per chunk
  uint2* chunk_pre;        // (generation offset, visible-list position) per chunk
  int64_t n_chunks;
  TileCounters cnt;        // pairs per tile; set to each copy's place in the list here
                           // (the scatter's cursors)
  uint32_t* tstart;        // list start per tile
  int64_t n_tiles;
  uint32_t* boff;          // splat-wise only (else null): bucket offset per tile, [T] = total
  uint32_t* order;         // work order of the render kernels: kOrderClasses rows of T
  uint4* long_list;        // (tile, list start, pairs, -) of the lists for the long-list sort
  // kScanBoth: chunks and tile counts (the projection's); kScanChunks: the
  // chunks alone (radix binning, before the pairs exist); kScanTiles: the
  // tiles alone from the list ends (cnt) and starts (tstart) that the radix
  // binning found in its sorted keys, with the counts written back to cnt
  int mode;
};
constexpr int kScanBoth = 0, kScanChunks = 1, kScanTiles = 2;

// Work order of the render kernels: the tiles by the length class of their
// lists, longest class first, in tile order within a class.  A wavefront
// composites a list serially, so what matters is that the longest ones start
// first.  A class has a row of its own in `order` (a tile's position in it
// is the scan's count of the class before it) and its size in the flags.
__device__ __forceinline__ int order_class(uint32_t c) {
  return c > 1024 ? 0 : c > 512 ? 1 : c > 256 ? 2 : c > kTileSortSmall ? 3 : c > 48 ? 4 : 5;
}
static_assert(kTileSortSmall == 128 && kOrderClasses == 6, "classes 0..3 are the long-list sort's");

// Block-wide exclusive scan of N64 64-bit and N32 32-bit per-thread sums
// (replaced by the thread's start); the carries (uniform) are added and
// advanced by the block totals.  The 64-bit channels count pairs (their
// totals decide the overflow); the 32-bit ones are exact whenever those fit
// the pair capacity.  w64 / w32 hold (NW + 1) entries per channel.  Every
// thread of the block must call.
template <int N64, int N32>
__device__ __forceinline__ void block_exscan(uint64_t (&s64)[N64], uint32_t (&s32)[N32],
                                             uint64_t (&c64)[N64], uint32_t (&c32)[N32],
                                             uint64_t* w64, uint32_t* w32) {
  constexpr int NW = kScanBlock / kWave;
  static_assert(NW == 16, "the wave sums are scanned within one 16-lane row");
  const int lane = lane_id(), w = threadIdx.x / kWave;
  uint64_t i64[N64];
  uint32_t i32[N32];
#pragma unroll
  for (int c = 0; c < N64; ++c) i64[c] = scan_dpp<6>(s64[c]);
#pragma unroll
  for (int c = 0; c < N32; ++c) i32[c] = scan_dpp<6>(s32[c]);
  if (lane == kWave - 1) {
#pragma unroll
    for (int c = 0; c < N64; ++c) w64[c * (NW + 1) + w] = i64[c];
#pragma unroll
    for (int c = 0; c < N32; ++c) w32[c * (NW + 1) + w] = i32[c];
  }
  __syncthreads();
  if (w == 0) {
    // lanes 0..15 of wave 0 scan the wave sums: exclusive offsets (plus the
    // carry) at [0, NW), the new carry at [NW]
#pragma unroll
    for (int c = 0; c < N64; ++c) {
      const uint64_t x = lane < NW ? w64[c * (NW + 1) + lane] : 0ull;
      const uint64_t j = scan_dpp<4>(x);
      if (lane < NW) w64[c * (NW + 1) + lane] = c64[c] + j - x;
      if (lane == NW - 1) w64[c * (NW + 1) + NW] = c64[c] + j;
    }
#pragma unroll
    for (int c = 0; c < N32; ++c) {
      const uint32_t x = lane < NW ? w32[c * (NW + 1) + lane] : 0u;
      const uint32_t j = scan_dpp<4>(x);
      if (lane < NW) w32[c * (NW + 1) + lane] = c32[c] + j - x;
      if (lane == NW - 1) w32[c * (NW + 1) + NW] = c32[c] + j;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < N64; ++c) {
    s64[c] = w64[c * (NW + 1) + w] + i64[c] - s64[c];
    c64[c] = w64[c * (NW + 1) + NW];
  }
#pragma unroll
  for (int c = 0; c < N32; ++c) {
    s32[c] = w32[c * (NW + 1) + w] + i32[c] - s32[c];
    c32[c] = w32[c * (NW + 1) + NW];
  }
  __syncthreads();  // the wave sums are rewritten by the next round
}

// Four consecutive u32 from a[i], zeros past n (a is 16-byte aligned, i a
// multiple of 4).
__device__ __forceinline__ uint4 load4(const uint32_t* __restrict__ a, int64_t i, int64_t n) {
  if (i + 4 <= n) return *reinterpret_cast<const uint4*>(a + i);
  uint4 x = make_uint4(0u, 0u, 0u, 0u);
  if (i < n) x.x = a[i];
  if (i + 1 < n) x.y = a[i + 1];
  if (i + 2 < n) x.z = a[i + 2];
  return x;
}

__device__ __forceinline__ void store4(uint32_t* __restrict__ a, int64_t i, int64_t n, uint4 x) {
  if (i + 4 <= n) {
    *reinterpret_cast<uint4*>(a + i) = x;
    return;
  }
  if (i < n) a[i] = x.x;
  if (i + 1 < n) a[i + 1] = x.y;
  if (i + 2 < n) a[i + 2] = x.z;
}

// Per-thread inputs of one round: 4 * kScanVec tiles and 2 * kScanVec
// chunks, and the thread's sums over them.  Channels: 64-bit tile pairs and
// chunk pairs; 32-bit buckets, visible records, and the tiles
// of each length class but the last (work order; the first four together are
// the lists of the long-list sort).
constexpr int kScanClass = 2;
constexpr int kScanN32 = kScanClass + kOrderClasses - 1;
// The 32-bit channels of a round, scanned packed: a round has at most
// kTileRound tiles, so its class counts fit 16 bits and go two to a word (the
// one-block scan of a small plan is a chain of these).  s: per-thread sums in,
// exclusive starts out (the carries c added); c advanced by the round's
// totals.
__device__ __forceinline__ void round_exscan(uint64_t (&s64)[2], uint32_t (&s)[kScanN32],
                                             uint64_t (&c64)[2], uint32_t (&c)[kScanN32],
                                             uint64_t* w64, uint32_t* w32) {
  static_assert(kScanN32 == 7 && kTileRound < 65536, "buckets, visible, five classes");
  uint32_t p[5] = {s[0], s[1], s[2] | s[3] << 16, s[4] | s[5] << 16, s[6]};
  uint32_t t[5] = {};
  block_exscan<2, 5>(s64, p, c64, t, w64, w32);
  const uint32_t e[7] = {p[0], p[1], p[2] & 0xFFFFu, p[2] >> 16, p[3] & 0xFFFFu, p[3] >> 16, p[4]};
  const uint32_t d[7] = {t[0], t[1], t[2] & 0xFFFFu, t[2] >> 16, t[3] & 0xFFFFu, t[3] >> 16, t[4]};
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    s[k] = c[k] + e[k];
    c[k] += d[k];
  }
}

struct ScanRound {
  static constexpr int NT = 4 * kScanVec, NC = 2 * kScanVec;
  int64_t it, ic;  // first tile and first chunk of the thread
  uint32_t tc[NT], nb[NT], cp[NC], cv[NC];
  uint64_t s64[2];
  uint32_t s32[kScanN32];
};

__device__ __forceinline__ void scan_load(const ScanArgs& A, int64_t r, ScanRound& R) {
  const int64_t T = A.n_tiles, C = A.n_chunks;
  R.it = r * kTileRound + (int64_t)ScanRound::NT * threadIdx.x;
  R.ic = r * kChunkRound + (int64_t)ScanRound::NC * threadIdx.x;
  const uint32_t* chunk_in = reinterpret_cast<const uint32_t*>(A.chunk_cnt);
#pragma unroll
  for (int k = 0; k < kScanVec; ++k) {
    uint4 x = load4(A.cnt.at, R.it + 4 * k, T);
    if (A.cnt.copies > 1) {
      uint4 y[kCountCopies];
#pragma unroll
      for (int j = 1; j < kCountCopies; ++j)
        y[j] = j < A.cnt.copies ? load4(A.cnt.at + j * A.cnt.stride, R.it + 4 * k, T)
                                : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int j = 1; j < kCountCopies; ++j)
        x = make_uint4(x.x + y[j].x, x.y + y[j].y, x.z + y[j].z, x.w + y[j].w);
    }
    if (A.mode == kScanTiles) {  // list end (0: no pairs) minus list start
      const uint4 st = load4(A.tstart, R.it + 4 * k, T);
      x = make_uint4(x.x ? x.x - st.x : 0u, x.y ? x.y - st.y : 0u, x.z ? x.z - st.z : 0u,
                     x.w ? x.w - st.w : 0u);
    }
    R.tc[4 * k] = x.x; R.tc[4 * k + 1] = x.y; R.tc[4 * k + 2] = x.z; R.tc[4 * k + 3] = x.w;
    const uint4 y = load4(chunk_in, 2 * (R.ic + 2 * k), 2 * C);
    R.cp[2 * k] = y.x; R.cv[2 * k] = y.y; R.cp[2 * k + 1] = y.z; R.cv[2 * k + 1] = y.w;
  }
  R.s64[0] = R.s64[1] = 0;
#pragma unroll
  for (int c = 0; c < kScanN32; ++c) R.s32[c] = 0;
#pragma unroll
  for (int k = 0; k < ScanRound::NT; ++k) {
    R.nb[k] = (R.tc[k] + kBucket - 1) / kBucket;
    R.s64[0] += R.tc[k];
    R.s32[0] += R.nb[k];
    const int oc = order_class(R.tc[k]);
#pragma unroll
    for (int c = 0; c < kOrderClasses - 1; ++c) R.s32[kScanClass + c] += oc == c ? 1u : 0u;
  }
#pragma unroll
  for (int k = 0; k < ScanRound::NC; ++k) {
    R.s64[1] += R.cp[k];
    R.s32[1] += R.cv[k];
  }
}

// Writes the round's outputs from the thread's exclusive starts (R.s64 /
// R.s32 after the block scan): list starts, bucket offsets and queue
// positions, work order, long-list entries (in tile order), chunk offsets;
// and sets the tile counters to the list starts (the scatter's cursors).
__device__ __forceinline__ void scan_emit(const ScanArgs& A, ScanRound& R) {
  const int64_t T = A.n_tiles, C = A.n_chunks;
  uint32_t* chunk_out = reinterpret_cast<uint32_t*>(A.chunk_pre);
#pragma unroll
  for (int k = 0; k < kScanVec; ++k) {
    uint32_t ts[4], bs[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t t = R.it + 4 * k + e;
      const uint32_t c = R.tc[4 * k + e];
      // work order: the tile's place in its class (the last class takes the
      // tiles that none of the others counts)
      const int oc = order_class(c);
      uint32_t counted = 0, place = 0;
#pragma unroll
      for (int k5 = 0; k5 < kOrderClasses - 1; ++k5) {
        counted += R.s32[kScanClass + k5];
        place = oc == k5 ? R.s32[kScanClass + k5] : place;
      }
      if (oc == kOrderClasses - 1) place = (uint32_t)t - counted;
      if (t < T) A.order[(int64_t)oc * T + place] = (uint32_t)t;
      // lists for the long-list sort (in tile order)
      if (t < T && c > kTileSortSmall)
        A.long_list[R.s32[kScanClass] + R.s32[kScanClass + 1] + R.s32[kScanClass + 2] +
                    R.s32[kScanClass + 3]] = make_uint4((uint32_t)t, (uint32_t)R.s64[0], c, 0u);
      ts[e] = (uint32_t)R.s64[0];
      bs[e] = R.s32[0];
      R.s64[0] += c;
      R.s32[0] += R.nb[4 * k + e];
#pragma unroll
      for (int k5 = 0; k5 < kOrderClasses - 1; ++k5) R.s32[kScanClass + k5] += oc == k5 ? 1u : 0u;
    }
    store4(A.tstart, R.it + 4 * k, T, make_uint4(ts[0], ts[1], ts[2], ts[3]));
    // the scatter's cursors start where the copy's pairs begin in the list;
    // the radix binning's per-tile pass reads the counts
    if (A.mode == kScanTiles) {
      store4(A.cnt.at, R.it + 4 * k, T,
             make_uint4(R.tc[4 * k], R.tc[4 * k + 1], R.tc[4 * k + 2], R.tc[4 * k + 3]));
    } else if (A.cnt.copies == 1) {
      store4(A.cnt.at, R.it + 4 * k, T, make_uint4(ts[0], ts[1], ts[2], ts[3]));
    } else {
      uint4 y[kCountCopies], at = make_uint4(ts[0], ts[1], ts[2], ts[3]);
#pragma unroll
      for (int j = 0; j < kCountCopies; ++j)
        if (j < A.cnt.copies) y[j] = load4(A.cnt.at + j * A.cnt.stride, R.it + 4 * k, T);
#pragma unroll
      for (int j = 0; j < kCountCopies; ++j)
        if (j < A.cnt.copies) {
          store4(A.cnt.at + j * A.cnt.stride, R.it + 4 * k, T, at);
          at = make_uint4(at.x + y[j].x, at.y + y[j].y, at.z + y[j].z, at.w + y[j].w);
        }
    }
    if (A.boff) store4(A.boff, R.it + 4 * k, T, make_uint4(bs[0], bs[1], bs[2], bs[3]));
    const uint32_t p0 = (uint32_t)R.s64[1], v0 = R.s32[1];
    const uint32_t p1 = p0 + R.cp[2 * k], v1 = v0 + R.cv[2 * k];
    store4(chunk_out, 2 * (R.ic + 2 * k), 2 * C, make_uint4(p0, v0, p1, v1));
    R.s64[1] = p1 + R.cp[2 * k + 1];
    R.s32[1] = v1 + R.cv[2 * k + 1];
  }
}

// Totals -> flags (one thread).  Both pair totals count the same pairs; a
// mismatch is reported as an overflow so that nothing is scattered.
__device__ __forceinline__ void scan_finish(const ScanArgs& A, const uint64_t (&c64)[2],
                                            const uint32_t (&c32)[kScanN32], int64_t cap,
                                            int32_t* __restrict__ fl, const StepAdvance& st) {
  const bool splat = A.boff != nullptr;
  const uint32_t long_lists =
      c32[kScanClass] + c32[kScanClass + 1] + c32[kScanClass + 2] + c32[kScanClass + 3];
  if (A.mode != kScanChunks)
    for (int c = 0; c < kOrderClasses - 1; ++c) fl[F_CLASS + c] = (int32_t)c32[kScanClass + c];
  if (A.mode == kScanTiles) {
    // the pair totals were settled by the chunk scan before
    const bool over = fl[F_OVERFLOW] != 0;
    fl[F_LONG_TILES] = over ? 0 : (int32_t)long_lists;
    fl[F_BUCKETS] = (over || !splat) ? 0 : (int32_t)c32[0];
    if (splat) A.boff[A.n_tiles] = c32[0];
    return;
  }
  const uint64_t tile_pairs = c64[0], chunk_pairs = c64[1];
  const bool chunks_only = A.mode == kScanChunks;
  const uint64_t pairs = chunks_only ? chunk_pairs : tile_pairs;
  const bool over = pairs > (uint64_t)cap || (!chunks_only && tile_pairs != chunk_pairs);
  fl[F_OVERFLOW] = over ? 1 : 0;
  fl[F_PAIRS] = over ? 0 : (int32_t)pairs;
  fl[F_PAIRS_WANTED] = pairs > 0x7FFFFFFFull ? 0x7FFFFFFF : (int32_t)pairs;
  fl[F_VISIBLE] = (int32_t)c32[1];
  fl[F_NONFINITE] = fl[F_NF_ACC];  // counted by the projection
  fl[F_NF_ACC] = 0;
  fl[F_HEAVY] = 0;  // counted by the kernel that lists the visible records
  if (!chunks_only) {
    // the bucket queue is filled by the tile sort at the positions scanned
    // here; the long lists are sorted by their own kernel (none on overflow)
    fl[F_LONG_TILES] = (int32_t)long_lists;
    fl[F_BUCKETS] = (over || !splat) ? 0 : (int32_t)c32[0];
    if (splat) A.boff[A.n_tiles] = c32[0];
  }
  // a whole iteration with Adam advances its step here, once the pairs are
  // known to fit: after an overflow the iteration's Adam launch changes
  // nothing, and neither does the step counter
  if (st.step && !over) advance_step(st);
}

// One block, all rounds in sequence (small plans: no extra launches).
__global__ void __launch_bounds__(kScanBlock) k_scans(ScanArgs A, int64_t cap,
                                                      int32_t* __restrict__ fl, StepAdvance st) {
  constexpr int NW = kScanBlock / kWave;
  __shared__ uint64_t w64[2 * (NW + 1)];
  __shared__ uint32_t w32[kScanN32 * (NW + 1)];
  uint64_t c64[2] = {0, 0};
  uint32_t c32[kScanN32] = {};
  const int64_t rt = (A.n_tiles + kTileRound - 1) / kTileRound;
  const int64_t rc = (A.n_chunks + kChunkRound - 1) / kChunkRound;
  const int64_t rounds = rt > rc ? rt : rc;
  for (int64_t r = 0; r < rounds; ++r) {
    ScanRound R;
    scan_load(A, r, R);
    round_exscan(R.s64, R.s32, c64, c32, w64, w32);
    scan_emit(A, R);
  }
  if (threadIdx.x == 0) scan_finish(A, c64, c32, cap, fl, st);
}

// Larger plans: one block per round in two launches.  Per-round totals of
// every channel (reduce), then every round again from its carry (down; the
// last block sets the flags).  The carries were scanned by a launch of one
// block in between: 23.3 -> 19.6 us for 12750 tiles and 4700 chunks.
struct ScanPart {
  uint64_t p64[2];
  uint32_t p32[kScanN32];
  uint32_t pad;
};

__global__ void __launch_bounds__(kScanBlock) k_scan_reduce(ScanArgs A,
                                                            ScanPart* __restrict__ part) {
  constexpr int NW = kScanBlock / kWave;
  __shared__ uint64_t w64[2 * (NW + 1)];
  __shared__ uint32_t w32[kScanN32 * (NW + 1)];
  uint64_t c64[2] = {0, 0};
  uint32_t c32[kScanN32] = {};
  ScanRound R;
  scan_load(A, blockIdx.x, R);
  round_exscan(R.s64, R.s32, c64, c32, w64, w32);  // c64 / c32: block totals
  if (threadIdx.x == 0) {
    ScanPart p;
    p.p64[0] = c64[0];
    p.p64[1] = c64[1];
#pragma unroll
    for (int c = 0; c < kScanN32; ++c) p.p32[c] = c32[c];
    p.pad = 0u;
    part[blockIdx.x] = p;
  }
}

// Each block adds up the partial sums before its own instead of waiting for
// a launch that scans them; the last block has the totals.
__global__ void __launch_bounds__(kScanBlock) k_scan_down(ScanArgs A,
                                                          const ScanPart* __restrict__ part,
                                                          int64_t cap, int32_t* __restrict__ fl,
                                                          StepAdvance st) {
  constexpr int NW = kScanBlock / kWave;
  __shared__ uint64_t w64[2 * (NW + 1)];
  __shared__ uint32_t w32[kScanN32 * (NW + 1)];
  ScanRound R;
  scan_load(A, blockIdx.x, R);  // (in flight while the partial sums are added)
  uint64_t c64[2] = {0, 0};
  uint32_t c32[kScanN32] = {};
  for (uint32_t base = 0; base < blockIdx.x; base += kScanBlock) {
    const uint32_t i = base + threadIdx.x;
    uint64_t s64[2] = {0, 0};
    uint32_t s32[kScanN32] = {};
    if (i < blockIdx.x) {
      const ScanPart p = part[i];
      s64[0] = p.p64[0];
      s64[1] = p.p64[1];
#pragma unroll
      for (int c = 0; c < kScanN32; ++c) s32[c] = p.p32[c];
    }
    block_exscan<2, kScanN32>(s64, s32, c64, c32, w64, w32);
  }
  round_exscan(R.s64, R.s32, c64, c32, w64, w32);
  scan_emit(A, R);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) scan_finish(A, c64, c32, cap, fl, st);
}

// ---------------------------------------------------------------- scatter
// One wavefront per chunk (64 Gaussians of one view, the projection's
// wavefront): the generation offsets of its records become absolute (poff),
// its visible records are listed in index order, and every pair gets the
// next free slot of its tile's list with key (depth bits << 32 | generation
// index); pair -> record is recorded.  The chunk's pairs are spread evenly
// over the lanes (exclusive scan of the pair counts, binary search of a
// pair's record in LDS), so a large Gaussian does not serialise its tiles'
// slot claims on one lane.
__global__ void __launch_bounds__(256) k_scatter(
    const uint32_t* __restrict__ tt, uint32_t* __restrict__ poff,
    const uint2* __restrict__ chunk_pre, int64_t chunks_per_view, int64_t n_chunks,
    const ushort4* __restrict__ rect, const uint32_t* __restrict__ zbits, int64_t n, ViewTable vt,
    int32_t* __restrict__ fl, HeavyList heavy, TileCounters cursors, uint64_t* __restrict__ skey, uint32_t* __restrict__ pair_rec,
    uint32_t* __restrict__ vis_list) {
  constexpr int NW = 256 / kWave;
  __shared__ uint32_t s_pre[NW][kWave];
  __shared__ uint32_t s_p0[NW][kWave], s_dbits[NW][kWave], s_x0y0[NW][kWave];
  __shared__ uint32_t s_tile0[NW][kWave];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  const int64_t gw = (int64_t)blockIdx.x * NW + w;  // chunk
  if (gw >= n_chunks) return;                       // whole wavefront; no block barrier below
  const int v = (int)(gw / chunks_per_view);
  const int64_t gi = (gw - (int64_t)v * chunks_per_view) * kWave + lane;  // Gaussian
  const int64_t ri = (int64_t)v * n + gi;                                 // record
  const uint64_t P = (uint64_t)fl[F_PAIRS];
  const bool over = fl[F_OVERFLOW] != 0;
  const uint32_t c = (gi < n && !over) ? tt[ri] : 0u;
  const uint2 cp = chunk_pre[gw];
  // the record's tile box and depth are fetched before the scan of the
  // counts, which then runs while they are in flight (DPP, no LDS)
  ushort4 r = make_ushort4(0, 0, 0, 0);
  uint32_t dbits = 0;
  if (c > 0) {
    r = rect[ri];
    dbits = zbits[ri];
  }
  const uint32_t incl = scan_dpp<6>(c);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  const uint64_t base64 = (uint64_t)cp.x + (incl - c);
  if ((uint64_t)cp.x + total > P) return;  // cannot happen without overflow (uniform)
  const uint64_t vmask = ballot64(c > 0);
  uint32_t p0 = 0, x0y0 = 0, tile0 = 0;
  if (c > 0) {
    p0 = (uint32_t)base64;
    poff[ri] = p0;
    const uint32_t vp = cp.y + (uint32_t)__popcll(vmask & lanemask_lt());
    vis_list[vp] = (uint32_t)ri;
    note_heavy(heavy, fl, c, (uint32_t)ri);
    x0y0 = (uint32_t)r.x | ((uint32_t)r.y << 16);
    tile0 = (uint32_t)(r.z - r.x);  // box width in tiles
  }
  if (total == 0) return;
  s_pre[w][lane] = incl - c;
  s_p0[w][lane] = p0;
  s_dbits[w][lane] = dbits;
  s_x0y0[w][lane] = x0y0;
  s_tile0[w][lane] = tile0;
  wave_lds_sync();
  const ViewInfo vi = vt.v[v];
  const uint32_t rec0 = (uint32_t)(ri - lane);
  uint32_t* cursor = count_copy(cursors, gw - (int64_t)v * chunks_per_view);
  for (uint32_t q = (uint32_t)lane; q < total; q += kWave) {
    // owner: the last lane whose prefix is <= q (it has pairs)
    int lo = 0, hi = kWave - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_pre[w][mid] <= q) lo = mid; else hi = mid - 1;
    }
    const uint32_t k = q - s_pre[w][lo];
    const uint32_t bw = s_tile0[w][lo], xy = s_x0y0[w][lo];
    const int x = (int)(xy & 0xFFFFu) + (int)(k % bw);
    const int y = (int)(xy >> 16) + (int)(k / bw);
    const int t = vi.tile_off + y * vi.tiles_x + x;
    const uint32_t p = s_p0[w][lo] + k;
    const uint32_t slot = atomicAdd(&cursor[t], 1u);
    if (slot < P) skey[slot] = ((uint64_t)s_dbits[w][lo] << 32) | p;
    pair_rec[p] = rec0 + (uint32_t)lo;
  }
}

// ---------------------------------------------------------------- tile sort
// (per-tile sort helpers in tilesort.h)

// Blocks [0, long_blocks): the listed long lists -- those beyond
// kTileSortMid pairs a workgroup each, the others a wavefront each.  The
// other blocks: the tiles, a wavefront each (the long lists' wavefronts only
// write the range and queue entries there).  One launch where there were
// three: the long lists, first in the grid, hide behind the short ones (with
// the networks still in LDS: 1200x680 view, 12750 lists of 34 pairs on
// average, 44 -> 35 us; in 16x16 tiles, 3225 lists of 194, 116 -> 64 us; a
// 128x96 view 30 -> 15 us).  Held to 64 registers so that two workgroups share
// a CU: the three now take 15, 32 and 6 us, with one workgroup a CU 17, 38 and
// 6; 2.7M pairs in 12900 lists 87 and 130.  Bound by VALU issue (some 450
// instructions a key of a list of 512) and the latency of its chain.
__global__ void __launch_bounds__(kSortWaves * kWave) __attribute__((amdgpu_waves_per_eu(8))) k_tile_sort(
    TileSortArgs A, uint64_t* __restrict__ skey, const uint4* __restrict__ long_list,
    int long_blocks, int n_tiles) {
  __shared__ uint64_t sk[kTileSortLong];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  uint64_t* wsk = sk + w * kTileSortMid;
  if ((int)blockIdx.x >= long_blocks) {
    const int t = ((int)blockIdx.x - long_blocks) * kSortWaves + w;
    if (t < n_tiles) sort_tile_wave(A, t, lane, wsk);
    return;
  }
  const int n_long = A.fl[F_OVERFLOW] ? 0 : A.fl[F_LONG_TILES];
  for (int li = blockIdx.x; li < n_long; li += long_blocks) {
    const uint4 e = long_list[li];  // the scan recorded (tile, list start, pairs, -)
    const uint32_t start = e.y, n = e.z;
    if (n <= kTileSortMid) continue;  // uniform: a wavefront's, below
    const uint64_t tkey = (uint64_t)e.x << 32;
    constexpr uint32_t NT = kSortWaves * kWave;
    if (n <= kTileSortLong) {
      sort_keys_block(skey + start, n, w, lane, sk);
      __syncthreads();
      for (uint32_t k = threadIdx.x; k < n; k += NT) emit_sorted(A.out, start + k, tkey, sk[k]);
    } else {
      bitonic_sort(skey + start, n, threadIdx.x, NT);
      for (uint32_t k = threadIdx.x; k < n; k += NT)
        emit_sorted(A.out, start + k, tkey, skey[start + k]);
    }
    __syncthreads();  // the LDS is reused
  }
  for (int li = blockIdx.x + w * long_blocks; li < n_long; li += long_blocks * kSortWaves) {
    const uint4 e = long_list[li];
    if (e.z <= kTileSortMid)
      sort_list_wave<kTileSortMid>(A.out, skey, (uint64_t)e.x << 32, e.y, e.z, lane, wsk);
  }
}

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int64_t blocks = (count + 255) / 256;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, value, count);
  return hipGetLastError();
}

hipError_t launch_rb_generate(const Plan& P, void* ws, hipStream_t s);
hipError_t launch_rb_tile_sort(const Plan& P, void* ws, hipStream_t s);
hipError_t launch_rb_runs(const Plan& P, void* ws, hipStream_t s);

hipError_t launch_clear_counters(const Plan& P, void* ws, hipStream_t s) {
  // per-iteration flags 0..10 and the per-tile pair counters
  const int64_t words = P.cnt_stride * P.cnt_copies;
  const int64_t m = std::max<int64_t>(words, F_NF_ACC + 1);
  hipLaunchKernelGGL(k_fill2_u32, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s,
                     ws_at<uint32_t>(ws, P.off_flags), (int64_t)(F_NF_ACC + 1),
                     ws_at<uint32_t>(ws, P.off_tile_cnt), words);
  return hipGetLastError();
}

// Arguments of the per-tile sort.
static TileSortArgs tile_sort_args(const Plan& P, void* ws) {
  const bool splat = P.splat != 0;
  TileSortArgs A{};
  A.cnt = tile_counters(P, ws);
  A.tstart = ws_at<uint32_t>(ws, P.off_tile_start);
  A.fl = ws_at<int32_t>(ws, P.off_flags);
  const bool radix = (P.cfg.flags & GS_RADIX_BIN) != 0;  // (no scattered keys, no copies)
  A.skey = radix ? nullptr : ws_at<uint64_t>(ws, P.off_scatter);
  A.out = TileSortOut{ws_at<uint64_t>(ws, P.off_keys), ws_at<uint32_t>(ws, P.off_vals),
                      ws_at<uint32_t>(ws, P.off_sorted_rec),
                      radix ? nullptr : ws_at<uint32_t>(ws, P.off_pair_rec)};
  A.ranges = ws_at<uint32_t>(ws, P.off_ranges);
  A.boff = splat ? ws_at<uint32_t>(ws, P.off_boff) : nullptr;
  A.bq = splat ? ws_at<uint2>(ws, P.off_bq) : nullptr;
  A.presorted = radix;
  return A;
}

hipError_t launch_bin_sort(const Plan& P, void* ws, hipStream_t s, const StepAdvance* step,
                           const Marks* marks) {
  const Marks none{};
  const Marks& mk = marks ? *marks : none;
  int32_t* fl = ws_at<int32_t>(ws, P.off_flags);
  uint32_t* tt = ws_at<uint32_t>(ws, P.off_tt);
  uint32_t* poff = ws_at<uint32_t>(ws, P.off_poff);
  uint32_t* tstart = ws_at<uint32_t>(ws, P.off_tile_start);
  const int T = P.vt.total_tiles;
  const uint2* chunk_cnt = ws_at<uint2>(ws, P.off_chunk_cnt);
  uint2* chunk_pre = ws_at<uint2>(ws, P.off_chunk_pre);
  uint4* long_list = ws_at<uint4>(ws, P.off_long);
  const bool radix = (P.cfg.flags & GS_RADIX_BIN) != 0;
  ScanArgs sa{chunk_cnt, chunk_pre, P.n_chunks, tile_counters(P, ws), tstart, (int64_t)T,
              P.splat ? ws_at<uint32_t>(ws, P.off_boff) : nullptr,
              ws_at<uint32_t>(ws, P.off_order), long_list, kScanBoth};
  // always launched, so that the flags are always set: one block for a
  // plan of one round, one block per round in two launches beyond
  const StepAdvance adv = step ? *step : StepAdvance{};
  auto scan = [&](const ScanArgs& a, const StepAdvance& st) {
    if (P.scan_rounds <= 1) {
      hipLaunchKernelGGL(k_scans, dim3(1), dim3(kScanBlock), 0, s, a, P.pair_cap, fl, st);
    } else {
      static_assert(sizeof(ScanPart) <= 64, "scan partial slot");
      ScanPart* part = ws_at<ScanPart>(ws, P.off_scan_part);
      const unsigned rounds = (unsigned)P.scan_rounds;
      hipLaunchKernelGGL(k_scan_reduce, dim3(rounds), dim3(kScanBlock), 0, s, a, part);
      hipLaunchKernelGGL(k_scan_down, dim3(rounds), dim3(kScanBlock), 0, s, a, part, P.pair_cap, fl,
                         st);
    }
  };
  if (radix) {
    ScanArgs sc = sa;
    sc.n_tiles = 0;
    sc.mode = kScanChunks;
    scan(sc, adv);
  } else {
    scan(sa, adv);
  }
  hipError_t e = mk.at(GS_MARK_BIN_SCAN, s);
  if (e != hipSuccess) return e;
  if (radix) {
    // records by depth, their pairs in that order, then the pairs by tile;
    // the list starts and ends found in the sorted keys give the per-tile
    // counts (the projection counted none), scanned like the projection's;
    // the per-tile pass writes the ranges and queue entries and zeroes the
    // counters
    if ((e = launch_rb_generate(P, ws, s)) != hipSuccess) return e;
    if ((e = mk.at(GS_MARK_BIN_SCATTER, s)) != hipSuccess) return e;
    if ((e = launch_rb_tile_sort(P, ws, s)) != hipSuccess) return e;
    if ((e = mk.at(GS_MARK_BIN_SHORT_SORT, s)) != hipSuccess) return e;
    if ((e = launch_rb_runs(P, ws, s)) != hipSuccess) return e;
    ScanArgs st = sa;
    st.n_chunks = 0;
    st.mode = kScanTiles;
    scan(st, StepAdvance{});
    if (T > 0)
      hipLaunchKernelGGL(k_tile_sort, dim3((unsigned)((T + kSortWaves - 1) / kSortWaves)),
                         dim3(kSortWaves * kWave), 0, s, tile_sort_args(P, ws), nullptr, long_list,
                         0, T);
    if ((e = mk.at(GS_MARK_BIN_LONG_SORT, s)) != hipSuccess) return e;
    return hipGetLastError();
  }
  uint64_t* skey = ws_at<uint64_t>(ws, P.off_scatter);
  uint32_t* pair_rec = ws_at<uint32_t>(ws, P.off_pair_rec);
  if (P.n_chunks > 0) {
    const int64_t blocks = (P.n_chunks + 3) / 4;
    hipLaunchKernelGGL(k_scatter, dim3((unsigned)blocks), dim3(256), 0, s, tt, poff, chunk_pre,
                       P.chunks_per_view, P.n_chunks, ws_at<ushort4>(ws, P.off_rect),
                       ws_at<uint32_t>(ws, P.off_zbits), P.n, P.vt, fl, heavy_list(P, ws), tile_counters(P, ws),
                       skey, pair_rec,
                       ws_at<uint32_t>(ws, P.off_vis_list));
  }
  if ((e = mk.at(GS_MARK_BIN_SCATTER, s)) != hipSuccess) return e;
  if (T > 0) {
    // the pass over the tiles zeroes the counters, so that every counter is
    // zero again after the binning of an iteration.  At most one long list
    // per kTileSortSmall + 1 pairs of capacity; two workgroups per CU are
    // resident and loop over the lists
    const int64_t max_long = std::min<int64_t>(T, P.pair_cap / (kTileSortSmall + 1) + 1);
    const int long_blocks = (int)std::min<int64_t>(max_long, 512);
    hipLaunchKernelGGL(k_tile_sort,
                       dim3((unsigned)(long_blocks + (T + kSortWaves - 1) / kSortWaves)),
                       dim3(kSortWaves * kWave), 0, s, tile_sort_args(P, ws), skey, long_list,
                       long_blocks, T);
  }
  if ((e = mk.at(GS_MARK_BIN_SHORT_SORT, s)) != hipSuccess) return e;
  if ((e = mk.at(GS_MARK_BIN_LONG_SORT, s)) != hipSuccess) return e;
  return hipGetLastError();
}

// Rounds of the binning scan for a plan (a round = one block's share).
int64_t scan_rounds(const Plan& P) {
  const int64_t rt = ((int64_t)P.vt.total_tiles + kTileRound - 1) / kTileRound;
  const int64_t rc = (P.n_chunks + kChunkRound - 1) / kChunkRound;
  return std::max<int64_t>(1, std::max(rt, rc));
}

// Sorted pair values (generation indices) after launch_bin_sort.
uint32_t* sorted_vals(const Plan& P, void* ws) { return ws_at<uint32_t>(ws, P.off_vals); }

}  // namespace gs
