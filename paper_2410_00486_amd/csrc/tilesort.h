// Per-tile list sort of the binning.
//
// Output per tile: sorted keys (tile << 32 | depth bits), generation
// indices, record ids, the records in list order, the [start, end) range
// ((0, 0) when empty) and, for the splat-wise backward, the tile's entries
// in the bucket queue.  Keys are unique, so any correct sort gives the
// same lists.  One launch: a wavefront sorts lists up to 64 keys in
// registers (rank = number of smaller keys) and up to kTileSortMid keys with a
// bitonic network in LDS; longer lists take a whole 1024-thread workgroup,
// with the same network in LDS up to kTileSortLong keys and in place in
// global memory beyond.  The workgroup's LDS holds kTileSortLong keys
// (64 KB), so that two share a CU (32 wavefronts, all it holds) and one's
// barrier waits overlap the other's compares.
//
// The network keeps every merge ascending (the first compare of a merge
// pairs i with its mirror in the block), so positions past the list end act
// as +infinity and are never touched: no padding is written.
#pragma once

#include "gs_internal.h"

namespace gs {

// lists of more pairs are listed by the binning scan and sorted apart from
// the pass over the tiles
constexpr uint32_t kTileSortSmall = 128;
constexpr uint32_t kTileSortLong = 8192;
constexpr int kSortWaves = 16;                                  // wavefronts per workgroup
constexpr uint32_t kTileSortMid = kTileSortLong / kSortWaves;   // 512: one wavefront's share

struct TileSortOut {
  uint64_t* keys;
  uint32_t* vals;
  uint32_t* sorted_rec;
  const uint32_t* pair_rec;
};

// Writes the pair of key (depth bits << 32 | generation index) at list
// position pos: sorted key, generation index, record id.
__device__ __forceinline__ void emit_sorted(const TileSortOut& o, uint32_t pos, uint64_t tkey,
                                            uint64_t key) {
  const uint32_t g = (uint32_t)key;
  const uint32_t r = o.pair_rec[g];
  o.keys[pos] = tkey | (key >> 32);
  o.vals[pos] = g;
  o.sorted_rec[pos] = r;
}

__device__ __forceinline__ void cmp_swap(uint64_t* k, uint32_t a, uint32_t b, uint32_t n) {
  if (b >= n) return;
  const uint64_t ka = k[a], kb = k[b];
  if (ka > kb) {
    k[a] = kb;
    k[b] = ka;
  }
}

// Sorts k[0, n) ascending (LDS or global memory) with nthreads threads of
// the block; every thread of the block must call it.
__device__ inline void bitonic_sort(uint64_t* k, uint32_t n, uint32_t tid, uint32_t nthreads) {
  uint32_t m = 1;
  while (m < n) m <<= 1;
  for (uint32_t size = 2; size <= m; size <<= 1) {
    const uint32_t half = size >> 1;
    for (uint32_t idx = tid; idx < m / 2; idx += nthreads) {
      const uint32_t blk = idx / half, off = idx % half;
      cmp_swap(k, blk * size + off, blk * size + size - 1 - off, n);
    }
    __syncthreads();
    for (uint32_t stride = size >> 2; stride > 0; stride >>= 1) {
      for (uint32_t idx = tid; idx < m / 2; idx += nthreads) {
        const uint32_t a = 2 * idx - (idx & (stride - 1));
        cmp_swap(k, a, a + stride, n);
      }
      __syncthreads();
    }
  }
}

// Sorts k[0, n) ascending in LDS with the 64 lanes of one wavefront and
// wavefront-level syncs only (the other wavefronts of its workgroup sort
// their own lists meanwhile).
__device__ inline void bitonic_sort_wave(uint64_t* k, uint32_t n, uint32_t lane) {
  uint32_t m = 1;
  while (m < n) m <<= 1;
  for (uint32_t size = 2; size <= m; size <<= 1) {
    const uint32_t half = size >> 1;
    for (uint32_t idx = lane; idx < m / 2; idx += kWave) {
      const uint32_t blk = idx / half, off = idx % half;
      cmp_swap(k, blk * size + off, blk * size + size - 1 - off, n);
    }
    wave_lds_sync();
    for (uint32_t stride = size >> 2; stride > 0; stride >>= 1) {
      for (uint32_t idx = lane; idx < m / 2; idx += kWave) {
        const uint32_t a = 2 * idx - (idx & (stride - 1));
        cmp_swap(k, a, a + stride, n);
      }
      wave_lds_sync();
    }
  }
}

// Everything a wavefront needs to sort one tile's list.
struct TileSortArgs {
  TileCounters cnt;        // pairs per tile (the scatter's cursors); cleared after use
  const uint32_t* tstart;  // list start per tile
  const int32_t* fl;
  const uint64_t* skey;    // scattered keys (depth bits << 32 | generation index)
  TileSortOut out;
  uint32_t* ranges;
  const uint32_t* boff;  // splat-wise only (bq non-null): the tile's first queue entry
  uint2* bq;
  // the lists were sorted by the radix binning: ranges, queue entries and
  // counter clears only
  bool presorted;
};

// Sorts the n <= MAX keys of a list with one wavefront and writes the sorted
// outputs: the lane's positions are written out and their record ids looked
// up all at once (one memory round trip for all of them instead of one per
// position).  sk: MAX keys of LDS of this wavefront.
template <uint32_t MAX>
__device__ inline void sort_list_wave(const TileSortOut& o, const uint64_t* __restrict__ skey,
                                      uint64_t tkey, uint32_t start, uint32_t n, int lane,
                                      uint64_t* sk) {
  constexpr int KMAX = MAX / kWave;
  for (uint32_t k = lane; k < n; k += kWave) sk[k] = skey[start + k];
  wave_lds_sync();
  bitonic_sort_wave(sk, n, (uint32_t)lane);
  uint32_t r[KMAX];
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    const uint32_t k = (uint32_t)lane + (uint32_t)q * kWave;
    r[q] = 0u;
    if (k < n) {
      const uint64_t key = sk[k];
      const uint32_t g = (uint32_t)key;
      o.keys[start + k] = tkey | (key >> 32);
      o.vals[start + k] = g;
      r[q] = o.pair_rec[g];
    }
  }
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    const uint32_t k = (uint32_t)lane + (uint32_t)q * kWave;
    if (k < n) o.sorted_rec[start + k] = r[q];
  }
  wave_lds_sync();  // every key read before the next list overwrites them
}

// One wavefront: range and bucket queue entries of tile t, then, for a list
// of at most kTileSortSmall pairs, the sort and the sorted outputs.  sk:
// kTileSortSmall keys of LDS of this wavefront.
__device__ inline void sort_tile_wave(const TileSortArgs& A, int t, int lane, uint64_t* sk) {
  const uint64_t P = (uint64_t)A.fl[F_PAIRS];
  // (radix binning: the count; else the last copy's cursor is the list's end)
  const uint32_t c = A.cnt.at[(A.cnt.copies - 1) * A.cnt.stride + t] -
                     (A.presorted ? 0u : A.tstart[t]);
  const uint32_t n = A.fl[F_OVERFLOW] ? 0u : c;
  const uint64_t start64 = A.tstart[t];
  const bool ok = n > 0 && start64 + n <= P;
  if (lane == 0) {
    A.ranges[2 * (int64_t)t] = ok ? (uint32_t)start64 : 0u;
    A.ranges[2 * (int64_t)t + 1] = ok ? (uint32_t)(start64 + n) : 0u;
  }
  // the counters are consumed: zero again for the next projection
  if (lane < A.cnt.copies) A.cnt.at[lane * A.cnt.stride + t] = 0u;
  if (A.bq && ok) {
    // splat-wise work queue: the tile's buckets of 64 pairs
    const uint32_t q0 = A.boff[t], nb = (n + kBucket - 1) / kBucket;
    for (uint32_t k = lane; k < nb; k += kWave) A.bq[q0 + k] = make_uint2((uint32_t)t, k);
  }
  if (!ok || n > kTileSortSmall || A.presorted) return;  // uniform
  const uint32_t start = (uint32_t)start64;
  const uint64_t tkey = (uint64_t)(uint32_t)t << 32;
  if (n <= (uint32_t)kWave) {
    const bool has = (uint32_t)lane < n;
    const uint64_t key = has ? A.skey[start + lane] : ~0ull;
    uint32_t rank = 0;
    for (uint32_t j = 0; j < n; ++j) {
      const uint64_t kj = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(key >> 32), j) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, j);
      rank += kj < key ? 1u : 0u;
    }
    if (has) emit_sorted(A.out, start + rank, tkey, key);
    return;
  }
  sort_list_wave<kTileSortSmall>(A.out, A.skey, tkey, start, n, lane, sk);
}

}  // namespace gs
