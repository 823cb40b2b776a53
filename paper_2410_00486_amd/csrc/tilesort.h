// Per-tile list sort of the binning.
//
// Output per tile: sorted keys (tile << 32 | depth bits), generation
// indices, record ids, the [start, end) range ((0, 0) when empty) and, for the
// splat-wise backward, the tile's entries in the bucket queue.  Keys are
// unique, so any correct sort gives the same lists.  One launch: a wavefront
// ranks lists of up to 64 keys (rank = number of smaller keys) and sorts up to
// kTileSortMid in its registers, a bitonic network padded with keys above any
// other; longer lists take a whole 1024-thread workgroup, the same network
// with its widest exchanges through LDS up to kTileSortLong keys, and one in
// place in global memory beyond.  The workgroup's LDS holds kTileSortLong keys
// (64 KB), so that two share a CU (32 wavefronts, all it holds) and one's
// barrier waits overlap the other's compares.
//
// The network in global memory keeps every merge ascending (the first compare
// of a merge pairs i with its mirror in the block), so positions past the list
// end act as +infinity and are never touched: no padding is written.
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

// Sorts k[0, n) ascending (global memory) with nthreads threads of
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

// Both keys of a compare-exchange between lanes a distance of X apart: the
// lane's own and its partner's, in either order.
template <int X>
__device__ __forceinline__ void lane_pair(uint32_t& a, uint32_t& b) {
  if constexpr (X == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    a = r[0];
    b = r[1];
  } else if constexpr (X == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    a = r[0];
    b = r[1];
  } else if constexpr (X == 8) {
    b = (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0x128, 0xF, 0xF, true);  // row_ror:8
  } else if constexpr (X == 4) {  // row_shl:4 into the lower four of eight lanes, row_shr:4 the upper
    b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, 0x104, 0xF, 0x5, true);
    b = (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x114, 0xF, 0xA, true);
  } else {  // quad_perm [1,0,3,2] or [2,3,0,1]
    b = (uint32_t)__builtin_amdgcn_mov_dpp((int)a, X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
  }
}

// Stages of the bitonic network over 64 E keys (element lane E + r is k[r]):
// elements STRIDE, STRIDE / 2 .. apart, ascending in every other run of SIZE;
// a run of all keys ascends if `whole_up`.
template <int E, int SIZE, int STRIDE>
__device__ __forceinline__ void bitonic_stage(uint64_t (&k)[E], int lane, bool whole_up) {
  const bool lane_up = SIZE == E * kWave ? whole_up : (lane & (SIZE / E)) == 0;
  if constexpr (STRIDE < E) {
#pragma unroll
    for (int r = 0; r < E; ++r)
      if ((r & STRIDE) == 0) {
        const bool up = SIZE < E ? (r & SIZE) == 0 : lane_up;
        const uint64_t x = k[r], y = k[r + STRIDE];
        const bool keep = (x < y) == up;
        k[r] = keep ? x : y;
        k[r + STRIDE] = keep ? y : x;
      }
  } else {
    constexpr int X = STRIDE / E;
    const bool low = lane_up == ((lane & X) == 0);  // keeps the smaller one
#pragma unroll
    for (int r = 0; r < E; ++r) {
      uint32_t al = (uint32_t)k[r], ah = (uint32_t)(k[r] >> 32), bl, bh;
      lane_pair<X>(al, bl);
      lane_pair<X>(ah, bh);
      const uint64_t x = (uint64_t)ah << 32 | al, y = (uint64_t)bh << 32 | bl;
      k[r] = (x < y) == low ? x : y;
    }
  }
  if constexpr (STRIDE > 1) bitonic_stage<E, SIZE, STRIDE / 2>(k, lane, whole_up);
}
template <int E, int SIZE = 2>
__device__ __forceinline__ void bitonic_regs(uint64_t (&k)[E], int lane, bool whole_up) {
  bitonic_stage<E, SIZE, SIZE / 2>(k, lane, whole_up);
  if constexpr (SIZE < E * kWave) bitonic_regs<E, 2 * SIZE>(k, lane, whole_up);
}

// Sorts n <= 64 E keys from src into sk (LDS) with one wavefront: the keys
// stay in registers through the network.  With the network in LDS (two reads
// and two writes a comparison) the sort was bound by it: 2.7M pairs in 12900
// lists 133 us, now 88 (110 with only the lists up to 512 in registers); 433k
// in 12750 lists 22.5 and 15.5; 12.5k in 192 lists 13.8 and 5.4.  Up to 64
// pairs counting the smaller keys is as fast (15.2 and 17.2 us for the 433k).
template <int E>
__device__ __forceinline__ void sort_keys_wave(const uint64_t* __restrict__ src, uint32_t n,
                                               int lane, uint64_t* sk) {
  uint64_t k[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t i = (uint32_t)(r * kWave + lane);
    k[r] = i < n ? src[i] : ~0ull;
  }
  bitonic_regs<E>(k, lane, true);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t i = (uint32_t)(lane * E + r);
    if (i < n) sk[i] = k[r];
  }
}

// Sorts 512 < n <= 512 kSortWaves keys from src into sk (LDS, as many keys)
// with the whole workgroup: 512 keys per wavefront, as above; only the stages
// that compare keys of different wavefronts go through LDS.
__device__ __forceinline__ void sort_keys_block(const uint64_t* __restrict__ src, uint32_t n,
                                                int w, int lane, uint64_t* sk) {
  constexpr int E = kTileSortMid / kWave;
  int waves = 2;
  while ((uint32_t)waves * kTileSortMid < n) waves <<= 1;
  const bool on = w < waves;
  uint64_t k[E];
  if (on) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t i = (uint32_t)w * kTileSortMid + (uint32_t)(r * kWave + lane);
      k[r] = i < n ? src[i] : ~0ull;
    }
    bitonic_regs<E>(k, lane, (w & 1) == 0);
  }
  for (int size = 2; size <= waves; size <<= 1) {
    const bool up = (w & size) == 0;
    for (int d = size >> 1; d > 0; d >>= 1) {
      if (on) {
#pragma unroll
        for (int r = 0; r < E; ++r) sk[w * (int)kTileSortMid + r * kWave + lane] = k[r];
      }
      __syncthreads();
      if (on) {
        const bool low = up == ((w & d) == 0);
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const uint64_t y = sk[(w ^ d) * (int)kTileSortMid + r * kWave + lane];
          k[r] = (k[r] < y) == low ? k[r] : y;
        }
      }
      __syncthreads();
    }
    if (on) bitonic_stage<E, E * kWave, E * kWave / 2>(k, lane, up);
  }
  if (on) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t i = (uint32_t)w * kTileSortMid + (uint32_t)(lane * E + r);
      if (i < n) sk[i] = k[r];
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
  if (MAX <= 2 * kWave || n <= 2 * kWave) sort_keys_wave<2>(skey + start, n, lane, sk);
  else if (MAX <= 4 * kWave || n <= 4 * kWave) sort_keys_wave<4>(skey + start, n, lane, sk);
  else sort_keys_wave<8>(skey + start, n, lane, sk);
  wave_lds_sync();
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
