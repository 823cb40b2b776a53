// Stable LSD radix sort of (uint64 key, uint32 value) pairs, 8-bit digits.
//
// Up to kBlockSort pairs: one workgroup keeps everything in LDS and runs
// every pass itself (one launch; small sorts are a chain of launches
// otherwise: 4096 pairs of 46 bits took 101 us in 12 launches, 43 in this one;
// 8192 took 136, now 49, and the passes below take 60 there).
//
// Larger: per pass the digit counts of each block of 1024 or 2048 keys, their scan
// over the blocks per digit, and a downsweep that ranks a block's keys
// (wave64 ballots, in index order: stable), reorders them in LDS and writes
// each digit's run contiguously.  Up to kFusedBlocks blocks the downsweep sums
// the counts itself, one launch fewer per pass: 20 000 pairs (20 blocks) 55 us
// so and 58 with the scan's own launch; at 30 blocks of 2048 it was 86 and 78.
// Before, every block summed up to 256 counts per digit in a serial loop and
// wrote each key where its rank put it: 2^20 pairs of 46 bits, 58 us a pass in
// the scatter alone; now 6 + 4 + 14 us a pass (eager), the whole sort 414 ->
// 116 us.  A pass moves 33 MB, 7 us at the rate of a large copy; the rest is
// the three launches and the chain of ranks within a block.
#include "sort.h"
#include "wavescan.h"

namespace gs {
namespace {

constexpr int kSortWaves = kSortThreads / kWave;
constexpr int64_t kFusedBlocks = 24;
constexpr int kBlockThreads = 1024;
constexpr int kBlockItems = 8;
constexpr int kBlockSort = kBlockThreads * kBlockItems;  // 8192 pairs
static_assert(kSortThreads == kSortRadix, "one digit per thread in the scans");

__device__ __forceinline__ uint32_t digit_of(uint64_t key, int shift) {
  return (uint32_t)(key >> shift) & (kSortRadix - 1);
}

// Lanes of the wavefront whose digit equals this lane's (among `valid`
// lanes), from one ballot per digit bit.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid) {
  uint64_t peers = ballot64(valid);
#pragma unroll
  for (int b = 0; b < kSortBits; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bb = ballot64(bit);
    peers &= bit ? bb : ~bb;
  }
  return peers;
}

// Exclusive scan over the first 256 threads of one value each (the first
// four wavefronts; every thread of the block must call).  ws: 4 words.
__device__ __forceinline__ uint32_t exscan256(uint32_t x, uint32_t* ws) {
  const int w = threadIdx.x / kWave, lane = lane_id();
  const uint32_t incl = scan_dpp<6>(x);
  if (lane == kWave - 1 && w < 4) ws[w] = incl;
  __syncthreads();
  uint32_t off = 0;
  for (int k = 0; k < w && k < 4; ++k) off += ws[k];
  __syncthreads();  // ws is reused by the caller's next scan
  return off + incl - x;
}

// Digit counts of each block, digit-major: hist[d * nb + block].
template <int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_sort_hist(const uint64_t* __restrict__ keys,
                                                            uint32_t n, uint32_t* __restrict__ hist,
                                                            uint32_t nb, int shift) {
  __shared__ uint32_t h[kSortWaves][kSortRadix];
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < kSortWaves; ++k) h[k][threadIdx.x] = 0u;
  __syncthreads();
  const uint32_t base = blockIdx.x * (uint32_t)(kSortThreads * ITEMS) + threadIdx.x;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t idx = base + r * kSortThreads;
    if (idx < n) atomicAdd(&h[w][digit_of(keys[idx], shift)], 1u);
  }
  __syncthreads();
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kSortWaves; ++k) s += h[k][threadIdx.x];
  hist[(size_t)threadIdx.x * nb + blockIdx.x] = s;
}

// One block per digit: exclusive scan of the digit's counts over the blocks
// (in place); the digit's total to dtot.
__global__ void __launch_bounds__(kSortThreads) k_sort_scan(uint32_t* __restrict__ hist,
                                                            uint32_t* __restrict__ dtot,
                                                            uint32_t nb) {
  uint32_t* row = hist + (size_t)blockIdx.x * nb;
  __shared__ uint32_t ws[4], tot;
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < nb; b0 += kSortThreads) {
    const uint32_t b = b0 + threadIdx.x;
    const uint32_t x = b < nb ? row[b] : 0u;
    const uint32_t ex = exscan256(x, ws);
    if (b < nb) row[b] = carry + ex;
    if (threadIdx.x == kSortThreads - 1) tot = ex + x;
    __syncthreads();
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

// Ranks of a wavefront's keys among its own of the same digit, in index
// order; counts the digits in wcnt (this wavefront's row, zero before).
template <int ITEMS>
__device__ __forceinline__ void rank_wave(const uint64_t (&key)[ITEMS], const bool (&valid)[ITEMS],
                                          int shift, uint32_t* wcnt, uint32_t (&rank)[ITEMS]) {
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t d = digit_of(key[r], shift);
    const uint64_t peers = digit_peers(d, valid[r]), below = peers & lt;
    uint32_t old = 0;
    if (valid[r]) old = wcnt[d];
    if (valid[r] && below == 0) wcnt[d] = old + (uint32_t)__popcll(peers);
    rank[r] = old + (uint32_t)__popcll(below);
  }
}

template <bool FUSED, int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_sort_scatter(
    const uint64_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
    uint64_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, uint32_t n,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ dtot, uint32_t nb, int shift) {
  __shared__ uint32_t wcnt[kSortWaves][kSortRadix];
  __shared__ uint32_t lstart[kSortRadix], gofs[kSortRadix], ws[4];
  constexpr int kTile = kSortThreads * ITEMS;
  __shared__ uint64_t sbuf[kTile];  // keys, then the values in their place
  const int w = threadIdx.x / kWave, lane = lane_id();
  const uint32_t d0 = threadIdx.x, base = blockIdx.x * (uint32_t)kTile;
#pragma unroll
  for (int k = 0; k < kSortWaves; ++k) wcnt[k][d0] = 0u;
  {
    uint32_t tot = 0, before = 0;
    if (FUSED) {
      for (uint32_t b = 0; b < nb; ++b) {
        const uint32_t h = hist[(size_t)d0 * nb + b];
        before += b < blockIdx.x ? h : 0u;
        tot += h;
      }
    } else {
      tot = dtot[d0];
      before = hist[(size_t)d0 * nb + blockIdx.x];
    }
    gofs[d0] = exscan256(tot, ws) + before;  // (its barriers also order the clear)
  }
  uint64_t key[ITEMS];
  bool valid[ITEMS];
  uint32_t rank[ITEMS];
  const uint32_t ibase = base + (uint32_t)w * (kWave * ITEMS) + (uint32_t)lane;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    valid[r] = ibase + r * kWave < n;
    key[r] = valid[r] ? keys_in[ibase + r * kWave] : 0ull;
  }
  rank_wave<ITEMS>(key, valid, shift, wcnt[w], rank);
  __syncthreads();
  {
    uint32_t run = 0;
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) {
      const uint32_t c = wcnt[k][d0];
      wcnt[k][d0] = run;
      run += c;
    }
    lstart[d0] = exscan256(run, ws);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t d = digit_of(key[r], shift);
    rank[r] += lstart[d] + wcnt[w][d];
    if (valid[r]) sbuf[rank[r]] = key[r];
  }
  uint32_t val[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) val[r] = valid[r] ? vals_in[ibase + r * kWave] : 0u;
  __syncthreads();
  const uint32_t nloc = min(n - base, (uint32_t)kTile);
  uint32_t opos[ITEMS];
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const uint32_t i = threadIdx.x + q * kSortThreads;
    opos[q] = 0u;
    if (i < nloc) {
      const uint64_t k = sbuf[i];
      const uint32_t d = digit_of(k, shift);
      opos[q] = gofs[d] + i - lstart[d];
      keys_out[opos[q]] = k;
    }
  }
  __syncthreads();
  uint32_t* svals = reinterpret_cast<uint32_t*>(sbuf);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (valid[r]) svals[rank[r]] = val[r];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const uint32_t i = threadIdx.x + q * kSortThreads;
    if (i < nloc) vals_out[opos[q]] = svals[i];
  }
}

// All passes of a small sort in one workgroup.
__global__ void __launch_bounds__(kBlockThreads) k_sort_block(uint64_t* __restrict__ keys,
                                                              uint32_t* __restrict__ vals, int n,
                                                              int key_bits) {
  constexpr int NW = kBlockThreads / kWave;
  __shared__ uint64_t sk[kBlockSort];
  __shared__ uint32_t sv[kBlockSort];
  __shared__ uint32_t wcnt[NW][kSortRadix];
  __shared__ uint32_t dstart[kSortRadix], ws[4];
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int ibase = w * (kWave * kBlockItems) + lane;
  uint64_t key[kBlockItems];
  uint32_t val[kBlockItems];
  bool valid[kBlockItems];
#pragma unroll
  for (int r = 0; r < kBlockItems; ++r) {
    const int i = ibase + r * kWave;
    valid[r] = i < n;
    key[r] = valid[r] ? keys[i] : 0ull;
    val[r] = valid[r] ? vals[i] : 0u;
  }
  for (int shift = 0; shift < key_bits; shift += kSortBits) {
    for (int k = threadIdx.x; k < NW * kSortRadix; k += kBlockThreads) (&wcnt[0][0])[k] = 0u;
    __syncthreads();
    uint32_t rank[kBlockItems];
    rank_wave<kBlockItems>(key, valid, shift, wcnt[w], rank);
    __syncthreads();
    uint32_t run = 0;
    if (threadIdx.x < kSortRadix) {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t c = wcnt[k][threadIdx.x];
        wcnt[k][threadIdx.x] = run;
        run += c;
      }
    }
    const uint32_t ex = exscan256(run, ws);
    if (threadIdx.x < kSortRadix) dstart[threadIdx.x] = ex;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kBlockItems; ++r)
      if (valid[r]) {
        const uint32_t d = digit_of(key[r], shift);
        const uint32_t at = dstart[d] + wcnt[w][d] + rank[r];
        sk[at] = key[r];
        sv[at] = val[r];
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kBlockItems; ++r)
      if (valid[r]) {
        key[r] = sk[ibase + r * kWave];
        val[r] = sv[ibase + r * kWave];
      }
  }
#pragma unroll
  for (int r = 0; r < kBlockItems; ++r)
    if (valid[r]) {
      keys[ibase + r * kWave] = key[r];
      vals[ibase + r * kWave] = val[r];
    }
}

template <int ITEMS>
void sort_pass(const uint64_t* kin, const uint32_t* vin, uint64_t* kout, uint32_t* vout, uint32_t n,
               uint32_t* hist, uint32_t* dtot, uint32_t nb, int shift, hipStream_t s) {
  const dim3 grid(nb), block(kSortThreads);
  hipLaunchKernelGGL(k_sort_hist<ITEMS>, grid, block, 0, s, kin, n, hist, nb, shift);
  if (nb <= kFusedBlocks) {
    hipLaunchKernelGGL((k_sort_scatter<true, ITEMS>), grid, block, 0, s, kin, vin, kout, vout, n,
                       hist, dtot, nb, shift);
  } else {
    hipLaunchKernelGGL(k_sort_scan, dim3(kSortRadix), block, 0, s, hist, dtot, nb);
    hipLaunchKernelGGL((k_sort_scatter<false, ITEMS>), grid, block, 0, s, kin, vin, kout, vout, n,
                       hist, dtot, nb, shift);
  }
}

}  // namespace

hipError_t launch_sort_pairs(uint64_t* keys, uint32_t* vals, int64_t n, int key_bits, void* tmp,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n <= kBlockSort) {
    hipLaunchKernelGGL(k_sort_block, dim3(1), dim3(kBlockThreads), 0, s, keys, vals, (int)n,
                       key_bits);
    return hipGetLastError();
  }
  const SortScratch L = sort_scratch(n);
  char* base = static_cast<char*>(tmp);
  uint64_t* kb[2] = {keys, reinterpret_cast<uint64_t*>(base + L.k1)};
  uint32_t* vb[2] = {vals, reinterpret_cast<uint32_t*>(base + L.v1)};
  uint32_t* hist = reinterpret_cast<uint32_t*>(base + L.hist);
  uint32_t* dtot = reinterpret_cast<uint32_t*>(base + L.dtot);
  const uint32_t nb = (uint32_t)sort_blocks(n);
  int cur = 0;
  for (int shift = 0; shift < key_bits; shift += kSortBits) {
    if (n <= kSortFew)
      sort_pass<kSortItemsFew>(kb[cur], vb[cur], kb[cur ^ 1], vb[cur ^ 1], (uint32_t)n, hist, dtot,
                               nb, shift, s);
    else
      sort_pass<kSortItemsMany>(kb[cur], vb[cur], kb[cur ^ 1], vb[cur ^ 1], (uint32_t)n, hist, dtot,
                                nb, shift, s);
    cur ^= 1;
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && cur == 1) {
    e = hipMemcpyAsync(keys, kb[1], (size_t)n * 8, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(vals, vb[1], (size_t)n * 4, hipMemcpyDeviceToDevice, s);
  }
  return e;
}

}  // namespace gs
