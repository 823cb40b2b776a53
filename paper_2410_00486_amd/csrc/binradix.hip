// a2, second form (GS_RADIX_BIN): tile binning by two stable radix sorts,
// with no per-tile atomics and no per-tile sorts.
//
// The lists must be ordered by (tile, depth, generation index) (Sec.
// III-C-1: per-tile lists in depth order).  A record meets a tile at most
// once, and its pairs carry consecutive generation indices that grow with
// the record index, so the order within a tile is also (depth, record
// index).  Hence:
//   1. the visible records are listed in record order with their depth
//      bits as keys (positive floats: the bits order like the values) and
//      a 16-byte generation payload each (tile box, first generation
//      index, record id);
//   2. a stable LSD radix sort orders their list positions by depth (ties
//      keep record order); its last pass writes the records' payloads in
//      that order, so the generation reads them in sequence;
//   3. their pairs are generated in that order (a scan of the pair counts
//      gives each record its first slot), key = global tile id, values =
//      generation index and record id;
//   4. a stable LSD radix sort by tile id (only the bits the plan's tile
//      count needs) then leaves every tile's pairs contiguous, in depth
//      order, at exactly the list starts the binning scan computed; its
//      last pass writes the sorted outputs (keys, values and record ids)
//      directly.
// Every pass is an upsweep (per-block digit counts), a per-digit scan over
// the blocks and a downsweep that ranks a block's keys (stable: wave64
// ballots, in index order), reorders them in LDS and writes each digit's
// run contiguously.  Counts are read on the device (flags), grids are sized
// for the plan's capacities; graph-capturable, no spin-waits.
#include "tilesort.h"
#include "wavescan.h"

namespace gs {
namespace {

constexpr int kRbThreads = 256;
constexpr int kRbItems = 12;
constexpr int kRbTile = kRbThreads * kRbItems;  // keys per block
constexpr int kRbWaves = kRbThreads / kWave;
constexpr int kRbMaxBits = 9;  // tile passes: 18 bits of tile id in two
constexpr int kRbMaxRadix = 1 << kRbMaxBits;
// depth-sorted records per group of the pair generation (4 per thread), and
// the pairs of a group that one workgroup writes
constexpr int kGenRecs = 1024;
constexpr int kGenPer = kGenRecs / kRbThreads;
constexpr uint32_t kGenPairs = 8192;
constexpr int kGenScanThreads = 1024;
constexpr int kRunsPer = 4;  // sorted keys per thread of the run search

static_assert(kRbMaxRadix == 2 * kRbThreads, "two digits per thread in the block scans");

// Number of keys a pass sorts: a flag of the workspace, zero after a pair
// overflow (then nothing is generated or written).
__device__ __forceinline__ int64_t rb_count(const int32_t* fl, int which) {
  return fl[F_OVERFLOW] ? 0 : (int64_t)fl[which];
}

// Lanes of the wavefront whose digit equals this lane's (among `valid`
// lanes), from one ballot per digit bit.
template <int BITS>
__device__ __forceinline__ uint64_t rb_peers(uint32_t d, bool valid) {
  uint64_t peers = ballot64(valid);
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bb = ballot64(bit);
    peers &= bit ? bb : ~bb;
  }
  return peers;
}

// Exclusive scan over the block's 256 threads of one value each; every
// thread of the block must call.  ws: kRbWaves words of LDS.
__device__ __forceinline__ uint32_t rb_block_exscan(uint32_t x, uint32_t* ws) {
  const int w = threadIdx.x / kWave, lane = lane_id();
  const uint32_t incl = scan_dpp<6>(x);
  if (lane == kWave - 1) ws[w] = incl;
  __syncthreads();
  uint32_t off = 0;
  for (int k = 0; k < w; ++k) off += ws[k];
  __syncthreads();  // ws is reused by the caller's next scan
  return off + incl - x;
}

// What the pair generation needs of a visible record, in one 16-byte word
// (one random read per record once the records are in depth order): its
// tile box (x0 | y0 << 16, x1 | y1 << 16), first generation index and
// record id.
__device__ __forceinline__ uint32_t pay_tiles(const uint4 p) {
  return ((p.y & 0xFFFFu) - (p.x & 0xFFFFu)) * ((p.y >> 16) - (p.x >> 16));
}

// 1. Visible records in record order: pair offset (first generation index),
// visible-list entry, depth key and generation payload.  One wavefront per
// chunk of 64 Gaussians of a view, at the positions the binning scan gave
// the chunk.  Bound by HBM: the depth and the box come from arrays of their
// own (a 64-byte record per visible Gaussian: 32M records, 6.1M of them
// visible, 173 us, now 101).
__global__ void __launch_bounds__(256) k_rb_visible(
    const uint32_t* __restrict__ tt, uint32_t* __restrict__ poff,
    const uint2* __restrict__ chunk_pre, int64_t chunks_per_view, int64_t n_chunks,
    const uint32_t* __restrict__ zbits, const uint2* __restrict__ rect, int64_t n,
    int32_t* __restrict__ fl, HeavyList heavy, uint32_t* __restrict__ vis_list,
    uint32_t* __restrict__ dkey, uint4* __restrict__ pay) {
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int64_t gw = (int64_t)blockIdx.x * (256 / kWave) + w;  // chunk
  if (gw >= n_chunks) return;
  const int v = (int)(gw / chunks_per_view);
  const int64_t gi = (gw - (int64_t)v * chunks_per_view) * kWave + lane;
  const int64_t ri = (int64_t)v * n + gi;
  const bool over = fl[F_OVERFLOW] != 0;
  const uint32_t c = (gi < n && !over) ? tt[ri] : 0u;
  uint32_t z = 0;
  uint2 b = make_uint2(0u, 0u);
  if (c > 0) {
    z = zbits[ri];
    b = rect[ri];
  }
  const uint32_t incl = scan_dpp<6>(c);
  const uint2 cp = chunk_pre[gw];
  const uint64_t vmask = ballot64(c > 0);
  if (c > 0) {
    const uint32_t p0 = cp.x + (incl - c);
    poff[ri] = p0;
    const uint32_t vp = cp.y + (uint32_t)__popcll(vmask & lanemask_lt());
    vis_list[vp] = (uint32_t)ri;
    note_heavy(heavy, fl, c, (uint32_t)ri);
    dkey[vp] = z;
    pay[vp] = make_uint4(b.x, b.y, p0, (uint32_t)ri);
  }
}

// Upsweep: per-block counts of the digit (key >> shift) & (2^bits - 1),
// stored digit-major: hist[d * nb_cap + block].  LDS atomics on a row per
// wavefront: ranking by ballots only to count, 25M pairs took 90 to 99 us,
// now 37 to 41 (1.5M keys 12 -> 5); conflicts cost most on the depth's top
// byte (few values: 8.5 us, 5 otherwise).  Neighbouring blocks on one XCD, as
// in the downsweep, so that their counts of a digit (one cache line) meet in
// one L2: 64 -> 40 us of that.
__global__ void __launch_bounds__(kRbThreads) k_rb_hist(const uint32_t* __restrict__ keys,
                                                        const int32_t* __restrict__ fl, int which,
                                                        uint32_t* __restrict__ hist,
                                                        int64_t nb_cap, int shift, int bits) {
  const int64_t cnt = rb_count(fl, which);
  const uint32_t blk = xcd_item(blockIdx.x, gridDim.x);
  const int64_t base = (int64_t)blk * kRbTile;
  if (base >= cnt) return;
  __shared__ uint32_t h[kRbWaves][kRbMaxRadix];
  const int w = threadIdx.x / kWave;
  for (int k = threadIdx.x; k < kRbWaves * kRbMaxRadix; k += kRbThreads) (&h[0][0])[k] = 0u;
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1u;
  uint32_t key[kRbItems];
#pragma unroll
  for (int r = 0; r < kRbItems; ++r) {
    const int64_t idx = base + r * kRbThreads + threadIdx.x;
    key[r] = idx < cnt ? keys[idx] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kRbItems; ++r)
    if (base + r * kRbThreads + threadIdx.x < cnt) atomicAdd(&h[w][(key[r] >> shift) & mask], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d <= (int)mask; d += kRbThreads) {
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kRbWaves; ++k) s += h[k][d];
    hist[(int64_t)d * nb_cap + blk] = s;
  }
}

// One block per digit: exclusive scan of the digit's counts over the active
// blocks (in place); the digit's total to dtot.
__global__ void __launch_bounds__(kRbThreads) k_rb_digit_scan(uint32_t* __restrict__ hist,
                                                              const int32_t* __restrict__ fl,
                                                              int which,
                                                              uint32_t* __restrict__ dtot,
                                                              int64_t nb_cap) {
  const int64_t cnt = rb_count(fl, which);
  const int64_t nb = (cnt + kRbTile - 1) / kRbTile;
  uint32_t* row = hist + (int64_t)blockIdx.x * nb_cap;
  // four counts per thread in flight (one at a time: 24 us for 8100 blocks,
  // now 11)
  constexpr int V = 4;
  const int w = threadIdx.x / kWave, lane = lane_id();
  __shared__ uint32_t ws[V][kRbWaves];
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += V * kRbThreads) {
    uint32_t x[V], incl[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const int64_t b = b0 + k * kRbThreads + threadIdx.x;
      x[k] = b < nb ? row[b] : 0u;
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      incl[k] = scan_dpp<6>(x[k]);
      if (lane == kWave - 1) ws[k][w] = incl[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const int64_t b = b0 + k * kRbThreads + threadIdx.x;
      uint32_t at = carry;
#pragma unroll
      for (int j = 0; j < kRbWaves; ++j) {
        at += j < w ? ws[k][j] : 0u;
        carry += ws[k][j];
      }
      if (b < nb) row[b] = at + incl[k] - x[k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

// Outputs of the last tile pass: the sorted lists.
struct RbEmit {
  uint64_t* keys;          // tile << 32 | depth bits
  uint32_t* vals;          // generation index
  uint32_t* sorted_rec;    // record id
  const uint32_t* zrec;    // depth bits by record id (gathered per pair)
  // the last depth pass instead (spay non-null): the generation payload of
  // each value's record in sorted order, no keys or values
  const uint4* pay;
  uint4* spay;
};

// Downsweep: stable ranking of the block's keys by digit, reorder in LDS,
// then each digit's run written contiguously at the digit's global offset
// (digit totals scanned over digits + the block's offset within the digit).
// A block's run of one digit is 24 to 48 bytes, part of a cache line whose
// rest the neighbouring blocks write, so 32 neighbours share an XCD: 25M pairs
// 332 -> 256 us and 297 -> 269 (emitting), the last depth pass of 6.1M
// records 140 -> 98.  Bound by those writes (12 to 16 bytes a pair; 600 to
// 700 MB in all, 120 us at the rate of a large copy).  Keys per block: 8 rows
// of 256 302 + 261 us, 12 259 + 271, 16 259 + 284, 20 249 + 317.
// EMIT: the last pass of the tile sort (keys are tile ids, values
// generation indices): writes the sorted lists instead of keys / values.
template <bool EMIT, bool TWO, int BITS>
__global__ void __launch_bounds__(kRbThreads) k_rb_scatter(
    const uint32_t* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
    const uint32_t* __restrict__ vals2_in, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, uint32_t* __restrict__ vals2_out, RbEmit E,
    const int32_t* __restrict__ fl, int which, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ dtot, int64_t nb_cap, int shift, int bits) {
  const int64_t cnt = rb_count(fl, which);
  const uint32_t blk = xcd_item(blockIdx.x, gridDim.x);
  const int64_t base = (int64_t)blk * kRbTile;
  if (base >= cnt) return;
  __shared__ uint32_t wcnt[kRbWaves][kRbMaxRadix];
  __shared__ uint32_t lstart[kRbMaxRadix];
  __shared__ uint32_t gofs[kRbMaxRadix];
  __shared__ uint32_t ws[kRbWaves];
  // one staging buffer, reused for the keys, the values and the second
  // values in turn (a third of the LDS of staging all three, so more
  // workgroups per CU hide the memory latency)
  __shared__ uint32_t sbuf[kRbTile];
  const int w = threadIdx.x / kWave, lane = lane_id();
  // the two consecutive digits this thread handles in the block scans
  const int d0 = 2 * (int)threadIdx.x, d1 = d0 + 1;
  const uint32_t mask = (1u << bits) - 1u;
  const bool h0 = d0 <= (int)mask, h1 = d1 <= (int)mask;
  for (int k = threadIdx.x; k < kRbWaves * kRbMaxRadix; k += kRbThreads) (&wcnt[0][0])[k] = 0u;
  {
    const uint32_t x0 = h0 ? dtot[d0] : 0u, x1 = h1 ? dtot[d1] : 0u;
    const uint32_t ex = rb_block_exscan(x0 + x1, ws);  // (its barrier also orders the clear)
    if (h0) gofs[d0] = ex + hist[(int64_t)d0 * nb_cap + blk];
    if (h1) gofs[d1] = ex + x0 + hist[(int64_t)d1 * nb_cap + blk];
  }
  // (the values are loaded only when they are staged: fewer registers held
  // through the ranking)
  uint32_t key[kRbItems], rank[kRbItems];
  const uint64_t lt = lanemask_lt();
  const int64_t ibase = base + (int64_t)w * (kWave * kRbItems) + lane;
#pragma unroll
  for (int r = 0; r < kRbItems; ++r) {
    const int64_t idx = ibase + r * kWave;
    const bool valid = idx < cnt;
    key[r] = valid ? keys_in[idx] : 0u;
    const uint32_t d = (key[r] >> shift) & mask;
    const uint64_t peers = rb_peers<BITS>(d, valid);
    const uint64_t below = peers & lt;
    uint32_t old = 0;
    if (valid) old = wcnt[w][d];
    if (valid && below == 0) wcnt[w][d] = old + (uint32_t)__popcll(peers);
    rank[r] = valid ? old + (uint32_t)__popcll(below) : 0xFFFFFFFFu;
  }
  __syncthreads();
  {
    // per digit: exclusive prefix over the waves, then the block-local
    // start of the digit's run
    uint32_t t0 = 0, t1 = 0;
#pragma unroll
    for (int k = 0; k < kRbWaves; ++k) {
      if (h0) {
        const uint32_t c = wcnt[k][d0];
        wcnt[k][d0] = t0;
        t0 += c;
      }
      if (h1) {
        const uint32_t c = wcnt[k][d1];
        wcnt[k][d1] = t1;
        t1 += c;
      }
    }
    const uint32_t ex = rb_block_exscan(t0 + t1, ws);
    if (h0) lstart[d0] = ex;
    if (h1) lstart[d1] = ex + t0;
  }
  __syncthreads();
  // each item's slot in the block's digit order (kRbTile: none)
#pragma unroll
  for (int r = 0; r < kRbItems; ++r) {
    if (rank[r] != 0xFFFFFFFFu) {
      const uint32_t d = (key[r] >> shift) & mask;
      rank[r] = lstart[d] + wcnt[w][d] + rank[r];
    } else {
      rank[r] = kRbTile;
    }
  }
  const int nloc = (int)((cnt - base) < kRbTile ? (cnt - base) : kRbTile);
  // keys: staged, then each slot's global position (kept for the values)
  // and the key itself (kept by the last pass for its output keys)
#pragma unroll
  for (int r = 0; r < kRbItems; ++r)
    if (rank[r] < (uint32_t)kRbTile) sbuf[rank[r]] = key[r];
  __syncthreads();
  uint32_t opos[kRbItems], okey[kRbItems];
#pragma unroll
  for (int q = 0; q < kRbItems; ++q) {
    const int i = threadIdx.x + q * kRbThreads;
    okey[q] = i < nloc ? sbuf[i] : 0u;
    const uint32_t d = (okey[q] >> shift) & mask;
    opos[q] = i < nloc ? gofs[d] + (uint32_t)i - lstart[d] : 0u;
    if (!EMIT && keys_out && i < nloc) keys_out[opos[q]] = okey[q];
  }
  __syncthreads();
  // values
  {
    uint32_t val[kRbItems];
#pragma unroll
    for (int r = 0; r < kRbItems; ++r)
      val[r] = rank[r] < (uint32_t)kRbTile
                   ? (vals_in ? vals_in[ibase + r * kWave] : (uint32_t)(ibase + r * kWave))
                   : 0u;
#pragma unroll
    for (int r = 0; r < kRbItems; ++r)
      if (rank[r] < (uint32_t)kRbTile) sbuf[rank[r]] = val[r];
  }
  __syncthreads();
  if (!EMIT && E.spay) {
    // the records' payloads in depth order: gathered four per thread in
    // flight, stored in place of the values
    constexpr int G = 4;
#pragma unroll
    for (int q0 = 0; q0 < kRbItems; q0 += G) {
      uint4 pv[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int i = threadIdx.x + (q0 + u) * kRbThreads;
        pv[u] = i < nloc ? E.pay[sbuf[i]] : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int i = threadIdx.x + (q0 + u) * kRbThreads;
        if (i < nloc) E.spay[opos[q0 + u]] = pv[u];
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < kRbItems; ++q) {
      const int i = threadIdx.x + q * kRbThreads;
      if (i < nloc) {
        if constexpr (EMIT) E.vals[opos[q]] = sbuf[i];
        else vals_out[opos[q]] = sbuf[i];
      }
    }
  }
  if constexpr (TWO) {
    {
      uint32_t val2[kRbItems];
#pragma unroll
      for (int r = 0; r < kRbItems; ++r)
        val2[r] = rank[r] < (uint32_t)kRbTile ? vals2_in[ibase + r * kWave] : 0u;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRbItems; ++r)
        if (rank[r] < (uint32_t)kRbTile) sbuf[rank[r]] = val2[r];
    }
    __syncthreads();
    if constexpr (!EMIT) {
#pragma unroll
      for (int q = 0; q < kRbItems; ++q) {
        const int i = threadIdx.x + q * kRbThreads;
        if (i < nloc) vals2_out[opos[q]] = sbuf[i];
      }
    } else {
      // the record ids came along as second values; each pair's key takes
      // the depth of its record (all of the thread's gathers in flight
      // before its stores)
      uint32_t rid[kRbItems], zb[kRbItems];
#pragma unroll
      for (int q = 0; q < kRbItems; ++q) {
        const int i = threadIdx.x + q * kRbThreads;
        rid[q] = i < nloc ? sbuf[i] : 0u;
        zb[q] = i < nloc ? E.zrec[rid[q]] : 0u;
      }
#pragma unroll
      for (int q = 0; q < kRbItems; ++q) {
        const int i = threadIdx.x + q * kRbThreads;
        if (i < nloc) {
          E.keys[opos[q]] = ((uint64_t)okey[q] << 32) | zb[q];
          E.sorted_rec[opos[q]] = rid[q];
        }
      }
    }
  } else {
    static_assert(TWO || !EMIT, "the last tile pass carries the record ids");
  }
}

// 3a. Pairs of each block of kGenRecs depth-sorted records.
__global__ void __launch_bounds__(kRbThreads) k_rb_gen_count(const uint4* __restrict__ spay,
                                                             const int32_t* __restrict__ fl,
                                                             uint32_t* __restrict__ part) {
  const int64_t V = rb_count(fl, F_VISIBLE);
  const int64_t base = (int64_t)blockIdx.x * kGenRecs;
  if (base >= V) return;
  __shared__ uint32_t ws[kRbWaves];
  uint32_t s = 0;
#pragma unroll
  for (int q = 0; q < kGenPer; ++q) {
    const int64_t j = base + q * kRbThreads + threadIdx.x;
    if (j < V) s += pay_tiles(spay[j]);
  }
  s = scan_dpp<6>(s);
  if (lane_id() == kWave - 1) ws[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
#pragma unroll
    for (int k = 0; k < kRbWaves; ++k) t += ws[k];
    part[blockIdx.x] = t;
  }
}

// 3b. One block: exclusive scan of the groups' pair counts (in place), and
// the work items of the generation: a group of p pairs is ceil(p / kGenPairs)
// items (group, first pair).  items[0].x holds their number, the items
// follow.  Near cameras the first groups in depth order hold splats over
// thousands of tiles each: one workgroup per group left the chip to the few
// heaviest (generation of 6.0M pairs of 8 close and overview views 470 us,
// with items 26 us; 25M pairs of 16 views 156 us, 82 us: 300 MB, 3.6 TB/s).
__global__ void __launch_bounds__(kGenScanThreads) k_rb_gen_scan(const int32_t* __restrict__ fl,
                                                                 uint32_t* __restrict__ part,
                                                                 uint2* __restrict__ items) {
  constexpr int NW = kGenScanThreads / kWave;
  const int64_t V = rb_count(fl, F_VISIBLE);
  const int64_t nb = (V + kGenRecs - 1) / kGenRecs;
  __shared__ uint64_t ws[NW];
  const int w = threadIdx.x / kWave, lane = lane_id();
  uint64_t carry = 0;  // items << 32 | pairs (each below 2^31)
  for (int64_t b0 = 0; b0 < nb; b0 += kGenScanThreads) {
    const int64_t b = b0 + threadIdx.x;
    const uint32_t p = b < nb ? part[b] : 0u;
    const uint64_t x = ((uint64_t)((p + kGenPairs - 1) / kGenPairs) << 32) | p;
    const uint64_t incl = scan_dpp<6>(x);
    if (lane == kWave - 1) ws[w] = incl;
    __syncthreads();
    uint64_t ex = carry + incl - x;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const uint64_t t = ws[k];
      if (k < w) ex += t;
      carry += t;
    }
    if (b < nb) {
      part[b] = (uint32_t)ex;
      uint2* dst = items + 1 + (ex >> 32);
      for (uint32_t k = 0; k < p; k += kGenPairs) *dst++ = make_uint2((uint32_t)b, k);
    }
    __syncthreads();  // ws is rewritten by the next round
  }
  if (threadIdx.x == 0) items[0] = make_uint2((uint32_t)(carry >> 32), 0u);
}

// 3c. Pair generation in depth order, one work item per workgroup: the
// group's records (4 consecutive per thread) get their first slots from a
// block scan plus the group's offset; the item's pairs are spread evenly
// over the threads, four consecutive 16-byte aligned output positions each
// (the first one's record by binary search of the slots in LDS, the others
// by walking on), so one large footprint does not serialise on one thread.
// Writes the tile key, the generation index and the record id of every pair.
__global__ void __launch_bounds__(kRbThreads) k_rb_generate(
    const uint4* __restrict__ spay, uint32_t n, ViewTable vt,
    const int32_t* __restrict__ fl, const uint32_t* __restrict__ part,
    const uint2* __restrict__ items, uint32_t* __restrict__ tkey, uint32_t* __restrict__ gidx,
    uint32_t* __restrict__ ridx) {
  if (blockIdx.x >= items[0].x) return;
  const uint2 item = items[1 + blockIdx.x];
  const int64_t V = rb_count(fl, F_VISIBLE);
  const int64_t base = (int64_t)item.x * kGenRecs;
  __shared__ uint32_t s_pre[kGenRecs + 1], s_p0[kGenRecs], s_t0[kGenRecs], s_rid[kGenRecs];
  __shared__ uint32_t s_bw[kGenRecs], s_tx[kGenRecs];
  __shared__ uint32_t ws[kRbWaves];
  uint32_t c[kGenPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kGenPer; ++q) {
    const int64_t j = base + (int64_t)threadIdx.x * kGenPer + q;
    const int l = threadIdx.x * kGenPer + q;
    c[q] = 0u;
    if (j < V) {
      const uint4 p = spay[j];
      const uint32_t r = p.w;
      const ViewInfo& vi = vt.v[r / n];
      c[q] = pay_tiles(p);
      s_rid[l] = r;
      s_p0[l] = p.z;
      s_bw[l] = (p.y & 0xFFFFu) - (p.x & 0xFFFFu);
      s_tx[l] = (uint32_t)vi.tiles_x;
      s_t0[l] = (uint32_t)(vi.tile_off + (int)(p.x >> 16) * vi.tiles_x + (int)(p.x & 0xFFFFu));
    }
    sum += c[q];
  }
  uint32_t run = rb_block_exscan(sum, ws);
#pragma unroll
  for (int q = 0; q < kGenPer; ++q) {
    // records past the end keep the group's total: never chosen below
    s_pre[threadIdx.x * kGenPer + q] = run;
    run += c[q];
  }
  if (threadIdx.x == kRbThreads - 1) s_pre[kGenRecs] = run;
  __syncthreads();
  const uint32_t total = s_pre[kGenRecs];
  const uint32_t q0 = part[item.x];
  const uint32_t g0 = q0 + item.y, g1 = q0 + min(total, item.y + kGenPairs);
  for (uint32_t g = g0 / 4 + threadIdx.x; 4 * g < g1; g += kRbThreads) {
    const uint32_t a = max(4 * g, g0), b = min(4 * g + 4, g1);
    const uint32_t q = a - q0;
    // owner: the last record whose first slot is <= q (every record here
    // has at least one pair, so the slots strictly increase)
    int lo = 0, hi = kGenRecs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_pre[mid] <= q) lo = mid; else hi = mid - 1;
    }
    uint32_t k = q - s_pre[lo], left = s_pre[lo + 1] - q, bw = s_bw[lo];
    uint32_t row = k / bw, col = k - row * bw;
    uint32_t t[4], gi[4], ri[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t at = 4 * g + (uint32_t)u;
      if (at >= a && at < b) {
        t[u] = s_t0[lo] + row * s_tx[lo] + col;
        gi[u] = s_p0[lo] + k;
        ri[u] = s_rid[lo];
        ++k;
        if (++col == bw) {
          col = 0u;
          ++row;
        }
        if (--left == 0u && at + 1 < b) {  // the next record begins
          ++lo;
          left = s_pre[lo + 1] - s_pre[lo];
          bw = s_bw[lo];
          k = row = col = 0u;
        }
      } else {
        t[u] = gi[u] = ri[u] = 0u;
      }
    }
    if (b - a == 4) {
      reinterpret_cast<uint4*>(tkey)[g] = make_uint4(t[0], t[1], t[2], t[3]);
      reinterpret_cast<uint4*>(gidx)[g] = make_uint4(gi[0], gi[1], gi[2], gi[3]);
      reinterpret_cast<uint4*>(ridx)[g] = make_uint4(ri[0], ri[1], ri[2], ri[3]);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t at = 4 * g + (uint32_t)u;
        if (at >= a && at < b) {
          tkey[at] = t[u];
          gidx[at] = gi[u];
          ridx[at] = ri[u];
        }
      }
    }
  }
}

// 5. Per-tile list bounds from the sorted keys (tile << 32 | depth): the
// first position of each tile's run to tstart, one past its last to cnt.
// Tiles without pairs keep cnt = 0 (the per-tile pass zeroed it).  A read of
// 8 bytes a pair: each key once (its neighbours come from the next lanes),
// four in flight; with three loads per key, 25M pairs took 81 us, now 37
// (5.3 TB/s).
__global__ void __launch_bounds__(kRbThreads) k_rb_runs(const uint64_t* __restrict__ keys,
                                                        const int32_t* __restrict__ fl,
                                                        uint32_t* __restrict__ tstart,
                                                        uint32_t* __restrict__ tend) {
  const int64_t P = rb_count(fl, F_PAIRS);
  const int64_t b0 = (int64_t)blockIdx.x * (kRbThreads * kRunsPer), q0 = b0 + threadIdx.x;
  if (b0 >= P) return;
  // (the first and last lane fetch the neighbour outside the wavefront)
  const uint32_t* tile = reinterpret_cast<const uint32_t*>(keys) + 1;
  constexpr uint32_t kNone = 0xFFFFFFFFu;  // (no tile id)
  const int lane = lane_id();
  uint32_t t[kRunsPer], side[kRunsPer];
#pragma unroll
  for (int k = 0; k < kRunsPer; ++k) {
    const int64_t q = q0 + k * kRbThreads, n = lane == 0 ? q - 1 : q + 1;
    t[k] = q < P ? tile[2 * q] : kNone;
    side[k] = (lane == 0 || lane == kWave - 1) && n >= 0 && n < P ? tile[2 * n] : kNone;
  }
#pragma unroll
  for (int k = 0; k < kRunsPer; ++k) {
    const int64_t q = q0 + k * kRbThreads;
    const uint32_t up = __shfl_up(t[k], 1, kWave), down = __shfl_down(t[k], 1, kWave);
    if (q < P) {
      if ((lane == 0 ? side[k] : up) != t[k]) tstart[t[k]] = (uint32_t)q;
      if ((lane == kWave - 1 ? side[k] : down) != t[k]) tend[t[k]] = (uint32_t)(q + 1);
    }
  }
}

}  // namespace

namespace {

struct RbBuffers {
  const int32_t* fl;
  uint32_t *tt, *poff, *vis, *dk[2], *rid[2], *tk[2], *gx[2], *rx[2], *hist, *dtot, *part;
  uint4 *pay, *spay;
  uint2* items;
  RbEmit emit;
};

RbBuffers rb_buffers(const Plan& P, void* ws) {
  RbBuffers B;
  B.fl = ws_at<int32_t>(ws, P.off_flags);
  B.tt = ws_at<uint32_t>(ws, P.off_tt);
  B.poff = ws_at<uint32_t>(ws, P.off_poff);
  B.vis = ws_at<uint32_t>(ws, P.off_vis_list);
  for (int k = 0; k < 2; ++k) {
    B.dk[k] = ws_at<uint32_t>(ws, P.off_rb_dkey[k]);
    B.rid[k] = ws_at<uint32_t>(ws, P.off_rb_rid[k]);
    B.tk[k] = ws_at<uint32_t>(ws, P.off_rb_tkey[k]);
    B.gx[k] = ws_at<uint32_t>(ws, P.off_rb_gidx[k]);
    B.rx[k] = ws_at<uint32_t>(ws, P.off_rb_ridx[k]);
  }
  B.hist = ws_at<uint32_t>(ws, P.off_rb_hist);
  B.dtot = ws_at<uint32_t>(ws, P.off_rb_dtot);
  B.part = ws_at<uint32_t>(ws, P.off_rb_part);
  B.pay = ws_at<uint4>(ws, P.off_rb_pay);
  B.spay = ws_at<uint4>(ws, P.off_rb_spay);
  B.items = ws_at<uint2>(ws, P.off_rb_items);
  B.emit = RbEmit{ws_at<uint64_t>(ws, P.off_keys), ws_at<uint32_t>(ws, P.off_vals),
                  ws_at<uint32_t>(ws, P.off_sorted_rec), ws_at<uint32_t>(ws, P.off_zbits),
                  nullptr, nullptr};
  return B;
}

// One stable pass over the keys counted by flag `which`; vin null: each
// key's value is its own position; vin2 / vout2: a second value array
// carried along (null: none); spay (no emit): write the payloads of the
// values' records in sorted order instead of keys and values.
void rb_pass(const RbBuffers& B, hipStream_t s, const uint32_t* kin, const uint32_t* vin,
             const uint32_t* vin2, uint32_t* kout, uint32_t* vout, uint32_t* vout2, bool emit,
             int which, int64_t nb_cap, int shift, int bits, uint4* spay = nullptr) {
  const dim3 grid((unsigned)nb_cap), block(kRbThreads);
  hipLaunchKernelGGL(k_rb_hist, grid, block, 0, s, kin, B.fl, which, B.hist, nb_cap, shift, bits);
  hipLaunchKernelGGL(k_rb_digit_scan, dim3(1u << bits), block, 0, s, B.hist, B.fl, which, B.dtot,
                     nb_cap);
#define GS_RB_SCATTER_N(E, T, N, OUT)                                                          \
  hipLaunchKernelGGL((k_rb_scatter<E, T, N>), grid, block, 0, s, kin, vin, vin2, kout, vout,  \
                     vout2, OUT, B.fl, which, B.hist, B.dtot, nb_cap, shift, bits)
#define GS_RB_SCATTER(E, T, OUT)             \
  if (bits > 8)                              \
    GS_RB_SCATTER_N(E, T, kRbMaxBits, OUT);  \
  else                                       \
    GS_RB_SCATTER_N(E, T, 8, OUT)
  if (emit) {  // (the lists' record ids come along as second values)
    GS_RB_SCATTER(true, true, B.emit);
  } else {
    if (vin2) {
      GS_RB_SCATTER(false, true, RbEmit{});
    } else {
      const RbEmit out{nullptr, nullptr, nullptr, nullptr, B.pay, spay};
      GS_RB_SCATTER(false, false, out);
    }
  }
#undef GS_RB_SCATTER
#undef GS_RB_SCATTER_N
}

}  // namespace

// Workspace blocks of the radix binning: (record blocks, pair blocks, gen
// blocks) for a plan's record and pair capacities.
int64_t rb_blocks(int64_t count) { return (count + kRbTile - 1) / kRbTile; }
int64_t rb_gen_blocks(int64_t records) { return (records + kGenRecs - 1) / kGenRecs; }
// Work items of the generation: each group's last item may be partial.
int64_t rb_gen_items(int64_t records, int64_t pairs) {
  return rb_gen_blocks(records) + pairs / kGenPairs;
}
int rb_max_radix() { return kRbMaxRadix; }

// Steps 1-3 of the radix binning (after the binning scan, which kept the
// per-tile counters): visible records, their depth sort, pair generation.
hipError_t launch_rb_generate(const Plan& P, void* ws, hipStream_t s) {
  const RbBuffers B = rb_buffers(P, ws);
  if (P.n_chunks <= 0 || P.rb_rec_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rb_visible, dim3((unsigned)((P.n_chunks + 3) / 4)), dim3(256), 0, s, B.tt,
                     B.poff, ws_at<uint2>(ws, P.off_chunk_pre), P.chunks_per_view, P.n_chunks,
                     ws_at<uint32_t>(ws, P.off_zbits), ws_at<uint2>(ws, P.off_rect), P.n,
                     ws_at<int32_t>(ws, P.off_flags), heavy_list(P, ws), B.vis,
                     B.dk[0], B.pay);
  // depth bits in four 8-bit passes; values: visible-list positions (the
  // first pass takes each key's own position); the last pass writes the
  // records' generation payloads in depth order instead
  // (dk0, -) -> (dk1, rid1) -> (dk0, rid0) -> (dk1, rid1) -> spay
  for (int p = 0; p < 4; ++p) {
    const uint32_t* kin = B.dk[p & 1];
    const uint32_t* vin = p == 0 ? nullptr : B.rid[p & 1];
    const bool last = p == 3;
    rb_pass(B, s, kin, vin, nullptr, last ? nullptr : B.dk[(p + 1) & 1],
            last ? nullptr : B.rid[(p + 1) & 1], nullptr, false, F_VISIBLE, P.rb_rec_blocks,
            8 * p, 8, last ? B.spay : nullptr);
  }
  const int64_t gb = rb_gen_blocks(P.n_rec);
  hipLaunchKernelGGL(k_rb_gen_count, dim3((unsigned)gb), dim3(kRbThreads), 0, s, B.spay, B.fl,
                     B.part);
  hipLaunchKernelGGL(k_rb_gen_scan, dim3(1), dim3(kGenScanThreads), 0, s, B.fl, B.part, B.items);
  hipLaunchKernelGGL(k_rb_generate, dim3((unsigned)rb_gen_items(P.n_rec, P.pair_cap)),
                     dim3(kRbThreads), 0, s, B.spay, (uint32_t)P.n, P.vt, B.fl, B.part, B.items,
                     B.tk[0], B.gx[0], B.rx[0]);
  return hipGetLastError();
}

// Step 4: the pairs by tile id, as many passes of at most 9 bits as the
// plan's tile bits need (equal widths); the last writes the sorted lists.
hipError_t launch_rb_tile_sort(const Plan& P, void* ws, hipStream_t s) {
  const RbBuffers B = rb_buffers(P, ws);
  if (P.rb_pair_blocks <= 0) return hipSuccess;
  const int tb = P.tile_bits;
  const int passes = (tb + kRbMaxBits - 1) / kRbMaxBits;
  const int width = (tb + passes - 1) / passes;
  int cur = 0;
  for (int p = 0; p < passes; ++p) {
    const int shift = p * width;
    const int bits = std::min(width, tb - shift);
    const bool last = p == passes - 1;
    rb_pass(B, s, B.tk[cur], B.gx[cur], B.rx[cur], last ? nullptr : B.tk[cur ^ 1],
            last ? nullptr : B.gx[cur ^ 1], last ? nullptr : B.rx[cur ^ 1], last, F_PAIRS,
            P.rb_pair_blocks, shift, bits);
    cur ^= 1;
  }
  return hipGetLastError();
}

// Step 5: list bounds per tile from the sorted keys (for the tile scan).
hipError_t launch_rb_runs(const Plan& P, void* ws, hipStream_t s) {
  if (P.rb_pair_blocks <= 0) return hipSuccess;
  constexpr int64_t per = kRbThreads * kRunsPer;
  const int64_t blocks = (P.rb_pair_blocks * kRbTile + per - 1) / per;
  hipLaunchKernelGGL(k_rb_runs, dim3((unsigned)blocks), dim3(kRbThreads), 0, s,
                     ws_at<uint64_t>(ws, P.off_keys), ws_at<int32_t>(ws, P.off_flags),
                     ws_at<uint32_t>(ws, P.off_tile_start), ws_at<uint32_t>(ws, P.off_tile_cnt));
  return hipGetLastError();
}

}  // namespace gs
