// Stable LSD radix sort of (uint64 key, uint32 value) pairs with caller
// scratch: the stand-alone sort and the pool's spatial order.
#pragma once

#include "gs_internal.h"

namespace gs {

constexpr int kSortThreads = 256;
// Keys per thread, few and many pairs: 4 and 8 take 58 and 67 us for 20 000
// pairs of 46 bits, 79 and 87 for 300 000, 124 and 115 for 2^20.
constexpr int kSortItemsFew = 4, kSortItemsMany = 8;
constexpr int64_t kSortFew = int64_t(1) << 19;
constexpr int kSortBits = 8;  // bits of a digit
constexpr int kSortRadix = 1 << kSortBits;

// Scratch of a sort of n pairs (bytes from a 256-byte aligned base): second
// key and value buffers, per-block digit counts, digit totals.  Nothing in
// it has to start at zero.
struct SortScratch {
  size_t k1, v1, hist, dtot, bytes;
};
constexpr size_t sort_align(size_t x) { return (x + 255) / 256 * 256; }
constexpr int64_t sort_blocks(int64_t n) {
  const int64_t tile = kSortThreads * (n <= kSortFew ? kSortItemsFew : kSortItemsMany);
  return n > tile ? (n + tile - 1) / tile : 1;
}
constexpr SortScratch sort_scratch(int64_t n) {
  SortScratch t{};
  t.k1 = 0;
  t.v1 = sort_align(t.k1 + (size_t)n * 8 + 8);
  t.hist = sort_align(t.v1 + (size_t)n * 4 + 4);
  // (never less than for fewer pairs)
  const int64_t few = n < kSortFew ? n : kSortFew;
  const int64_t blocks = sort_blocks(few) > sort_blocks(n) ? sort_blocks(few) : sort_blocks(n);
  t.dtot = sort_align(t.hist + (size_t)kSortRadix * blocks * 4);
  t.bytes = sort_align(t.dtot + kSortRadix * 4);
  return t;
}

// Sorts keys / vals [n] in place on the low key_bits bits (1..64), rounded up
// to whole digits.
hipError_t launch_sort_pairs(uint64_t* keys, uint32_t* vals, int64_t n, int key_bits, void* tmp,
                             hipStream_t s);

}  // namespace gs
