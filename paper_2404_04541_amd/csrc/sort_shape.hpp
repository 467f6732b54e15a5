// How the radix sort of n entries is cut (plain C++: the host's arithmetic, without HIP).
#pragma once
#include <cstddef>
#include <cstdint>

namespace spg {

constexpr int kSortThreads = 512;      // of a workgroup that counts
constexpr int kScatterThreads = 1024;  // of one that scatters
constexpr int kSortItems = 8;          // entries of a thread in a tile
constexpr int kSortFewItems = 2;       // ranges of so few a thread (sorts of at most 2^20 entries) take a variant that ranks no more: 200 003 entries 46 | 27 us
constexpr int kSortTile = kScatterThreads * kSortItems;
constexpr int kSortBins = 256;
constexpr int kSortMaxRanges = 1024;

// Passes over digits of `bits` bits; ranges of whole steps of kScatterThreads entries, each taken in equal tiles.
struct SortShape {
  int passes, bits, ranges, first_bit;   // (bits below first_bit are not sorted by)
  int64_t per_range;
};

// A compute unit holds two workgroups that scatter.  Up to a tile for every place on the chip the ranges share the entries evenly
// (small sorts too are spread over the chip: 200 003 entries 57 us for four passes as 25 whole tiles, 27 us as 196 ranges), beyond
// there are up to kSortMaxRanges of them.
constexpr int64_t kSortPlaces = 512;
inline SortShape sort_shape(int64_t n, int nbits, int first_bit = 0) {
  SortShape sh{};
  sh.first_bit = first_bit;
  if (nbits < 1) nbits = 1;
  sh.passes = (nbits + 7) / 8;
  sh.bits = (nbits + sh.passes - 1) / sh.passes;
  if (n < 1) n = 1;
  const int64_t most = n <= kSortPlaces * kSortTile ? kSortPlaces : kSortMaxRanges;
  const int64_t even = (n + most - 1) / most;
  sh.per_range = (even + kScatterThreads - 1) / kScatterThreads * kScatterThreads;
  sh.ranges = (int)((n + sh.per_range - 1) / sh.per_range);
  return sh;
}

// Sorts of many bits: passes over the upper ones only, as many as leave kBucketMean entries on average with the same ones, and such a bucket is then
// sorted by its lower bits at once (k_sort_buckets).  That is one pass in place of all over the lower bits: where it saves two at least.
constexpr int kBucketMean = 192;
constexpr int kBucketBits = 20;     // lower bits at most: with an entry's place (11 bits) they make a word that is not the largest
struct SortPlan {
  SortShape sh;
  int low;   // lower bits left to the buckets (0: the passes sort by all)
};
inline SortPlan sort_plan(int64_t n, int nbits, bool plain) {
  SortPlan p{sort_shape(n, nbits), 0};
  if (plain) return p;
  int top = 1;
  while (top < 24 && ((int64_t)kBucketMean << top) < n) ++top;
  if (top > 16 && ((int64_t)kBucketMean << 16) * 3 / 2 >= n) top = 16;   // (a third pass is not worth buckets of less than 288)
  if (top < nbits - kBucketBits) top = nbits - kBucketBits;
  if ((top + 7) / 8 + 2 > p.sh.passes || top > 24 || ((int64_t)1 << top) > n / 16 + 1024) return p;   // (a wave for every bucket, empty ones too)
  p.low = nbits - top;
  p.sh = sort_shape(n, top, p.low);
  return p;
}

// Counters of sorts of up to n entries: one per digit value and range, and the digits' totals.  The number of ranges does not
// grow with n throughout, so the room is for as many ranges as any smaller sort takes.
constexpr size_t sort_counter_bytes(int64_t n) {
  const int64_t steps = ((n > 0 ? n : 1) + kScatterThreads - 1) / kScatterThreads;
  return (size_t)((steps < kSortMaxRanges ? steps : kSortMaxRanges) + 1) * kSortBins * 4;
}

}  // namespace spg
