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
constexpr int kBucketGroup = 2048;  // entries of a bucket at most: one that has more makes the sort begin again, by passes alone
// So that this hardly ever happens, an entry of every kSampleStride is counted in its bucket beforehand, and where one of them is met kSampleCrowded
// times (an estimate of 1800 entries) the passes sort by all bits from the start.  A bucket of 3000 entries is met so often in 98 of 100 sorts, one
// of 2100 in 7 of 10; where keys are spread evenly (288 a bucket at most) one sort in 100 takes a bucket for crowded.
constexpr int64_t kSampleStride = 128;
constexpr unsigned kSampleCrowded = 14;
// Buckets only where they gain more than the sample costs where it finds them crowded: from a million entries of more than 32 bits on (passes of
// 64-bit keys).
// Unfolding, us passes alone | buckets with the sample, keys spread evenly and crowded (coordinates drawn as cubes): 33 bits, 1 M entries 220 | 175
// and 256 | 278, 3 M 275 | 218 and 297 | 322, 10 M 725 | 540 and 743 | 792 (sorted twice, without the sample: 1416), 20 M 1294 | 1089 and 1317 |
// 1390; but 29 bits, 200 000 entries 115 | 111 and 128 | 152, 3 M 186 | 173 and 217 | 255, 20 M 679 | 685.  Outer product of 32 M products 3300 |
// 2260, with a row of 80 000 of them 3300 | 3050 (sorted twice: 3800).
constexpr int64_t kBucketMinEntries = (1 << 20) + 1;
static_assert(kBucketMinEntries / 16 + 1025 <= kBucketMinEntries, "the sample's counts fit a buffer of keys");
inline bool buckets_pay(int64_t n, int nbits) { return n >= kBucketMinEntries && nbits > 32; }
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
