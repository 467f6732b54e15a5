// How the radix sort of n entries is cut (plain C++: the host's arithmetic, without HIP).
#pragma once
#include <cstddef>
#include <cstdint>

namespace spg {

constexpr int kSortThreads = 512;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kSortBins = 256;
constexpr int kSortMaxRanges = 1024;

// Passes over digits of `bits` bits, ranges of whole tiles.
struct SortShape {
  int passes, bits, ranges, first_bit;   // (bits below first_bit are not sorted by)
  int64_t per_range;
};

inline SortShape sort_shape(int64_t n, int nbits, int first_bit = 0) {
  SortShape sh{};
  sh.first_bit = first_bit;
  if (nbits < 1) nbits = 1;
  sh.passes = (nbits + 7) / 8;
  sh.bits = (nbits + sh.passes - 1) / sh.passes;
  const int64_t tiles = ((n > 0 ? n : 1) + kSortTile - 1) / kSortTile;
  const int64_t tiles_per = (tiles + kSortMaxRanges - 1) / kSortMaxRanges;
  sh.ranges = (int)((tiles + tiles_per - 1) / tiles_per);
  sh.per_range = tiles_per * kSortTile;
  return sh;
}

// Counters of sorts of up to n entries: one per digit value and range, and the digits' totals.  The number of ranges does not
// grow with n throughout (1024 tiles make 1024 ranges, 1025 make 513), so the room is for as many ranges as any smaller sort takes.
inline size_t sort_counter_bytes(int64_t n) {
  const int64_t tiles = ((n > 0 ? n : 1) + kSortTile - 1) / kSortTile;
  return (size_t)((tiles < kSortMaxRanges ? tiles : kSortMaxRanges) + 1) * kSortBins * 4;
}

}  // namespace spg
