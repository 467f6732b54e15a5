// A sort of distinct words in LDS, shared by the hash workspace and the buckets of the radix sort.
#pragma once
#include "common.hpp"

namespace spg {

// Sorts the first n of GROUP * KPL distinct 32-bit words in LDS (by a wave or a workgroup): every wave 64 * KPL of them in
// registers, then each word goes to its position in its share plus the number of words below it in the other shares (bisected).
// A bitonic network of the whole table through LDS took 45 to 66 barriers: rows of 193 to 1536 entries of R-MAT scale 14 squared
// 160 us, here 98; of a 5003 x 3001 x 7777 product 108 and 72.  All threads call; ends with a barrier.
template <int GROUP, int KPL>
__device__ __forceinline__ void sort_shares(int* keys, int n) {
  constexpr int kShare = kWave * KPL, kShares = GROUP / kWave;
  const int wave = GROUP > kWave ? threadIdx.x >> 6 : 0, lane = lane_id();
  unsigned key[KPL];
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int t = wave * kShare + lane * KPL + i;
    key[i] = t < n ? (unsigned)keys[t] : ~0u;
  }
  lane_sort<kShare, KPL>(key, lane);
#pragma unroll
  for (int i = 0; i < KPL; ++i) keys[wave * kShare + lane * KPL + i] = (int)key[i];
  group_sync<GROUP>();
  int rank[KPL];
#pragma unroll
  for (int i = 0; i < KPL; ++i) rank[i] = lane * KPL + i;
  for (int w = 1; w < kShares; ++w) {
    const int* other = keys + ((wave + w) & (kShares - 1)) * kShare;
    int lo[KPL] = {};
#pragma unroll
    for (int step = kShare / 2; step > 0; step >>= 1) {   // the bisections of a thread advance together
#pragma unroll
      for (int i = 0; i < KPL; ++i) lo[i] += (unsigned)other[lo[i] + step - 1] < key[i] ? step : 0;
    }
#pragma unroll
    for (int i = 0; i < KPL; ++i) rank[i] += lo[i] + ((unsigned)other[lo[i]] < key[i] ? 1 : 0);
  }
  group_sync<GROUP>();
#pragma unroll
  for (int i = 0; i < KPL; ++i)
    if (key[i] != ~0u) keys[rank[i]] = (int)key[i];
  group_sync<GROUP>();
}

}  // namespace spg
