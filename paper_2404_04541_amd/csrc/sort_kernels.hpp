// Stable least-significant-digit radix sort of (key, payload) pairs and exclusive scans, used by the
// tensor unfolding, the doubly compressed formats and the outer-product workspace.
//
// One pass over a digit of at most 8 bits:
//   k_sort_hist     entries per digit of every range of consecutive entries (at most kSortMaxRanges ranges)
//   k_sort_scan     exclusive scan over the ranges, one workgroup per digit
//   (the last bits of long keys: k_sort_buckets)
//   k_sort_scatter  a workgroup walks its range tile by tile: ranks its entries (ballots inside a wave,
//                   counters per wave in LDS), puts the tile into digit order in LDS and writes every
//                   digit's entries as one run
// Bound: memory.  A pass moves key + payload once in and once out and the keys once more for the counts.
// Carrying the payload (the value itself) costs at most 8 bytes an entry and pass and saves the gather
// through a permutation at the end, which costs a 128-byte line per entry.  Tiles of 8192 entries keep the
// runs of a digit at 32 entries (256 bytes of keys) on average; a wave that scattered its own 64 entries
// without the exchange in LDS wrote 4-byte pieces to as many lines.
// 10^7 tensor entries of 33 key bits and double values, kernel time per pass over a digit: scatter 92 us (3.5 TB/s of key and value
// moved), counts 18 us, scan of the counters 5 us; unfolding as a whole 0.7 ms.  16.8 M components of 36 bits: scatter 140 us (3.8 TB/s).
// Two workgroups of 16 waves, 64 registers each, hold a compute unit's LDS; with 8 waves of 16 entries a lane each it was 105 and
// 163 us.  Payloads are loaded when the keys have left their registers, so that little spills: the figures above are with 32 bytes a lane (keys of 64
// bits, of which nine registers go to memory), with 60 bytes a pass takes 118 us; keys of 32 bits spill two registers or none.
#pragma once
#include "common.hpp"
#include "sort_shape.hpp"
#include "share_sort.hpp"

namespace spg {

constexpr int kSortWaves = kScatterThreads / kWave;

// Adds the digit counts of this workgroup's LDS histogram copies up and writes them for range r of nr.
constexpr int kHistCopies = 4;
__device__ __forceinline__ void sort_hist_out(const unsigned (*cnt)[kSortBins], int nbins, int r, int nr, unsigned* __restrict__ hist) {
  __syncthreads();
  for (int d = threadIdx.x; d < nbins; d += kSortThreads) {
    unsigned s = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) s += cnt[c][d];
    hist[(int64_t)d * nr + r] = s;
  }
}

// hist[digit * gridDim.x + range] = entries of the range whose digit (bits [shift, shift + bits) of the key) is `digit`
template <typename K>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(int64_t n, int64_t per_range, int shift, int bits, const K* __restrict__ keys,
                                                            unsigned* __restrict__ hist) {
  __shared__ unsigned cnt[kHistCopies][kSortBins];
  for (int d = threadIdx.x; d < kHistCopies * kSortBins; d += kSortThreads) (&cnt[0][0])[d] = 0;
  __syncthreads();
  const unsigned mask = (1u << bits) - 1;
  const int64_t lo = (int64_t)blockIdx.x * per_range, hi = lo + per_range < n ? lo + per_range : n;
  unsigned* mine = cnt[threadIdx.x & (kHistCopies - 1)];
  for (int64_t p = lo + threadIdx.x; p < hi; p += kSortThreads * 4) {
    K k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = p + u * kSortThreads < hi ? keys[p + u * kSortThreads] : K(0);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p + u * kSortThreads < hi) atomicAdd(&mine[(unsigned)(k[u] >> shift) & mask], 1u);
  }
  sort_hist_out(cnt, 1 << bits, blockIdx.x, gridDim.x, hist);
}

// Workgroup d: exclusive scan of hist[d * nr .. (d + 1) * nr) in place, total of the digit to totals[d].
__global__ __launch_bounds__(256) void k_sort_scan(int nr, unsigned* __restrict__ hist, unsigned* __restrict__ totals) {
  constexpr int kPer = kSortMaxRanges / 256;
  __shared__ unsigned ws[4];
  unsigned* h = hist + (int64_t)blockIdx.x * nr;
  const int base = threadIdx.x * kPer;
  unsigned v[kPer], s = 0;
#pragma unroll
  for (int t = 0; t < kPer; ++t) { v[t] = base + t < nr ? h[base + t] : 0u; s += v[t]; }
  const unsigned incl = (unsigned)wave_incl_scan((int)s);
  if (lane_id() == kWave - 1) ws[threadIdx.x >> 6] = incl;
  __syncthreads();
  unsigned run = incl - s;
  for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) run += ws[w];
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    if (base + t < nr) h[base + t] = run;
    run += v[t];
  }
  if (threadIdx.x == 255) totals[blockIdx.x] = run;
}

// Exclusive scan of one value per thread over the first 256 threads of the workgroup; all threads call.
__device__ __forceinline__ unsigned scan_bins(unsigned v, unsigned* ws) {
  const unsigned incl = (unsigned)wave_incl_scan((int)v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane_id() == kWave - 1 && wave < kSortBins / kWave) ws[wave] = incl;
  __syncthreads();
  unsigned before = 0;
#pragma unroll
  for (int w = 0; w < kSortBins / kWave; ++w) before += w < wave ? ws[w] : 0u;
  return before + incl - v;
}

// One pass.  P: payload.  col_out (optional): the low bits of the key (key & col_mask), written with the last pass.
template <typename K, typename P, int ITEMS>
__global__ __launch_bounds__(kScatterThreads, 8) void k_sort_scatter(int64_t n, int64_t per_range, int shift, int bits, const K* __restrict__ keys,
                                                                  const P* __restrict__ pay, const unsigned* __restrict__ hist,
                                                                  const unsigned* __restrict__ totals, K* __restrict__ keys_out,
                                                                  P* __restrict__ pay_out, int32_t* __restrict__ col_out, K col_mask) {
  constexpr int kTile = kScatterThreads * ITEMS;
  constexpr size_t kSlot = sizeof(K) > sizeof(P) ? sizeof(K) : sizeof(P);
  __shared__ __align__(16) unsigned char s_tile[kTile * kSlot];   // the tile in digit order: keys, then payloads
  __shared__ __align__(16) unsigned short s_cnt[kSortWaves][kSortBins];   // entries of a digit in every wave, then their prefix over the waves
  __shared__ unsigned s_to[kSortBins];                // global position of a digit's run minus its position in the tile
  __shared__ unsigned short s_at[kSortBins];          // position of a digit's run in the tile
  __shared__ unsigned ws[kSortBins / kWave];
  static_assert(kTile <= 65535, "a position in the tile fits two bytes");
  K* s_key = reinterpret_cast<K*>(s_tile);
  P* s_pay = reinterpret_cast<P*>(s_tile);
  const int tid = threadIdx.x;
  const int nbins = 1 << bits;
  const unsigned mask = (unsigned)nbins - 1;
  unsigned at_global = 0;   // (thread d < nbins) where the next entry of digit d goes
  {
    const unsigned mine = tid < nbins ? totals[tid] : 0u;
    const unsigned before = scan_bins(mine, ws);
    if (tid < nbins) at_global = before + hist[(int64_t)tid * gridDim.x + blockIdx.x];
  }
  const int64_t lo = (int64_t)blockIdx.x * per_range, hi = lo + per_range < n ? lo + per_range : n;
  // tiles of equal size, whole steps of a thread's entry each
  const int tiles = (int)((per_range + kTile - 1) / kTile);
  const int per_tile = (int)((per_range / kScatterThreads + tiles - 1) / tiles) * kScatterThreads;
  for (int64_t t0 = lo; t0 < hi; t0 += per_tile) {
    int tl = tid;
    asm volatile("" : "+v"(tl));   // (no code: keeps what follows from the thread's number from being computed before the loop and held in registers)
    const int lane = tl & (kWave - 1), wave = tl >> 6;
    const int count = (int)(hi - t0 < per_tile ? hi - t0 : per_tile);
    const int items = (count + kScatterThreads - 1) / kScatterThreads;
    // a wave owns items * 64 consecutive entries, 64 at a time
    const int first = wave * (items * kWave) + lane, mine = items * kWave < count - first + lane ? items * kWave : count - first + lane;
    K key[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      key[i] = i * kWave + lane < mine ? (keys + t0 + first)[i * kWave] : K(~K(0));   // (behind the end: the last digit, behind every real entry)
    }
    for (int d = tid; d < kSortWaves * kSortBins / 2; d += kScatterThreads) reinterpret_cast<unsigned*>(&s_cnt[0][0])[d] = 0;
    __syncthreads();
    int pos[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {   // (items that the tile does not have are ranked too, but leave no trace: a branch around them makes the registers spill)
      const unsigned d = (unsigned)(key[i] >> shift) & mask;
      unsigned long long peers = ~0ULL;
#pragma unroll
      for (int b = 0; b < 8; ++b) {   // (all eight: a bit that no digit has excludes nobody, and a branch for every bit costs more)
        const unsigned long long m = __ballot((d >> b) & 1u);
        peers &= ((d >> b) & 1u) ? m : ~m;
      }
      const unsigned before = s_cnt[wave][d];
      const int below = lanes_below(peers);
      pos[i] = (int)before + below;
      wave_sync_lds();
      if (below == 0 && i < items) s_cnt[wave][d] = (unsigned short)(before + (unsigned)__popcll(peers));
      wave_sync_lds();
    }
    __syncthreads();
    unsigned total = 0;
    if (tid < nbins) {
#pragma unroll
      for (int w0 = 0; w0 < kSortWaves; w0 += 4) {
        unsigned c[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) c[w] = s_cnt[w0 + w][tl];
#pragma unroll
        for (int w = 0; w < 4; ++w) { s_cnt[w0 + w][tl] = (unsigned short)total; total += c[w]; }
      }
    }
    const unsigned at = scan_bins(total, ws);
    if (tid < nbins) {
      s_at[tid] = (unsigned short)at;
      s_to[tid] = at_global - at;
      at_global += total;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const unsigned d = (unsigned)(key[i] >> shift) & mask;
      pos[i] += s_at[d] + s_cnt[wave][d];
      if (i < items) s_key[pos[i]] = key[i];
    }
    P val[ITEMS];   // (the keys have left their registers: 64 of them allow two workgroups on a compute unit)
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      val[i] = i * kWave + lane < mine ? (pay + t0 + first)[i * kWave] : P(0);
    }
    __syncthreads();
    unsigned to[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int e = i * kScatterThreads + tl;
      const K k = s_key[e];   // (behind the tile's entries: anything)
      to[i] = s_to[(unsigned)(k >> shift) & mask] + (unsigned)e;
      if (e < count) {
        keys_out[to[i]] = k;
        if (col_out) col_out[to[i]] = (int32_t)(k & col_mask);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (i < items) s_pay[pos[i]] = val[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int e = i * kScatterThreads + tl;
      if (e < count) pay_out[to[i]] = s_pay[e];
    }
    __syncthreads();
  }
}

// The first r of [0, n] whose before(r) is false (before holds up to some r and not from there on), by a wave: 64 probes a round.
template <class F>
__device__ __forceinline__ int64_t wave_first_not(int64_t n, F before) {
  int64_t lo = 0, hi = n;   // the answer is in [lo, hi]
  while (lo < hi) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t at = lo + (lane_id() + 1) * step - 1;   // (every lane's stretch ends with its probe)
    const int held = __popcll(__ballot(at < hi && before(at)));
    lo += held * step;
    if (lo > hi) lo = hi;
    hi = lo + step - 1 < hi ? lo + step - 1 : hi;
  }
  return lo;
}

// Keys that the passes have sorted by their upper bits (key >> low) are sorted by all, with their payloads: a wave takes a bucket of at most
// kBucketWave entries with the same upper bits, the workgroup one of at most kBucketGroup.  An entry's lower bits and its place in the bucket make
// one word, so that a sort of distinct words (registers, lane_sort; sort_shares) is a stable one of the entries; the words then say
// where payloads come from.  *too_long is set where a bucket has more entries, and its entries are left out: the caller sorts again by passes alone.
// Bound: the loads that find a bucket (three to five that wait for each other), then the network and memory.  16.8 M components of 36 bits: three
// passes of 188 us each with their counts | one of these kernels 135 to 150 us (166 to 210 with a search of all keys, 64 probes a round, for either
// end); 10^7 tensor entries of 33 bits 345 | 118 us.
constexpr int kBucketWave = 512;
static_assert(kBucketWave * 4 == kBucketGroup, "the waves' buckets and the workgroup's share LDS");
template <typename P>
struct BucketLds {
  P pay[kBucketGroup];
  int words[kBucketGroup];
  int64_t begin[5];
};

template <typename K, typename P>
__global__ __launch_bounds__(256) void k_sort_buckets(int64_t n, int64_t buckets, int low, const K* __restrict__ keys, const P* __restrict__ pay,
    K* __restrict__ keys_out, P* __restrict__ pay_out, int32_t* __restrict__ col_out, K col_mask, int* __restrict__ too_long) {
  __shared__ BucketLds<P> lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  const int64_t b0 = (int64_t)blockIdx.x * 4;
  {
    // Where the wave's bucket begins and where it ends: half of the lanes look for either, 32 probes a round.  First around the place where it is if
    // the keys are spread evenly up to the largest (a round of loads less, mostly two), otherwise everywhere.
    const int64_t b = b0 + wave + (lane >> 5);
    const int probe = lane & 31;
    auto before = [&](int64_t p) { return (int64_t)(keys[p] >> low) < b; };
    auto held_of = [&](bool held) { const unsigned long long m = __ballot(held); return __popc((unsigned)(lane < 32 ? m : m >> 32)); };
    constexpr int64_t kNear = 256;
    const int64_t guess = (int64_t)((double)b * ((double)n / ((double)(int64_t)(keys[n - 1] >> low) + 1.0))) + (probe - 16) * kNear;
    const int64_t near = guess < 0 ? 0 : (guess < n ? guess : n - 1);
    const int held = held_of(before(near));
    const int src = (lane & 32) + (held > 0 ? held - 1 : 0), dst = (lane & 32) + (held < 32 ? held : 31);
    // the first position that is not before is in [lo, hi]
    int64_t lo = __shfl((long long)near, src, kWave) + 1, hi = __shfl((long long)near, dst, kWave);
    if (held == 0) lo = 0;
    if (held == 32) hi = n;
    if (lo > hi) lo = hi;
    while (__any(lo < hi)) {
      const int64_t step = (hi - lo + 31) / 32;
      const int64_t at = lo + (probe + 1) * step - 1;   // (every lane's stretch ends with its probe)
      const int64_t n_held = held_of(lo < hi && at < hi && before(at));
      if (lo < hi) {
        lo += n_held * step;
        if (lo > hi) lo = hi;
        hi = lo + step - 1 < hi ? lo + step - 1 : hi;
      }
    }
    if ((lane & 31) == 0 && (lane == 0 || wave == 3)) lds.begin[wave + (lane >> 5)] = lo;
  }
  __syncthreads();
  const K low_mask = (K)(((K)1 << low) - 1);
  // entry `at` of bucket b goes where its word stands
  auto put = [&](int64_t b, int64_t to, unsigned word, int place_bits, P v) {
    const K k = ((K)b << low) | (K)(word >> place_bits);
    keys_out[to] = k;
    pay_out[to] = v;
    if (col_out) col_out[to] = (int32_t)(k & col_mask);
  };
  {
    const int64_t from = lds.begin[wave];
    const int count = lds.begin[wave + 1] - from <= kBucketWave ? (int)(lds.begin[wave + 1] - from) : 0;
    P* w_pay = lds.pay + wave * kBucketWave;
    int* w_words = lds.words + wave * kBucketWave;
    constexpr int kPlaceBits = 9;
    auto sort = [&](auto per_lane) {
      constexpr int kPer = decltype(per_lane)::value;
      unsigned word[kPer];
      P v[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int t = q * kWave + lane;
        const bool on = t < count;
        const K k = on ? keys[from + t] : K(0);
        v[q] = on ? pay[from + t] : P(0);
        word[q] = on ? ((unsigned)(k & low_mask) << kPlaceBits) | (unsigned)t : ~0u;
      }
#pragma unroll
      for (int q = 0; q < kPer; ++q) w_pay[q * kWave + lane] = v[q];
      lane_sort<kPer * kWave, kPer>(word, lane);
#pragma unroll
      for (int q = 0; q < kPer; ++q) w_words[lane * kPer + q] = (int)word[q];
      wave_sync_lds();
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int t = q * kWave + lane;
        if (t < count) {
          const unsigned w = (unsigned)w_words[t];
          put(b0 + wave, from + t, w, kPlaceBits, w_pay[w & (kBucketWave - 1)]);
        }
      }
    };
    if (count > 4 * kWave) sort(std::integral_constant<int, 8>{});
    else if (count > 2 * kWave) sort(std::integral_constant<int, 4>{});
    else if (count > 0) sort(std::integral_constant<int, 2>{});
  }
  for (int w = 0; w < 4; ++w) {
    const int64_t from = lds.begin[w], count = lds.begin[w + 1] - from;   // (the same for the workgroup)
    if (count <= kBucketWave) continue;
    if (count > kBucketGroup) {
      if (threadIdx.x == 0) __hip_atomic_store(too_long, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      continue;
    }
    constexpr int kPlaceBits = 11;
    static_assert(kBucketBits + kPlaceBits < 32 && kBucketGroup == 1 << kPlaceBits, "lower bits and place make a word");
    __syncthreads();   // (the waves' buckets, or the long one before, have left LDS)
    for (int t = threadIdx.x; t < kBucketGroup; t += 256) {
      const bool on = t < (int)count;
      lds.words[t] = on ? (int)(((unsigned)(keys[from + t] & low_mask) << kPlaceBits) | (unsigned)t) : -1;
      if (on) lds.pay[t] = pay[from + t];
    }
    __syncthreads();
    sort_shares<256, kBucketGroup / 256>(lds.words, (int)count);
    for (int t = threadIdx.x; t < (int)count; t += 256) {
      const unsigned word = (unsigned)lds.words[t];
      put(b0 + w, from + t, word, kPlaceBits, lds.pay[word & (kBucketGroup - 1)]);
    }
  }
}

// Counts a sample of the keys (key_at(p): the key of entry p) by their upper bits in counts[buckets + 1], which are cleared; *crowded (in host
// memory, cleared) is set where one is met kSampleCrowded times (once: what goes to the host is slow; the last of the counts says that it is on its
// way).  Of every kSampleStride consecutive entries one at a changing place: one in order, or with a period, is seen as it is.  A workgroup's
// entries are counted in LDS first: atomics on one counter in memory take 12 ns each.
// Bound by its chain of loads, LDS and atomics: 10^7 tensor entries 14 us, 27 where they crowd (one of 64 entries 24 and 47), 16 M products of an
// outer product 29.
constexpr int kSampleThreads = 256;
constexpr int kSamplePer = 2;
__global__ __launch_bounds__(kSampleThreads) void k_sample_clear(unsigned buckets, unsigned* __restrict__ counts) {
  const unsigned b = blockIdx.x * kSampleThreads + threadIdx.x;
  if (b <= buckets) counts[b] = 0;
}
template <class KeyAt>
__global__ __launch_bounds__(kSampleThreads) void k_sort_sample(int64_t n, const KeyAt key_at, int low, unsigned buckets,
    unsigned* __restrict__ counts, int* __restrict__ crowded) {
  constexpr unsigned kSlots = 2 * kSampleThreads * kSamplePer, kFree = ~0u;
  __shared__ unsigned bucket[kSlots], met[kSlots];
  for (unsigned t = threadIdx.x; t < kSlots; t += kSampleThreads) { bucket[t] = kFree; met[t] = 0; }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {
    const int64_t t = ((int64_t)blockIdx.x * kSamplePer + u) * kSampleThreads + threadIdx.x;
    const int64_t p = t * kSampleStride + ((unsigned)t * 2654435761u >> 25);
    if (p >= n) continue;
    const unsigned long long b = (unsigned long long)key_at(p) >> low;
    if (b >= buckets) continue;   // (a coordinate out of range)
    unsigned slot = ((unsigned)b * 2654435761u >> 16) & (kSlots - 1);
    while (true) {   // (half of the slots stay free)
      const unsigned old = atomicCAS(&bucket[slot], kFree, (unsigned)b);
      if (old == kFree || old == (unsigned)b) break;
      slot = (slot + 1) & (kSlots - 1);
    }
    atomicAdd(&met[slot], 1u);
  }
  __syncthreads();
  bool seen = false;
  for (unsigned t = threadIdx.x; t < kSlots; t += kSampleThreads) {
    const unsigned c = met[t];
    if (c) seen = seen || atomicAdd(&counts[bucket[t]], c) + c >= kSampleCrowded;
  }
  if (__syncthreads_or(seen) && threadIdx.x == 0 && atomicAdd(&counts[buckets], 1u) == 0)
    __hip_atomic_store(crowded, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ptr[r] = first position of the sorted keys whose high part (key >> shift) is r or more (r = 0 .. rows).  A workgroup takes
// kPtrRows consecutive values and finds the stretch of keys they fall into.  A stretch of at most kPtrKeys keys is read once, in
// order: where the high part changes its position goes to LDS, and values that no key has take the next one's from a scan.  Behind
// a longer stretch (some rows of very many entries) every value is bisected.
// Bound: reading the keys.  A bisection for every value (13 dependent loads and more) | now: 10^7 keys of 4.2 M rows 85 | 42 us,
// 200 003 keys of 700 891 rows 24.6 | 7.1 us, 32 M keys of 10^6 rows and 8 M keys of as many columns together 169 | 115 us.  The line at
// 64 keys a row: there a stretch is 32 rounds of loads that do not wait for each other, as many as four bisections have that do.
constexpr int kPtrRows = 1024;
constexpr int kPtrKeys = 64 * kPtrRows;
template <typename K>
__global__ __launch_bounds__(256) void k_key_ptr(int64_t n, int64_t rows, int shift, const K* __restrict__ keys, int64_t* __restrict__ ptr) {
  constexpr int kPer = kPtrRows / 256;
  __shared__ int64_t bound[2];
  __shared__ __align__(16) int s_at[kPtrRows];   // position in the stretch of a value's first key
  __shared__ int s_min[4];
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t r0 = (int64_t)blockIdx.x * kPtrRows;
  if (wave < 2) {
    const int64_t r = r0 + wave * (int64_t)kPtrRows;
    const int64_t at = wave_first_not(n, [&](int64_t p) { return (int64_t)(keys[p] >> shift) < r; });
    if (lane == 0) bound[wave] = at;
  }
#pragma unroll
  for (int t = 0; t < kPer; ++t) s_at[t * 256 + threadIdx.x] = kPtrKeys;
  __syncthreads();
  const int64_t lo = bound[0], hi = bound[1];
  if (hi - lo > kPtrKeys) {
    for (int64_t r = r0 + threadIdx.x; r < r0 + kPtrRows && r <= rows; r += 256) {
      int64_t l = lo, h = hi;
      while (l < h) {
        const int64_t mid = l + ((h - l) >> 1);
        if ((int64_t)(keys[mid] >> shift) < r) l = mid + 1; else h = mid;
      }
      ptr[r] = l;
    }
    return;
  }
  const int len = (int)(hi - lo);
  constexpr int kAhead = 4;
  for (int x0 = 0; x0 < len; x0 += 256 * kAhead) {
    K k[kAhead], before[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int x = x0 + u * 256 + threadIdx.x;
      k[u] = x < len ? keys[lo + x] : K(0);
      before[u] = x > 0 && x < len ? keys[lo + x - 1] : K(0);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int x = x0 + u * 256 + threadIdx.x;
      const uint64_t r = (uint64_t)(k[u] >> shift) - (uint64_t)r0;   // (keys that do not ascend, of indices beyond their range: nowhere)
      if (x < len && r < kPtrRows && (x == 0 || (k[u] >> shift) != (before[u] >> shift))) s_at[r] = x;
    }
  }
  __syncthreads();
  // smallest position from a value on: positions ascend, so it is the next value's that has a key
  int at[kPer], next = len;
  const int4 v = reinterpret_cast<const int4*>(s_at)[threadIdx.x];
  static_assert(kPer == 4, "a thread takes four values");
  at[0] = v.x; at[1] = v.y; at[2] = v.z; at[3] = v.w;
  int mine = at[0] < at[1] ? at[0] : at[1];
  mine = mine < at[2] ? mine : at[2];
  mine = mine < at[3] ? mine : at[3];
  int after = mine;   // minimum from this lane to the wave's last
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int o = __shfl_down(after, d, kWave);
    if (lane + d < kWave && o < after) after = o;
  }
  if (lane == 0) s_min[wave] = after;
  __syncthreads();
  for (int w = wave + 1; w < 4; ++w) next = s_min[w] < next ? s_min[w] : next;
  const int beyond = __shfl_down(after, 1, kWave);
  if (lane < kWave - 1 && beyond < next) next = beyond;
  const int64_t r = r0 + threadIdx.x * kPer;
#pragma unroll
  for (int t = kPer - 1; t >= 0; --t) {
    next = at[t] < next ? at[t] : next;
    if (r + t <= rows) ptr[r + t] = lo + next;
  }
}

// ---- exclusive scan in place, v[n] = total: sums of tiles, scan of the sums by one workgroup, scan inside the tiles ----
constexpr int kScanV = 16;
constexpr int kScanTileN = 256 * kScanV;

template <typename T>
__device__ __forceinline__ T scan_wave(T v) {   // inclusive, over the wave
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const T o = __shfl_up(v, d, kWave);
    if (lane_id() >= d) v += o;
  }
  return v;
}

// exclusive over a workgroup of 256 threads, with the total
template <typename T>
__device__ __forceinline__ T scan_256(T v, T& total, T* ws) {
  const T incl = scan_wave(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane_id() == kWave - 1) ws[wave] = incl;
  __syncthreads();
  T before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) { const T x = ws[w]; if (w < wave) before += x; total += x; }
  return before + incl - v;
}

template <typename T>
__global__ __launch_bounds__(256) void k_scan_sums(int64_t n, const T* __restrict__ v, T* __restrict__ sums) {
  __shared__ T ws[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTileN;
  T s = 0;
#pragma unroll
  for (int t = 0; t < kScanV; ++t) {
    const int64_t i = base + (int64_t)t * 256 + threadIdx.x;
    if (i < n) s += v[i];
  }
  T total;
  (void)scan_256(s, total, ws);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// total (optional, in host memory): the sum of all.
template <typename T>
__global__ __launch_bounds__(256) void k_scan_top(int64_t n, T* __restrict__ sums, T* __restrict__ total_out) {
  __shared__ T ws[4];
  T carry = 0;
  for (int64_t b = 0; b < n; b += kScanTileN) {
    const int64_t base = b + (int64_t)threadIdx.x * kScanV;
    T x[kScanV], s = 0;
#pragma unroll
    for (int t = 0; t < kScanV; ++t) { x[t] = base + t < n ? sums[base + t] : T(0); s += x[t]; }
    T total;
    T run = carry + scan_256(s, total, ws);
#pragma unroll
    for (int t = 0; t < kScanV; ++t) { if (base + t < n) sums[base + t] = run; run += x[t]; }
    carry += total;
  }
  if (threadIdx.x == 0) {
    sums[n] = carry;
    if (total_out) __hip_atomic_store(total_out, carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_scan_tiles(int64_t n, T* __restrict__ v, const T* __restrict__ sums) {
  __shared__ T ws[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTileN + (int64_t)threadIdx.x * kScanV;   // a thread owns 16 consecutive values
  T x[kScanV], s = 0;
#pragma unroll
  for (int t = 0; t < kScanV; ++t) { x[t] = base + t < n ? v[base + t] : T(0); s += x[t]; }
  T total;
  T run = sums[blockIdx.x] + scan_256(s, total, ws);
#pragma unroll
  for (int t = 0; t < kScanV; ++t) { if (base + t < n) v[base + t] = run; run += x[t]; }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) v[n] = sums[gridDim.x];
}

}  // namespace spg
