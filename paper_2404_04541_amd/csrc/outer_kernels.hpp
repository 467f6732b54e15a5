// Outer-product sparse x sparse product with a second-order (coordinate) sparse workspace: the
// paper's leading example (sections 1 and 4.1, the algorithm template of section 4.3, evaluated
// in section 7.3).  Loop order k -> i -> j over A in doubly compressed sparse columns and B in
// doubly compressed sparse rows; consecutive products land on unrelated coordinates (i, j), so
// they pass through a workspace of whole components:
//   insert   a batch of products fills the accumulation array: coordinate (i above the bits of j, one 64-bit key) and a_ik * b_kj
//   sort     the accumulation array goes into result order (stable radix sort by coordinate, values along)
//   merge    the first batch's array becomes the all array; every other sorted batch is merged into it, and the first component of a
//            coordinate takes the values of all others along, whichever array holds them (a single batch is added up instead: the first
//            component of a run walks it, in order)
//   compress the last of these stages writes columns and values of C, the row pointer comes from the coordinates
// On the GPU a batch is inserted by one launch, a workgroup taking a range of the sort and finding the columns of A of a tile of
// products once, and the merge is cut into tiles along the diagonals of the two arrays; the stages and the two arrays are the
// paper's.
#pragma once
#include "sort_kernels.hpp"

namespace spg {

// Sort key of every entry of a CSR matrix, (column << row_bits) | row: 16 lanes a row.
__global__ __launch_bounds__(256) void k_column_keys(int64_t rows, int row_bits, const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                     unsigned long long* __restrict__ keys) {
  const int64_t stride = (int64_t)gridDim.x * (blockDim.x / 16);
  const int lane = threadIdx.x & 15;
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / 16) + (threadIdx.x >> 4); r < rows; r += stride)
    for (int64_t p = rowptr[r] + lane; p < rowptr[r + 1]; p += 16) keys[p] = ((unsigned long long)(unsigned)col[p] << row_bits) | (unsigned long long)r;
}

// flag[v] = 1 when vector v (a row, or a column) has entries.
__global__ __launch_bounds__(256) void k_dcs_flags(int64_t n, const int64_t* __restrict__ ptr, unsigned* __restrict__ flag) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) flag[v] = ptr[v + 1] > ptr[v] ? 1u : 0u;
}

// pos = exclusive scan of the flags: the non-empty vectors move up, in order.
__global__ __launch_bounds__(256) void k_dcs_fill(int64_t n, const int64_t* __restrict__ ptr, const unsigned* __restrict__ pos,
                                                  int32_t* __restrict__ vec, int64_t* __restrict__ out_ptr, int64_t nnz, int64_t nvec) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride)
    if (ptr[v + 1] > ptr[v]) { vec[pos[v]] = (int32_t)v; out_ptr[pos[v]] = ptr[v]; }
  if (blockIdx.x == 0 && threadIdx.x == 0) out_ptr[nvec] = nnz;
}

// cnt[p] = products of A's p-th kept column: its length times the length of the B row of the same
// index k (0 when B has no such row); match[p] = that row's position in B's list, or -1.
__global__ __launch_bounds__(256) void k_outer_count(int64_t na, const int32_t* __restrict__ a_vec, const int64_t* __restrict__ a_ptr,
                                                     int64_t nb, const int32_t* __restrict__ b_vec, const int64_t* __restrict__ b_ptr,
                                                     long long* __restrict__ cnt, int32_t* __restrict__ match) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < na; p += stride) {
    const int k = a_vec[p];
    const int64_t q = lower_bound_i32(b_vec, 0, nb, k);
    const bool hit = q < nb && b_vec[q] == k;
    match[p] = hit ? (int32_t)q : -1;
    cnt[p] = hit ? (a_ptr[p + 1] - a_ptr[p]) * (b_ptr[q + 1] - b_ptr[q]) : 0;
  }
}

// The coordinate of product t0 + x of the k -> i -> j order, by a bisection of all offsets (for a few of them).
struct OuterKey {
  int64_t t0, na;
  int col_bits;
  const long long* off;
  const int32_t* match;
  const int64_t *a_ptr, *b_ptr;
  const int32_t *a_idx, *b_idx;
  __device__ __forceinline__ unsigned long long operator()(int64_t x) const {
    const int64_t t = t0 + x;
    int64_t l = 0, h = na;
    while (h - l > 1) {
      const int64_t mid = l + ((h - l) >> 1);
      if (off[mid] <= t) l = mid; else h = mid;
    }
    const int64_t q = match[l], b0 = b_ptr[q], lb = b_ptr[q + 1] - b0, local = t - off[l];
    return ((unsigned long long)(unsigned)a_idx[a_ptr[l] + local / lb] << col_bits) | (unsigned)b_idx[b0 + local % lb];
  }
};

// Insert stage: products [t0, t0 + n) of the k -> i -> j order fill the accumulation array.  A workgroup takes one range of the
// sort that follows, kInsertTile products at a time: the columns of A that a tile touches are found once (two bisections of the
// offsets), a product then only looks among those, in LDS when they are few; the first digit's counts of the range on the way.
// 16.8 M products over 10^6 columns: 338 us with a bisection of all offsets per product (and 27 for the counts), 162 with the two per tile by a
// thread each (twenty loads that wait for one another), 144 by a wave each.
constexpr int kInsertTile = 4096;
constexpr int kInsertCols = 2048;
template <typename T>
__global__ __launch_bounds__(kSortThreads) void k_outer_insert(int64_t t0, int64_t n, int64_t per_range, int shift, int bits, int64_t na,
    const long long* __restrict__ off, const int32_t* __restrict__ match, const int64_t* __restrict__ a_ptr, const int32_t* __restrict__ a_idx,
    const T* __restrict__ a_val, const int64_t* __restrict__ b_ptr, const int32_t* __restrict__ b_idx, const T* __restrict__ b_val, int col_bits,
    unsigned long long* __restrict__ keys, double* __restrict__ vals, unsigned* __restrict__ hist) {
  __shared__ unsigned cnt[kHistCopies][kSortBins];
  __shared__ long long s_off[kInsertCols];
  __shared__ long long bound[2];
  for (int d = threadIdx.x; d < kHistCopies * kSortBins; d += kSortThreads) (&cnt[0][0])[d] = 0;
  unsigned* mine = cnt[threadIdx.x & (kHistCopies - 1)];
  const unsigned mask = (1u << bits) - 1;
  const int64_t lo = (int64_t)blockIdx.x * per_range, hi = lo + per_range < n ? lo + per_range : n;
  for (int64_t x0 = lo; x0 < hi; x0 += kInsertTile) {
    const int64_t x1 = x0 + kInsertTile < hi ? x0 + kInsertTile : hi;
    __syncthreads();   // (the counters are cleared; the tile before has left the offsets)
    if (threadIdx.x < 2 * kWave) {   // a wave an end: last column whose first product is <= t, in 64 parts at a time
      const int64_t t = t0 + (threadIdx.x < kWave ? x0 : x1 - 1);
      int64_t l = 0, h = na;
      while (h - l > 1) {
        const int64_t step = (h - l + kWave - 1) / kWave, c = l + lane_id() * step;
        const unsigned long long below = __ballot(c < h && off[c < h ? c : l] <= t);
        l += (63 - __clzll((long long)(below | 1))) * step;
        h = l + step < h ? l + step : h;
      }
      if (lane_id() == 0) bound[threadIdx.x / kWave] = l;
    }
    __syncthreads();
    const int64_t c0 = bound[0], c1 = bound[1] + 1;
    const bool cached = c1 - c0 <= kInsertCols;
    if (cached) {
      for (int64_t c = c0 + threadIdx.x; c < c1; c += kSortThreads) s_off[c - c0] = off[c];
      __syncthreads();
    }
    for (int64_t x = x0 + threadIdx.x; x < x1; x += kSortThreads) {
      const int64_t t = t0 + x;
      int64_t col, first;
      if (cached) {
        int l = 0, h = (int)(c1 - c0);
        while (h - l > 1) {
          const int mid = (l + h) >> 1;
          if (s_off[mid] <= t) l = mid; else h = mid;
        }
        col = c0 + l;
        first = s_off[l];
      } else {
        int64_t l = c0, h = c1;
        while (h - l > 1) {
          const int64_t mid = l + ((h - l) >> 1);
          if (off[mid] <= t) l = mid; else h = mid;
        }
        col = l;
        first = off[l];
      }
      const int64_t q = match[col];
      const int64_t b0 = b_ptr[q], lb = b_ptr[q + 1] - b0, local = t - first;
      int64_t i, j;
      if (local <= 0xffffffffLL && lb <= 0xffffffffLL) { const unsigned d = (unsigned)local / (unsigned)lb; i = d; j = (unsigned)local - d * (unsigned)lb; }
      else { i = local / lb; j = local % lb; }
      const int64_t pa = a_ptr[col] + i, pb = b0 + j;
      const unsigned long long key = ((unsigned long long)(unsigned)a_idx[pa] << col_bits) | (unsigned)b_idx[pb];
      keys[x] = key;
      vals[x] = (double)a_val[pa] * (double)b_val[pb];
      atomicAdd(&mine[(unsigned)(key >> shift) & mask], 1u);
    }
  }
  sort_hist_out(cnt, 1 << bits, blockIdx.x, gridDim.x, hist);
}

// Where components go: coordinate and sum of the all array or, with the last stage, the row (the row pointer comes from
// it: four bytes written and read in place of the coordinate's eight), the column and the value of C.
template <typename T>
struct OuterOut {
  unsigned long long* keys;
  double* vals;     // keys, vals: null with the last stage
  uint32_t* row;
  int32_t* col;     // row, col, val: null before it
  T* val;
  int col_bits;
  __device__ __forceinline__ void put(int64_t at, unsigned long long key, double v) const {
    if (vals) {
      keys[at] = key;
      vals[at] = v;
    } else {
      row[at] = (uint32_t)(key >> col_bits);
      col[at] = (int32_t)(key & ((1ULL << col_bits) - 1));
      val[at] = (T)v;
    }
  }
};

// Equal neighbours of a sorted array are added up, in their order, by the thread of the run's first component.  A wave owns
// kRunItems * 64 consecutive components of a tile; heads are ballots, so no flags go through memory (flags, their scan and the
// walk took 450 us for 16.8 M components, the two passes here 140).
constexpr int kRunItems = 16;
constexpr int kRunTile = 256 * kRunItems;
__device__ __forceinline__ int run_heads(int64_t n, const unsigned long long* __restrict__ keys, int64_t first, unsigned long long (&key)[kRunItems],
                                         unsigned long long (&heads)[kRunItems]) {
  int total = 0;
#pragma unroll
  for (int t = 0; t < kRunItems; ++t) {
    const int64_t x = first + t * kWave + lane_id();
    key[t] = x < n ? keys[x] : 0ULL;
    heads[t] = __ballot(x < n && (x == 0 || keys[x - 1] != key[t]));
    total += __popcll(heads[t]);
  }
  return total;
}

// sums[tile] = runs that begin in the tile
__global__ __launch_bounds__(256) void k_run_count(int64_t n, const unsigned long long* __restrict__ keys, unsigned* __restrict__ sums) {
  __shared__ int part[4];
  const int wave = threadIdx.x >> 6;
  unsigned long long key[kRunItems], heads[kRunItems];
  const int mine = run_heads(n, keys, (int64_t)blockIdx.x * kRunTile + wave * (kRunItems * kWave), key, heads);
  if (lane_id() == 0) part[wave] = mine;
  __syncthreads();
  if (threadIdx.x == 0) sums[blockIdx.x] = (unsigned)(part[0] + part[1] + part[2] + part[3]);
}

template <typename T>
__global__ __launch_bounds__(256) void k_run_sum(int64_t n, const unsigned long long* __restrict__ keys, const double* __restrict__ vals,
                                                 const unsigned* __restrict__ sums, OuterOut<T> out) {
  __shared__ int part[4];
  const int wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * kRunTile + wave * (kRunItems * kWave);
  unsigned long long key[kRunItems], heads[kRunItems];
  const int mine = run_heads(n, keys, first, key, heads);
  if (lane_id() == 0) part[wave] = mine;
  __syncthreads();
  int64_t at = sums[blockIdx.x];
  for (int w = 0; w < wave; ++w) at += part[w];
#pragma unroll
  for (int t = 0; t < kRunItems; ++t) {
    const int64_t x = first + t * kWave + lane_id();
    if ((heads[t] >> lane_id()) & 1ULL) {
      double s = vals[x];
      for (int64_t y = x + 1; y < n && keys[y] == key[t]; ++y) s += vals[y];
      out.put(at + lanes_below(heads[t]), key[t], s);
    }
    at += __popcll(heads[t]);
  }
}

// Merge stage: the sorted batch (b) into the all array (a), equal coordinates added.  The
// merged order (a's components first where both hold a coordinate) is cut into tiles of kMergeTile; a tile's share of either
// array comes from a bisection along the diagonal, and so does a thread's share of a tile.  Either array may hold a coordinate
// several times: the first component of the merged order that has it stays and takes the others' values along, a's in their order, then b's.
// (So the batches need not be added up by themselves first, which took a pass over their keys, one over all, and a wait of the host each: 16.8 M
// components 145 us and the wait.)  Bound by reading and writing the components (four arrays of 8 bytes in, 20 to 24 bytes out).
// Two sorted arrays of 16.7 M components each: bisection of the other array per component, head flags, their scan and a walk
// over the runs 1.47 ms, tiles with a bisection in LDS per component 0.61 (count 137 us, put 437), here 0.35 (92, 228).
constexpr int kMergeTile = 2048;

// split[t] = components of a among the first t * kMergeTile of the merged order
__global__ __launch_bounds__(256) void k_merge_split(int64_t na, const unsigned long long* __restrict__ ka, int64_t nb, const unsigned long long* __restrict__ kb,
                                                     int64_t tiles, int64_t* __restrict__ split) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t > tiles) return;
  const int64_t d = t * kMergeTile < na + nb ? t * kMergeTile : na + nb;
  int64_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
  while (lo < hi) {   // the smallest i with a[i] > b[d - 1 - i]: a's component goes first on equal coordinates
    const int64_t i = lo + ((hi - lo) >> 1);
    if (ka[i] <= kb[d - 1 - i]) lo = i + 1; else hi = i;
  }
  split[t] = lo;
}

struct MergeLds {
  unsigned long long key[kMergeTile];   // a's components of the tile, then b's
  unsigned from[kMergeTile];            // of every component that stays: how many of a's and of b's lie before it, and whether it is a's
  int part[4];
};
constexpr unsigned kFromBits = 12;
constexpr unsigned kFromA = 1u << (2 * kFromBits);
static_assert((1u << kFromBits) > kMergeTile, "places of a tile");

// Loads the tile's keys and merges them, kPer consecutive components of the merged order to a thread: a bisection along its diagonal, then a step
// each.  Returns how many stay; PUT: lists them in ml->from.
template <bool PUT>
__device__ __forceinline__ int merge_tile(int64_t na, const unsigned long long* __restrict__ ka, int64_t nb,
    const unsigned long long* __restrict__ kb, int64_t a0, int an, int64_t b0, int bn, MergeLds* ml) {
  constexpr int kPer = kMergeTile / 256;
  for (int x = threadIdx.x; x < an; x += 256) ml->key[x] = ka[a0 + x];
  for (int x = threadIdx.x; x < bn; x += 256) ml->key[an + x] = kb[b0 + x];
  // the components in front of the tile
  const unsigned long long a_front = a0 > 0 ? ka[a0 - 1] : 0ULL, b_front = b0 > 0 ? kb[b0 - 1] : 0ULL;
  __syncthreads();
  const int n = an + bn, d = (int)threadIdx.x * kPer < n ? (int)threadIdx.x * kPer : n;
  int i = d > bn ? d - bn : 0, hi = d < an ? d : an;
  while (i < hi) {   // (as in k_merge_split)
    const int mid = (i + hi) >> 1;
    if (ml->key[mid] <= ml->key[an + d - 1 - mid]) i = mid + 1; else hi = mid;
  }
  int j = d - i;
  // the component before the thread's first: the larger one of both arrays
  bool have = a0 + i > 0 || b0 + j > 0;
  const unsigned long long a_last = i > 0 ? ml->key[i - 1] : a_front, b_last = j > 0 ? ml->key[an + j - 1] : b_front;
  unsigned long long before = a_last > b_last ? a_last : b_last;
  unsigned long long x = i < an ? ml->key[i] : 0ULL, y = j < bn ? ml->key[an + j] : 0ULL;
  unsigned from[kPer], stay = 0;
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    from[t] = 0;
    if (d + t >= n) continue;
    const bool of_a = i < an && (j >= bn || x <= y);
    const unsigned long long key = of_a ? x : y;
    from[t] = (unsigned)i | ((unsigned)j << kFromBits) | (of_a ? kFromA : 0u);
    if (!(have && before == key)) stay |= 1u << t;
    have = true;
    before = key;
    if (of_a) {
      if (++i < an) x = ml->key[i];
    } else {
      if (++j < bn) y = ml->key[an + j];
    }
  }
  const int mine = __popc(stay);
  const int incl = wave_incl_scan(mine);
  if (lane_id() == kWave - 1) ml->part[threadIdx.x >> 6] = incl;
  __syncthreads();
  int at = incl - mine, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) { const int c = ml->part[w]; if (w < (int)(threadIdx.x >> 6)) at += c; total += c; }
  if (PUT) {
#pragma unroll
    for (int t = 0; t < kPer; ++t)
      if (stay >> t & 1) ml->from[at++] = from[t];
    __syncthreads();
  }
  return total;
}

// sums[tile] = components that stay
__global__ __launch_bounds__(256) void k_merge_count(int64_t na, const unsigned long long* __restrict__ ka, int64_t nb, const unsigned long long* __restrict__ kb,
                                                     const int64_t* __restrict__ split, unsigned* __restrict__ sums) {
  __shared__ MergeLds ml;
  const int64_t d0 = (int64_t)blockIdx.x * kMergeTile, d1 = d0 + kMergeTile < na + nb ? d0 + kMergeTile : na + nb;
  const int64_t a0 = split[blockIdx.x], a1 = split[blockIdx.x + 1];
  const int stay = merge_tile<false>(na, ka, nb, kb, a0, (int)(a1 - a0), d0 - a0, (int)((d1 - a1) - (d0 - a0)), &ml);
  if (threadIdx.x == 0) sums[blockIdx.x] = (unsigned)stay;
}

// Adds the values of the components from p on that have this coordinate, in their order.  The chain of a load and a comparison per component is what a
// coordinate that is there hundreds of times costs, so kAhead of them are loaded at a time; the first few come one by one (most coordinates have no more,
// and their neighbours' values need not be read for nothing).  32 M products in two batches, whole calls, us with batches added up by themselves (k_run_sum) |
// merged one by one | 4 | 8 | 16 at a time: 53 of each coordinate 2854 | 1937 | 1755 | 1732 | 1726, 1600 of each 4547 | 6277 | 3216 | 2553 | 2683, 20 000
// 8545 | 12 959 | 5074 | 3867 | 4037; coordinates that hardly repeat 2218 | 1815 | 1774 | 1772 | 1775.
constexpr int kNear = 4, kAhead = 8;
__device__ __forceinline__ double add_equal(const unsigned long long* __restrict__ keys, const double* __restrict__ vals, int64_t p, int64_t n,
                                            unsigned long long key, double sum) {
  for (int64_t near = p + kNear; p < near; ++p) {
    if (p >= n || keys[p] != key) return sum;
    sum += vals[p];
  }
  for (; p + kAhead <= n; p += kAhead) {
    unsigned long long k[kAhead];
    double v[kAhead];
#pragma unroll
    for (int t = 0; t < kAhead; ++t) { k[t] = keys[p + t]; v[t] = vals[p + t]; }
#pragma unroll
    for (int t = 0; t < kAhead; ++t)
      if (k[t] == key) sum += v[t];   // (sorted: those of the coordinate come first)
    if (k[kAhead - 1] != key) return sum;
  }
  for (; p < n && keys[p] == key; ++p) sum += vals[p];
  return sum;
}

template <typename T>
__global__ __launch_bounds__(256) void k_merge_put(int64_t na, const unsigned long long* __restrict__ ka, const double* __restrict__ va, int64_t nb,
                                                   const unsigned long long* __restrict__ kb, const double* __restrict__ vb,
                                                   const int64_t* __restrict__ split, const unsigned* __restrict__ sums, OuterOut<T> out) {
  __shared__ MergeLds ml;
  const int64_t d0 = (int64_t)blockIdx.x * kMergeTile, d1 = d0 + kMergeTile < na + nb ? d0 + kMergeTile : na + nb;
  const int64_t a0 = split[blockIdx.x], a1 = split[blockIdx.x + 1];
  const int64_t b0 = d0 - a0;
  const int an = (int)(a1 - a0), bn = (int)((d1 - a1) - b0);
  const int stay = merge_tile<true>(na, ka, nb, kb, a0, an, b0, bn, &ml);
  const int64_t at = sums[blockIdx.x];
  for (int x = threadIdx.x; x < stay; x += 256) {
    const unsigned w = ml.from[x];
    int i = (int)(w & ((1u << kFromBits) - 1)), j = (int)((w >> kFromBits) & ((1u << kFromBits) - 1));
    const bool of_a = (w & kFromA) != 0;
    const unsigned long long key = ml.key[of_a ? i : an + j];
    double v = of_a ? va[a0 + i] : vb[b0 + j];
    if (of_a) ++i; else ++j;
    // the others: a's (none where the first is b's), then b's; one by one in the tile, behind it and where there are many kAhead at a time
    if (of_a) {
      const int near = i + kNear < an ? i + kNear : an;
      while (i < near && ml.key[i] == key) v += va[a0 + i++];
      if (i == near) v = add_equal(ka, va, a0 + i, na, key, v);
    }
    const int near = j + kNear < bn ? j + kNear : bn;
    while (j < near && ml.key[an + j] == key) v += vb[b0 + j++];
    if (j == near) v = add_equal(kb, vb, b0 + j, nb, key, v);
    out.put(at + x, key, v);
  }
}

}  // namespace spg
