// Mode-3 unfolding of a sparse 3-tensor given as coordinates (the "index folding" route to a
// sparse tensor-times-matrix product, paper section 7.4): X(i,j,k) becomes row i*J + j, column k
// of a CSR matrix, so that Y(i,j,l) = sum_k X(i,j,k) M(k,l) is one row-wise product whose CSR
// result is the unfolding of Y.  Coordinates may come in any order; repeated coordinates stay
// separate entries (the product adds them).
//   keys     row << (bits of k) | k per entry, 32 bits wide when that is enough, and the first digit's counts
//   sort     stable radix sort by key with the values as payload (sort_kernels.hpp)
//   compress columns with the sort's last pass, the row pointer from the sorted keys
#pragma once
#include "sort_kernels.hpp"

namespace spg {

// The key of the entry (i, j, k); false: a coordinate is out of range, the key 0.
template <typename Key>
__device__ __forceinline__ bool tensor_key(int i, int j, int k, int64_t I, int64_t J, int64_t K, int col_bits, Key* key) {
  *key = 0;
  if (i < 0 || i >= I || j < 0 || j >= J || k < 0 || k >= K) return false;
  *key = ((Key)((long long)i * J + j) << col_bits) | (Key)(unsigned)k;
  return true;
}

template <typename Key>
struct TensorKey {   // of entry p
  int64_t I, J, K;
  int col_bits;
  const int32_t *xi, *xj, *xk;
  __device__ __forceinline__ Key operator()(int64_t p) const {
    Key key;
    (void)tensor_key<Key>(xi[p], xj[p], xk[p], I, J, K, col_bits, &key);
    return key;
  }
};

// A workgroup takes one range of entries of the sort: keys and the range's counts of the first digit.
template <typename Key>
__global__ __launch_bounds__(kSortThreads) void k_tensor_keys(int64_t nnz, int64_t per_range, int64_t I, int64_t J, int64_t K, int col_bits,
    int shift, int bits, const int32_t* __restrict__ xi, const int32_t* __restrict__ xj, const int32_t* __restrict__ xk, Key* __restrict__ keys,
    unsigned* __restrict__ hist, int* __restrict__ bad) {
  __shared__ unsigned cnt[kHistCopies][kSortBins];
  for (int d = threadIdx.x; d < kHistCopies * kSortBins; d += kSortThreads) (&cnt[0][0])[d] = 0;
  __syncthreads();
  const unsigned mask = (1u << bits) - 1;
  const int64_t lo = (int64_t)blockIdx.x * per_range, hi = lo + per_range < nnz ? lo + per_range : nnz;
  unsigned* mine = cnt[threadIdx.x & (kHistCopies - 1)];
#pragma unroll 4
  for (int64_t p = lo + threadIdx.x; p < hi; p += kSortThreads) {
    Key key;
    if (!tensor_key<Key>(xi[p], xj[p], xk[p], I, J, K, col_bits, &key)) *bad = 1;
    keys[p] = key;
    atomicAdd(&mine[(unsigned)(key >> shift) & mask], 1u);
  }
  sort_hist_out(cnt, 1 << bits, blockIdx.x, gridDim.x, hist);
}

// Rows of an unfolded result back to coordinates: per entry the row's two folded coordinates (row / B, row % B) and, when asked
// for, the column as the third.  Row ends and entries together are cut into equal tiles, so a workgroup's share is the same whether
// rows are empty, short or long: it finds its first row and entry, leaves every row's number at its first entry in LDS, and a
// running maximum gives each entry its row.
// Bound: memory, 4 bytes read and 12 written per entry.  700 891 rows (a quarter of them not empty) of 1.6 M entries: a wave for every
// row, with divisions of 64 bits, 47 us; here 15 us.
constexpr int kFoldTile = 4096;
__global__ __launch_bounds__(256) void k_tensor_fold(int64_t rows, int64_t B, const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                     int32_t* __restrict__ ya, int32_t* __restrict__ yb, int32_t* __restrict__ yc) {
  constexpr int kPer = kFoldTile / 256;
  __shared__ __align__(16) int s_row[kFoldTile];   // row of an entry minus the tile's first: at a row's first entry, then everywhere
  __shared__ int64_t bound[2];
  __shared__ int s_max[4];
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int64_t p0 = rowptr[0], total = rows + (rowptr[rows] - p0);
  int4* mine4 = reinterpret_cast<int4*>(s_row) + threadIdx.x * (kPer / 4);
  for (int64_t d0 = (int64_t)blockIdx.x * kFoldTile; d0 < total; d0 += (int64_t)gridDim.x * kFoldTile) {
    const int64_t d1 = d0 + kFoldTile < total ? d0 + kFoldTile : total;
    if (wave < 2) {   // rows whose end, the rows before them counted, is at or before the tile's edge
      const int64_t d = wave ? d1 : d0;
      const int64_t r = wave_first_not(rows, [&](int64_t i) { return i + 1 + (rowptr[i + 1] - p0) <= d; });
      if (lane == 0) bound[wave] = r;
    }
#pragma unroll
    for (int t = 0; t < kPer / 4; ++t) reinterpret_cast<int4*>(s_row)[t * 256 + threadIdx.x] = make_int4(0, 0, 0, 0);
    __syncthreads();
    const int64_t r0 = bound[0], e0 = d0 - r0;
    const int nr = (int)(bound[1] - r0), left = (int)(d1 - d0) - nr;
    const int ne = left < kFoldTile ? left : kFoldTile;
    for (int i = 1 + threadIdx.x; i <= nr; i += 256) {
      if (r0 + i >= rows) break;
      const Run<int64_t, 2> v = load_run<int64_t, 2>(rowptr + r0 + i);
      const int64_t at = v.v[0] - p0 - e0;   // (the last of these rows may begin behind the tile's entries)
      if (v.v[0] < v.v[1] && at >= 0 && at < ne) s_row[at] = i;
    }
    __syncthreads();
    int x[kPer], top = 0;
#pragma unroll
    for (int t = 0; t < kPer / 4; ++t) {
      const int4 v = mine4[t];
      x[t * 4] = v.x; x[t * 4 + 1] = v.y; x[t * 4 + 2] = v.z; x[t * 4 + 3] = v.w;
    }
#pragma unroll
    for (int t = 0; t < kPer; ++t) top = x[t] > top ? x[t] : top;
    const int incl = group_max_scan<kWave>(top);
    if (lane == kWave - 1) s_max[wave] = incl;
    int before = __shfl_up(incl, 1, kWave);
    if (lane == 0) before = 0;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before = s_max[w] > before ? s_max[w] : before;
#pragma unroll
    for (int t = 0; t < kPer; ++t) { before = x[t] > before ? x[t] : before; x[t] = before; }
#pragma unroll
    for (int t = 0; t < kPer / 4; ++t) mine4[t] = make_int4(x[t * 4], x[t * 4 + 1], x[t * 4 + 2], x[t * 4 + 3]);
    __syncthreads();
    // (there are less than 2^31 rows and B is one of their divisors)
    const unsigned a0 = (unsigned)r0 / (unsigned)B, b0 = (unsigned)r0 - a0 * (unsigned)B;
#pragma unroll 4
    for (int e = threadIdx.x; e < ne; e += 256) {
      const unsigned b = b0 + (unsigned)s_row[e], q = b / (unsigned)B;
      const int64_t p = p0 + e0 + e;
      ya[p] = (int32_t)(a0 + q);
      yb[p] = (int32_t)(b - q * (unsigned)B);
      if (yc) yc[p] = colidx[p];
    }
    __syncthreads();
  }
}

}  // namespace spg
