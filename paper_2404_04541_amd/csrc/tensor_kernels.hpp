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

// A workgroup takes one range of entries of the sort: keys and the range's counts of the first digit.
template <typename Key>
__global__ __launch_bounds__(kSortThreads) void k_tensor_keys(int64_t nnz, int64_t per_range, int64_t I, int64_t J, int64_t K, int col_bits, int bits,
                                                              const int32_t* __restrict__ xi, const int32_t* __restrict__ xj,
                                                              const int32_t* __restrict__ xk, Key* __restrict__ keys, unsigned* __restrict__ hist,
                                                              int* __restrict__ bad) {
  __shared__ unsigned cnt[kHistCopies][kSortBins];
  for (int d = threadIdx.x; d < kHistCopies * kSortBins; d += kSortThreads) (&cnt[0][0])[d] = 0;
  __syncthreads();
  const unsigned mask = (1u << bits) - 1;
  const int64_t lo = (int64_t)blockIdx.x * per_range, hi = lo + per_range < nnz ? lo + per_range : nnz;
  unsigned* mine = cnt[threadIdx.x & (kHistCopies - 1)];
#pragma unroll 4
  for (int64_t p = lo + threadIdx.x; p < hi; p += kSortThreads) {
    const int i = xi[p], j = xj[p], k = xk[p];
    Key key = 0;
    if (i < 0 || i >= I || j < 0 || j >= J || k < 0 || k >= K) *bad = 1;
    else key = ((Key)((long long)i * J + j) << col_bits) | (Key)(unsigned)k;
    keys[p] = key;
    atomicAdd(&mine[(unsigned)key & mask], 1u);
  }
  sort_hist_out(cnt, 1 << bits, blockIdx.x, gridDim.x, hist);
}

// A row of an unfolded result back to coordinates: per entry the row's two folded coordinates
// (row / B, row % B) and, when asked for, the column as the third.
__global__ __launch_bounds__(256) void k_tensor_fold(int64_t rows, int64_t B, const int64_t* __restrict__ rowptr,
                                                     const int32_t* __restrict__ colidx, int32_t* __restrict__ ya,
                                                     int32_t* __restrict__ yb, int32_t* __restrict__ yc) {
  const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kWave);
  const int lane = threadIdx.x & 63;
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x >> 6); r < rows; r += stride) {
    const int64_t lo = rowptr[r], hi = rowptr[r + 1];
    const int32_t a = (int32_t)(r / B), b = (int32_t)(r % B);
    for (int64_t p = lo + lane; p < hi; p += kWave) {
      ya[p] = a;
      yb[p] = b;
      if (yc) yc[p] = colidx[p];
    }
  }
}

}  // namespace spg
