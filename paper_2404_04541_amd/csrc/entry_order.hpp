// The order of the operands' entries.  What short rows leave in the plan (sorted words, records, descriptions) goes by the position
// of an entry in its row, but a plan holds for operands of the same structure whatever the order of a row's entries.  So the
// columns of both operands are summed with a weight per position (the weights of any two positions differ), once for a plan that
// its caller holds and again in every numeric phase on it; where the sum is another one, the kernels that go by the plan's order
// end at once and k_other_order does their rows without it.  The plan's tiles go by it too where B ascends (which part of a row of B a
// tile holds): rows of numeric class 3 are then done without tiles, whereas the rows of the dense classes have no other way, which is
// why the order of an ascending B may not change where there are any.
// Bound: memory, one pass over the columns (of one operand where both are the same array), and the launches.  Numeric phase on a
// kept plan, 27-point stencil (fp64): 61^3 rows 256 -> 268 us, 128^3 rows 2.19 -> 2.24 ms; in another order 475 us and 4.36 ms
// (without any plan of the order, 546 us and 4.79 ms).
#pragma once
#include "common.hpp"

namespace spg {

__device__ __forceinline__ unsigned order_weight(int64_t p) {   // a bijection of 32 bits
  unsigned x = (unsigned)p ^ ((unsigned)((unsigned long long)p >> 32) * 0x51ED2705u);
  x = (x ^ (x >> 16)) * 0x9E3779B1u;
  return (x ^ (x >> 15)) * 0x85157AF5u;
}

constexpr int kOrderThreads = 1024;
constexpr int kOrderQuads = 4;   // loads in flight per thread
constexpr int kOrderTile = kOrderThreads * kOrderQuads * 4;

// This thread's share (workgroup part of parts, THREADS threads) of the sum over n columns.
template <int THREADS>
__device__ __forceinline__ unsigned long long order_sum_of(int64_t n, const int32_t* __restrict__ col, int part, int parts) {
  constexpr int kTile = THREADS * kOrderQuads * 4;
  unsigned long long s = 0;
  for (int64_t t0 = (int64_t)part * kTile; t0 < n; t0 += (int64_t)parts * kTile) {
    Run<int32_t, 4> c[kOrderQuads];
    const int64_t p = t0 + threadIdx.x * 4;
    if (t0 + kTile <= n) {
#pragma unroll
      for (int u = 0; u < kOrderQuads; ++u) c[u] = load_run<int32_t, 4>(col + p + u * THREADS * 4);
    } else {
#pragma unroll
      for (int u = 0; u < kOrderQuads; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t q = p + u * THREADS * 4 + i;
          c[u].v[i] = q < n ? col[q] : 0;
        }
    }
#pragma unroll
    for (int u = 0; u < kOrderQuads; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) s += (unsigned long long)order_weight(p + u * THREADS * 4 + i) * (unsigned)c[u].v[i];
  }
  return s;
}

// b_col null: B's columns are A's.
template <int THREADS>
__device__ __forceinline__ unsigned long long order_share(int64_t na, const int32_t* __restrict__ a_col, int64_t nb, const int32_t* __restrict__ b_col, int part,
                                                          int parts) {
  const unsigned long long a = order_sum_of<THREADS>(na, a_col, part, parts);
  unsigned long long s = a + (b_col ? order_sum_of<THREADS>(nb, b_col, part, parts) : a) * 0x9E3779B97F4A7C15ULL;
  for (int d = kWave / 2; d > 0; d >>= 1) s += __shfl_xor(s, d, kWave);
  return s;   // (of the wave)
}

// One word for both operands: their sums' low 56 bits above the number of workgroups that have
// added theirs, so that a workgroup sends one atomic and the last one knows the whole (three atomics each, to sums and a counter:
// 11 us for 6 M entries, and 15 us with twice the workgroups; now 8 us).  s: a wave's share, from every wave of the workgroup.  plan:
// the word is the plan's, otherwise it is compared with it, and *differs says how that came out.
constexpr int kOrderParts = 128;   // at most
static_assert(kOrderParts < 256, "the count has eight bits");
template <int THREADS>
__device__ __forceinline__ void order_add(unsigned long long s, int parts, Control* ctl, int plan, int* differs) {
  __shared__ unsigned long long part[THREADS / kWave];
  if (lane_id() == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < THREADS / kWave; ++w) s += part[w];
    const unsigned long long mine = (s << 8) + 1, before = atomicAdd(&ctl->order_now, mine);
    if ((before & 255) == (unsigned long long)(parts - 1)) {
      ctl->order_now = 0;   // (for the next time)
      const unsigned long long all = (before + mine) & ~255ULL;
      if (plan) ctl->order = all;
      else *differs = all != ctl->order ? 1 : 0;
    }
  }
}

__global__ __launch_bounds__(kOrderThreads) void k_order_sum(int64_t na, const int32_t* __restrict__ a_col, int64_t nb, const int32_t* __restrict__ b_col,
                                                             Control* ctl, int plan) {
  order_add<kOrderThreads>(order_share<kOrderThreads>(na, a_col, nb, b_col, blockIdx.x, gridDim.x), gridDim.x, ctl, plan, &ctl->order_differs);
}

// What the numeric kernel of recorded rows needs to look at the order with `parts` workgroups of its own (it does its rows meanwhile:
// whatever the order, they stay in bounds, for what they index comes from the plan and from row lengths).
struct OrderOperands {
  int parts;
  int64_t na, nb;
  const int32_t *a_col, *b_col;   // b_col null: as a_col
};
// What a numeric phase knows of the order when its kernels run: nobody has looked (or need not), k_order_sum has, k_num_recorded has.
enum { kOrderNotLooked = 0, kOrderSummed = 1, kOrderBeside = 2 };
__device__ __forceinline__ bool other_order(const Control* ctl, int looked) {
  return looked == kOrderSummed ? ctl->order_differs != 0 : looked == kOrderBeside && ctl->order_later != 0;
}

// Up to this many entries that saves the launch of k_order_sum; beyond, the rows' kernel loses more (its code with the sum in it takes
// a tenth longer for the rows).  Numeric phase of stencils, us with the launch | inside | without any check: 10 600 entries 19.0 | 13.6 | 11.6,
// 0.10 M 21.6 | 16.1 | 13.5, 0.83 M 47.9 | 44.7 | 39.1, 1.6 M 71.7 | 71.3 | 63.1, 2.9 M 144 | 148 | 133.
constexpr int64_t kOrderInside = 1 << 20;
constexpr int kOrderInsideTile = 256 * kOrderQuads * 4;

}  // namespace spg
