// What the kernels over short rows share: the chain of loads that leads to a row's products, and loads of four entries.
#pragma once
#include "common.hpp"

namespace spg {

// Up to four entries of an array of b_nnz elements from position p on (n of them are wanted; 0: lane is off): one load where
// four elements exist behind every lane's position.
template <typename E>
__device__ __forceinline__ void load_quad(const E* __restrict__ a, int64_t p, int n, int64_t b_nnz, E (&out)[4]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) out[u] = E(0);
  if (!__any(n > 0 && p + 4 > b_nnz)) {
    if (n > 0) {
      const Run<E, 4> r = load_run<E, 4>(a + p);
#pragma unroll
      for (int u = 0; u < 4; ++u) out[u] = r.v[u];
    }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < n) out[u] = a[p + u];
  }
}

// The loads that lead to a row's products depend on each other (row number, range in A, entry, bounds of the B row): a group of
// GROUP lanes keeps four rows in flight, one load of the chain each, so that a row waits for none of them.
template <int GROUP>
struct RowChain {
  const int* perm;
  const int64_t* a_rp;
  const int32_t* a_col;
  const int64_t* b_rp;
  const unsigned long long* desc;   // (optional) per A entry: where its B row begins, how long it is
  unsigned nrows, step, at;   // at: the row being fetched now
  int row, row1, row2, row3;  // rows of the bin: in the works, next, ...
  int64_t a0, a01, a02;
  int d, d1, d2;
  int k1;                     // this lane's entry of the next row
  Run<int64_t, 2> bounds;     // of this lane's entry of the row in the works

  static __device__ __forceinline__ int gl() { return lane_id() & (GROUP - 1); }
  __device__ __forceinline__ int fetch_row() {
    const int r = at < nrows ? perm[at] : -1;
    at += step;
    return r;
  }
  __device__ __forceinline__ void fetch_range(int r, int64_t& a, int& n) const {
    a = 0; n = 0;
    if (r >= 0) { const Run<int64_t, 2> v = load_run<int64_t, 2>(a_rp + r); a = v.v[0]; n = (int)(v.v[1] - v.v[0]); }
  }
  __device__ __forceinline__ int fetch_entry(int64_t a, int n) const { return !desc && gl() < n ? a_col[a + gl()] : -1; }
  // bounds of the B row of this lane's entry: the entry's column is key, or its description is at a + gl()
  __device__ __forceinline__ void fetch_bounds(int64_t a, int n, int key, Run<int64_t, 2>& v) const {
    if (desc) v = desc_bounds(gl() < n ? desc[a + gl()] : 0ULL);
    else fetch_bounds(key, v);
  }
  // the same for entry c + gl() of the row in the works
  __device__ __forceinline__ void fetch_more(int c) {
    if (desc) bounds = desc_bounds(c + gl() < d ? desc[a0 + c + gl()] : 0ULL);
    else fetch_bounds(c + gl() < d ? a_col[a0 + c + gl()] : -1, bounds);
  }
  __device__ __forceinline__ void fetch_bounds(int key, Run<int64_t, 2>& v) const {
    v.v[0] = 0; v.v[1] = 0;
    if (key >= 0) v = load_run<int64_t, 2>(b_rp + key);
  }
  __device__ __forceinline__ void start(unsigned first) {
    at = first;
    row = fetch_row(); row1 = fetch_row(); row2 = fetch_row(); row3 = fetch_row();
    fetch_range(row, a0, d);
    fetch_range(row1, a01, d1);
    fetch_range(row2, a02, d2);
    const int k = fetch_entry(a0, d);
    k1 = fetch_entry(a01, d1);
    fetch_bounds(a0, d, k, bounds);
  }

  // One load further for each of the rows ahead; advance() takes what they brought when the row in the works is done.
  struct Ahead {
    Run<int64_t, 2> bounds;
    int64_t a0;
    int k, d, row;
  };
  __device__ __forceinline__ Ahead fetch() {
    Ahead n;
    fetch_bounds(a01, d1, k1, n.bounds);
    n.k = fetch_entry(a02, d2);
    fetch_range(row3, n.a0, n.d);
    n.row = fetch_row();
    return n;
  }
  __device__ __forceinline__ void advance(const Ahead& n) {
    row = row1; row1 = row2; row2 = row3; row3 = n.row;
    a0 = a01; a01 = a02; a02 = n.a0;
    d = d1; d1 = d2; d2 = n.d;
    k1 = n.k;
    bounds = n.bounds;
  }
};

// The rows of a list that a wave takes, for a grid of whole multiples of kDies workgroups of four waves that stays on the chip: a die's
// waves take stretches of consecutive rows, `rounds` rows a wave, and the dies take the stretches in turn.  Neighbouring rows mostly want
// the same rows of B, which then come into one die's L2 cache instead of all of them (27-point stencil of 128^3 rows, numeric phase: 6.7 -> 3.6
// GB read from behind the caches); the stretches are short enough that a list that begins with its heaviest rows is shared out evenly.
constexpr unsigned kDies = 8;   // (workgroups are dealt to the dies in turn)
struct DieRows {
  unsigned waves, rounds, first, count;   // count: rows of this wave
  __device__ __forceinline__ DieRows(unsigned wg, unsigned wgs, int wave, unsigned nrows) {
    waves = wgs / kDies * 4;
    rounds = nrows / (waves * kDies * 8);
    rounds = rounds < 1 ? 1 : (rounds < 32 ? rounds : 32);
    first = wg % kDies * waves * rounds + wg / kDies * 4 + wave;
    const unsigned all = waves * rounds * kDies, left = nrows % all;
    const unsigned more = left > first ? (left - first + waves - 1) / waves : 0;
    count = nrows / all * rounds + (more < rounds ? more : rounds);
  }
  __device__ __forceinline__ unsigned at(unsigned t) const { return first + t / rounds * (waves * rounds * kDies) + t % rounds * waves; }   // the wave's t-th row
};

// What is known of a wave's rows, 64 of them at a time, row t in lane t mod 64 (Row: its numbers): the loads that lead to it are paid once
// for 32 rows, and they are loads of the vector kind: scalar ones are waited for together with LDS, in no order.
template <class Row>
struct RowRing {
  Row rows;
  unsigned t;   // the row in the works
  template <class Load>   // load(t): what is known of the wave's row t
  __device__ __forceinline__ void start(Load load) { t = 0; rows = load((unsigned)lane_id()); }
  template <class Load>
  __device__ __forceinline__ void step(Load load) {
    ++t;
    if ((t & (kWave / 2 - 1)) == 0) {   // (the rows of half of the lanes are done)
      const unsigned mine = (unsigned)lane_id();
      if (((mine ^ t) & (kWave / 2)) != 0) rows = load((t & ~(unsigned)(kWave - 1)) + kWave + mine - ((t & (kWave / 2)) ? 0 : kWave));
    }
  }
  template <class F>   // a number of the row `ahead` rows behind the one in the works (at most 31)
  __device__ __forceinline__ int get(int ahead, F number) const { return __builtin_amdgcn_readlane(number(rows), (int)((t + ahead) & (kWave - 1))); }
  template <class F>
  __device__ __forceinline__ int64_t get64(int ahead, F number) const {
    const unsigned lo = (unsigned)get(ahead, [&](const Row& r) { return (int)(unsigned)(unsigned long long)number(r); });
    const unsigned hi = (unsigned)get(ahead, [&](const Row& r) { return (int)(unsigned)((unsigned long long)number(r) >> 32); });
    return (int64_t)(((unsigned long long)hi << 32) | lo);
  }
};

}  // namespace spg
