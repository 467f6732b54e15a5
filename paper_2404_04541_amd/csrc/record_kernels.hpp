// Short rows of the hash class (at most kSymHashSmall products), one wave per row, and the record that the symbolic pass
// leaves of them for the numeric pass.
//
// Products are taken four at a time: a "quad" is up to four consecutive entries of one B row, so the search for the A entry,
// the address arithmetic and the load are paid once per quad instead of once per product.
//
// Symbolic: an LDS hash set of the columns.  A new column gets the next free number of the row; when the row has at most
//   kNumHashSmall of them, the (column, number) words are sorted in registers and the row's record is written:
//   one byte per product (the rank of its column in the row, in quad order) and the columns in ascending order.
// Numeric: with the record a product is one byte, one multiplication and one addition at its rank; nothing is hashed,
//   searched or sorted again.  Rows without a record take the hash workspace.
// The record costs one byte per product and four per entry, written and read once; finding the ranks again costs a
// compare-and-swap loop per product (the slowest of 64 lanes decides) and a sort per row.
// Bounds: the symbolic kernel issues about 600 vector instructions per row (insertion 300, sort and ranks 160; vector units 0.6, LDS
// 0.66 of the cycles on the stencil below); the numeric one is bound by memory: 9.9 GB between L2 and memory in 2.2 ms, 4.5 TB/s of
// the 4.7 that a large copy reaches (records 3.2, C 3.1, A 0.7 GB, the rest B's values, which every die fetches for itself), with LDS
// active for half of the cycles.
// 27-point stencil of 128^3 rows, fp64 (729 products and 125 entries per row): hash workspace 2.39 + 4.80 ms, here 3.13 + 2.22 ms;
// of 61^3 rows, numeric phase on a kept plan: 480 -> 255 us.
#pragma once
#include "common.hpp"
#include "entry_order.hpp"
#include "row_chain.hpp"

namespace spg {

constexpr int kQuadEntries = 64;                               // A entries of a recorded row: a lane each
constexpr int kQuadRounds = 4;
static_assert(kSymHashSmall / 4 + kQuadEntries * 3 / 4 <= kQuadRounds * kWave, "the quads of 64 entries of a row fit four rounds of a wave");
constexpr int kRecRankWords = kQuadRounds * kWave;
constexpr int kRecWords = kRecRankWords + kNumHashSmall;       // 32-bit words of a record: ranks by quad, then columns
constexpr int kRecColBits = 23;                                // a column and its number (8 bits) share 31 bits
static_assert(kNumHashSmall <= 256, "a rank fits a byte");
static_assert(kRecWords % 4 == 0 && kRecRankWords % 4 == 0, "records and their column lists start on 16 bytes");
constexpr int kSymLogSlots = 10;
constexpr int kSymSlots = 1 << kSymLogSlots;
constexpr int kNumQuads = 2;                                   // quads in flight per lane (numeric)

struct __align__(16) QuadEntry { int first, len; int64_t bs; };   // first quad of an A entry, its products, the start of its B row

// The entry that quad q belongs to (q below the number of quads): with B rows of similar length it sits where the quad's
// share of all quads points, or next to it; otherwise it is bisected.  Returns its position.
__device__ __forceinline__ int find_quad(const QuadEntry* ent, int q, float per_quad, QuadEntry& en) {
  int lo = (int)((float)q * per_quad);
  lo = lo < kQuadEntries - 1 ? lo : kQuadEntries - 1;
  en = ent[lo];
  if (en.first > q) en = ent[--lo];
  else if (en.first + ((en.len + 3) >> 2) <= q && lo < kQuadEntries - 1) en = ent[++lo];
  if (en.first > q || en.first + ((en.len + 3) >> 2) <= q) {
    int hi = kQuadEntries;
    lo = 0;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (ent[mid].first <= q) lo = mid; else hi = mid;
    }
    en = ent[lo];
  }
  return lo;
}


// The quads of the entries that the wave's lanes hold (len products from bs on each), described in LDS: at most kQuadRounds * 64.
struct QuadMap {
  int nq;           // quads
  float per_quad;   // entries per quad
};

// extra(): called by every lane between the barriers, for what else it leaves in LDS.
template <class F>
__device__ __forceinline__ QuadMap quad_map(int64_t bs, int len, int nent, QuadEntry* ent, F extra) {
  QuadMap m;
  const int quads = (len + 3) >> 2;
  const int incl = wave_incl_scan(quads);
  m.nq = __builtin_amdgcn_readlane(incl, kWave - 1);
  m.nq = m.nq < kQuadRounds * kWave ? m.nq : kQuadRounds * kWave;
  wave_sync_lds();   // (the entries of the pass before have been read)
  ent[lane_id()] = QuadEntry{incl - quads, len, bs};
  extra();
  wave_sync_lds();
  m.per_quad = m.nq > 0 ? (float)nent / (float)m.nq : 0.0f;
  return m;
}

// Quad q of the map (below nq): the position of its entry, the products left in the entry from the quad on, and where they are.
__device__ __forceinline__ int quad_entry(const QuadMap& m, int q, const QuadEntry* ent, int& left, int64_t& at) {
  QuadEntry en;
  const int pos = find_quad(ent, q, m.per_quad, en);
  const int off = (q - en.first) * 4;
  left = en.len - off;
  at = en.bs + off;
  return pos;
}

// Home slot of a column (24-bit multiplication: a 32-bit one takes four issue slots).
__device__ __forceinline__ unsigned set_home(int col) {
  return (__umul24((unsigned)col ^ ((unsigned)col >> 20), 0x9E3779u) >> (32 - kSymLogSlots)) & (kSymSlots - 1);
}

__global__ __launch_bounds__(256) void k_sym_wave(const int* __restrict__ perm, Control* __restrict__ ctl, int bin,
                                                  const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                                  const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col, int64_t b_nnz,
                                                  int* __restrict__ cnt, unsigned* __restrict__ records, unsigned record_rows,
                                                  int* __restrict__ record_of) {
  __shared__ __align__(16) int s_table[4][kSymSlots];
  __shared__ QuadEntry s_ent[4][kQuadEntries];
  __shared__ unsigned short s_slot[4][kNumHashSmall];   // slot of the column with a number
  if (ctl->error) return;
  const unsigned first = ctl->offset[0][bin];
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  int* table = s_table[g];
  QuadEntry* ent = s_ent[g];
  unsigned* words = reinterpret_cast<unsigned*>(s_ent[g]);   // (column, number) by number, once the entries are no longer needed
  static_assert(sizeof(QuadEntry) * kQuadEntries >= kNumHashSmall * sizeof(unsigned), "the words fit the entries' space");
  unsigned short* slot_of = s_slot[g];
  unsigned kept = 0;
  RowChain<kWave> ch{perm + first, a_rp, a_col, b_rp, nullptr, nrows, gridDim.x * 4};
  unsigned row_at = blockIdx.x * 4 + g;
  ch.start(row_at);
  for (; row_at < nrows; row_at += gridDim.x * 4) {
    const int row = ch.row, d = ch.d;
    const RowChain<kWave>::Ahead nx = ch.fetch();
    {
      int4* t4 = reinterpret_cast<int4*>(table);
#pragma unroll
      for (int t = 0; t < kSymSlots / 4 / kWave; ++t) t4[t * kWave + lane] = make_int4(kEmptyKey, kEmptyKey, kEmptyKey, kEmptyKey);
    }
    const bool want = row_at < record_rows && d <= kQuadEntries;
    int found = 0;                                 // (wave-uniform) distinct columns so far
    unsigned slots[kQuadRounds][2] = {};           // of a recorded row's products, two to a word
    int nq_row = 0;
    for (int base = 0; base < d; base += kQuadEntries) {
      if (base > 0) ch.fetch_more(base);
      const QuadMap map = quad_map(ch.bounds.v[0], (int)(ch.bounds.v[1] - ch.bounds.v[0]), d - base < kQuadEntries ? d - base : kQuadEntries, ent, [] {});
      nq_row = map.nq;
      int col[kQuadRounds][4];
      int n_of[kQuadRounds];
#pragma unroll
      for (int r = 0; r < kQuadRounds; ++r) {
        n_of[r] = 0;
        if (r * kWave < map.nq) {
          int64_t p = 0;
          if (r * kWave + lane < map.nq) (void)quad_entry(map, r * kWave + lane, ent, n_of[r], p);
          load_quad<int32_t>(b_col, p, n_of[r], b_nnz, col[r]);
        }
      }
      wave_sync_lds();   // (the entries have been read: a recorded row's words take their place)
#pragma unroll
      for (int r = 0; r < kQuadRounds; ++r) {
        if (r * kWave >= map.nq) break;
        unsigned slot[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          slot[u] = set_home(col[r][u]);
          bool is_new = false;
          if (u < n_of[r]) {
            while (true) {
              const int old = atomicCAS(&table[slot[u]], kEmptyKey, col[r][u]);
              if (old == kEmptyKey) { is_new = true; break; }
              if (old == col[r][u]) break;
              slot[u] = (slot[u] + 1) & (kSymSlots - 1);
            }
          }
          const unsigned long long fresh = __ballot(is_new);
          if (fresh) {
            const int at = found + lanes_below(fresh);
            if (want && is_new && at < kNumHashSmall) {
              words[at] = ((unsigned)col[r][u] << 8) | (unsigned)at;
              slot_of[at] = (unsigned short)slot[u];
            }
            found += __popcll(fresh);
          }
        }
        slots[r][0] = slot[0] | (slot[1] << 16);
        slots[r][1] = slot[2] | (slot[3] << 16);
      }
    }
    const bool keep = want && found <= kNumHashSmall;
    if (lane == 0) {
      cnt[row] = found;
      if (record_of) record_of[row] = keep ? (int)row_at : -1;
    }
    if (keep) {
      ++kept;
      unsigned* rec = records + (size_t)row_at * kRecWords;
      wave_sync_lds();
      auto ranks = [&](auto per_lane) {
        constexpr int kPer = decltype(per_lane)::value;
        unsigned key[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) key[i] = lane * kPer + i < found ? words[lane * kPer + i] : 0xffffffffu;
        lane_sort<kPer * kWave, kPer>(key, lane);
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          if (lane * kPer + i < found) {
            table[slot_of[key[i] & 255u]] = lane * kPer + i;   // the set's slot now holds the rank of its column
            key[i] >>= 8;
          }
        if (lane * kPer < found) {   // (a record has room for whole groups of kPer columns)
          Run<unsigned, kPer> out;
#pragma unroll
          for (int i = 0; i < kPer; ++i) out.v[i] = key[i];
          *reinterpret_cast<Run<unsigned, kPer>*>(rec + kRecRankWords + lane * kPer) = out;
        }
      };
      if (found <= 2 * kWave) ranks(std::integral_constant<int, 2>{});
      else ranks(std::integral_constant<int, 4>{});
      wave_sync_lds();
#pragma unroll
      for (int r = 0; r < kQuadRounds; ++r) {
        const int q = r * kWave + lane;
        if (q < nq_row) {
          unsigned w = 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned slot = (u & 1) ? slots[r][u >> 1] >> 16 : slots[r][u >> 1] & 0xffffu;
            w |= ((unsigned)table[slot] & 255u) << (8 * u);
          }
          rec[q] = w;
        }
      }
    }
    wave_sync_lds();
    ch.advance(nx);
  }
  if (lane == 0 && kept) atomicAdd(&ctl->recorded, kept);
}

// Numeric pass over the recorded rows of a bin, a wave per row; rows without a record are left to the hash workspace.
// SUM: the first order.parts workgroups look at the order of the entries (order_later) while the others do the rows.
template <typename T, bool SUM>
__global__ __launch_bounds__(256) void k_num_recorded(const int* __restrict__ perm, std::conditional_t<SUM, Control, const Control>* __restrict__ ctl, int bin, const int* __restrict__ ip_row,
                                                      const unsigned* __restrict__ records, const int* __restrict__ record_of,
                                                      const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const T* __restrict__ a_val,
                                                      const int64_t* __restrict__ b_rp, const T* __restrict__ b_val, int64_t b_nnz,
                                                      const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val, const OrderOperands order) {
  __shared__ double s_acc[4][256];   // (a rank is a byte)
  __shared__ QuadEntry s_ent[4][kQuadEntries];
  __shared__ T s_av[4][kQuadEntries];
  if (ctl->error || (!SUM && ctl->order_differs)) return;
  unsigned wg = blockIdx.x, wgs = gridDim.x;
  if constexpr (SUM) {
    if ((int)wg < order.parts) {
      order_add<256>(order_share<256>(order.na, order.a_col, order.nb, order.b_col, wg, order.parts), order.parts, ctl, 0, &ctl->order_later);
      return;
    }
    wg -= order.parts;
    wgs -= order.parts;
  }
  const unsigned first = ctl->offset[1][bin];
  const unsigned nrows = ctl->offset[1][bin + 1] - first;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  double* acc = s_acc[g];
  QuadEntry* ent = s_ent[g];
  T* s_a = s_av[g];
  auto record = [&](int row) { return row >= 0 && ip_row[row] <= kSymHashSmall ? record_of[row] : -1; };
  auto range = [&](int row, int64_t& lo, int& n) {
    lo = 0; n = 0;
    // (a recorded row has no more entries than that, whatever room the row pointer leaves behind them)
    if (row >= 0) { const Run<int64_t, 2> v = load_run<int64_t, 2>(c_rp + row); lo = v.v[0]; n = v.v[1] - v.v[0] < kNumHashSmall ? (int)(v.v[1] - v.v[0]) : kNumHashSmall; }
  };
  auto value = [&](int64_t a, int n) { return lane < n ? a_val[a + lane] : T(0); };
  RowChain<kWave> ch{perm + first, a_rp, a_col, b_rp, nullptr, nrows, wgs * 4};
  unsigned row_at = wg * 4 + g;
  ch.start(row_at);
  int at0 = record(ch.row), at1 = record(ch.row1), at2 = record(ch.row2);
  int64_t out0, out1, out2;
  int n0, n1, n2;
  range(ch.row, out0, n0);
  range(ch.row1, out1, n1);
  range(ch.row2, out2, n2);
  T av0 = value(ch.a0, ch.d), av1 = value(ch.a01, ch.d1);
  for (; row_at < nrows; row_at += wgs * 4) {
    const RowChain<kWave>::Ahead nx = ch.fetch();
    int64_t out3;
    int n3;
    const T av2 = value(ch.a02, ch.d2);
    range(ch.row3, out3, n3);
    const int at3 = record(ch.row3);
    if (at0 >= 0) {
      const unsigned* rec = records + (size_t)at0 * kRecWords;
      for (int t = lane; t < n0; t += kWave) acc[t] = 0.0;
      // (operands of another structure than the plan's read no further than the record)
      const QuadMap map = quad_map(ch.bounds.v[0], (int)(ch.bounds.v[1] - ch.bounds.v[0]), ch.d, ent, [&] { s_a[lane] = av0; });
#pragma unroll
      for (int r0 = 0; r0 < kQuadRounds; r0 += kNumQuads) {
        if (r0 * kWave >= map.nq) break;
        T b[kNumQuads][4];
        unsigned w[kNumQuads];
        int left[kNumQuads];
        double a[kNumQuads];
#pragma unroll
        for (int i = 0; i < kNumQuads; ++i) {
          const int q = (r0 + i) * kWave + lane;
          left[i] = 0;
          w[i] = 0;
          a[i] = 0.0;
          int64_t p = 0;
          if (q < map.nq) {
            w[i] = rec[q];
            const int at = quad_entry(map, q, ent, left[i], p);
            a[i] = (double)s_a[at];
          }
          load_quad<T>(b_val, p, left[i], b_nnz, b[i]);
        }
#pragma unroll
        for (int i = 0; i < kNumQuads; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (u < left[i])
              __hip_atomic_fetch_add(&acc[(w[i] >> (8 * u)) & 255u], a[i] * (double)b[i][u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      wave_sync_lds();
      for (int t = lane; t < n0; t += kWave) {
        c_col[out0 + t] = (int32_t)rec[kRecRankWords + t];
        c_val[out0 + t] = (T)acc[t];
      }
      wave_sync_lds();
    }
    ch.advance(nx);
    out0 = out1; out1 = out2; out2 = out3;
    n0 = n1; n1 = n2; n2 = n3;
    at0 = at1; at1 = at2; at2 = at3;
    av0 = av1; av1 = av2;
  }
}

}  // namespace spg
