// Short rows of the hash class (at most kSymHashSmall products), one wave per row, and the record that the symbolic pass
// leaves of them for the numeric pass.
//
// Products are taken four at a time: a "quad" is up to four consecutive entries of one B row, so the search for the A entry,
// the address arithmetic and the load are paid once per quad instead of once per product.
//
// Symbolic: an LDS hash set of the columns.  A new column gets the next free number of the row; when the row has at most
//   kNumHashSmall of them, the (column, number) words are sorted in registers and the row's record is written:
//   one byte per product (the rank of its column in the row, in quad order) and the columns in ascending order.
//   Rows of discretised operators are mostly the same row moved to other columns.  A wave keeps a row as its model; a later row with as many
//   entries and as many products of each has its columns compared with the model's, and where all differ by the same shift nothing is
//   inserted, sorted or written: the row takes the model's record and the shift.  (Where the row count has seen that rows are mostly like the ones
//   before them; otherwise the model's registers cost a fifth of the waves.)
// Numeric: with the record a product is one byte, one multiplication and one addition at its rank; nothing is hashed,
//   searched or sorted again.  The record stays in registers as long as the wave's rows have the same one.  Rows without a record take the
//   hash workspace.
// The record costs one byte per product and four per entry, written and read once; finding the ranks again costs a
// compare-and-swap loop per product (the slowest of 64 lanes decides) and a sort per row.
// Bounds: the symbolic kernel issues about 600 vector instructions for a row by itself (insertion 300, sort and ranks 160) and 140 for one
// that is the model moved; the numeric one adds 729 products a row in 250 LDS cycles of 500 (without the stores 1.35 of 2.02 ms, without
// additions 1.95): what it waits for is memory, C's 3.1 GB written and 2.7 GB of A and B read.
// 27-point stencil of 128^3 rows, fp64 (729 products and 125 entries per row), every row by itself | with models: symbolic 3.08 | 1.12 ms,
// numeric 2.20 | 2.02 ms; of 61^3 rows 463 | 212 us and 255 | 190 us.  (Hash workspace: 2.39 + 4.80 ms.)  Of that, rows dealt to all dies in turn |
// neighbouring ones to one die: symbolic 1.45 | 1.12 ms, numeric 2.14 | 2.02; stores through the caches | past them: numeric 2.32 | 2.02 ms, 61^3
// 244 | 190 us.
// Measured and not kept in the numeric kernel: the next row's values asked for before this one's stores, with the loads free of conditions
// (2.08 ms: 142 registers); two products a load (2.08); 24 or 32 waves on a compute unit (2.36, 2.40).
#pragma once
#include "common.hpp"
#include "entry_order.hpp"
#include "quad_reads.hpp"
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
constexpr int kRecordGroups = 4;                               // workgroups of these kernels on a compute unit
// Slots of the set: 2048, 2.7 times the most products (with 1024 the slowest lane of an insertion walked over twenty taken ones and more, and a row of
// 768 products took 35 us: whole calls, us with 1024 | 2048: ragged 5003 rows 236 | 216, R-MAT squared scale 12 210 | 201, 14 444 | 432).  That is
// 38 KB a workgroup, four of which fit a compute unit, where rows of few products would rather have more: with 1024 (22 KB) they do.  So 1024 where rows
// differ and the class's have kFewProducts or fewer on average and no more than one of kFewLongShare has more than kLongProducts (any row is still
// right).  300 000 rows, this kernel, us with 1024 | 2048: 144 products a row 354 | 390, 196 265 | 272, 240 288 | 282, 256 293 | 285, 324 554 |
// 476, 400 648 | 512, 576 1412 | 831, 756 2362 | 986; 2 M rows of 130 products 1831 | 2130.  200 000 rows of 143, whole calls, one of 50 of 767 704 | 650, of
// 400 633 | 592, of 1000 574 | 568, of 4000 562 | 563; one of 20 of 390 627 | 636, one of four (205 on average)
// 947 | 932.  Where the classes of shorter rows share a launch, which the slowest row
// ends, not a single one may be long: 60 000 rows 234 | 241, 40 000 189 | 194, 20 000 153 | 154, with one of 4000 of 767 40 000 223 | 210.
// (The number of slots by the row, in the LDS of 2048, gains nothing: what counts is the fifth workgroup.)
constexpr int kSymLogSlots = 11, kFewLogSlots = 10;
constexpr int kFewGroups = 5;
constexpr int64_t kFewProducts = 200;
constexpr unsigned kFewLongShare = 4096;
// sums of a row in LDS (a rank is a byte), and a place for every lane's missing products
constexpr int kRecSums = 256 + kWave;
static_assert(4 * kRecSums * 8 <= 65536, "a sum's place in the workgroup's LDS fits 16 bits");

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

__device__ __forceinline__ QuadMap quad_map(int64_t bs, int len, int nent, QuadEntry* ent) {
  QuadMap m;
  const int quads = (len + 3) >> 2;
  const int incl = wave_incl_scan(quads);
  m.nq = __builtin_amdgcn_readlane(incl, kWave - 1);
  m.nq = m.nq < kQuadRounds * kWave ? m.nq : kQuadRounds * kWave;
  wave_sync_lds();   // (the entries of the pass before have been read)
  ent[lane_id()] = QuadEntry{incl - quads, len, bs};
  wave_sync_lds();
  m.per_quad = m.nq > 0 ? (float)nent / (float)m.nq : 0.0f;
  return m;
}

// Home slot of a column (24-bit multiplication: a 32-bit one takes four issue slots).
template <int LOG_SLOTS>
__device__ __forceinline__ unsigned set_home(int col) {
  return (__umul24((unsigned)col ^ ((unsigned)col >> 20), 0x9E3779u) >> (32 - LOG_SLOTS)) & ((1 << LOG_SLOTS) - 1);
}

struct NumRow {   // record (-1: no row, -2: none), how far its columns are from the row's, entries of A, entries of C
  int record = -1, shift = 0, d = 0, n = 0;
  int64_t a0 = 0, out = 0;
  __device__ __forceinline__ bool there() const { return record != -1; }
};
struct SymRow {   // a row, its entries of A (none: row < 0)
  int row = -1, d = 0;
  int64_t a0 = 0;
  __device__ __forceinline__ bool there() const { return row >= 0; }
};
constexpr int kAlikeTries = 8;   // rows that only look alike a wave compares in vain before it stops

template <int LOG_SLOTS>
struct SymWaveLds {
  __align__(16) int table[4][1 << LOG_SLOTS];
  QuadEntry ent[4][kQuadEntries];
  unsigned short slot[4][kNumHashSmall];   // slot of the column with a number
  unsigned kept, done;                     // rows with a record, waves that have no more rows
};
static_assert(kRecordGroups * sizeof(SymWaveLds<kSymLogSlots>) <= 160 * 1024 && kFewGroups * sizeof(SymWaveLds<kFewLogSlots>) <= 160 * 1024, "workgroups on a compute unit");

template <bool ALIKE, int LOG_SLOTS>
__device__ __forceinline__ void sym_wave_rows(SymWaveLds<LOG_SLOTS>* lds, unsigned wg, unsigned wgs, const int* __restrict__ perm, Control* __restrict__ ctl,
    int bin, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const int64_t* __restrict__ b_rp,
    const int32_t* __restrict__ b_col, int64_t b_nnz, int* __restrict__ cnt, unsigned* __restrict__ records, unsigned record_rows,
    int* __restrict__ record_of, int* __restrict__ shift_of) {
  constexpr int kSlots = 1 << LOG_SLOTS;
  if (threadIdx.x == 0) { lds->kept = 0; lds->done = 0; }
  __syncthreads();
  const unsigned first = ctl->offset[0][bin];
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  int* table = lds->table[g];
  QuadEntry* ent = lds->ent[g];
  unsigned* words = reinterpret_cast<unsigned*>(lds->ent[g]);   // (column, number) by number, once the entries are no longer needed
  static_assert(sizeof(QuadEntry) * kQuadEntries >= kNumHashSmall * sizeof(unsigned), "the words fit the entries' space");
  unsigned short* slot_of = lds->slot[g];
  unsigned kept = 0;
  // The model: the row that later ones are compared with.  Its entries and their products (d < 0: there is none), where its quads
  // come from and their columns, what became of it, and how the comparisons with it went.
  int m_d = -1, m_len = 0, m_nq = 0, m_found = 0, m_rec = -1, m_hits = 0, m_missed = 0, vain = 0;
  unsigned m_quad[kQuadRounds] = {};
  int m_col[kQuadRounds][4] = {};
  const DieRows order(wg, wgs, g, nrows);
  // One atomic a workgroup that has kept rows: they come from all workgroups to one counter, about 12 ns each (one a wave: 300 000 rows of 256
  // products 470 us, of which the rows are 250).
  auto finish = [&] {
    if (lane != 0) return;
    if (kept) atomicAdd(&lds->kept, kept);
    // (the last one sees what all have added)
    if (__hip_atomic_fetch_add(&lds->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) != 3) return;
    const unsigned all = __hip_atomic_load(&lds->kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (all) atomicAdd(&ctl->recorded, all);
  };
  if (order.count == 0) {   // (the wave)
    finish();
    return;
  }
  auto load = [&](unsigned t) {
    SymRow r;
    const unsigned at = order.at(t);
    if (at < nrows) {
      r.row = perm[first + at];
      const Run<int64_t, 2> v = load_run<int64_t, 2>(a_rp + r.row);
      r.a0 = v.v[0];
      r.d = (int)(v.v[1] - v.v[0]);
    }
    return r;
  };
  RowRing<SymRow> rows;
  rows.start(load);
  auto entries = [&](int ahead) { return rows.get(ahead, [](const SymRow& r) { return r.d; }); };
  // The loads of the rows to come have no conditions (lanes without an entry load the row's first), so that it is known how many are on
  // their way when one is waited for: loads and stores return in order, and a wait that does not know what is behind waits for everything.
  auto place = [&](int ahead) { return rows.get64(ahead, [](const SymRow& r) { return r.a0; }) + (lane < entries(ahead) ? lane : 0); };
  auto bounds_of = [&](int k) { return load_run<int64_t, 2>(b_rp + k); };
  int col[kQuadRounds][4];
  unsigned quad[kQuadRounds];
  const int32_t* const from = b_nnz >= 4 ? b_col : reinterpret_cast<const int32_t*>(ctl);
  const int64_t last = b_nnz >= 4 ? b_nnz - 4 : 0;
  int k2 = a_col[place(0)];
  const int k1 = a_col[place(1)];
  Run<int64_t, 2> bounds1 = bounds_of(k2);
  k2 = k1;
  int64_t bs = 0;         // of the row in the works: where the lane's entry's products begin, and how many there are
  int len = 0;
  bool compare = false;   // it has as many entries as the model, and they as many products: its quads are the model's, its columns are on their way
  auto begin = [&] {
    const int d = entries(0);
    bs = bounds1.v[0];
    len = lane < d ? (int)(bounds1.v[1] - bs) : 0;
    if constexpr (ALIKE) {
    // (a quad that reaches behind the end of B is loaded further in front: such a row is not compared)
    compare = d == m_d && vain < kAlikeTries && !__any(len != m_len || (len > 0 && bs + len + 3 > b_nnz));
    wave_sync_lds();
    ent[lane].bs = bs;
    wave_sync_lds();
    auto fetch = [&](int r) {
      const int64_t p = ent[quad_src(m_quad[r])].bs + quad_off(m_quad[r]);
      const Run<int32_t, 4> v = load_run<int32_t, 4>(from + (p < last ? p : last));
#pragma unroll
      for (int u = 0; u < 4; ++u) col[r][u] = v.v[u];
    };
    static_assert(kQuadRounds == 4, "two rounds that rows may not have, two that are loaded always");
    if (m_nq > 3 * kWave) fetch(3);
    if (m_nq > 2 * kWave) fetch(2);
    fetch(1);
    fetch(0);
    wave_sync_lds();
    }
    bounds1 = bounds_of(k2);
    k2 = a_col[place(2)];
  };
  begin();
  while (rows.t < order.count) {
    const unsigned row_at = order.at(rows.t);
    const int row = rows.get(0, [](const SymRow& r) { return r.row; }), d = entries(0);
    const bool want = row_at < record_rows && d <= kQuadEntries;
    int found = 0;                                 // (wave-uniform) distinct columns so far
    int in_record = -1, shift = 0;
    unsigned slots[kQuadRounds][2] = {};           // of a recorded row's products, two to a word
    int nq_row = 0;
    bool alike = false;
    if (ALIKE && compare) {   // is the row the model moved to other columns?
      shift = __builtin_amdgcn_readfirstlane(col[0][0]) - __builtin_amdgcn_readfirstlane(m_col[0][0]);
      bool other = false;
#pragma unroll
      for (int r = 0; r < kQuadRounds; ++r)
        if (r * kWave < m_nq) {
#pragma unroll
          for (int u = 0; u < 4; ++u) other = other || (u < quad_count(m_quad[r]) && col[r][u] - m_col[r][u] != shift);
        }
      alike = !__any(other);
      if (alike) {
        ++m_hits;
        m_missed = 0;
        found = m_found;
        in_record = m_rec;
      } else {
        shift = 0;
        if (m_hits == 0) ++vain;
      }
    }
    for (int base = 0; base < d && !alike; base += kQuadEntries) {
      int nq = m_nq;
      if (!ALIKE || base > 0 || !compare) {
        int64_t from_here = bs;
        int n_here = len;
        if (base > 0) {
          const int64_t a0 = rows.get64(0, [](const SymRow& r) { return r.a0; });
          Run<int64_t, 2> v;
          v.v[0] = 0; v.v[1] = 0;
          if (base + lane < d) v = bounds_of(a_col[a0 + base + lane]);
          from_here = v.v[0];
          n_here = (int)(v.v[1] - v.v[0]);
        }
        const QuadMap map = quad_map(from_here, n_here, d - base < kQuadEntries ? d - base : kQuadEntries, ent);
        nq = map.nq;
#pragma unroll
        for (int r = 0; r < kQuadRounds; ++r) {
          quad[r] = 0;
          if (r * kWave < nq) {
            int64_t p = 0;
            if (r * kWave + lane < nq) {
              QuadEntry en;
              const int q = r * kWave + lane, src = find_quad(ent, q, map.per_quad, en), off = (q - en.first) * 4;
              quad[r] = pack_quad(src, en.len - off, off);
              p = en.bs + off;
            }
            load_quad<int32_t>(b_col, p, quad_count(quad[r]), b_nnz, col[r]);
          }
        }
        wave_sync_lds();   // (the entries have been read: a recorded row's words take their place)
      } else {
#pragma unroll
        for (int r = 0; r < kQuadRounds; ++r) quad[r] = m_quad[r];
      }
      nq_row = nq;
      if (base == 0) {
        int4* t4 = reinterpret_cast<int4*>(table);
#pragma unroll
        for (int t = 0; t < kSlots / 4 / kWave; ++t) t4[t * kWave + lane] = make_int4(kEmptyKey, kEmptyKey, kEmptyKey, kEmptyKey);
        wave_sync_lds();
        if (ALIKE && d <= kQuadEntries && (m_hits == 0 || ++m_missed > 1)) {   // (one row at an edge leaves the model what it is)
          m_d = d; m_len = len; m_nq = nq; m_hits = 0; m_missed = 0;
#pragma unroll
          for (int r = 0; r < kQuadRounds; ++r) {
            m_quad[r] = quad[r];
#pragma unroll
            for (int u = 0; u < 4; ++u) m_col[r][u] = col[r][u];
          }
          m_rec = -2;
        }
      }
#pragma unroll
      for (int r = 0; r < kQuadRounds; ++r) {
        if (r * kWave >= nq) break;
        unsigned slot[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          slot[u] = set_home<LOG_SLOTS>(col[r][u]);
          bool is_new = false;
          if (u < quad_count(quad[r])) {
            while (true) {
              const int old = atomicCAS(&table[slot[u]], kEmptyKey, col[r][u]);
              if (old == kEmptyKey) { is_new = true; break; }
              if (old == col[r][u]) break;
              slot[u] = (slot[u] + 1) & (kSlots - 1);
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
    const bool keep = !alike && want && found <= kNumHashSmall;
    if (keep) in_record = (int)row_at;
    if (ALIKE && m_rec == -2) {   // the row is the model
      m_found = found;
      m_rec = in_record;
    }
    if (in_record >= 0) ++kept;
    if (keep) {
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
    rows.step(load);
    begin();
    // (behind the loads of the rows to come, which are waited for in order with the stores)
    if (lane == 0) {
      cnt[row] = found;
      if (record_of) record_of[row] = in_record;
      if (ALIKE && shift_of) shift_of[row] = shift;
    }
  }
  finish();
}

// ALIKE: rows are compared with a model.  (Bounds: as many workgroups as LDS holds.)
template <bool ALIKE, int LOG_SLOTS>
__global__ __launch_bounds__(256, LOG_SLOTS == kSymLogSlots ? kRecordGroups : kFewGroups) void k_sym_wave(const int* __restrict__ perm, Control* __restrict__ ctl, int bin,
                                                  const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                                  const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col, int64_t b_nnz,
                                                  int* __restrict__ cnt, unsigned* __restrict__ records, unsigned record_rows,
                                                  int* __restrict__ record_of, int* __restrict__ shift_of) {
  __shared__ SymWaveLds<LOG_SLOTS> lds;
  if (ctl->error) return;
  sym_wave_rows<ALIKE, LOG_SLOTS>(&lds, blockIdx.x, gridDim.x, perm, ctl, bin, a_rp, a_col, b_rp, b_col, b_nnz, cnt, records, record_rows, record_of, shift_of);
}

// Numeric pass over the recorded rows of a bin, a wave per row; rows without a record are left to the hash workspace.
template <typename T>
struct NumRecordedLds {
  double acc[4][kRecSums];
  QuadEntry ent[4][kQuadEntries];
  T av[4][kQuadEntries];
};

// ALIKE: neighbouring rows of a wave have the same record; otherwise fewer registers (two quads in flight a lane) and more waves are worth more.
template <bool ALIKE, typename T>
__device__ __forceinline__ void num_recorded_rows(NumRecordedLds<T>* lds, unsigned wg, unsigned wgs, const int* __restrict__ perm,
    const Control* __restrict__ ctl, int bin, const unsigned* __restrict__ records, const int* __restrict__ record_of,
    const int* __restrict__ shift_of, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const T* __restrict__ a_val,
    const int64_t* __restrict__ b_rp, const T* __restrict__ b_val, int64_t b_nnz, const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col,
    T* __restrict__ c_val) {
  const unsigned first = ctl->offset[0][bin];   // (the order of the symbolic kernel: a wave meets the rows of a record one after the other)
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  double* acc = lds->acc[g];
  QuadEntry* ent = lds->ent[g];
  T* s_a = lds->av[g];
  const DieRows in_order(wg, wgs, g, nrows);
  auto load = [&](unsigned t) {
    NumRow r;
    const unsigned at = in_order.at(t);
    if (at < nrows) {
      const int row = perm[first + at];
      const int of = record_of[row];
      const Run<int64_t, 2> a = load_run<int64_t, 2>(a_rp + row), c = load_run<int64_t, 2>(c_rp + row);
      r.record = of >= 0 ? of : -2;
      if (ALIKE) r.shift = shift_of ? shift_of[row] : 0;
      r.a0 = a.v[0];
      r.d = (int)(a.v[1] - a.v[0]);
      r.out = c.v[0];
      // (a recorded row has no more entries than that, whatever room the row pointer leaves behind them)
      r.n = c.v[1] - c.v[0] < kNumHashSmall ? (int)(c.v[1] - c.v[0]) : kNumHashSmall;
    }
    return r;
  };
  if (in_order.count == 0) return;   // (the wave)
  RowRing<NumRow> rows;
  rows.start(load);
  auto record = [&](int ahead) { return rows.get(ahead, [](const NumRow& r) { return r.record; }); };
  auto entries = [&](int ahead) { return rows.get(ahead, [](const NumRow& r) { return r.d; }); };
  // (lanes without an entry load the row's first)
  auto place = [&](int ahead) { return rows.get64(ahead, [](const NumRow& r) { return r.a0; }) + (lane < entries(ahead) ? lane : 0); };
  auto bounds_of = [&](int k) { return load_run<int64_t, 2>(b_rp + k); };
  // The record in registers: which one, of a row with how many entries (and products of this lane's), its quads (the lane of the entry,
  // the place inside it and how many there are), where in LDS their products are added up (two 16-bit offsets a word; what a quad has
  // not goes to a place of its own behind the row's sums) and the columns.
  int h_rec = -1, h_n = 0, h_d = 0, h_len = 0, h_nq = 0, h_col[kNumHashSmall / kWave] = {};
  unsigned h_quad[kQuadRounds] = {}, h_sum[kQuadRounds][2] = {};
  // (the loads that lead to a row's products depend on each other: each is on its way while the rows before are in the works)
  int k1 = a_col[place(0)], k2 = a_col[place(1)];
  Run<int64_t, 2> bounds = bounds_of(k1);
  T av = a_val[place(0)];
  for (; rows.t < in_order.count; rows.step(load)) {
    const int at = record(0), n = rows.get(0, [](const NumRow& r) { return r.n; }), d = entries(0);
    const int64_t bs = bounds.v[0];
    const int len = lane < d ? (int)(bounds.v[1] - bs) : 0;
    if (at >= 0) {
#pragma unroll
      for (int i = 0; i < kNumHashSmall / kWave; ++i)
        if (i * kWave < n) acc[i * kWave + lane] = 0.0;
      // (operands of another structure than the plan's read no further than the record)
      if (at != h_rec || n != h_n || d != h_d || __any(len != h_len)) {
        const unsigned* rec = records + (size_t)at * kRecWords;
        const QuadMap map = quad_map(bs, len, d, ent);
        h_rec = at; h_n = n; h_d = d; h_len = len; h_nq = map.nq;
#pragma unroll
        for (int r = 0; r < kQuadRounds; ++r) {
          const int q = r * kWave + lane;
          unsigned rank = 0;
          h_quad[r] = 0;
          if (r * kWave < map.nq && q < map.nq) {
            rank = rec[q];
            QuadEntry en;
            const int src = find_quad(ent, q, map.per_quad, en), off = (q - en.first) * 4;
            h_quad[r] = pack_quad(src, en.len - off, off);
          }
          unsigned to[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned place = u < quad_count(h_quad[r]) ? (rank >> (8 * u)) & 255u : 256u + lane;
            to[u] = g * (unsigned)sizeof(lds->acc[0]) + place * 8u;
          }
          h_sum[r][0] = to[0] | (to[1] << 16);
          h_sum[r][1] = to[2] | (to[3] << 16);
        }
#pragma unroll
        for (int i = 0; i < kNumHashSmall / kWave; ++i) h_col[i] = i * kWave + lane < n ? (int)rec[kRecRankWords + i * kWave + lane] : 0;
      }
      const bool tight = __any(quads_leave(lane, bs, len, b_nnz));   // (a quad might reach behind the end of B)
      wave_sync_lds();
      ent[lane].bs = bs;
      s_a[lane] = av;
      wave_sync_lds();
      constexpr int kAhead = ALIKE ? kQuadRounds : 2;   // quads in flight a lane
#pragma unroll
      for (int r0 = 0; r0 < kQuadRounds; r0 += kAhead) {
        if (r0 * kWave >= h_nq) break;
        T b[kAhead][4];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
          const int r = r0 + i;
          if (r * kWave >= h_nq) break;
          const int64_t p = ent[quad_src(h_quad[r])].bs + quad_off(h_quad[r]);
          if (!tight) {
            const Run<T, 4> v = load_run<T, 4>(b_val + p);
#pragma unroll
            for (int u = 0; u < 4; ++u) b[i][u] = v.v[u];
          } else {
            int n4 = quad_count(h_quad[r]);
            asm volatile("" : "+v"(n4));   // (no code: keeps this first load from being shared with the wide one, which then is three)
#pragma unroll
            for (int u = 0; u < 4; ++u) b[i][u] = u < n4 ? b_val[p + u] : T(0);
          }
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
          const int r = r0 + i;
          if (r * kWave >= h_nq) break;
          const double a = (double)s_a[quad_src(h_quad[r])];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned to = (h_sum[r][u >> 1] >> (16 * (u & 1))) & 0xffffu;
            double* sum = static_cast<double*>(__builtin_assume_aligned(reinterpret_cast<unsigned char*>(lds->acc) + to, 8));
            __hip_atomic_fetch_add(sum, a * (double)b[i][u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      wave_sync_lds();
      const int shift = rows.get(0, [](const NumRow& r) { return r.shift; });
      const int64_t out = rows.get64(0, [](const NumRow& r) { return r.out; });
#pragma unroll
      for (int i = 0; i < kNumHashSmall / kWave; ++i) {
        const int t = i * kWave + lane;
        if (t < n) {
          __builtin_nontemporal_store(h_col[i] + shift, &c_col[out + t]);
          __builtin_nontemporal_store((T)acc[t], &c_val[out + t]);
        }
      }
      wave_sync_lds();
    }
    // a step further for the rows behind
    bounds = bounds_of(k2);
    av = a_val[place(1)];
    k2 = a_col[place(2)];
  }
}

// SUM: the first order.parts workgroups look at the order of the entries (order_later) while the others do the rows.
template <typename T, bool SUM, bool ALIKE>
__global__ __launch_bounds__(256, ALIKE ? kRecordGroups : 8) void k_num_recorded(const int* __restrict__ perm,
                                                      std::conditional_t<SUM, Control, const Control>* __restrict__ ctl, int bin,
                                                          const unsigned* __restrict__ records, const int* __restrict__ record_of,
                                                          const int* __restrict__ shift_of, const int64_t* __restrict__ a_rp,
                                                          const int32_t* __restrict__ a_col, const T* __restrict__ a_val,
                                                          const int64_t* __restrict__ b_rp, const T* __restrict__ b_val, int64_t b_nnz,
                                                          const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val,
                                                          const OrderOperands order) {
  __shared__ NumRecordedLds<T> lds;
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
  num_recorded_rows<ALIKE, T>(&lds, wg, wgs, perm, ctl, bin, records, record_of, shift_of, a_rp, a_col, a_val, b_rp, b_val, b_nnz, c_rp, c_col,
      c_val);
}

}  // namespace spg
