// Dense LDS workspaces for long rows (Gustavson's flag list / coordinate list of the
// paper's section 4.4, and the dense first-order workspace of section 7.2): the symbolic
// kernel and what it shares with the numeric ones (tile_kernels.hpp, wide_kernels.hpp).
//
// Symbolic (k_sym_dense), a workgroup per row: a flag list with one bit per column (up to 2^20 columns per span in
//   128 KB of LDS); products set bits, the row's size is the population count.  From the
//   finished flag list the kernel also plans the row's numeric work: the column space is cut
//   at multiples of kBlkCols columns into tiles, each small enough for the numeric workspace,
//   and the row's column structure goes to the plan (decoded columns, or the flag words of
//   direct blocks), so that the numeric phase need not find it again.
//   The flag list takes the LDS that the matrix's width needs, and the workgroups are as many as hold 32 waves a compute unit in 64 registers
//   each (sym_dense_shape): what a row costs beside its products (clearing and counting the flags, planning, the round trips for its entries and
//   its shares of the lists, decoding) is waiting for the most part, which other workgroups fill.  The flags are counted with a lane on every
//   fourth word, a block per wave (32 consecutive words per thread collided on the banks).
//   Up to 2^18 columns, workgroups of 8 waves, four on a compute unit (three at 2^18), where there are 32 rows or more for a compute unit, otherwise two of 16:
//   us with 16 | 8: R-MAT squared scale 12 34 | 48, scale 14 (5277 rows) 111 | 120, 15 (16 500) 244 | 206, 17 1391 | 990, 18 3435 | 2990; deduplication sweep
//   of 10 000 columns 533 | 487; 1071 rows of 4400 products 35 | 46; 60 000 of 3600 837 | 671.  With 4 waves 15 and 16 lose (362, 508).
//   Up to 2^19 two of 16 with 512 A entries described at a time: scale 19 9.3 ms, with two of 8 waves in 84 registers 10.2.
//   Beyond that one of 16 waves has a compute unit to itself.
// Numeric (k_num_tiles, or k_num_wide), one tile at a time, one pass over the tile's products:
//   direct tile (one block of kBlkCols columns in which the row is dense): sums live in a
//     dense array indexed by column; the flags say which exist; flags and sums are compressed
//     at the end ("boolean indexing" in the paper's words).
//   ranked tile (a run of blocks in which the row is sparse): an exclusive prefix over the flag
//     words gives every present column its rank; a product adds a_ik * b_kj at the rank of
//     column j - LDS holds only columns that exist in C and the finished tile is already in
//     ascending column order.  Flags and ranks come from the plan's column list; without one,
//     a first pass over the products rebuilds them.
//   searched tile (a short row, or half of one): the row's columns sit in LDS and a product finds its
//     rank by bisection, so the tile's width does not matter.
//   The piece of B row k that falls into a tile is found with two loads from a table of
//   per-row block offsets (ascending B rows), so a pass touches only its own products.
#pragma once
#include "common.hpp"
#include "piece_pass.hpp"

namespace spg {

constexpr int kSymFlagWords = 32768;    // 2^20 columns per symbolic span (128 KB)
constexpr int kBlkCols = 8192;          // tile boundaries are multiples of this many columns
constexpr int kBlkShift = 13;
constexpr int kSpanBlocks = kSymFlagWords * 32 / kBlkCols;   // 128 blocks per symbolic span
constexpr int kTileBudget = 66 * 1024; // LDS bytes of one numeric tile (flags + ranks + sums): two workgroups on a compute unit
constexpr int kWideTileBudget = 135 * 1024;   // ... of a wide one: one workgroup (wide_tiles_from says which products)
constexpr int kRankBlkBytes = kBlkCols / 32 * 8;   // flag word + rank per 32 columns of a ranked tile
constexpr int kRankEntryBytes = 8;                // sum per entry of a ranked tile (its column goes straight to C)
constexpr int kDirectMinDefault = 6144; // a block with at least this many entries becomes a direct tile
constexpr int kRunTiles = 16;           // tiles handed to a workgroup at a time
constexpr int kListSlab = 1 << 20;      // list entries and tile records that a symbolic workgroup draws at a time
constexpr int kTileSlab = 512;
constexpr int kDirectBit = 1 << 30;     // in TileRec::cnt
constexpr int kSearchBit = 1 << 29;     // in TileRec::cnt: a searched tile (ranks by bisection of the column list)
constexpr int kCountMask = kSearchBit - 1;
constexpr int kSearchCap = 5632;      // entries of a searched tile (column 4 B + sum 8 B each)
constexpr int kSearchRow = 2 * kSearchCap;   // entries of a row that becomes searched tiles: one, or two (one wide one)
constexpr int kBlkWords = kBlkCols / 32;
// every tile kind must fit the tile area of the numeric kernel
static_assert((long long)kSearchCap * 12 <= kTileBudget && (long long)kSearchRow * 12 <= kWideTileBudget, "searched tile: 4 B column + 8 B sum per entry");
static_assert((long long)kBlkCols * 8 + kBlkCols / 8 <= kTileBudget, "direct tile: sums, flag words");
static_assert(kRankBlkBytes + 8LL * kBlkCols <= kTileBudget, "ranked tile: one block must fit even when it is full");
constexpr long long kListBias = 1LL << 40;   // RunRec::list holds position + bias (so that -1 can mean "none")
constexpr long long kListFlagWords = 1LL << 60;   // RunRec::list: the row's structure is kept as flag words, not as columns
constexpr int kFlagWordsNum = 1, kFlagWordsDen = 1;   // flag words are kept when words * Num <= entries * Den (measured: best near one entry per word)
constexpr int kGrpWords = 64;                // flag words per group: the plan keeps the rank of every group's first entry
constexpr int kSpanGroups = kSymFlagWords / kGrpWords;

// Layout of a span's structure kept as flag words: first the group ranks (row-relative rank of the first
// entry of every group of kGrpWords words, padded to 16 bytes), then the flag words themselves.
__host__ __device__ __forceinline__ int span_flag_words(int64_t n_cols, int64_t c0) {
  const int64_t left = n_cols - c0, span = (int64_t)kSymFlagWords * 32;
  return (int)(((left < span ? left : span) + 31) >> 5);
}
// Flag words that the symbolic kernel keeps in LDS: those of a span, in whole blocks.
__host__ __device__ __forceinline__ int sym_flag_words(int64_t n_cols) { return (span_flag_words(n_cols, 0) + kBlkWords - 1) / kBlkWords * kBlkWords; }
__host__ __device__ __forceinline__ int span_rank_slots(int words) { return (((words + kGrpWords - 1) / kGrpWords) + 3) & ~3; }

// Stores and loads of data that passes through the numeric kernel once (the result, the plan's
// column list): the non-temporal hint keeps it from displacing B, which is re-read all the time,
// from the caches.  (Not for the symbolic kernel's list writes: partial lines written with the
// hint are not combined, which costs more than it saves.)
template <typename V>
__device__ __forceinline__ void stream_store(V* p, V v) { __builtin_nontemporal_store(v, p); }
template <typename V>
__device__ __forceinline__ V stream_load(const V* p) { return __builtin_nontemporal_load(p); }

// List entries that a symbolic workgroup draws at a time, at most: together a quarter of the list, so that a short list is not
// spent on slack.
__host__ __device__ __forceinline__ unsigned long long list_slab_of(unsigned long long list_cap, int64_t workgroups) {
  const unsigned long long s = (list_cap / (4ULL * (unsigned long long)workgroups)) & ~3ULL;
  return s < (unsigned long long)kListSlab ? s : (unsigned long long)kListSlab;
}

struct TileRec { int b0, b1, cnt, out; };     // blocks [b0, b1), entries (| kDirectBit), offset inside the row of C
// tiles [first, first + count) of one row; its A entries [a0, a0 + d); list (-1: the row has no list):
// where entry 0 of the row sits in the plan's list, plus kListBias - or, with kListFlagWords set,
// where the flag word of column 0 sits (the row's structure is kept as one bit per column)
struct RunRec { int row; unsigned first; int count, d; long long a0, list; };

// Per-workgroup bookkeeping of the piece walker below.
template <int WAVES, int PIECES>
struct __align__(16) RowScratch {   // (the tile planner's arrays, written 16 bytes at a time, lie behind it)
  static constexpr int kPieces = PIECES;              // A entries described in LDS at a time, at most one per thread
  static constexpr int kListStage = 5 * PIECES / WAVES;   // entries that a wave gathers here, when the pieces are done with, before writing them to the column list
  long long start[kPieces];   // first B entry of each A entry's piece
  int plen[kPieces];          // piece length
  int cpre[kPieces + 1];      // exclusive prefix of chunk counts
  int red[kPieces + 1];       // (the column decode stages kListStage entries per wave from `start` to here)
  int s_row;
  int pad;
  unsigned long long span_ip;       // products streamed since the owner last cleared it
  SPG_CLK(ClkLds clk;)
};

// block_excl_scan of two ints, by name.
template <int WAVES>
__device__ __forceinline__ void block_excl_scan2(int a, int b, int& ea, int& eb, int& ta, int& tb, int* red) {
  const int v[2] = {a, b};
  int e[2], t[2];
  block_excl_scan<WAVES>(v, e, t, red);
  ea = e[0]; eb = e[1];
  ta = t[0]; tb = t[1];
}

// Visits every element of the pieces once (k_num_wide; cpre counts quads here).  A piece is cut into quads; the quads of all pieces are dealt to the waves
// in contiguous shares of whole batches of 64, a lane takes a quad: one load of four columns and one of four values.  Which piece a lane's quad belongs to:
// lane i looks at where the i-th piece behind the one in hand begins and pushes i + 1 to the lane whose quad that is; a running maximum spreads it to the
// lanes behind.  g(quad) is called per lane and batch (a, b only meaningful when WITH_VALUES).
// What bounds the numeric pass is neither traffic nor its instructions (a search for every 64 chunks, as in piece_pass, is slower here: rows in any order 577 |
// 634 us) but the chain of loads and LDS steps of a batch.  Chunks of 64 elements with wave-uniform descriptors took about 35 scalar and 10 vector
// instructions a chunk and were 70 % full with pieces of 122 entries; quads are 98 % full and take about 45 per 256 elements.  R-MAT scale 19 squared
// (fp32), k_num_wide 27.9 -> 25.9 ms; scale 14: numeric 218 -> 190 us; deduplication sweep (fp64) 1.64 -> 1.59 ms.  With values one batch at a time is best
// (two in flight 26.5 ms, three 29.7, four 31.8: registers; the next one prefetched 25.9, but 1.69 for the sweep).
template <int WAVES, bool WITH_VALUES, typename T, class G>
__device__ __forceinline__ void quad_pass(int np, int nq, const PieceList<T> pl, const int32_t* __restrict__ b_col,
                                          const T* __restrict__ b_val, int64_t b_nnz, G g) {
  const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
  np = uni(np);
  nq = uni(nq);
  const int nb = (nq + kWave - 1) >> 6;
  const int per = (nb + WAVES - 1) / WAVES;
  int c = wave * per * kWave;
  const int cend = c + per * kWave < nq ? c + per * kWave : nq;
  if (c >= cend) return;
  int p;   // last piece whose first quad is <= c: among every sixteenth piece first, then among the sixteen
  {
    static_assert(WAVES <= 16, "64 steps of sixteen pieces");
    const int i0 = lane * 16;
    const int hi = __popcll(__ballot(i0 < np && pl.cpre[i0 < np ? i0 : 0] <= c)) - 1;
    const int i1 = hi * 16 + lane;
    p = hi * 16 + __popcll(__ballot(lane < 16 && i1 < np && pl.cpre[i1 < np ? i1 : 0] <= c)) - 1;
  }
  auto fetch = [&](int cu, Quad<T>& o) {
    const int ahead = p + 1 + lane;
    const int begins = (ahead < np ? pl.cpre[ahead] : 0x7fffffff) - cu;   // (1 or more: piece p holds quad cu)
    int m = __builtin_amdgcn_ds_permute(begins < kWave ? begins * 4 : 0, lane + 1);   // (the others push to lane 0, which does not look)
    m = group_max_scan<kWave>(lane == 0 ? 0 : m);
    const int piece = p + m;
    const int q = cu + lane;
    const int off = (q - pl.cpre[piece]) * 4;
    const int len = pl.len[piece];
    const int64_t at = pl.s[piece] + off;
    if (WITH_VALUES) o.a = pl.av[piece];
    o.n = q < cend ? len - off : 0;
    p += __popcll(__ballot(begins <= kWave));
    if (!__any(o.n > 0 && at + 4 > b_nnz)) {
      if (o.n > 0) {
        o.col = load_run<int32_t, 4>(b_col + at);
        if (WITH_VALUES) o.b = load_run<T, 4>(b_val + at);
      }
    } else {   // (fewer than four elements behind some lane's position)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < o.n) {
          o.col.v[i] = b_col[at + i];
          if (WITH_VALUES) o.b.v[i] = b_val[at + i];
        }
    }
  };
  Quad<T> now;
  if constexpr (WITH_VALUES) {
    for (; c < cend; c += kWave) {
      now = Quad<T>{};
      fetch(c, now);
      g(now);
    }
  } else {
    fetch(c, now);
    while (true) {   // (the next batch is on its way while g works on this one)
      Quad<T> next;
      const bool more = c + kWave < cend;
      if (more) fetch(c + kWave, next);
      g(now);
      if (!more) break;
      now = next;
      c += kWave;
    }
  }
}

// Walks every pair (A entry p of the row, B entry q of row a_col[p]) and hands the columns to f, a quad per lane at a time.
// range(k, s, en) may narrow the piece [s, en) of B row k first.  As many A entries as the workgroup has threads are described
// at once.  Contains barriers: every thread of the workgroup must call it.
template <int WAVES, int PIECES, class Range, class F>
__device__ __forceinline__ void stream_columns(int64_t a0, int d, const int32_t* __restrict__ a_col,
                                               const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col, int64_t b_nnz,
                                               RowScratch<WAVES, PIECES>* rs, Range range, F f) {
  const int tid = threadIdx.x, lane = tid & 63;
  for (int base = 0; base < d; base += PIECES) {
    const int e = PIECES >= WAVES * kWave || tid < PIECES ? base + tid : d;
    int64_t s = 0;
    int len = 0;
    if (e < d) {
      const int k = a_col[a0 + e];
      const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k);
      s = bounds.v[0];
      int64_t en = bounds.v[1];
      range(k, s, en);
      len = (int)(en - s);
    }
    if (Range::kNarrows) {   // (a narrowed walk covers a part of the row: its products are counted for the caller)
      unsigned long long wl = (unsigned long long)len;
#pragma unroll
      for (int sh = 1; sh < kWave; sh <<= 1) wl += __shfl_xor(wl, sh, kWave);
      if (lane == 0 && wl) atomicAdd(&rs->span_ip, wl);
    }
    const PieceCut cut = piece_chunks<WAVES>(len, rs->red);
    if (len > 0) {
      rs->start[cut.idx] = s;
      rs->plen[cut.idx] = len;
      rs->cpre[cut.idx] = cut.first;
    }
    __syncthreads();
    SPG_CLK(clk_mark(&rs->clk, 2); clk_add(&rs->clk, 18, 1); clk_add(&rs->clk, 19, (unsigned long long)cut.chunks << cut.lanes);)
    if (cut.chunks > 0)
      piece_pass<WAVES>(cut.pieces, cut.chunks, cut.lanes, PieceList<int>{rs->start, rs->cpre, rs->plen, nullptr}, b_col, b_nnz, f);
    SPG_CLK(clk_mark(&rs->clk, 3);)
    __syncthreads();
    SPG_CLK(clk_mark(&rs->clk, 4);)
  }
}

// For ascending B rows: bp[k * nb1 + b] = number of entries of row k with a column below
// b * kBlkCols (b = nb1 - 1 gives the row length).  One thread per table slot, each bisecting its
// row (the threads of a row read the same few lines, and the table leaves in coalesced stores).
__global__ __launch_bounds__(256) void k_block_ptrs(int64_t rows, int nb1, const int64_t* __restrict__ b_rp,
                                                    const int32_t* __restrict__ b_col, const Control* __restrict__ ctl,
                                                    int* __restrict__ bp) {
  if (ctl->error || !ctl->b_sorted) return;
  const int64_t total = rows * nb1;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int64_t k = i / nb1;
    const int b = (int)(i - k * nb1);
    const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k);
    const int64_t s = bounds.v[0], en = bounds.v[1];
    int off;
    if (b == 0 || en == s) off = 0;
    else if (b == nb1 - 1) off = (int)(en - s);
    else off = (int)(lower_bound_i32(b_col, s, en, b << kBlkShift) - s);
    bp[i] = off;
  }
}

struct NoRange {
  static constexpr bool kNarrows = false;
  __device__ __forceinline__ void operator()(int, int64_t&, int64_t&) const {}
};

struct TableRange {   // ascending rows with the block-offset table: the entries in blocks [b0, b1)
  static constexpr bool kNarrows = true;
  const int* bp; int nb1; int b0, b1;
  __device__ __forceinline__ void operator()(int k, int64_t& s, int64_t& en) const {
    const int* row = bp + (int64_t)k * nb1;
    en = s + row[b1];
    s += row[b0];
  }
};

struct SearchRange {   // binary search in an ascending row
  static constexpr bool kNarrows = true;
  const int32_t* b_col; int lo; int64_t hi;
  __device__ __forceinline__ void operator()(int, int64_t& s, int64_t& en) const {
    if (en > s) {
      s = lower_bound_i32(b_col, s, en, lo);
      if (hi <= 0x7fffffff) en = lower_bound_i32(b_col, s, en, (int)hi);
    }
  }
};

// What a workgroup has left of the slabs drawn from the plan's lists, and what its rows have taken.
struct Slabs {
  unsigned long long list_used;         // list entries taken
  unsigned long long sl_pos, sl_left;   // left: list entries,
  unsigned st_pos, st_left;             // tile records
  unsigned used_tiles, used_runs;
};

// LDS of the tile planner.
struct __align__(16) TilePlan {
  int grp[kSpanGroups];   // entries per group of kGrpWords flag words
  int blk_cnt[kSpanBlocks];
  int cum[kSpanBlocks + 1];
  int nxt[kSpanBlocks];
  TileRec rec[kSpanBlocks];
  int ntiles, ndirect, nruns;
  int next_block;         // list decode: the next block to hand to a wave
  unsigned tile_base;
  unsigned place;         // of the row among the rows
  unsigned run_first, run_base;   // where the span's first run goes, and its others
  int row_out;
  int span_out0;          // row_out when the span began
  long long list_base;    // position of the span's first entry (or first flag word) in the plan's list, -1 = none
  int list_words;         // > 0: the span's structure goes to the list as that many flag words instead of columns
  Slabs slabs;
};

// index of the lowest set bit at or above position b in the 128-bit mask (hi:lo); 128 when none
__device__ __forceinline__ int next_bit128(unsigned long long lo, unsigned long long hi, int b) {
  if (b < 64) {
    const unsigned long long m = lo >> b;
    if (m) return b + __ffsll((long long)m) - 1;
    if (hi) return 64 + __ffsll((long long)hi) - 1;
    return 128;
  }
  if (b >= 128) return 128;
  const unsigned long long m = hi >> (b - 64);
  return m ? b + __ffsll((long long)m) - 1 : 128;
}

// index of the highest set bit below position e; -1 when none
__device__ __forceinline__ int prev_bit128(unsigned long long lo, unsigned long long hi, int e) {
  if (e > 64) {
    const unsigned long long m = e >= 128 ? hi : (hi & ((1ULL << (e - 64)) - 1ULL));
    if (m) return 127 - __clzll((long long)m);
    e = 64;
  }
  if (e <= 0) return -1;
  const unsigned long long m = e >= 64 ? lo : (lo & ((1ULL << e) - 1ULL));
  return m ? 63 - __clzll((long long)m) : -1;
}

// Cuts the nb blocks of one span (counts in tp->blk_cnt) into tiles; run by wave 0.
// A block with at least direct_min entries is a direct tile of its own; the blocks between
// are grouped greedily into ranked tiles of at most `budget` bytes
// (kRankBlkBytes per block + kRankEntryBytes per entry).  Records land in tp->rec, their number in tp->ntiles.
// First part (wave 0): entry prefix over the blocks and the span's total.
constexpr bool kSpanTwoHalves = kSpanBlocks > kWave;   // a lane plans one block, or two
static_assert(kSpanBlocks == kWave || kSpanBlocks == 2 * kWave, "a span of 64 or 128 blocks");
__device__ __forceinline__ void plan_head(TilePlan* tp, int nb, bool count_only) {
  const int l = lane_id();
  const int c0 = l < nb ? tp->blk_cnt[l] : 0;
  const int c1 = (kSpanTwoHalves && l + 64 < nb) ? tp->blk_cnt[l + 64] : 0;
  const int i0 = wave_incl_scan(c0);
  const int t0 = __builtin_amdgcn_readlane(i0, 63);
  const int i1 = kSpanTwoHalves ? wave_incl_scan(c1) : 0;
  tp->cum[l] = i0 - c0;
  if (kSpanTwoHalves) tp->cum[l + 64] = t0 + i1 - c1;
  if (l == 63) {
    const int total = t0 + i1;
    tp->cum[kSpanBlocks] = total;
    tp->ntiles = 0;
    tp->ndirect = 0;
    if (count_only) tp->row_out += total;   // the row's numeric class needs no tiles
  }
}

// Second part (wave 0): the tile records (direct and ranked tiles).
__device__ __forceinline__ void plan_tail(TilePlan* tp, int nb, int block0, int direct_min, int budget) {
  const int l = lane_id();
  const int c0 = l < nb ? tp->blk_cnt[l] : 0;
  const int c1 = (kSpanTwoHalves && l + 64 < nb) ? tp->blk_cnt[l + 64] : 0;
  const unsigned long long dm0 = __ballot(c0 >= direct_min), dm1 = __ballot(c1 >= direct_min);
  const unsigned long long nm0 = __ballot(c0 > 0), nm1 = __ballot(c1 > 0);
#pragma unroll
  for (int half = 0; half < (kSpanTwoHalves ? 2 : 1); ++half) {
    const int b = l + 64 * half;
    if (b < nb) {
      int lim = next_bit128(dm0, dm1, b);   // first direct block at or behind b
      if (lim > nb) lim = nb;
      const int base = tp->cum[b];
      int lo = b + 1, hi = lim;             // largest e in [b+1, lim] that fits
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((long long)(mid - b) * kRankBlkBytes + (long long)kRankEntryBytes * (tp->cum[mid] - base) <= budget) lo = mid; else hi = mid - 1;
      }
      tp->nxt[b] = lo;
    }
  }
  wave_sync();
  if (l == 0) {
    int n = 0, nd = 0, out = tp->row_out;
    int b = next_bit128(nm0, nm1, 0);
    while (b < nb) {
      const int cb = tp->blk_cnt[b];
      if (cb >= direct_min) {
        tp->rec[n++] = TileRec{block0 + b, block0 + b + 1, cb | kDirectBit, out};
        ++nd;
        out += cb;
        b = b + 1;
      } else {
        const int e = tp->nxt[b];
        const int c = tp->cum[e] - tp->cum[b];
        const int et = prev_bit128(nm0, nm1, e) + 1;   // drop empty blocks at the end
        tp->rec[n++] = TileRec{block0 + b, block0 + et, c, out};
        out += c;
        b = e;
      }
      b = next_bit128(nm0, nm1, b);
    }
    tp->ntiles = n;
    tp->ndirect = nd;
    tp->row_out = out;
  }
}

// The numeric kernels' runs lie in the order of the symbolic kernel's rows, the first of every row, the heaviest first, and behind them the further runs of
// rows that have several; workgroups draw them by number.  Where there are few for a workgroup they are taken in that order, so that no workgroup is left with
// a long row at the end.  Where there are many, every draw of four is from the front and the others are from the back: heavy rows use the memory, light ones
// wait for it, and both kinds do better beside the other.  k_num_tiles of R-MAT squared, us in order | from both ends: scale 14 146 | 161, scale 16 746 | 768
// (53 runs a workgroup), scale 17 2812 | 2774 (97), 18 8886 | 7827, 19 25364 | 23041; 60 000 rows of 3600 products 1443 | 1409.  One of two and one
// of eight do less for the larger ones (19: 23413, 23494).
// k_num_wide takes the further runs before all others (`rows` first runs; they belong to the heaviest rows, and in k_num_tiles it makes no difference).
// k_num_wide, ms in order | from both ends | so: R-MAT squared scale 20 (fp32) 74.4 | 71.9 | 71.5, fp64 90.9 | 85.4 | 85.8, 8 edges 29.3 | 27.1 | 27.0,
// scale 21 with 6 edges 78.5 | 78.9 | 78.5; 20 000 unordered rows of 120 x 120 products 2.57 | 2.55 | 2.56.  (In the order in which the symbolic
// workgroups drew records, 256 at a time: 70.0, 86.4, 27.0, 79.2, 2.57.  That order over the rows as they lie now 71.0, 86.2, 27.3, 79.7, 2.59; halves from
// either end 71.3, 86.1, 26.9, 83.6, 2.57; 4, 16 or 64 stretches side by side 74 and more, -, 29.)
constexpr unsigned kManyRuns = 64;
__device__ __forceinline__ unsigned run_of(unsigned draw, unsigned nruns, unsigned rows) {
  if (nruns < kManyRuns * gridDim.x || draw >= nruns) return draw;
  const unsigned more = nruns - rows;
  if (draw < more) return rows + draw;
  const unsigned q = (draw - more) / 4, r = (draw - more) % 4;
  return r == 0 ? q : rows - 3 * q - r;
}

// Takes `amount` from a shared cursor if that stays within `cap` (compare and advance: the cursor never
// passes the capacity, so a request that does not fit costs later, smaller requests nothing).
__device__ __forceinline__ bool reserve_below(unsigned long long* cursor, unsigned long long amount, unsigned long long cap,
                                              unsigned long long& base) {
  unsigned long long cur = __hip_atomic_load(cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (cur + amount <= cap) {
    const unsigned long long seen = atomicCAS(cursor, cur, cur + amount);
    if (seen == cur) { base = cur; return true; }
    cur = seen;
  }
  return false;
}

// Draws up to `amount` from a shared cursor by addition and returns how much it got; nothing where less than that is left.  (Workgroups
// with rows of similar length draw at the same moment, and of hundreds that compare and exchange one gets through at a time: 12 770 rows
// of 3700 entries, 300 000 columns, 512 workgroups, symbolic kernel 5250 | 365 us.)  A draw may take the cursor beyond the capacity, where it
// stays: nobody begins there, and who began before it has what is left.  look: for an amount that would take much room with it that
// way (every look and every draw costs all workgroups together about 12 ns: 640 us with both for every row).
__device__ __forceinline__ unsigned long long draw_below(unsigned long long* cursor, unsigned long long amount, unsigned long long cap,
                                                         bool look, unsigned long long& base) {
  if (look && __hip_atomic_load(cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + amount > cap) return 0;
  base = atomicAdd(cursor, amount);
  return base >= cap ? 0 : (cap - base < amount ? cap - base : amount);
}

// PER_SIMD 4: LDS leaves room for one workgroup on a compute unit, so it may take the registers it wants (R-MAT scale 20: 45.8 ms in 64
// registers, with spills, 44.4 in 75).  The other forms spill nine registers (40 bytes a lane), outside their loops over products.
template <int WAVES, int PER_SIMD, int PIECES>
__global__ __launch_bounds__(WAVES * kWave, PER_SIMD) void k_sym_dense(const int* __restrict__ perm, Control* ctl,
                                                             const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                                             const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col,
                                                             int64_t n_cols, const int* __restrict__ ip, int* __restrict__ cnt,
                                                             TileRec* __restrict__ tiles, RunRec* __restrict__ runs,
                                                             int32_t* __restrict__ col_list, int direct_min, int no_tiles_ip,
                                                             int search_ratio, const int* __restrict__ bp, int nb1, int64_t b_nnz, int run_tiles, int wide) {
  constexpr int kThreads = WAVES * kWave;
  constexpr bool ALONE = PER_SIMD == 4;
  constexpr bool kLook = !ALONE;
  extern __shared__ __align__(16) unsigned char smem[];
  const int flag_words = sym_flag_words(n_cols);
  unsigned* flags = reinterpret_cast<unsigned*>(smem);                               // flag_words
  using Scratch = RowScratch<WAVES, PIECES>;
  constexpr int kListStage = Scratch::kListStage;
  Scratch* rs = reinterpret_cast<Scratch*>(smem + (size_t)flag_words * 4);
  TilePlan* tp = reinterpret_cast<TilePlan*>(smem + (size_t)flag_words * 4 + sizeof(Scratch));
  if (ctl->error) return;
  const bool sorted = ctl->b_sorted != 0;
  const int64_t span = (int64_t)kSymFlagWords * 32;
  const int tid = threadIdx.x;
  const unsigned row_lo = ctl->offset[0][4], row_hi = ctl->offset[0][7];   // the dense bins, heaviest class last
  const unsigned tile_cap = ctl->tile_cap, run_cap = ctl->run_cap;
  const unsigned long long list_cap = ctl->list_cap;
  SPG_CLK(clk_begin(&rs->clk);)
  // The first row of a workgroup is its own by its number, the others are drawn from a counter.  A row's place among the rows is
  // the place of its first run too.
  const unsigned nrows = row_hi - row_lo;
  const bool one = !ALONE || n_cols <= span;   // every column is in the span
  int row = blockIdx.x < nrows ? perm[row_hi - 1 - blockIdx.x] : -1;
  if (tid == 0) tp->place = blockIdx.x;
  // Thread 0's slabs of the plan's lists are in LDS (its registers would be everybody's), but where there are registers to spare (R-MAT
  // scale 20: 44.6 | 43.0 ms).  The first slab of
  // every workgroup is its own by its number (the cursors start behind these: k_set_caps); when all workgroups drew their
  // first slab from the shared cursors at the same moment, the compare-and-swaps of 256 of them took 0.2 ms (1071 rows: 366 -> 73 us).
  const unsigned long long list_slab = list_slab_of(list_cap, gridDim.x);
  Slabs own{};
  Slabs& sl = ALONE ? own : tp->slabs;
  if (tid == 0)
    sl = Slabs{0, blockIdx.x * list_slab, list_slab, blockIdx.x * (unsigned)kTileSlab, (unsigned)kTileSlab, 0, 0};
  int next_row = -1;   // (thread 0) the row after this one
  while (row >= 0) {
    unsigned nx = 0;   // (thread 0) the draw for the row after this one: on its way while this row is in the works
    if (tid == 0) nx = atomicAdd(&ctl->work[0], 1u);
    const int64_t a0 = a_rp[row];
    const int d = (int)(a_rp[row + 1] - a0);
    if (tid == 0) tp->row_out = 0;
    SPG_CLK(clk_mark(&rs->clk, 0); clk_add(&rs->clk, 16, 1);)
    for (int64_t c0 = 0; c0 < n_cols; c0 += span) {
      const int64_t c1 = (c0 + span < n_cols) ? c0 + span : n_cols;
      const int words = (int)((c1 - c0 + 31) >> 5);
      const int nb = (int)((c1 - c0 + kBlkCols - 1) >> kBlkShift);
      {
        uint4* f4 = reinterpret_cast<uint4*>(flags);
        for (int w = tid; w < flag_words / 4; w += kThreads) f4[w] = make_uint4(0, 0, 0, 0);
      }
      if (tid == 0) { tp->span_out0 = tp->row_out; tp->list_base = -1; rs->span_ip = 0; }
      __syncthreads();
      SPG_CLK(clk_mark(&rs->clk, 1); clk_add(&rs->clk, 17, 1);)
      const int lo = (int)c0;
      const int64_t hi = c1;
      auto mark = [&](const Quad<int>& q, auto full) {
        constexpr bool kFull = decltype(full)::value;
        if (kFull && one) {
          // (looking at the flag words first, so that only bits that are not set yet go through the atomic, gains where hub columns are hit by
          // most pieces or columns many times - us without | with: R-MAT scale 17 1515 | 1450, dedup sweep of 30000 4390 | 4270, of 10000 2035 |
          // 2060 - and loses where there are 16 waves on a compute unit: scale 19 36.0 | 36.4 ms)
          unsigned w[4];
          if (kLook) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = flags[(unsigned)q.col.v[i] >> 5];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const unsigned bit = 1u << (q.col.v[i] & 31);
            if (!kLook || !(w[i] & bit)) atomicOr(&flags[(unsigned)q.col.v[i] >> 5], bit);
          }
          return;
        }
        unsigned w[4];
        bool ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ok[i] = i < q.n && (one || (q.col.v[i] >= lo && (int64_t)q.col.v[i] < hi));
          w[i] = flags[ok[i] ? (q.col.v[i] - lo) >> 5 : 0];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned bit = 1u << ((q.col.v[i] - lo) & 31);
          if (ok[i] && !(w[i] & bit)) atomicOr(&flags[(q.col.v[i] - lo) >> 5], bit);
        }
      };
      if (!one && sorted && bp)
        stream_columns(a0, d, a_col, b_rp, b_col, b_nnz, rs, TableRange{bp, nb1, (int)(c0 >> kBlkShift), (int)((c1 + kBlkCols - 1) >> kBlkShift)}, mark);
      else if (!one && sorted)
        stream_columns(a0, d, a_col, b_rp, b_col, b_nnz, rs, SearchRange{b_col, lo, hi}, mark);
      else
        stream_columns(a0, d, a_col, b_rp, b_col, b_nnz, rs, NoRange{}, mark);
      const bool last_span = c1 >= n_cols;
      const int ip_row = tid < kWave ? ip[row] : 0;   // (on its way while the entries are counted)
      // entries per block and per group: a wave takes a block, a lane four words of it, a group is a row of 16 lanes
      {
        static_assert(kBlkWords == 4 * kWave && kGrpWords == 64, "four words per lane, sixteen lanes per group");
        const int lane = tid & 63;
        for (int blk = uni(tid >> 6); blk < nb; blk += WAVES) {
          const uint4 v = reinterpret_cast<const uint4*>(flags)[blk * kWave + lane];
          const int incl = wave_incl_scan(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w));
          const int t0 = __builtin_amdgcn_readlane(incl, 15), t1 = __builtin_amdgcn_readlane(incl, 31);
          const int t2 = __builtin_amdgcn_readlane(incl, 47), t3 = __builtin_amdgcn_readlane(incl, 63);
          if (lane == 0) {
            *reinterpret_cast<int4*>(&tp->grp[blk * 4]) = make_int4(t0, t1 - t0, t2 - t1, t3 - t2);
            tp->blk_cnt[blk] = t3;
          }
        }
      }
      __syncthreads();
      SPG_CLK(clk_mark(&rs->clk, 5);)
      const bool count_only = ip_row <= no_tiles_ip;
      const int block0 = (int)(c0 >> kBlkShift);
      if (tid < kWave) {
        plan_head(tp, nb, count_only);
        if (!count_only) plan_tail(tp, nb, block0, direct_min, wide ? kWideTileBudget : kTileBudget);
        wave_sync_lds();
      }
      SPG_CLK(clk_mark(&rs->clk, 6);)
      if (tid == 0) {
        // Everything this span needs from the plan's shared lists, and the next row, in one round trip:
        // room for the entries in the column list (without it the numeric kernel rebuilds the flags
        // itself), tile and run records.  A span that got room in the list and has at
        // most search_ratio products per entry becomes searched tiles (the records planned above then stay unused): one of at most
        // kSearchCap entries, or two of an ascending B, where that is less than half of the tiles planned: a bisection costs
        // three times the look-up in a ranked tile (R-MAT scale 17, searched wherever a tile was saved: row blocks 7.27 ms, now 6.83).
        // Wide tiles: one of at most kSearchRow entries wherever a tile is saved.
        const int total = tp->cum[kSpanBlocks];
        const int nt = tp->ntiles;
        const bool want_list = !count_only && total > 0 && list_cap > 0;
        // a short row with little deduplication becomes one searched tile and needs its columns; every
        // other row keeps its flag words as they are (no decoding here, and far less memory for rows
        // with many entries) unless they would take much more room than the columns
        // (products of the span: counted by the walk when it covered a part of the row)
        const long long span_products = (n_cols > span && sorted) ? (long long)rs->span_ip : (long long)ip_row;
        // (a searched tile takes every product of its pieces: with unordered B rows the pieces are whole rows,
        // so the tile must be the whole row)
        bool search_row = (sorted || n_cols <= span) && total <= kSearchRow && nt > (wide ? 1 : total <= kSearchCap ? 2 : 4) && span_products <= (long long)search_ratio * total;
        int cut = nb;   // where the second searched tile begins
        if (search_row && !wide && total > kSearchCap) {
          int e = 0;   // as many blocks as one tile holds
          for (int step = kSpanBlocks / 2; step > 0; step >>= 1)
            if (e + step < nb && tp->cum[e + step] <= kSearchCap) e += step;
          search_row = sorted && total - tp->cum[e] <= kSearchCap;
          cut = e;
        }
        const int fwords = (words + 3) & ~3;
        const bool as_words = !search_row && (long long)fwords * kFlagWordsNum <= (long long)kFlagWordsDen * total;
        const unsigned long long need = as_words ? (unsigned long long)(span_rank_slots(words) + fwords)
                                                 : (unsigned long long)((total + 3) & ~3);   // (16-byte granules)
        // The shares come out of slabs that the workgroup draws from the shared cursors now and then: a round
        // trip to a counter that every workgroup hits costs microseconds, a row needs its answer at once.
        unsigned long long at = 0;
        unsigned tb = 0, rb = 0;
        bool listed = false;
        if (want_list) {
          if (need <= sl.sl_left) {
            at = sl.sl_pos; sl.sl_pos += need; sl.sl_left -= need; listed = true;
          } else {
            // (room for a power of two of rows like this one: rows are of similar length, and what is left of the old slab stays
            // unused; a row that takes more than half of a slab draws for itself alone)
            unsigned grab = (unsigned)need;
            while ((unsigned long long)grab * 2 <= list_slab) grab *= 2;
            const bool alone = grab == (unsigned)need;
            unsigned long long base;
            const unsigned long long got = draw_below(&ctl->list_cursor, grab, list_cap, alone, base);
            if (got >= need) {
              at = base; listed = true;
              if (!alone) { sl.sl_pos = base + need; sl.sl_left = got - need; }
            } else {
              if (got > sl.sl_left) { sl.sl_pos = base; sl.sl_left = got; }   // (the end of the list, for a shorter row)
              if (reserve_below(&ctl->list_cursor, need, list_cap, base)) { at = base; listed = true; }   // (no room for a slab, but for the row alone)
            }
          }
        }
        // (a searched tile pays a bisection per product: only for rows with little deduplication, and
        // only where it saves tiles - a row that is one ranked or direct tile anyway stays that)
        const bool as_searched = listed && search_row;
        const int ntiles = as_searched ? (cut < nb ? 2 : 1) : nt;
        const int nr = (ntiles + run_tiles - 1) / run_tiles;
        const int placed = c0 == 0 ? 1 : 0;   // a row's first run has its place, so that the numeric kernel takes the rows in the same order
        bool room = true;
        if (ntiles > 0) {
          if ((unsigned)ntiles > sl.st_left) {
            sl.st_pos = atomicAdd(&ctl->tile_cursor, (unsigned)kTileSlab);
            room = sl.st_pos + (unsigned)kTileSlab <= tile_cap;
            sl.st_left = room ? (unsigned)kTileSlab : 0u;
          }
          if (room) {
            tb = sl.st_pos; sl.st_pos += (unsigned)ntiles; sl.st_left -= (unsigned)ntiles;
            if (nr > placed) {
              rb = atomicAdd(&ctl->run_cursor, (unsigned)(nr - placed));
              room = rb + (unsigned)(nr - placed) <= run_cap;
            }
          }
        }
        if (listed) sl.list_used += need;
        else if (total > 0 && !count_only) ctl->unlisted = 1;
        tp->list_base = listed ? (long long)at : -1;
        tp->list_words = listed && as_words ? fwords : 0;
        tp->tile_base = tb;
        tp->run_base = rb - (unsigned)placed;
        tp->run_first = placed ? tp->place : rb;
        tp->next_block = 0;
        tp->nruns = nr > placed ? nr : placed;   // (a row without tiles leaves an empty record)
        tp->ntiles = ntiles;
        if (!room) {
          ctl->error = 3;   // cannot happen when the host sized the lists from the bound
          tp->ntiles = 0;
          tp->nruns = placed;
        } else if (as_searched) {
          const int c0 = cut < nb ? tp->cum[cut] : total;
          tp->rec[0] = TileRec{block0, block0 + cut, c0 | kSearchBit, tp->span_out0};
          if (cut < nb) tp->rec[1] = TileRec{block0 + cut, block0 + nb, (total - c0) | kSearchBit, tp->span_out0 + c0};
          atomicAdd(&ctl->search_tiles, 1u);
        } else if (tp->ndirect > 0) {
          atomicAdd(&ctl->direct_tiles, (unsigned)tp->ndirect);
        }
        sl.used_tiles += (unsigned)tp->ntiles;
        sl.used_runs += (unsigned)(room ? nr : 0);
        if (last_span) {
          tp->place = gridDim.x + nx;
          next_row = gridDim.x + nx < nrows ? perm[row_hi - 1 - (gridDim.x + nx)] : -1;
        }
      }
      __syncthreads();
      SPG_CLK(clk_mark(&rs->clk, 7);)
      const long long lb = tp->list_base;
      const int nt = tp->ntiles;
      if (nt > 0 || tp->nruns > 0) {
        if (tid < nt) tiles[tp->tile_base + tid] = tp->rec[tid];
        if (tid < tp->nruns) {
          const int left = nt - tid * run_tiles;
          // (flag words: the position of the word of column 0, which may lie before the span's words)
          const long long lpos = lb < 0 ? -1LL : (tp->list_words ? (lb + kListBias) | kListFlagWords : lb - tp->span_out0 + kListBias);
          runs[tid == 0 ? tp->run_first : tp->run_base + tid] = RunRec{row, tp->tile_base + (unsigned)(tid * run_tiles), left < 0 ? 0 : (left < run_tiles ? left : run_tiles), d, a0, lpos};
        }
      }
      if (lb >= 0 && tp->list_words) {
        // the flag list leaves as it is (one coalesced copy), behind the rank of every group's first entry
        static_assert(kGrpWords * 4 == kBlkWords, "four groups per block");
        const int nslots = span_rank_slots(words);
        for (int t = tid; t < nslots; t += kThreads) {
          int r = tp->span_out0 + tp->cum[(t >> 2) < kSpanBlocks ? (t >> 2) : kSpanBlocks];
          for (int g = t & ~3; g < t; ++g) r += tp->grp[g];
          col_list[lb + t] = r;
        }
        const uint4* f4 = reinterpret_cast<const uint4*>(flags);
        uint4* o4 = reinterpret_cast<uint4*>(col_list + lb + nslots);
        const int n4 = tp->list_words >> 2;
        for (int w = tid; w < n4; w += kThreads) o4[w] = f4[w];
      } else if (lb >= 0) {
        // The list position of a block's first entry is its entry prefix.  Sparse blocks: the columns are decoded, a round
        // with few entries is gathered in LDS first and leaves as one coalesced run.
        // Direct blocks: the numeric kernel wants the flag words themselves (their 256 words fit
        // in the space of the block's entries).
        const int wave = tid >> 6, lane = tid & 63;
        const bool searched = (tp->rec[0].cnt & kSearchBit) != 0;
        int* wst = reinterpret_cast<int*>(rs) + wave * kListStage;   // the piece walker's scratch is free now
        // (blocks are handed out one at a time: their entry counts differ by orders of magnitude,
        // so a fixed share per wave would leave most waves waiting for the one with the dense blocks)
        while (true) {
          int blk = 0;
          if (lane == 0) blk = atomicAdd(&tp->next_block, 1);
          blk = __builtin_amdgcn_readfirstlane(blk);
          if (blk >= nb) break;
          const int cb = tp->blk_cnt[blk];
          if (cb == 0) continue;
          int running = tp->cum[blk];
          if (cb >= direct_min && !searched) {
#pragma unroll
            for (int q = 0; q < kBlkWords; q += kWave) col_list[lb + running + q + lane] = (int)flags[blk * kBlkWords + q + lane];
            continue;
          }
          if (cb <= kListStage) {
            // a sparse block in one round: lane l decodes words 4 l .. 4 l + 3
            const uint4 v = reinterpret_cast<const uint4*>(flags)[blk * (kBlkWords / 4) + lane];
            const int c = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
            int excl = wave_incl_scan(c) - c;
            const int cbase = lo + (blk * kBlkWords + lane * 4) * 32;
            if (c) {
              unsigned wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                unsigned bits = wd[k];
                while (bits) {
                  const int b = __ffs((int)bits) - 1;
                  bits &= bits - 1;
                  wst[excl++] = cbase + k * 32 + b;
                }
              }
            }
            wave_sync_lds();
            for (int j = lane; j < cb; j += kWave) col_list[lb + running + j] = wst[j];
            wave_sync_lds();
            continue;
          }
          for (int q = 0; q < kBlkWords; q += kWave) {
            const int w = blk * kBlkWords + q + lane;
            unsigned bits = flags[w];
            const int c = __popc(bits);
            const int incl = wave_incl_scan(c);
            const int tot = __builtin_amdgcn_readlane(incl, kWave - 1);
            if (tot == 0) continue;
            int excl = incl - c;
            const int cbase = lo + w * 32;
            if (tot <= kListStage) {
              while (bits) {
                const int b = __ffs((int)bits) - 1;
                bits &= bits - 1;
                wst[excl++] = cbase + b;
              }
              wave_sync_lds();
              for (int j = lane; j < tot; j += kWave) col_list[lb + running + j] = wst[j];
              wave_sync_lds();   // (the stores themselves need not have left before the next round)
            } else {
              while (bits) {
                const int b = __ffs((int)bits) - 1;
                bits &= bits - 1;
                col_list[lb + running + excl++] = cbase + b;
              }
            }
            running += tot;
          }
        }
      }
      if (tid == 0 && last_span) {
        cnt[row] = tp->row_out;
        rs->s_row = next_row;
      }
      __syncthreads();
      SPG_CLK(clk_mark(&rs->clk, 8);)
    }
    row = rs->s_row;
  }
  if (tid == 0) {
    if (sl.used_tiles) atomicAdd(&ctl->tiles_used, sl.used_tiles);
    if (sl.used_runs) atomicAdd(&ctl->runs_used, sl.used_runs);
    if (sl.list_used) atomicAdd(&ctl->list_used, sl.list_used);
  }
  SPG_CLK(clk_mark(&rs->clk, 9); clk_flush(&rs->clk, ctl->clk[0]);)
}

static_assert(sizeof(RowScratch<8, 512>) % 16 == 0 && sizeof(RowScratch<16, 1024>) % 16 == 0 && alignof(TilePlan) == 16, "the planner's arrays start on 16 bytes");
template <int WAVES, int PIECES>
constexpr size_t sym_dense_lds(int64_t flag_words) { return (size_t)flag_words * 4 + sizeof(RowScratch<WAVES, PIECES>) + sizeof(TilePlan); }
// Half a span of flag words (64 KB): up to that many columns two workgroups of 16 waves share a compute unit, with 512 pieces described at a time.
constexpr int64_t kSymNarrowCols = (int64_t)kSymFlagWords * 16;
// A quarter: two of 16 waves with 1024 pieces or, where rows are many, four of 8 waves.
constexpr int64_t kSymShortCols = (int64_t)kSymFlagWords * 8;

}  // namespace spg
