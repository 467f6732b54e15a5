// The dense numeric workspace for wide tiles (k_num_wide): a workgroup of 16 waves has a compute unit to itself, its tiles take up to
// 135 KB.  It does every plan that k_num_tiles does not take: B rows in any order (a tile then filters the products of whole rows),
// pieces by bisection, rows without structure (a first pass over the products marks the flags), and the products of wide_tiles_from.
// Against two workgroups with tiles of half the size: half as many times through the entries of a row of A, which cost more than the
// products where a tile holds few of each; two segments of A entries in registers (2048), the next tile's bounds and the structure's
// words fetched ahead; but nobody accumulates while a tile is set up or leaves.
#pragma once
#include "common.hpp"
#include "entry_order.hpp"
#include "dense_kernels.hpp"

namespace spg {

constexpr int kWideThreads = 1024;
constexpr int kWideWaves = kWideThreads / kWave;
constexpr int kSegCap = 1024;           // A entries described in LDS at a time
constexpr int kListBatch = 4;           // column-list loads in flight per thread
constexpr int kRegSegs = 2;             // segments of A entries that stay in registers
static_assert((long long)kBlkCols * 12 + kBlkCols / 8 <= kWideTileBudget, "direct tile: sums, columns by rank, flag words");

// LDS behind the tile area of the numeric kernel.
template <typename T>
struct WideScratch {
  long long c_s[kSegCap];      // first B entry of every non-empty piece of the tile
  int c_cpre[kSegCap + 1];     // exclusive prefix of the pieces' quad counts
  int c_len[kSegCap];          // piece length
  T c_av[kSegCap];             // a_ik of the piece
  TileRec rec[kRunTiles];
  RunRec rr;                   // the run in the works
  int red[2 * kWideWaves];
  int s_run;
  int pad;
  SPG_CLK(ClkLds clk;)
};

// The piece [s, s + len) of B row k that falls into the tile (blocks [b0, b1), columns [t_lo, t_hi)).
__device__ __forceinline__ void piece_range(int k, long long rs, long long re, int b0, int b1, int t_lo, int64_t t_hi, bool sorted,
                                            const int* __restrict__ bp, int nb1, const int32_t* __restrict__ b_col,
                                            long long& s, int& len) {
  if (sorted && bp) {
    const int* row = bp + (int64_t)k * nb1;
    const int o0 = row[b0], o1 = row[b1];
    s = rs + o0;
    len = o1 - o0;
  } else {
    int64_t st = rs, en = re;
    if (sorted) SearchRange{b_col, t_lo, t_hi}(k, st, en);
    s = st;
    len = (int)(en - st);
  }
}

// Compacts the non-empty pieces of the workgroup's threads into c_s / c_cpre / c_len / c_av.
// Returns their number and the quad total.  Contains barriers.
template <typename T>
__device__ __forceinline__ void tile_pieces(WideScratch<T>* ns, long long s, int len, T av, int& np, int& nquads) {
  int idx, cpre;
  block_excl_scan2<kWideWaves>(len > 0 ? 1 : 0, (len + 3) >> 2, idx, cpre, np, nquads, ns->red);
  if (len > 0) {
    ns->c_s[idx] = s;
    ns->c_cpre[idx] = cpre;
    ns->c_len[idx] = len;
    ns->c_av[idx] = av;
  }
  __syncthreads();
  SPG_CLK(clk_add(&ns->clk, 20, (unsigned long long)nquads); clk_add(&ns->clk, 21, (unsigned long long)np);)
}

template <typename T, bool CHECK>
__device__ __forceinline__ void wide_run(const RunRec rr, WideScratch<T>* ns, unsigned char* tile, bool sorted,
                                              const int32_t* __restrict__ a_col, const T* __restrict__ a_val,
                                              const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col,
                                              const T* __restrict__ b_val, int64_t n_cols, const int* __restrict__ bp, int nb1,
                                              const int32_t* __restrict__ col_list,
                                              int64_t b_nnz, int64_t out_row, int32_t* __restrict__ c_col, T* __restrict__ c_val,
                                              const int (&pre_k)[kRegSegs], const T (&pre_av)[kRegSegs]) {
  const int tid = threadIdx.x;
  // the row's structure in the plan: none, its columns, or its flag words
  const bool have_words = rr.list >= 0 && (rr.list & kListFlagWords) != 0;
  const bool have_list = rr.list >= 0 && !have_words;
  const long long list_at = (rr.list & (kListFlagWords - 1)) - kListBias;   // entry 0 of the row, or the span's kept structure
  const int64_t a0 = rr.a0;
  const int d = rr.d;
  const int nseg = (d + kSegCap - 1) / kSegCap;
  // with few segments, thread e keeps its A entry of every segment in registers for the whole
  // run, together with the block offsets of the coming tile inside the entry's B row (fetched
  // while the current tile is in the works)
  const bool use_table = sorted && bp != nullptr;
  const bool cached = nseg == 1 || (use_table && nseg <= kRegSegs);
  int ck[kRegSegs], pf0[kRegSegs], pf1[kRegSegs];
  long long crs[kRegSegs];
  T cav[kRegSegs];
  long long my_re = 0;
#pragma unroll
  for (int g = 0; g < kRegSegs; ++g) {
    ck[g] = 0; pf0[g] = 0; pf1[g] = 0; crs[g] = 0; cav[g] = T(0);
    const int e = g * kSegCap + tid;
    if (cached && e < d) {
      ck[g] = pre_k[g];     // (fetched by the caller together with the run's tile records)
      cav[g] = pre_av[g];
      crs[g] = b_rp[ck[g]];
      if (!use_table) my_re = b_rp[ck[g] + 1];
      if (use_table) {
        const TileRec nx = ns->rec[0];
        const int* row = bp + (int64_t)ck[g] * nb1;
        pf0[g] = row[nx.b0];
        pf1[g] = row[nx.b1];
      }
    }
  }
  SPG_CLK(clk_mark(&ns->clk, 1);)
  for (int t = 0; t < rr.count; ++t) {
    const TileRec tr = ns->rec[t];
    const bool direct = (tr.cnt & kDirectBit) != 0;
    const bool searched = (tr.cnt & kSearchBit) != 0;
    const int count = tr.cnt & kCountMask;
    const int t_lo = tr.b0 << kBlkShift;
    int64_t t_hi = (int64_t)tr.b1 << kBlkShift;
    if (t_hi > n_cols) t_hi = n_cols;
    const int64_t out = out_row + tr.out;
    // kept flag words of the tile's span: group ranks first, then the words (indexed here by absolute word)
    const int64_t span_c0 = (int64_t)(tr.b0 / kSpanBlocks) * kSpanBlocks * kBlkCols;
    const int32_t* kept_ranks = col_list + list_at;
    const int32_t* kept_words = col_list + list_at + span_rank_slots(span_flag_words(n_cols, span_c0)) - (span_c0 >> 5);
    // this thread's pieces of the tile, one per cached segment
    int off_c[kRegSegs], len_c[kRegSegs];
#pragma unroll
    for (int g = 0; g < kRegSegs; ++g) {
      off_c[g] = 0; len_c[g] = 0;
      const int e = g * kSegCap + tid;
      if (cached && e < d) {
        if (use_table) {
          off_c[g] = pf0[g];
          len_c[g] = pf1[g] - pf0[g];
          if (t + 1 < rr.count) {
            const TileRec nx = ns->rec[t + 1];
            const int* row = bp + (int64_t)ck[g] * nb1;
            pf0[g] = nx.b0 == tr.b1 ? pf1[g] : row[nx.b0];
            pf1[g] = row[nx.b1];
          }
        } else {   // one segment, no table
          long long ps;
          piece_range(ck[g], crs[g], my_re, tr.b0, tr.b1, t_lo, t_hi, sorted, bp, nb1, b_col, ps, len_c[g]);
          off_c[g] = (int)(ps - crs[g]);
        }
      }
    }
    // piece of segment sg for this thread
    auto seg_piece = [&](int sg, long long& ps, int& plen, T& pav) {
      if (cached) {
        static_assert(kRegSegs == 2, "the selects below cover two segments");
        const int o = sg == 0 ? off_c[0] : off_c[1];
        plen = sg == 0 ? len_c[0] : len_c[1];
        ps = (sg == 0 ? crs[0] : crs[1]) + o;
        pav = sg == 0 ? cav[0] : cav[1];
        return;
      }
      ps = 0; plen = 0; pav = T(0);
      const int e = sg * kSegCap + tid;
      if (e < d && e < (sg + 1) * kSegCap) {
        const int k = a_col[a0 + e];
        pav = a_val[a0 + e];
        piece_range(k, b_rp[k], b_rp[k + 1], tr.b0, tr.b1, t_lo, t_hi, sorted, bp, nb1, b_col, ps, plen);
      }
    };
    long long s = 0;
    int len = 0;
    T my_av = T(0);
    if (nseg == 1) seg_piece(0, s, len, my_av);
    __syncthreads();   // the previous tile's output has left the tile area
    SPG_CLK(clk_mark(&ns->clk, 2); clk_add(&ns->clk, 22, (unsigned long long)count);)
    if (searched) {
      // the tile's columns (from the plan's list) and their sums, by rank; a product finds the rank of
      // its column by bisection, so the tile may be as wide as the matrix
      int* cols = reinterpret_cast<int*>(tile);
      double* acc = reinterpret_cast<double*>(tile + (((size_t)count * 4 + 7) & ~(size_t)7));
      const int32_t* lst = col_list + list_at + tr.out;
      for (int j0 = 0; j0 < count; j0 += kListBatch * kWideThreads) {
        int lc[kListBatch];
#pragma unroll
        for (int i = 0; i < kListBatch; ++i) {
          const int j = j0 + i * kWideThreads + tid;
          lc[i] = j < count ? stream_load(&lst[j]) : -1;
        }
#pragma unroll
        for (int i = 0; i < kListBatch; ++i) {
          const int j = j0 + i * kWideThreads + tid;
          if (j < count) {
            cols[j] = lc[i];
            acc[j] = 0.0;
            stream_store(&c_col[out + j], lc[i]);
          }
        }
      }
      SPG_CLK(clk_mark(&ns->clk, 10); clk_add(&ns->clk, 19, 1);)
      int top = 1;   // largest power of two below count
      while (top * 2 < count) top *= 2;
      for (int sg = 0; sg < nseg; ++sg) {
        T av = my_av;
        if (nseg > 1) seg_piece(sg, s, len, av);
        int np, nquads;
        tile_pieces(ns, s, len, av, np, nquads);   // (its barriers also publish cols and the cleared sums)
        quad_pass<kWideWaves, true, T>(np, nquads, PieceList<T>{ns->c_s, ns->c_cpre, ns->c_len, ns->c_av}, b_col, b_val, b_nnz,
                               [&](const Quad<T>& q) {
          // last position whose column is <= c (the column is in the list); the four bisections of a quad
          // advance in lockstep so that their LDS reads overlap
          int lo[4] = {0, 0, 0, 0};
          for (int step = top; step > 0; step >>= 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int mid = lo[i] + step;
              if (mid < count && cols[mid < count ? mid : 0] <= q.col.v[i]) lo[i] = mid;
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i < q.n)
              __hip_atomic_fetch_add(&acc[lo[i]], (double)q.a * (double)q.b.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        });
        if (nseg > 1) __syncthreads();
      }
      __syncthreads();
      SPG_CLK(clk_mark(&ns->clk, 11);)
      for (int r = tid; r < count; r += kWideThreads) stream_store(&c_val[out + r], (T)acc[r]);
      SPG_CLK(clk_mark(&ns->clk, 12);)
    } else if (direct) {
      double* acc = reinterpret_cast<double*>(tile);                      // kBlkCols sums, indexed by column
      int* stage = reinterpret_cast<int*>(tile + (size_t)kBlkCols * 8);   // kBlkCols columns, by rank
      unsigned* flags = reinterpret_cast<unsigned*>(tile + (size_t)kBlkCols * 12);   // kBlkCols / 32
      {
        double2* a2 = reinterpret_cast<double2*>(acc);
        for (int r = tid; r < kBlkCols / 2; r += kWideThreads) a2[r] = make_double2(0.0, 0.0);
      }
      // which columns exist: the flag words are in the plan's list, or are rebuilt by the pass
      if (tid < kBlkCols / 32)   // (the last block of the matrix may be cut short: no flag words are kept behind its end)
        flags[tid] = have_words ? (tid < (int)((t_hi - t_lo + 31) >> 5) ? (unsigned)kept_words[(long long)tr.b0 * kBlkWords + tid] : 0u)
                                : (have_list ? (unsigned)col_list[list_at + tr.out + tid] : 0u);
      SPG_CLK(clk_add(&ns->clk, 18, 1);)
      for (int sg = 0; sg < nseg; ++sg) {
        T av = my_av;
        if (nseg > 1) seg_piece(sg, s, len, av);
        int np, nquads;
        tile_pieces(ns, s, len, av, np, nquads);
        SPG_CLK(clk_mark(&ns->clk, 7);)
        quad_pass<kWideWaves, true, T>(np, nquads, PieceList<T>{ns->c_s, ns->c_cpre, ns->c_len, ns->c_av}, b_col, b_val, b_nnz,
                               [&](const Quad<T>& q) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i < q.n && (!CHECK || (q.col.v[i] >= t_lo && (int64_t)q.col.v[i] < t_hi))) {
                const int rel = q.col.v[i] - t_lo;
                if (!have_list && !have_words) atomicOr(&flags[rel >> 5], 1u << (rel & 31));
                __hip_atomic_fetch_add(&acc[rel], (double)q.a * (double)q.b.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              }
        });
        if (nseg > 1) __syncthreads();
      }
      __syncthreads();
      SPG_CLK(clk_mark(&ns->clk, 8);)
      // compress: thread t owns columns [8 t, 8 t + 8)
      const unsigned byte = (flags[tid >> 2] >> ((tid & 3) * 8)) & 255u;
      double v[8];
      {
        const double2* a2 = reinterpret_cast<const double2*>(acc) + tid * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) { const double2 x = a2[i]; v[2 * i] = x.x; v[2 * i + 1] = x.y; }
      }
      int base, dummy_e, tot, dummy_t;
      block_excl_scan2<kWideWaves>(__popc(byte), 0, base, dummy_e, tot, dummy_t, ns->red);   // barriers: every sum has been read
      (void)tot;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (byte & (1u << i)) {
          acc[base] = v[i];
          stage[base] = t_lo + tid * 8 + i;
          ++base;
        }
      }
      __syncthreads();
      for (int r = tid; r < count; r += kWideThreads) {
        stream_store(&c_val[out + r], (T)acc[r]);
        stream_store(&c_col[out + r], stage[r]);
      }
      SPG_CLK(clk_mark(&ns->clk, 9);)
    } else {
      const int nw = (tr.b1 - tr.b0) * (kBlkCols / 32);                   // 32-bit flag words
      uint2* fc = reinterpret_cast<uint2*>(tile);                         // per word: .x flag bits, .y rank of its first column
      double* acc = reinterpret_cast<double*>(tile + (size_t)nw * 8);     // count sums, by rank
      // with a column list: the first batch of its entries is on its way while the workspace is set up
      const int32_t* lst = col_list + (have_list ? list_at + tr.out : 0);
      int lc[kListBatch], lp[kListBatch];   // kListBatch loads in flight per thread
      auto fetch_list = [&](int j0) {
#pragma unroll
        for (int i = 0; i < kListBatch; ++i) {
          const int j = j0 + i * kWideThreads + tid;
          lc[i] = j < count ? stream_load(&lst[j]) : -1;
          lp[i] = ((tid & 63) == 0 && j > 0 && j < count) ? lst[j - 1] : -1;   // left neighbour of the wave's first entry
        }
      };
      if (have_list) fetch_list(0);
      int np = 0, nquads = 0;
      int* stage = reinterpret_cast<int*>(acc);   // columns by rank, in the space of the sums, on their way to C
      if (!have_words)
        for (int w = tid; w < nw; w += kWideThreads) fc[w] = make_uint2(0u, 0u);
      if (have_list) {
        // the symbolic phase left the tile's columns (ascending) in the plan: flag bits and ranks
        // come from that list, and the list is this tile's run of C's column indices
        for (int r = tid; r < count; r += kWideThreads) acc[r] = 0.0;
        if (nseg == 1) tile_pieces(ns, s, len, my_av, np, nquads); else __syncthreads();
        SPG_CLK(clk_mark(&ns->clk, 3); clk_add(&ns->clk, 17, 1);)
        for (int j0 = 0; j0 < count; j0 += kListBatch * kWideThreads) {
          if (j0 > 0) fetch_list(j0);
#pragma unroll
          for (int i = 0; i < kListBatch; ++i) {
            const int j = j0 + i * kWideThreads + tid;
            const int c = lc[i];
            int prev = __shfl_up(c, 1, kWave);
            if ((tid & 63) == 0) prev = lp[i];
            if (c >= 0) {
              const int rel = c - t_lo;
              flags_or_combined(rel >> 5, 1u << (rel & 31), [&](int w) { return &fc[w].x; });
              if (prev < 0 || ((prev - t_lo) >> 5) != (rel >> 5)) fc[rel >> 5].y = (unsigned)j;
              stream_store(&c_col[out + j], c);
            }
          }
        }
        __syncthreads();
        SPG_CLK(clk_mark(&ns->clk, 4);)
      } else if (have_words) {
        // the symbolic phase left the span's flag words in the plan, with the rank of the first entry of
        // every group of kGrpWords words: groups are dealt to the waves in turn (entries thin out with the
        // column, so neighbouring groups cost about the same), a lane takes a word, ranks follow from one
        // scan over the wave, and the columns are decoded ("boolean indexing") by rank into LDS
        const int wave = tid >> 6, lane = tid & 63;
        const int ngrp = nw / kGrpWords;
        const int nw_kept = (int)((t_hi - t_lo + 31) >> 5);   // (the last block of the matrix may be cut short)
        const int32_t* tw = kept_words + (long long)tr.b0 * kBlkWords;
        const int32_t* tr_ranks = kept_ranks + (int)((t_lo - span_c0) >> 5) / kGrpWords;
        constexpr int kGrpBatch = 4;
        int wd[kGrpBatch], rk[kGrpBatch];
        auto fetch_groups = [&](int g0) {
#pragma unroll
          for (int i = 0; i < kGrpBatch; ++i) {
            const int g = g0 + i * kWideWaves;
            const int w = g * kGrpWords + lane;
            wd[i] = (g < ngrp && w < nw_kept) ? stream_load(&tw[w]) : 0;
            rk[i] = g < ngrp ? tr_ranks[g] : 0;
          }
        };
        fetch_groups(wave);
        for (int g0 = wave; g0 < ngrp; g0 += kWideWaves * kGrpBatch) {
          int cw[kGrpBatch], cr[kGrpBatch];
#pragma unroll
          for (int i = 0; i < kGrpBatch; ++i) { cw[i] = wd[i]; cr[i] = rk[i]; }
          if (g0 + kWideWaves * kGrpBatch < ngrp) fetch_groups(g0 + kWideWaves * kGrpBatch);   // the next batch, while this one is decoded
#pragma unroll
          for (int i = 0; i < kGrpBatch; ++i) {
            const int g = g0 + i * kWideWaves;
            if (g < ngrp) {
              const int w = g * kGrpWords + lane;
              unsigned bits = (unsigned)cw[i];
              const int c = __popc(bits);
              int excl = cr[i] - tr.out + wave_incl_scan(c) - c;   // rank inside the tile
              fc[w] = make_uint2(bits, (unsigned)excl);
              const int cbase = t_lo + w * 32;
              while (bits) {
                const int b = __ffs((int)bits) - 1;
                bits &= bits - 1;
                stage[excl++] = cbase + b;
              }
            }
          }
        }
        __syncthreads();
        for (int r = tid; r < count; r += kWideThreads) stream_store(&c_col[out + r], stage[r]);
        __syncthreads();
        for (int r = tid; r < count; r += kWideThreads) acc[r] = 0.0;
        if (nseg == 1) tile_pieces(ns, s, len, my_av, np, nquads); else __syncthreads();
        SPG_CLK(clk_mark(&ns->clk, 15); clk_add(&ns->clk, 17, 1);)
      } else {
      // pass 1: which columns of the tile exist in the row
      for (int sg = 0; sg < nseg; ++sg) {
        T av = my_av;
        if (nseg > 1) seg_piece(sg, s, len, av);
        tile_pieces(ns, s, len, av, np, nquads);
        quad_pass<kWideWaves, false, T>(np, nquads, PieceList<T>{ns->c_s, ns->c_cpre, ns->c_len, ns->c_av}, b_col, b_val, b_nnz,
                                [&](const Quad<T>& q) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i < q.n && (!CHECK || (q.col.v[i] >= t_lo && (int64_t)q.col.v[i] < t_hi))) {
                const int rel = q.col.v[i] - t_lo;
                atomicOr(&fc[rel >> 5].x, 1u << (rel & 31));
              }
        });
        if (nseg > 1) __syncthreads();
      }
      // exclusive prefix of the flag-word populations: every wave owns a contiguous share of
      // the words and walks it 64 words at a time (lane = word, so LDS reads do not collide);
      // the columns are decoded from the flag words into the space of the sums, by rank, and
      // leave from there as one coalesced run of C's column indices
      const int wave = tid >> 6, lane = tid & 63;
      const int wper = ((nw + kWideThreads - 1) / kWideThreads) * kWave;
      const int wbase = wave * wper;
      __syncthreads();
      int mine = 0;
      for (int i = lane; i < wper; i += kWave) {
        const int w = wbase + i;
        if (w < nw) mine += __popc(fc[w].x);
      }
      mine = wave_sum(mine);
      if (lane == 0) ns->red[wave] = mine;
      __syncthreads();
      int running = 0;
#pragma unroll
      for (int w = 0; w < kWideWaves; ++w) running += w < wave ? ns->red[w] : 0;
      for (int i0 = 0; i0 < wper; i0 += kWave) {
        const int w = wbase + i0 + lane;
        unsigned bits = w < nw ? fc[w].x : 0u;
        const int c = __popc(bits);
        const int incl = wave_incl_scan(c);
        int excl = running + incl - c;
        running += __builtin_amdgcn_readlane(incl, kWave - 1);
        if (w < nw) fc[w].y = (unsigned)excl;
        const int cbase = t_lo + w * 32;
        while (bits) {
          const int b = __ffs((int)bits) - 1;
          bits &= bits - 1;
          stage[excl++] = cbase + b;
        }
      }
      __syncthreads();
      for (int r = tid; r < count; r += kWideThreads) stream_store(&c_col[out + r], stage[r]);
      __syncthreads();
      for (int r = tid; r < count; r += kWideThreads) acc[r] = 0.0;
      __syncthreads();
      SPG_CLK(clk_mark(&ns->clk, 13);)
      }
      // pass 2: accumulate a_ik * b_kj at the rank of column j
      for (int sg = 0; sg < nseg; ++sg) {
        if (nseg > 1) {
          T av;
          seg_piece(sg, s, len, av);
          tile_pieces(ns, s, len, av, np, nquads);
        }
        quad_pass<kWideWaves, true, T>(np, nquads, PieceList<T>{ns->c_s, ns->c_cpre, ns->c_len, ns->c_av}, b_col, b_val, b_nnz,
                               [&](const Quad<T>& q) {
          // the four flag words of a quad first, so that their reads overlap
          uint2 w[4];
          bool ok[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ok[i] = i < q.n && (!CHECK || (q.col.v[i] >= t_lo && (int64_t)q.col.v[i] < t_hi));
            w[i] = fc[ok[i] ? (q.col.v[i] - t_lo) >> 5 : 0];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (ok[i]) {
              const int rank = (int)w[i].y + __popc(w[i].x & ((1u << ((q.col.v[i] - t_lo) & 31)) - 1u));
              __hip_atomic_fetch_add(&acc[rank], (double)q.a * (double)q.b.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        });
        if (nseg > 1) __syncthreads();
      }
      __syncthreads();
      SPG_CLK(clk_mark(&ns->clk, 5);)
      // compress: sums and columns are already in ascending column order
      for (int r = tid; r < count; r += kWideThreads) stream_store(&c_val[out + r], (T)acc[r]);
      SPG_CLK(clk_mark(&ns->clk, 6);)
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kWideThreads) void k_num_wide(Control* ctl, const unsigned char* __restrict__ numbin,
                                                             const TileRec* __restrict__ tiles, const RunRec* __restrict__ runs,
                                                             const int32_t* __restrict__ a_col,
                                                             const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                                             const int32_t* __restrict__ b_col, const T* __restrict__ b_val,
                                                             int64_t n_cols, const int* __restrict__ bp, int nb1,
                                                             const int32_t* __restrict__ col_list, int64_t b_nnz,
                                                             const int64_t* __restrict__ c_rp,
                                                             int32_t* __restrict__ c_col, T* __restrict__ c_val, int tiles3, int looked) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* tile = smem;                                                         // kWideTileBudget bytes
  WideScratch<T>* ns = reinterpret_cast<WideScratch<T>*>(smem + kWideTileBudget);
  if (ctl->error) return;
  const bool sorted = ctl->b_sorted != 0;
  const bool class3 = tiles3 != 0 && !other_order(ctl, looked);   // (as in k_num_tiles)
  const int tid = threadIdx.x;
  const unsigned nruns = ctl->run_cursor, nrows = ctl->offset[0][7] - ctl->offset[0][4];   // (and as many first runs)
  // Thread 0 draws runs ahead of their use: the counter value for the run after next and the record
  // of the next run are on their way while the current run is in the works.
  unsigned drawn = 0;
  RunRec coming{};
  bool have_coming = false;
  SPG_CLK(clk_begin(&ns->clk);)
  if (tid == 0) {
    drawn = atomicAdd(&ctl->work[1], 1u);
    have_coming = blockIdx.x < nruns;   // (the first draw is the workgroup's own)
    if (have_coming) coming = runs[run_of(blockIdx.x, nruns, nrows)];
  }
  while (true) {
    __syncthreads();
    if (tid == 0) {
      ns->s_run = have_coming ? 1 : -1;
      if (have_coming) ns->rr = coming;
      const unsigned next = gridDim.x + drawn;
      have_coming = next < nruns;
      if (have_coming) {
        coming = runs[run_of(next, nruns, nrows)];
        drawn = atomicAdd(&ctl->work[1], 1u);
      }
    }
    __syncthreads();
    if (ns->s_run < 0) break;
    const RunRec rr = ns->rr;
    if (rr.count == 0) continue;   // a record that its row did not need
    // one round trip: the row's class and position in C, the run's tile records, its A entries
    const int cls = numbin[rr.row];
    const int64_t out_row = c_rp[rr.row];
    if (tid < rr.count) ns->rec[tid] = tiles[rr.first + tid];
    int pre_k[kRegSegs];
    T pre_av[kRegSegs];
#pragma unroll
    for (int g = 0; g < kRegSegs; ++g) {
      pre_k[g] = 0; pre_av[g] = T(0);
      const int e = g * kSegCap + tid;
      if (e < rr.d && rr.d <= kRegSegs * kSegCap) {
        pre_k[g] = a_col[rr.a0 + e];
        pre_av[g] = a_val[rr.a0 + e];
      }
    }
    if (!(cls == 3 && class3) && cls != 5 && cls != 6) continue;   // the row's numeric class is not this kernel's
    __syncthreads();
    SPG_CLK(clk_mark(&ns->clk, 0); clk_add(&ns->clk, 16, 1);)
    if (sorted)
      wide_run<T, false>(rr, ns, tile, true, a_col, a_val, b_rp, b_col, b_val, n_cols, bp, nb1, col_list, b_nnz, out_row, c_col, c_val, pre_k, pre_av);
    else
      wide_run<T, true>(rr, ns, tile, false, a_col, a_val, b_rp, b_col, b_val, n_cols, bp, nb1, col_list, b_nnz, out_row, c_col, c_val, pre_k, pre_av);
  }
  SPG_CLK(clk_mark(&ns->clk, 14); clk_flush(&ns->clk, ctl->clk[1]);)
}

template <typename T>
constexpr size_t num_wide_lds() { return (size_t)kWideTileBudget + sizeof(WideScratch<T>); }

}  // namespace spg
