// The dense numeric workspace (k_num_tiles): runs of tiles that the symbolic kernel has planned, one tile at a time.
//
// A workgroup of 1024 threads works on a tile of at most 66 KB; two of them share a compute unit, so that one accumulates
// products while the other waits for flag words, decodes columns or writes its tile out.  That takes 64 registers a thread and 80
// KB of LDS a workgroup, which is enough where B's rows ascend, the block-offset table is there, B has fewer than 2^30 entries, and
// every row of the dense classes has its structure in the plan; other plans, and some of these, are k_num_wide's (wide_tiles_from).
// Ranked tiles take 50 to 55 LDS cycles for 64 products (a look-up of 14, an addition of 27, the search for the piece), wide
// matrices beside that what the tile costs by itself: reads and writes run at 5.8 TB/s at scale 19 (B's entries come from behind
// the L2 caches).  The 64 registers fall 15 (fp32) or 22 (fp64) short: a run's and a tile's numbers stay in memory and are read once or
// twice a tile, none inside a loop over products.  Before, one workgroup of 16 waves with a tile of 135 KB had a compute unit to itself
// and accumulated products
// for 36 % of its time.  us before | two workgroups of 8 waves | of 16 waves: R-MAT squared (fp32) scale 14 192 | 158 | 158, scale 19
// 25871 | 23670 | 23400; deduplication sweep, 10000 columns (fp64), 1586 | 1360 | 1390; four row blocks of scale 17, whole call,
// 7710 | 7280 | 6840.
#pragma once
#include "common.hpp"
#include "entry_order.hpp"
#include "dense_kernels.hpp"

namespace spg {

constexpr int kTileThreads = 1024;
constexpr int kTileWaves = kTileThreads / kWave;
constexpr int64_t kTileMaxNnz = int64_t(1) << 30;   // a piece's start shares 32 bits with two others

// WHOLE: a tile is a whole row, without structure in the plan (k_row_tiles).
template <typename T, bool WHOLE, int WAVES = kTileWaves>
struct TileScratch {
  using Start = std::conditional_t<WHOLE, unsigned long long, unsigned>;
  static constexpr int kPieces = WHOLE ? WAVES * kWave : 768;   // pieces of B rows described at a time
  Start s[kPieces];               // a piece's first B entry, shifted left by two; entries missing in its last quad below
  int cpre[kPieces + 1];          // exclusive prefix of the pieces' quad counts
  T av[kPieces];                  // a_ik of the piece
  TileRec rec[kRunTiles];
  RunRec rr;                      // the run in the works
  int red[2 * WAVES];
  int s_run;
  int split;                      // quads before the pieces of the second round
  SPG_CLK(ClkLds clk;)
};

// Records of a run and of a tile, the same for the whole workgroup, in scalar registers (read from LDS they took 30 vector registers).
__device__ __forceinline__ RunRec uni_run(const RunRec& r) {
  return RunRec{uni(r.row), (unsigned)uni((int)r.first), uni(r.count), uni(r.d), uni64(r.a0), uni64(r.list)};
}
__device__ __forceinline__ TileRec uni_tile(const TileRec& t) { return TileRec{uni(t.b0), uni(t.b1), uni(t.cnt), uni(t.out)}; }

// A finished direct tile to C: every wave takes groups of 64 columns in turn; the group's entries follow each other in C, and
// where they begin comes from a scan over all flag words, four to a lane.
template <int WAVES, typename T>
__device__ __forceinline__ void direct_out(const double* acc, const unsigned* flags, int t_lo, int64_t out, int32_t* __restrict__ c_col, T* __restrict__ c_val) {
  static_assert(kBlkWords == 4 * kWave, "four flag words per lane");
  const int wave = uni(threadIdx.x >> 6), lane = lane_id();
  const uint4 f = reinterpret_cast<const uint4*>(flags)[lane];
  const int c0 = __popc(f.x) + __popc(f.y), c = c0 + __popc(f.z) + __popc(f.w);
  const int e0 = wave_incl_scan(c) - c, e1 = e0 + c0;
  for (int g = wave; g < kBlkCols / kWave; g += WAVES) {
    const unsigned long long mask = reinterpret_cast<const unsigned long long*>(flags)[g];
    const int at = __builtin_amdgcn_readlane((g & 1) ? e1 : e0, g >> 1) + lanes_below(mask);
    if ((mask >> lane) & 1) {
      c_val[out + at] = (T)acc[g * kWave + lane];
      c_col[out + at] = t_lo + g * kWave + lane;
    }
  }
}

// Visits every product of np pieces (nq quads) once, g(quad) per lane: as quad_pass, with the pieces' values and without their
// lengths (a piece's last quad says how many of its entries are missing).
template <int WAVES, bool WITH_VALUES, typename T, bool WHOLE, class G>
__device__ __forceinline__ void tile_pass(int np, int nq, const TileScratch<T, WHOLE, WAVES>* ts, const int32_t* __restrict__ b_col,
                                          const T* __restrict__ b_val, int64_t b_nnz, G g) {
  using Start = typename TileScratch<T, WHOLE, WAVES>::Start;
  const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nb = (nq + kWave - 1) >> 6;
  const int per = (nb + WAVES - 1) / WAVES;
  int c = wave * per * kWave;
  const int cend = c + per * kWave < nq ? c + per * kWave : nq;
  if (c >= cend) return;
  int p;   // last piece whose first quad is <= c: among every sixteenth piece first, then among the sixteen
  {
    static_assert(TileScratch<T, WHOLE, WAVES>::kPieces <= 16 * kWave, "64 steps of sixteen pieces");
    const int i0 = lane * 16;
    const int hi = __popcll(__ballot(i0 < np && ts->cpre[i0 < np ? i0 : 0] <= c)) - 1;
    const int i1 = hi * 16 + lane;
    p = hi * 16 + __popcll(__ballot(lane < 16 && i1 < np && ts->cpre[i1 < np ? i1 : 0] <= c)) - 1;
  }
  for (; c < cend; c += kWave) {
    const int ahead = p + 1 + lane;
    const int begins = (ahead < np ? ts->cpre[ahead] : 0x7fffffff) - c;   // (1 or more: piece p holds quad c)
    int m = __builtin_amdgcn_ds_permute(begins < kWave ? begins * 4 : 0, lane + 1);   // (the others push to lane 0, which does not look)
    m = group_max_scan<kWave>(lane == 0 ? 0 : m);
    const int piece = p + m;
    const int q = c + lane;
    const int q0 = ts->cpre[piece], q1 = ts->cpre[piece + 1];
    const Start sp = ts->s[piece];
    const Start at = (sp >> 2) + (Start)((q - q0) * 4);
    Quad<T> o;
    if (WITH_VALUES) o.a = ts->av[piece];
    o.n = q < cend ? (q + 1 == q1 ? 4 - (int)(sp & 3) : 4) : 0;
    p += __popcll(__ballot(begins <= kWave));
    if (!__any(o.n > 0 && at + 4 > (Start)b_nnz)) {
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
    g(o);
  }
}

// The tiles of one run; k, av: this thread's A entry, in rows of at most kThreads of them.
template <int WAVES, typename T, bool WHOLE>
__device__ __forceinline__ void tile_run(const RunRec rr, TileScratch<T, WHOLE, WAVES>* ts, unsigned char* tile, const int32_t* __restrict__ a_col,
                                         const T* __restrict__ a_val, const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col,
                                         const T* __restrict__ b_val, int64_t n_cols, const int* __restrict__ bp, int nb1,
                                         const int32_t* __restrict__ col_list, int64_t b_nnz, int64_t out_row, int32_t* __restrict__ c_col,
                                         T* __restrict__ c_val, int k, T av) {
  using Start = typename TileScratch<T, WHOLE, WAVES>::Start;
  constexpr int kPieces = TileScratch<T, WHOLE, WAVES>::kPieces;
  constexpr int kThreads = WAVES * kWave;
  const int tid = threadIdx.x;
  // the row's structure in the plan: its columns, its flag words, or (whole rows) none
  constexpr bool have = !WHOLE;
  const bool have_words = have && (rr.list & kListFlagWords) != 0;
  const long long list_at = (rr.list & (kListFlagWords - 1)) - kListBias;   // entry 0 of the row, or the span's kept structure
  const int nseg = (rr.d + kThreads - 1) / kThreads;
  // this thread's A entry (rows of at most kThreads entries keep it for the whole run) and the place of the coming tile in
  // its B row
  unsigned crs = 0;
  int pf0 = 0, pf1 = 0;
  const bool mine = nseg == 1 && tid < rr.d;
  if (!WHOLE && mine) {
    const TileRec nx = uni_tile(ts->rec[0]);
    crs = (unsigned)b_rp[k];
    const int* row = bp + (int64_t)k * nb1;
    pf0 = row[nx.b0];
    pf1 = row[nx.b1];
  }
  SPG_CLK(clk_mark(&ts->clk, 1);)
  for (int t = 0; t < rr.count; ++t) {
    const TileRec tr = uni_tile(ts->rec[t]);
    const bool direct = have && (tr.cnt & kDirectBit) != 0;
    const bool searched = have && (tr.cnt & kSearchBit) != 0;
    const int count = tr.cnt & kCountMask;
    const int t_lo = tr.b0 << kBlkShift;
    int64_t t_hi = (int64_t)tr.b1 << kBlkShift;
    if (t_hi > n_cols) t_hi = n_cols;
    const int64_t out = out_row + tr.out;
    Start s = 0;
    int len = 0;
    if (WHOLE && mine) {
      const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k);
      s = (Start)bounds.v[0];
      len = (int)(bounds.v[1] - bounds.v[0]);
    } else if (mine) {
      s = crs + (unsigned)pf0;
      len = pf1 - pf0;
      if (t + 1 < rr.count) {
        const TileRec nx = uni_tile(ts->rec[t + 1]);
        const int* row = bp + (int64_t)k * nb1;
        pf0 = nx.b0 == tr.b1 ? pf1 : row[nx.b0];
        pf1 = row[nx.b1];
      }
    }
    // All products of the tile, acc(quad) per lane.  Begins with a barrier; every product is in the tile behind it, but where the
    // last entries of A have none, waves may still be reading the totals in ts->red.
    auto products = [&](auto with_values, auto acc) {
      for (int sg = 0; sg < nseg; ++sg) {
        if (nseg > 1) {
          const int e = sg * kThreads + tid;
          len = 0;
          if (e < rr.d) {
            const int ke = a_col[rr.a0 + e];
            av = a_val[rr.a0 + e];
            if (WHOLE) {
              const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + ke);
              s = (Start)bounds.v[0];
              len = (int)(bounds.v[1] - bounds.v[0]);
            } else {
              const int* row = bp + (int64_t)ke * nb1;
              const int o0 = row[tr.b0];
              s = (Start)b_rp[ke] + (Start)o0;
              len = row[tr.b1] - o0;
            }
          }
        }
        int idx, cpre, np, nq;
        block_excl_scan2<WAVES>(len > 0 ? 1 : 0, (len + 3) >> 2, idx, cpre, np, nq, ts->red);
        np = uni(np);
        nq = uni(nq);
        SPG_CLK(clk_add(&ts->clk, 20, (unsigned long long)nq); clk_add(&ts->clk, 21, (unsigned long long)np);)
        for (int i0 = 0; i0 < np; i0 += kPieces) {   // (more pieces than are described at a time: the first of them, then the others)
          static_assert(2 * kPieces >= kThreads, "two rounds");
          const int i1 = np < i0 + kPieces ? np : i0 + kPieces;
          const int q0 = i0 ? uni(ts->split) : 0;
          if (len > 0) {
            if (idx >= i0 && idx < i1) {
              ts->s[idx - i0] = (s << 2) | (Start)(-len & 3);
              ts->cpre[idx - i0] = cpre - q0;
              ts->av[idx - i0] = av;
            }
            if (idx == i1) { ts->cpre[i1 - i0] = cpre - q0; ts->split = cpre; }
          }
          if (tid == 0 && i1 == np) ts->cpre[i1 - i0] = nq - q0;
          __syncthreads();
          const int q1 = i1 == np ? nq : uni(ts->split);
          tile_pass<WAVES, decltype(with_values)::value, T, WHOLE>(i1 - i0, q1 - q0, ts, b_col, b_val, b_nnz, acc);
          __syncthreads();
        }
      }
    };
    // (whole rows: operands of another structure than the plan's stay inside the tile)
    auto in_tile = [&](const Quad<T>& q, int i) { return i < q.n && (!WHOLE || (q.col.v[i] >= t_lo && (int64_t)q.col.v[i] < t_hi)); };
    __syncthreads();   // the previous tile's output has left the tile area
    SPG_CLK(clk_mark(&ts->clk, 2); clk_add(&ts->clk, 22, (unsigned long long)count);)
    if (searched) {
      // the tile's columns (from the plan's list) and their sums, by rank; a product finds the rank of
      // its column by bisection, so the tile may be as wide as the matrix
      int* cols = reinterpret_cast<int*>(tile);
      double* acc = reinterpret_cast<double*>(tile + (((size_t)count * 4 + 7) & ~(size_t)7));
      const int32_t* lst = col_list + list_at + tr.out;
      for (int j = tid; j < count; j += kThreads) {
        const int c = stream_load(&lst[j]);
        cols[j] = c;
        acc[j] = 0.0;
        stream_store(&c_col[out + j], c);
      }
      SPG_CLK(clk_mark(&ts->clk, 10); clk_add(&ts->clk, 19, 1);)
      int top = 1;   // largest power of two below count
      while (top * 2 < count) top *= 2;
      products(std::true_type{}, [&](const Quad<T>& q) {
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
      SPG_CLK(clk_mark(&ts->clk, 11);)
      for (int r = tid; r < count; r += kThreads) stream_store(&c_val[out + r], (T)acc[r]);
      SPG_CLK(clk_mark(&ts->clk, 12);)
    } else if (direct) {
      double* acc = reinterpret_cast<double*>(tile);                      // kBlkCols sums, indexed by column
      unsigned* flags = reinterpret_cast<unsigned*>(tile + (size_t)kBlkCols * 8);   // kBlkCols / 32
      {
        double2* a2 = reinterpret_cast<double2*>(acc);
        for (int r = tid; r < kBlkCols / 2; r += kThreads) a2[r] = make_double2(0.0, 0.0);
      }
      if (tid < kBlkWords) {   // (the last block of the matrix may be cut short: no flag words are kept behind its end)
        const int64_t span_c0 = (int64_t)(tr.b0 / kSpanBlocks) * kSpanBlocks * kBlkCols;
        const int32_t* words = have_words ? col_list + list_at + span_rank_slots(span_flag_words(n_cols, span_c0)) + ((t_lo - span_c0) >> 5)
                                          : col_list + list_at + tr.out;
        flags[tid] = !have_words || tid < (int)((t_hi - t_lo + 31) >> 5) ? (unsigned)words[tid] : 0u;
      }
      SPG_CLK(clk_mark(&ts->clk, 7); clk_add(&ts->clk, 18, 1);)
      products(std::true_type{}, [&](const Quad<T>& q) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (in_tile(q, i)) {
            const int rel = q.col.v[i] - t_lo;
            __hip_atomic_fetch_add(&acc[rel], (double)q.a * (double)q.b.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
      });
      SPG_CLK(clk_mark(&ts->clk, 8);)
      direct_out<WAVES>(acc, flags, t_lo, out, c_col, c_val);
      SPG_CLK(clk_mark(&ts->clk, 9);)
    } else {
      const int nw = (tr.b1 - tr.b0) * kBlkWords;                         // 32-bit flag words
      uint2* fc = reinterpret_cast<uint2*>(tile);                         // per word: .x flag bits, .y rank of its first column
      double* acc = reinterpret_cast<double*>(tile + (size_t)nw * 8);     // count sums, by rank
      int* stage = reinterpret_cast<int*>(acc);                           // columns by rank, in the space of the sums, on their way to C
      if (have_words) {
        // the symbolic phase left the span's flag words in the plan, with the rank of the first entry of
        // every group of kGrpWords words: groups are dealt to the waves in turn (entries thin out with the
        // column, so neighbouring groups cost about the same), a lane takes a word, ranks follow from one
        // scan over the wave, and the columns are decoded ("boolean indexing") by rank into LDS
        const int wave = uni(tid >> 6), lane = tid & 63;
        const int64_t span_c0 = (int64_t)(tr.b0 / kSpanBlocks) * kSpanBlocks * kBlkCols;
        const int rel = (int)((t_lo - span_c0) >> 5);
        const int32_t* ranks = col_list + list_at + rel / kGrpWords;
        const int32_t* words = col_list + list_at + span_rank_slots(span_flag_words(n_cols, span_c0)) + rel;
        const int ngrp = nw / kGrpWords;
        const int nw_kept = (int)((t_hi - t_lo + 31) >> 5);   // (the last block of the matrix may be cut short)
        // (loads of two groups in flight: R-MAT squared, whole calls, us with one | two | four | eight: scale 14 456 | 455 | 457 | 473, scale 17
        // 4364 | 4312 | 4390 | 4609, scale 16 (fp64) 1425 | 1409 | 1418 | -)
        constexpr int kGrpBatch = 2;
        for (int g0 = wave; g0 < ngrp; g0 += WAVES * kGrpBatch) {
          int wd[kGrpBatch], rk[kGrpBatch];
#pragma unroll
          for (int i = 0; i < kGrpBatch; ++i) {
            const int g = g0 + i * WAVES;
            const int w = g * kGrpWords + lane;
            wd[i] = (g < ngrp && w < nw_kept) ? stream_load(&words[w]) : 0;
            rk[i] = g < ngrp ? ranks[g] : 0;
          }
#pragma unroll
          for (int i = 0; i < kGrpBatch; ++i) {
            const int g = g0 + i * WAVES;
            if (g < ngrp) {
              const int w = g * kGrpWords + lane;
              unsigned bits = (unsigned)wd[i];
              const int c = __popc(bits);
              int excl = rk[i] - tr.out + wave_incl_scan(c) - c;   // rank inside the tile
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
        for (int r = tid; r < count; r += kThreads) stream_store(&c_col[out + r], stage[r]);
        __syncthreads();
        for (int r = tid; r < count; r += kThreads) acc[r] = 0.0;
        SPG_CLK(clk_mark(&ts->clk, 15); clk_add(&ts->clk, 17, 1);)
      } else if (!have) {
        // a pass over the products: which columns of the tile exist in the row
        for (int w = tid; w < nw; w += kThreads) fc[w] = make_uint2(0u, 0u);
        products(std::false_type{}, [&](const Quad<T>& q) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (in_tile(q, i)) {
              const int rel = q.col.v[i] - t_lo;
              atomicOr(&fc[rel >> 5].x, 1u << (rel & 31));
            }
        });
        // exclusive prefix of the flag-word populations: every wave owns a contiguous share of
        // the words and walks it 64 words at a time (lane = word, so LDS reads do not collide);
        // the columns are decoded from the flag words into the space of the sums, by rank, and
        // leave from there as one coalesced run of C's column indices
        const int wave = uni(tid >> 6), lane = tid & 63;
        const int wper = ((nw + kThreads - 1) / kThreads) * kWave;
        const int wbase = wave * wper;
        int in_share = 0;
        for (int i = lane; i < wper; i += kWave) {
          const int w = wbase + i;
          if (w < nw) in_share += __popc(fc[w].x);
        }
        in_share = wave_sum(in_share);
        __syncthreads();   // (the totals in ts->red have been read by all waves)
        if (lane == 0) ts->red[wave] = in_share;
        __syncthreads();
        int running = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) running += w < wave ? ts->red[w] : 0;
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
        for (int r = tid; r < count; r += kThreads) stream_store(&c_col[out + r], stage[r]);
        __syncthreads();
        for (int r = tid; r < count; r += kThreads) acc[r] = 0.0;
        SPG_CLK(clk_mark(&ts->clk, 13);)
      } else {
        // the symbolic phase left the tile's columns (ascending) in the plan: flag bits and ranks
        // come from that list, and the list is this tile's run of C's column indices
        const int32_t* lst = col_list + list_at + tr.out;
        for (int w = tid; w < nw; w += kThreads) fc[w] = make_uint2(0u, 0u);
        for (int r = tid; r < count; r += kThreads) acc[r] = 0.0;
        __syncthreads();
        SPG_CLK(clk_mark(&ts->clk, 3); clk_add(&ts->clk, 17, 1);)
        for (int j = tid; j < count; j += kThreads) {
          const int c = stream_load(&lst[j]);
          int prev = __shfl_up(c, 1, kWave);
          if ((tid & 63) == 0) prev = j > 0 ? lst[j - 1] : -1;   // left neighbour of the wave's first entry
          const int rel = c - t_lo;
          flags_or_combined(rel >> 5, 1u << (rel & 31), [&](int w) { return &fc[w].x; });
          if (prev < 0 || ((prev - t_lo) >> 5) != (rel >> 5)) fc[rel >> 5].y = (unsigned)j;
          stream_store(&c_col[out + j], c);
        }
        SPG_CLK(clk_mark(&ts->clk, 4);)
      }
      // accumulate a_ik * b_kj at the rank of column j
      products(std::true_type{}, [&](const Quad<T>& q) {
        // the four flag words of a quad first, so that their reads overlap
        uint2 w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = fc[in_tile(q, i) ? (q.col.v[i] - t_lo) >> 5 : 0];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (in_tile(q, i)) {
            const int rank = (int)w[i].y + __popc(w[i].x & ((1u << ((q.col.v[i] - t_lo) & 31)) - 1u));
            __hip_atomic_fetch_add(&acc[rank], (double)q.a * (double)q.b.v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
      });
      SPG_CLK(clk_mark(&ts->clk, 5);)
      // compress: sums and columns are already in ascending column order
      for (int r = tid; r < count; r += kThreads) stream_store(&c_val[out + r], (T)acc[r]);
      SPG_CLK(clk_mark(&ts->clk, 6);)
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kTileThreads, 8) void k_num_tiles(Control* ctl, const unsigned char* __restrict__ numbin, const TileRec* __restrict__ tiles,
                                                               const RunRec* __restrict__ runs, const int32_t* __restrict__ a_col,
                                                               const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                                               const int32_t* __restrict__ b_col, const T* __restrict__ b_val, int64_t n_cols,
                                                               const int* __restrict__ bp, int nb1, const int32_t* __restrict__ col_list, int64_t b_nnz,
                                                               const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val, int tiles3, int looked) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* tile = smem;                                                         // kTileBudget bytes
  TileScratch<T, false>* ts = reinterpret_cast<TileScratch<T, false>*>(smem + kTileBudget);
  if (ctl->error) return;
  const bool class3 = tiles3 != 0 && !other_order(ctl, looked);   // (in another order, or where hashing is asked for, k_row_tiles or the hash workspace does these rows)
  const int tid = threadIdx.x;
  const unsigned nruns = ctl->run_cursor;
  // The first lanes draw runs ahead of their use: the counter value for the run after next and the record of the next run, a word
  // to a lane, are on their way while the current run is in the works.
  constexpr int kRunWords = sizeof(RunRec) / 4;
  const int* run_words = reinterpret_cast<const int*>(runs);
  unsigned drawn = 0;
  int coming = 0;
  bool have_coming = false;
  SPG_CLK(clk_begin(&ts->clk);)
  if (tid < kRunWords) {
    if (tid == 0) drawn = atomicAdd(&ctl->work[1], 1u);
    have_coming = blockIdx.x < nruns;   // (the first draw is the workgroup's own)
    if (have_coming) coming = run_words[(size_t)run_of(blockIdx.x, nruns, nruns) * kRunWords + tid];
  }
  while (true) {
    __syncthreads();
    if (tid < kRunWords) {
      if (tid == 0) ts->s_run = have_coming ? 1 : -1;
      if (have_coming) reinterpret_cast<int*>(&ts->rr)[tid] = coming;
      const unsigned next = gridDim.x + (unsigned)uni((int)drawn);
      have_coming = next < nruns;
      if (have_coming) {
        coming = run_words[(size_t)run_of(next, nruns, nruns) * kRunWords + tid];
        if (tid == 0) drawn = atomicAdd(&ctl->work[1], 1u);
      }
    }
    __syncthreads();
    if (uni(ts->s_run) < 0) break;
    const RunRec rr = uni_run(ts->rr);
    if (rr.count == 0) continue;   // a record that its row did not need
    // one round trip: the row's class and position in C, the run's tile records, its A entries
    const int cls = numbin[rr.row];
    const int64_t out_row = c_rp[rr.row];
    if (tid < rr.count) ts->rec[tid] = tiles[rr.first + tid];
    int k = 0;
    T av = T(0);
    if (rr.d <= kTileThreads && tid < rr.d) {
      k = a_col[rr.a0 + tid];
      av = a_val[rr.a0 + tid];
    }
    if (!(cls == 3 && class3) && cls != 5 && cls != 6) continue;   // the row's numeric class is not this kernel's
    __syncthreads();
    SPG_CLK(clk_mark(&ts->clk, 0); clk_add(&ts->clk, 16, 1);)
    tile_run<kTileWaves, T, false>(rr, ts, tile, a_col, a_val, b_rp, b_col, b_val, n_cols, bp, nb1, col_list, b_nnz, out_row, c_col, c_val, k, av);
  }
  SPG_CLK(clk_mark(&ts->clk, 14); clk_flush(&ts->clk, ctl->clk[1]);)
}

// The rows of numeric class 3 without a tile in the plan (at most kSymHashLarge products; all of them where the entries of an ascending
// B come in another order than the plan's: a row as a whole is the same in any order), where the matrix has few columns: a row
// is one tile without structure, a workgroup of four waves each, several on a compute unit.  Marking the columns and ranking
// them by counting costs two passes over the products, the hash workspace its table, the slowest of 64 compare-and-swap loops
// and a sort: us hash (all rows of the class) | these kernels (with the rows that have tiles in k_num_tiles): R-MAT scale 14 (fp32)
// 101 | 46 + 2, of 5003 x 3001 x 7777 rows in any order 70 | 22 + 6, whole call of the numeric phase at scale 11 (fp64) 85 | 57.
// Up to 65536 columns (16 KB of flag words and ranks, four workgroups on a compute unit); wider matrices take the hash workspace.
constexpr int kRowTileWaves = 4;
constexpr int64_t kRowTileMaxCols = 8 * kBlkCols;
template <typename T>
__host__ __device__ constexpr size_t row_tile_bytes(int64_t n_cols) {   // flag words and ranks, sums
  return (size_t)((n_cols + kBlkCols - 1) / kBlkCols) * kRankBlkBytes + (size_t)kNumHashLarge * 8;
}
template <typename T>
constexpr size_t row_tile_lds(int64_t n_cols) { return row_tile_bytes<T>(n_cols) + sizeof(TileScratch<T, true, kRowTileWaves>); }

template <typename T>
__device__ __forceinline__ void row_tiles_rows(unsigned char* smem, unsigned wg, unsigned wgs, const int* __restrict__ perm,
    const Control* __restrict__ ctl, const int* __restrict__ ip_row, int most_ip, const int64_t* __restrict__ a_rp,
    const int32_t* __restrict__ a_col, const T* __restrict__ a_val, const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col,
    const T* __restrict__ b_val, int64_t b_nnz, int64_t n_cols, const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val,
    int looked) {
  TileScratch<T, true, kRowTileWaves>* ts = reinterpret_cast<TileScratch<T, true, kRowTileWaves>*>(smem + row_tile_bytes<T>(n_cols));
  if (other_order(ctl, looked)) most_ip = 0x7fffffff;
  const unsigned first = ctl->offset[1][3], nrows = ctl->offset[1][4] - first;
  const int tid = threadIdx.x;
  for (unsigned i = wg; i < nrows; i += wgs) {
    const int row = perm[first + i];
    if (ip_row[row] > most_ip) continue;   // done by its tiles
    const int64_t a0 = a_rp[row], out = c_rp[row];
    const int d = (int)(a_rp[row + 1] - a0);
    const int64_t n = c_rp[row + 1] - out;
    const int cnt = n < kNumHashLarge ? (int)n : kNumHashLarge;
    if (tid == 0) ts->rec[0] = TileRec{0, (int)((n_cols + kBlkCols - 1) >> kBlkShift), cnt, 0};
    int k = 0;
    T av = T(0);
    if (d <= kRowTileWaves * kWave && tid < d) { k = a_col[a0 + tid]; av = a_val[a0 + tid]; }
    __syncthreads();
    tile_run<kRowTileWaves, T, true>(RunRec{row, 0, 1, d, a0, -1}, ts, smem, a_col, a_val, b_rp, b_col, b_val, n_cols, (const int*)nullptr, 0,
                                     (const int32_t*)nullptr, b_nnz, out, c_col, c_val, k, av);
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(kRowTileWaves * kWave, 4) void k_row_tiles(const int* __restrict__ perm, const Control* __restrict__ ctl, const int* __restrict__ ip_row, int most_ip,
                                                                        const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                                                        const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                                                        const int32_t* __restrict__ b_col, const T* __restrict__ b_val, int64_t b_nnz, int64_t n_cols,
                                                                        const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val, int looked) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (ctl->error) return;
  row_tiles_rows<T>(smem, blockIdx.x, gridDim.x, perm, ctl, ip_row, most_ip, a_rp, a_col, a_val, b_rp, b_col, b_val, b_nnz, n_cols, c_rp, c_col,
      c_val, looked);
}

template <typename T>
constexpr size_t num_tiles_lds() { return (size_t)kTileBudget + sizeof(TileScratch<T, false>); }

}  // namespace spg
