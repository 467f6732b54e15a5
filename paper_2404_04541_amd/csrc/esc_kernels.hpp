// Sorted-list (sparse) workspace for short rows: every intermediate product of a row is
// appended to a small coordinate list (insert), the list is put in column order (sort) and runs
// of equal columns are summed (merge).  This is the expand / sort / reduce-by-key policy of the
// paper's table of library algorithms (section 4.4) run at wavefront level, one row per GROUP lanes.
//
// Symbolic (k_esc_sym): the columns, each with its position in the list below it in one word, are
//   sorted in registers; the row's size is the number of different columns, and the sorted words
//   stay in the plan.
// Numeric with the plan's words (k_esc_num): the products go to LDS by position and every sorted
//   word fetches its own; neither the columns nor their order is found again.
// Numeric without them (k_esc; no room in the plan, or columns too large for a shared word): insert,
//   a count of the entries before each entry, merge.
// Bound: the gathers of B, a 128-byte line per A entry and array: 4.2 M rows of 8 entries times 4.2 M rows of 4 (fp64) move
// 55 to 59 G missed lines a second (7 TB/s) in the row count and in both kernels here.  So nothing is gathered twice: the
// columns by the symbolic kernel, the values by the numeric one, B's row pointer by the row count (wants_desc).  That
// product: symbolic 1.26 -> 0.73 ms, numeric 2.51 -> 1.17 ms (with the row pointer gathered again 1.31 and 1.63 ms).
// Where B stays in the caches the loads still depend on each other, hence the chain kept four rows deep: 2048 x 2048 rows of
// 2.4 entries times rows of 16 (fp64): symbolic 1.34 -> 0.93 ms, numeric 1.83 -> 1.33 ms.
#pragma once
#include "common.hpp"
#include "row_chain.hpp"

namespace spg {

// ---- with the plan's sorted words -------------------------------------------------------

// Products of one chunk of a row's A entries: the lane's entry has len products from position bs of B on, the first of them
// is product pos of the row.  With B rows of at most four entries a lane takes its own entry's products; otherwise the quads (up to four consecutive
// products) of all entries are dealt to the lanes: ent and map describe them in LDS.
struct __align__(16) EscEntry { unsigned bs_lo, bs_hi; int len; int first_pos; };   // first quad | first product << 16

template <int GROUP, int CAP>
struct EscLds {
  EscEntry ent[GROUP];
  unsigned char map[CAP];   // lane + 1 of the entry whose first quad this is, 0: a later quad of the entry before
};

// The value of the group's last lane.
template <int GROUP>
__device__ __forceinline__ int group_last(int v) {
  if constexpr (GROUP == kWave) return __builtin_amdgcn_readlane(v, kWave - 1);
  else return __shfl(v, GROUP - 1, GROUP);
}

// Calls quad(lane of the entry inside the group, first product's position in the row, its index in B's arrays, products) for
// quads of the chunk; all lanes of the wave call together, lanes without a quad with 0 products.
template <int GROUP, int CAP, class F>
__device__ __forceinline__ void esc_quads(int64_t bs, int len, int pos, EscLds<GROUP, CAP>* lds, F quad) {
  const int gl = lane_id() & (GROUP - 1);
  if (!__any(len > 4)) {
    quad(gl, pos, bs, len);
    return;
  }
  const int quads = (len + 3) >> 2;
  const int incl = group_incl_scan<GROUP>(quads);
  const int nq = group_last<GROUP>(incl);
  const int first = incl - quads;
  for (int t = gl; t < CAP; t += GROUP) lds->map[t] = 0;
  group_sync<GROUP>();
  if (quads > 0 && first < CAP) {
    *reinterpret_cast<int4*>(&lds->ent[gl]) = make_int4((int)(unsigned)(unsigned long long)bs, (int)((unsigned long long)bs >> 32), len, first | (pos << 16));
    lds->map[first] = (unsigned char)(gl + 1);
  }
  group_sync<GROUP>();
  int carry = 0;
  for (int t0 = 0; __any(t0 < nq); t0 += GROUP) {
    const int t = t0 + gl;
    int m = group_max_scan<GROUP>((int)lds->map[t < CAP ? t : CAP - 1]);
    m = m > carry ? m : carry;
    carry = group_last<GROUP>(m);
    const bool on = t < nq;
    const int src = on ? m - 1 : 0;
    const int4 e = *reinterpret_cast<const int4*>(&lds->ent[src]);
    const int off = (t - (e.w & 0xffff)) * 4;
    const int64_t q = (int64_t)(((unsigned long long)(unsigned)e.y << 32) | (unsigned)e.x) + off;
    quad(src, (e.w >> 16) + off, on ? q : 0, on ? (e.z - off < 4 ? e.z - off : 4) : 0);
  }
  group_sync<GROUP>();
}

template <int GROUP>
__device__ __forceinline__ int group_number() {   // (wave-uniform where a group is a wave: its row's description then stays in scalar registers)
  const int g = threadIdx.x / GROUP;
  return GROUP == kWave ? __builtin_amdgcn_readfirstlane(g) : g;
}

// cnt[row] = different columns of the row; words (optional): CAP per row of the bin, (column << log2 CAP) | position, sorted.
// DESC: the row count has left the B rows of A's entries (desc).  pack != 0: such words fit 32 bits with the padding behind them.
// (the register bounds are the smallest that spill nothing to speak of: one step further costs half of the speed)
template <int GROUP, int CAP>
struct EscSymLds {
  __align__(16) unsigned keys[256 / GROUP][CAP];
  EscLds<GROUP, CAP> quads[256 / GROUP];
};

template <int GROUP, int CAP, bool DESC>
__device__ __forceinline__ void esc_sym_rows(EscSymLds<GROUP, CAP>* lds, unsigned wg, unsigned wgs, const int* __restrict__ perm,
    const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const int64_t* __restrict__ b_rp,
    const unsigned long long* __restrict__ desc, const int32_t* __restrict__ b_col, int64_t b_nnz, int pack, int* __restrict__ cnt,
    unsigned* __restrict__ words) {
  static_assert(CAP == 2 * GROUP && (CAP == 32 || CAP == 128), "each lane owns two list positions");
  constexpr int kGroups = 256 / GROUP;
  constexpr int kLogCap = CAP == 32 ? 5 : 7;
  const unsigned first = ctl->offset[0][bin];
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = group_number<GROUP>(), gl = threadIdx.x % GROUP;
  unsigned* keys = lds->keys[g];
  const int shift = pack ? kLogCap : 0, pmask = pack ? CAP - 1 : 0;
  const unsigned ngroups = wgs * kGroups;
  RowChain<GROUP> ch{perm + first, a_rp, a_col, b_rp, DESC ? desc : nullptr, nrows, ngroups};
  unsigned slot = wg * kGroups + g;
  ch.start(slot);
  const unsigned rounds = (nrows + ngroups - 1) / ngroups;   // (the same for every group: the wave's lanes stay together)
  for (unsigned r = 0; r < rounds; ++r, slot += ngroups) {
    const typename RowChain<GROUP>::Ahead nx = ch.fetch();
    const int row = ch.row, d = ch.d;
    int filled = 0;
    for (int c = 0; __any(c < d || c == 0); c += GROUP) {
      if (c > 0) ch.fetch_more(c);
      const int len = (int)(ch.bounds.v[1] - ch.bounds.v[0]);
      const int incl = group_incl_scan<GROUP>(len);
      esc_quads<GROUP, CAP>(ch.bounds.v[0], len, filled + incl - len, &lds->quads[g], [&](int, int pos, int64_t q, int n) {
        int col[4];
        load_quad<int32_t>(b_col, q, n, b_nnz, col);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u < n) keys[(pos + u) & (CAP - 1)] = ((unsigned)col[u] << shift) | (unsigned)((pos + u) & pmask);
      });
      filled += group_last<GROUP>(incl);
    }
    group_sync<GROUP>();
    int heads;
    const bool two = __any(filled > GROUP);
    if (two) {
      const uint2 v = *reinterpret_cast<const uint2*>(&keys[2 * gl]);
      unsigned k[2] = {2 * gl < filled ? v.x : ~0u, 2 * gl + 1 < filled ? v.y : ~0u};
      lane_sort<CAP, 2>(k, gl);
      const unsigned before = (unsigned)__shfl_up((int)k[1], 1, GROUP) >> shift;
      heads = ((2 * gl < filled && (gl == 0 || k[0] >> shift != before)) ? 1 : 0) + ((2 * gl + 1 < filled && k[1] >> shift != k[0] >> shift) ? 1 : 0);
      if (words && 2 * gl < filled) *reinterpret_cast<uint2*>(words + (size_t)slot * CAP + 2 * gl) = make_uint2(k[0], k[1]);
    } else {
      unsigned k[1] = {gl < filled ? keys[gl] : ~0u};
      lane_sort<GROUP, 1>(k, gl);
      const unsigned before = (unsigned)__shfl_up((int)k[0], 1, GROUP) >> shift;
      heads = (gl < filled && (gl == 0 || k[0] >> shift != before)) ? 1 : 0;
      if (words && gl < filled) words[(size_t)slot * CAP + gl] = k[0];
    }
    const int total = group_incl_scan<GROUP>(heads);
    if (row >= 0 && gl == GROUP - 1) cnt[row] = total;
    group_sync<GROUP>();
    ch.advance(nx);
  }
}

template <int GROUP, int CAP, bool DESC>
__global__ __launch_bounds__(256, 6) void k_esc_sym(const int* __restrict__ perm, const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp,
                                                 const int32_t* __restrict__ a_col, const int64_t* __restrict__ b_rp, const unsigned long long* __restrict__ desc, const int32_t* __restrict__ b_col,
                                                 int64_t b_nnz, int pack, int* __restrict__ cnt, unsigned* __restrict__ words) {
  __shared__ EscSymLds<GROUP, CAP> lds;
  if (ctl->error) return;
  esc_sym_rows<GROUP, CAP, DESC>(&lds, blockIdx.x, gridDim.x, perm, ctl, bin, a_rp, a_col, b_rp, desc, b_col, b_nnz, pack, cnt, words);
}

// The rows of C from the plan's sorted words.  Lane gl owns the sorted positions gl and gl + GROUP.
template <int GROUP, int CAP>
struct EscNumLds {
  double vals[256 / GROUP][CAP];
  unsigned cols[256 / GROUP][CAP];
  EscLds<GROUP, CAP> quads[256 / GROUP];
  double av[256 / GROUP][GROUP];
};

template <int GROUP, int CAP, typename T, bool DESC>
__device__ __forceinline__ void esc_num_rows(EscNumLds<GROUP, CAP>* lds, unsigned wg, unsigned wgs, const int* __restrict__ perm,
    const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const T* __restrict__ a_val,
    const int64_t* __restrict__ b_rp, const unsigned long long* __restrict__ desc, const T* __restrict__ b_val, int64_t b_nnz,
    const unsigned* __restrict__ words, const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val) {
  static_assert(CAP == 2 * GROUP && (CAP == 32 || CAP == 128), "each lane owns two list positions");
  constexpr int kGroups = 256 / GROUP;
  constexpr int kLogCap = CAP == 32 ? 5 : 7;
  const unsigned first = ctl->offset[0][bin];   // (the bins of rows this short are the same in both phases)
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = group_number<GROUP>(), gl = threadIdx.x % GROUP;
  double* vals = lds->vals[g];
  unsigned* cols = lds->cols[g];
  double* s_a = lds->av[g];
  const unsigned ngroups = wgs * kGroups;
  auto value = [&](int64_t a, int n) { return gl < n ? a_val[a + gl] : T(0); };
  auto position = [&](int row) { return row >= 0 ? c_rp[row] : 0; };
  RowChain<GROUP> ch{perm + first, a_rp, a_col, b_rp, DESC ? desc : nullptr, nrows, ngroups};
  unsigned slot = wg * kGroups + g;
  ch.start(slot);
  T av0 = value(ch.a0, ch.d), av1 = value(ch.a01, ch.d1);
  int64_t out0 = position(ch.row), out1 = position(ch.row1), out2 = position(ch.row2);
  const unsigned rounds = (nrows + ngroups - 1) / ngroups;
  for (unsigned r = 0; r < rounds; ++r, slot += ngroups) {
    const typename RowChain<GROUP>::Ahead nx = ch.fetch();
    const T av2 = value(ch.a02, ch.d2);
    const int64_t out3 = position(ch.row3);
    const int d = ch.d;
    const unsigned* w = words + (size_t)slot * CAP;
    // (the row's words are on their way while its products are formed; what lies behind the row's last product is not used)
    const bool live = ch.row >= 0;
    const unsigned w0 = live ? w[gl] : ~0u, w1 = live ? w[gl + GROUP] : ~0u;
    int filled = 0;
    for (int c = 0; __any(c < d || c == 0); c += GROUP) {
      T av = av0;
      if (c > 0) {
        ch.fetch_more(c);
        av = c + gl < d ? a_val[ch.a0 + c + gl] : T(0);
      }
      const int len = (int)(ch.bounds.v[1] - ch.bounds.v[0]);
      const int incl = group_incl_scan<GROUP>(len);
      s_a[gl] = (double)av;
      group_sync<GROUP>();
      esc_quads<GROUP, CAP>(ch.bounds.v[0], len, filled + incl - len, &lds->quads[g], [&](int src, int pos, int64_t q, int n) {
        T b[4];
        load_quad<T>(b_val, q, n, b_nnz, b);
        const double a = s_a[src];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u < n) vals[(pos + u) & (CAP - 1)] = a * (double)b[u];
      });
      filled += group_last<GROUP>(incl);
      group_sync<GROUP>();
    }
    group_sync<GROUP>();
    const int n = filled < CAP ? filled : CAP;
    const bool in0 = gl < n, in1 = gl + GROUP < n;
    const unsigned c0 = in0 ? w0 >> kLogCap : ~0u, c1 = in1 ? w1 >> kLogCap : ~0u;
    const unsigned p0 = (unsigned)__shfl_up((int)c0, 1, GROUP), p1s = (unsigned)__shfl_up((int)c1, 1, GROUP), last = (unsigned)__shfl((int)c0, GROUP - 1, GROUP);
    const bool h0 = in0 && (gl == 0 || c0 != p0), h1 = in1 && c1 != (gl == 0 ? last : p1s);
    double v0 = vals[w0 & (CAP - 1)], v1 = vals[w1 & (CAP - 1)];
    int r0 = gl, r1 = gl + GROUP;
    if (__any((in0 && !h0) || (in1 && !h1))) {   // some row of the wave has a column twice: runs are summed in the order of their products
      if (in0) cols[gl] = w0;
      if (in1) cols[gl + GROUP] = w1;
      const int i0 = group_incl_scan<GROUP>(h0 ? 1 : 0), i1 = group_incl_scan<GROUP>(h1 ? 1 : 0);
      r0 = i0 - 1;
      r1 = __shfl(i0, GROUP - 1, GROUP) + i1 - 1;
      group_sync<GROUP>();
      if (h0) for (int t = gl + 1; t < n && cols[t] >> kLogCap == c0; ++t) v0 += vals[cols[t] & (CAP - 1)];
      if (h1) for (int t = gl + GROUP + 1; t < n && cols[t] >> kLogCap == c1; ++t) v1 += vals[cols[t] & (CAP - 1)];
    }
    if (h0) { c_col[out0 + r0] = (int32_t)c0; c_val[out0 + r0] = (T)v0; }
    if (h1) { c_col[out0 + r1] = (int32_t)c1; c_val[out0 + r1] = (T)v1; }
    group_sync<GROUP>();
    ch.advance(nx);
    av0 = av1; av1 = av2;
    out0 = out1; out1 = out2; out2 = out3;
  }
}

template <int GROUP, int CAP, typename T, bool DESC>
__global__ __launch_bounds__(256, GROUP == kWave ? 6 : 5) void k_esc_num(const int* __restrict__ perm, const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp,
                                                 const int32_t* __restrict__ a_col, const T* __restrict__ a_val, const int64_t* __restrict__ b_rp, const unsigned long long* __restrict__ desc,
                                                 const T* __restrict__ b_val, int64_t b_nnz, const unsigned* __restrict__ words,
                                                 const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val) {
  __shared__ EscNumLds<GROUP, CAP> lds;
  if (ctl->error || ctl->order_differs) return;
  esc_num_rows<GROUP, CAP, T, DESC>(&lds, blockIdx.x, gridDim.x, perm, ctl, bin, a_rp, a_col, a_val, b_rp, desc, b_val, b_nnz, words, c_rp, c_col,
      c_val);
}

// ---- without them --------------------------------------------------------------------------

// Number of list entries before entry e with key k: those with a smaller key, and with TIE also those
// with the same key at an earlier position (without TIE the keys are distinct).  The lanes of a group
// read the list together, four keys at a time (one address for the group: no bank conflicts).
template <bool TIE>
__device__ __forceinline__ int count_before(const int* keys, int nscan, unsigned k, int e) {
  int r = 0;
#pragma unroll 2
  for (int j = 0; j < nscan; j += 4) {
    const int4 q = *reinterpret_cast<const int4*>(&keys[j]);
    r += (unsigned)q.x < k + ((TIE && j + 0 < e) ? 1u : 0u) ? 1 : 0;
    r += (unsigned)q.y < k + ((TIE && j + 1 < e) ? 1u : 0u) ? 1 : 0;
    r += (unsigned)q.z < k + ((TIE && j + 2 < e) ? 1u : 0u) ? 1 : 0;
    r += (unsigned)q.w < k + ((TIE && j + 3 < e) ? 1u : 0u) ? 1 : 0;
  }
  return r;
}

// GROUP lanes per row (16 or 64), list capacity CAP = 2 * GROUP products; workgroup wg of wgs.
// Writes the merged (column, value) run at c_rp[row]; pack != 0: every column shifted left by
// log2(CAP) stays below the padding key, so a key can carry its list position.
template <int GROUP, int CAP, typename T>
struct EscRowsLds {
  __align__(16) int keys[256 / GROUP][CAP];
  double vals[256 / GROUP][CAP];
};

template <int GROUP, int CAP, typename T>
__device__ __forceinline__ void esc_rows(EscRowsLds<GROUP, CAP, T>* lds, unsigned wg, unsigned wgs, const int* __restrict__ perm, const Control* __restrict__ ctl,
                                         int phase, int bin, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                         const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                         const int32_t* __restrict__ b_col, const T* __restrict__ b_val,
                                         const int64_t* __restrict__ c_rp,
                                         int32_t* __restrict__ c_col, T* __restrict__ c_val, int pack, int64_t b_nnz) {
  static_assert(CAP == 2 * GROUP, "each lane owns two list positions");
  constexpr int kGroups = 256 / GROUP;
  constexpr int kLogCap = CAP == 32 ? 5 : 7;
  static_assert((1 << kLogCap) == CAP, "list capacities 32 and 128");
  const int shift = pack ? kLogCap : 0;   // a numeric key: (column << shift) | position
  const int pmask = pack ? CAP - 1 : 0;
  constexpr int kSpreadMax = 16;   // A entries up to which a wave deals a row's products, not its entries, to its lanes
  const unsigned first = ctl->offset[phase][bin];
  const unsigned nrows = ctl->offset[phase][bin + 1] - first;
  const int g = threadIdx.x / GROUP;   // group inside the workgroup
  const int gl = threadIdx.x % GROUP;  // lane inside the group
  int* keys = lds->keys[g];
  double* vals = lds->vals[g];
  const unsigned ngroups = wgs * kGroups;
  // every wave iterates the same number of times so that the shuffles below always see
  // all 64 lanes; groups past the end of the bin run on an empty row
  const unsigned rounds = (nrows + ngroups - 1) / ngroups;
  for (unsigned r = 0; r < rounds; ++r) {
    const unsigned slot = r * ngroups + wg * kGroups + g;
    const bool live = slot < nrows;
    const int row = live ? perm[first + slot] : 0;
    const int64_t a0 = live ? a_rp[row] : 0;
    const int d = live ? (int)(a_rp[row + 1] - a0) : 0;
    // ---- insert: lane-per-A-entry, positions from a running prefix of B row lengths
    int filled = 0;
    int dmax = d;
#pragma unroll
    for (int s = GROUP; s < kWave; s <<= 1) { int o = __shfl_xor(dmax, s, kWave); dmax = o > dmax ? o : dmax; }
    for (int c = 0; c < dmax; c += GROUP) {
      const int e = c + gl;
      int64_t bs = 0; int len = 0; double av = 0.0;
      if (e < d) {
        const int k = a_col[a0 + e];
        const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k);
        bs = bounds.v[0];
        len = (int)(bounds.v[1] - bs);
        av = (double)a_val[a0 + e];
      }
      const int incl = group_incl_scan<GROUP>(len);
      if constexpr (GROUP == kWave) {
        // one row per wave: with few A entries most lanes would idle while a few walk their B rows, so
        // the products themselves are dealt to the lanes (at most two each); a lane finds the entry of
        // its product by counting the entries that end at or before it
        const int nent = __builtin_amdgcn_readfirstlane(d - c);
        if (nent <= kSpreadMax) {
          const int batch = __builtin_amdgcn_readlane(incl, kWave - 1);
          int cc[2];
          T vv[2];
          double aa[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int t = gl + u * kWave;
            const bool ok = t < batch;
            int ent = 0;
            for (int x = 0; x < nent; ++x) ent += __builtin_amdgcn_readlane(incl, x) <= t ? 1 : 0;
            if (!ok) ent = 0;
            const int ent_first = __shfl(incl - len, ent, kWave);
            const long long ent_bs = __shfl((long long)bs, ent, kWave);
            aa[u] = __shfl(av, ent, kWave);
            const long long q = ent_bs + (t - ent_first);
            cc[u] = ok ? b_col[q] : 0;
            vv[u] = ok ? b_val[q] : T(0);
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int t = gl + u * kWave;
            if (t < batch) {
              keys[filled + t] = (cc[u] << shift) | ((filled + t) & pmask);
              vals[filled + t] = aa[u] * (double)vv[u];
            }
          }
          filled += batch;
          continue;
        }
      }
      int pos = filled + incl - len;
      for (int t0 = 0; t0 < len; t0 += 4) {   // four loads in flight per lane
        int cc[4];
        T vv[4];
        if (bs + t0 + 4 <= b_nnz) {   // four elements exist behind the position, whatever the row's length
          const Run<int32_t, 4> qc = load_run<int32_t, 4>(b_col + bs + t0);
#pragma unroll
          for (int u = 0; u < 4; ++u) cc[u] = qc.v[u];
          const Run<T, 4> qv = load_run<T, 4>(b_val + bs + t0);
#pragma unroll
          for (int u = 0; u < 4; ++u) vv[u] = qv.v[u];
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const bool ok = t0 + u < len;
            cc[u] = ok ? b_col[bs + t0 + u] : 0;
            vv[u] = ok ? b_val[bs + t0 + u] : T(0);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (t0 + u < len) {
            keys[pos + t0 + u] = (cc[u] << shift) | ((pos + t0 + u) & pmask);
            vals[pos + t0 + u] = av * (double)vv[u];
          }
        }
      }
      filled += __shfl(incl, GROUP - 1, GROUP);
    }
    // pad the tail so that it sorts behind every real column
    for (int t = filled + gl; t < CAP; t += GROUP) keys[t] = kPadKey;
    group_sync<GROUP>();
    // ---- sort and merge.  With values, an exchange in a sorting network would carry 12 bytes through
    // LDS per entry and stage; instead every lane looks at its two entries (positions gl and gl + GROUP;
    // the second only when some row of the wave has that many) against the whole list.
    const int e0 = gl, e1 = gl + GROUP;
    const bool two = __any(filled > GROUP);
    int nscan = CAP;
    if constexpr (GROUP == kWave) nscan = __builtin_amdgcn_readfirstlane((filled + 3) & ~3);
    {
      // an entry's place in column order is the number of entries before it (smaller column,
      // or the same column and an earlier position); entries go there, then runs of equal columns are summed
      const unsigned ka = (unsigned)keys[e0], kb = (unsigned)keys[e1];
      const double va = vals[e0], vb = vals[e1];
      int ra = 0, rb = 0;
      if (pack) {
        ra = count_before<false>(keys, nscan, ka, e0);
        if (two) rb = count_before<false>(keys, nscan, kb, e1);
      } else {
        ra = count_before<true>(keys, nscan, ka, e0);
        if (two) rb = count_before<true>(keys, nscan, kb, e1);
      }
      group_sync<GROUP>();
      // (positions from `filled` on hold padding and stay as they are)
      if (e0 < filled) { keys[ra] = (int)(ka >> shift); vals[ra] = va; }
      if (e1 < filled) { keys[rb] = (int)(kb >> shift); vals[rb] = vb; }
      group_sync<GROUP>();
      // a list position is a head when its column differs from its left neighbour
      const int i0 = 2 * gl, i1 = 2 * gl + 1;
      const int k0 = keys[i0], k1 = keys[i1];
      const int kprev = i0 > 0 ? keys[i0 - 1] : -1;
      const int h0 = (i0 < filled && k0 != kprev) ? 1 : 0;
      const int h1 = (i1 < filled && k1 != k0) ? 1 : 0;
      const int incl = group_incl_scan<GROUP>(h0 + h1);
      if (live) {
        const int64_t out = c_rp[row];
        int rank = incl - (h0 + h1);
        if (h0) {
          double s = vals[i0];
          for (int t = i0 + 1; t < filled && keys[t] == k0; ++t) s += vals[t];
          c_col[out + rank] = k0;
          c_val[out + rank] = (T)s;
          ++rank;
        }
        if (h1) {
          double s = vals[i1];
          for (int t = i1 + 1; t < filled && keys[t] == k1; ++t) s += vals[t];
          c_col[out + rank] = k1;
          c_val[out + rank] = (T)s;
        }
      }
    }
    group_sync<GROUP>();
  }
}

template <int GROUP, int CAP, typename T>
__global__ __launch_bounds__(256) void k_esc(const int* __restrict__ perm, const Control* __restrict__ ctl, int phase, int bin,
                                              const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
                                              const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                              const int32_t* __restrict__ b_col, const T* __restrict__ b_val,
                                              const int64_t* __restrict__ c_rp,
                                              int32_t* __restrict__ c_col, T* __restrict__ c_val, int pack, int64_t b_nnz) {
  __shared__ EscRowsLds<GROUP, CAP, T> lds;
  if (ctl->error) return;
  esc_rows<GROUP, CAP, T>(&lds, blockIdx.x, gridDim.x, perm, ctl, phase, bin, a_rp, a_col, a_val, b_rp, b_col, b_val, c_rp, c_col, c_val, pack, b_nnz);
}

}  // namespace spg
