// Flag-list workspace for short rows of a product with few columns: one bit per column of B in LDS, 16 lanes per row.  The row's
// size is the number of set bits, a column's place in the row the number of bits before it: nothing is sorted, hashed or kept
// between the phases (the numeric one marks the columns again, which is why B's columns have to be close by: flag_rows_ok).
// This is Gustavson's flag list of the paper's section 4.4 at the scale of a DPP row.
//
// Bound: vector instructions (0.9 of the issue slots in the sorted-list kernels, whose bitonic networks these replace).
// 2048 x 2048 rows of 2.4 entries times 2048 rows of 16 entries (fp64, 2048 columns), us sorted list | flags: symbolic 234 + 644 |
// 129 + 147, numeric 437 + 886 | 460 + 779 (rows of at most 32 and of at most 128 products); the whole product 3324 | 2669.
#pragma once
#include "common.hpp"
#include "row_chain.hpp"
#include "esc_kernels.hpp"

namespace spg {

constexpr int kFlagGroup = 16;                                  // lanes per row
constexpr int kFlagRows = 256 / kFlagGroup;                     // rows of a workgroup in the works
// 8192: sixteen words of flags per lane.  With 32 (16000 columns, as at kFlagMaxNnz) 8 times 4 took 611 us against 572 with the
// sorted list, 8 times 12 1112 against 1231: the flags' LDS leaves two workgroups on a compute unit.
constexpr int64_t kFlagMaxCols = 16 * kFlagGroup * 32;

// Words of flags per lane for a matrix of so many columns (4, 8 or 16).
inline int flag_words_per_lane(int64_t cols) {
  int words = 4;
  while (cols > words * kFlagGroup * 32) words *= 2;
  return words;
}

// The flags of a group: lane gl owns words 4 (16 j + gl) .. + 3 for j below WPL / 4.
template <int WPL>
__device__ __forceinline__ void flags_clear(unsigned* flags, int gl) {
#pragma unroll
  for (int j = 0; j < WPL / 4; ++j) reinterpret_cast<uint4*>(flags)[j * kFlagGroup + gl] = make_uint4(0, 0, 0, 0);
}

// The quads (up to four consecutive products) of a chunk of a row's A entries, an entry to a lane: with B rows of at most four
// entries a lane takes its own, otherwise the quads of all entries are dealt to the lanes.
// (described in LDS as the sorted list does it: EscEntry, EscLds)
template <int CAP>
using FlagLds = EscLds<kFlagGroup, CAP>;

template <int CAP>
struct FlagWalk {
  FlagLds<CAP>* lds;
  int64_t bs;
  int len, pos, quads, carry;
  bool own;
  // All lanes of the wave together; the lane's entry has n products from position p of B on, the first of them is product at of
  // the row.
  __device__ __forceinline__ void begin(int64_t p, int n, int at) {
    const int gl = lane_id() & (kFlagGroup - 1);
    bs = p; len = n; pos = at; carry = 0;
    own = !__any(n > 4);
    quads = kFlagGroup;
    if (own) return;
    const int mine = (n + 3) >> 2;
    const int incl = group_incl_scan<kFlagGroup>(mine);
    const int first = incl - mine;
    quads = group_last<kFlagGroup>(incl);
    using Clear = std::conditional_t<CAP == 32, unsigned short, unsigned long long>;
    static_assert(sizeof(Clear) * kFlagGroup == CAP, "one store a lane");
    group_sync<kFlagGroup>();
    reinterpret_cast<Clear*>(lds->map)[gl] = 0;
    group_sync<kFlagGroup>();
    if (mine > 0 && first < CAP) {
      *reinterpret_cast<int4*>(&lds->ent[gl]) = make_int4((int)(unsigned)(unsigned long long)p, (int)((unsigned long long)p >> 32), n, first | (at << 16));
      lds->map[first] = (unsigned char)(gl + 1);
    }
    group_sync<kFlagGroup>();
  }
  // Quad t0 + gl, in order from t0 = 0 on: the lane of its entry, its first product's number, its place in B, its products (0: none).
  __device__ __forceinline__ void next(int t0, int& src, int& at, int64_t& q, int& n) {
    const int gl = lane_id() & (kFlagGroup - 1);
    if (own) { src = gl; at = pos; q = bs; n = len; return; }
    const int t = t0 + gl;
    int m = group_max_scan<kFlagGroup>((int)lds->map[t < CAP ? t : CAP - 1]);
    m = m > carry ? m : carry;
    carry = group_last<kFlagGroup>(m);
    const bool on = t < quads && m > 0;
    src = on ? m - 1 : 0;
    const int4 e = *reinterpret_cast<const int4*>(&lds->ent[src]);
    const int off = (t - (e.w & 0xffff)) * 4;
    at = (e.w >> 16) + off;
    q = on ? (int64_t)(((unsigned long long)(unsigned)e.y << 32) | (unsigned)e.x) + off : 0;
    n = on ? (e.z - off < 4 ? e.z - off : 4) : 0;
  }
};

template <int WPL>
__device__ __forceinline__ void flags_mark(unsigned* flags, const int (&col)[4], int n) {
#pragma unroll
  for (int u = 0; u < 4; ++u)   // (operands of another structure than the plan's stay inside LDS, here and below)
    if (u < n) atomicOr(&flags[((unsigned)col[u] >> 5) & (WPL * kFlagGroup - 1)], 1u << (col[u] & 31));
}

// cnt[row] = different columns of the row.
template <int CAP, int WPL>
__global__ __launch_bounds__(256, 6) void k_flag_sym(const int* __restrict__ perm, const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp,
                                                     const int32_t* __restrict__ a_col, const int64_t* __restrict__ b_rp, const int32_t* __restrict__ b_col,
                                                     int64_t b_nnz, int* __restrict__ cnt) {
  __shared__ __align__(16) unsigned s_flags[kFlagRows][WPL * kFlagGroup];
  __shared__ FlagLds<CAP> s_lds[kFlagRows];
  if (ctl->error) return;
  const unsigned first = ctl->offset[0][bin];
  const unsigned nrows = ctl->offset[0][bin + 1] - first;
  const int g = threadIdx.x / kFlagGroup, gl = threadIdx.x % kFlagGroup;
  unsigned* flags = s_flags[g];
  const unsigned ngroups = gridDim.x * kFlagRows;
  RowChain<kFlagGroup> ch{perm + first, a_rp, a_col, b_rp, nullptr, nrows, ngroups};
  ch.start(blockIdx.x * kFlagRows + g);
  FlagWalk<CAP> walk{&s_lds[g]};
  const unsigned rounds = (nrows + ngroups - 1) / ngroups;   // (the same for every group: the wave's lanes stay together)
  for (unsigned r = 0; r < rounds; ++r) {
    const RowChain<kFlagGroup>::Ahead nx = ch.fetch();
    flags_clear<WPL>(flags, gl);
    group_sync<kFlagGroup>();
    for (int c = 0; __any(c < ch.d || c == 0); c += kFlagGroup) {
      if (c > 0) ch.fetch_more(c);
      walk.begin(ch.bounds.v[0], (int)(ch.bounds.v[1] - ch.bounds.v[0]), 0);
      for (int t0 = 0; __any(t0 < walk.quads); t0 += kFlagGroup) {
        int src, at, n, col[4];
        int64_t q;
        walk.next(t0, src, at, q, n);
        load_quad<int32_t>(b_col, q, n, b_nnz, col);
        flags_mark<WPL>(flags, col, n);
      }
    }
    group_sync<kFlagGroup>();
    int mine = 0;
#pragma unroll
    for (int j = 0; j < WPL / 4; ++j) {
      const uint4 v = reinterpret_cast<const uint4*>(flags)[j * kFlagGroup + gl];
      mine += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    const int total = group_incl_scan<kFlagGroup>(mine);
    if (ch.row >= 0 && gl == kFlagGroup - 1) cnt[ch.row] = total;
    group_sync<kFlagGroup>();
    ch.advance(nx);
  }
}

// The rows of C.  The products go to LDS by number while their columns are marked; with the places known every lane takes its
// share of them back (kept in registers as quads instead they spill: 32-product rows 484 -> 1330 us) and puts them there, or
// adds them where a column comes twice.
// (Four waves a SIMD by registers for rows of 128 products; with 16 words of flags a lane the 48 KB of LDS leave three.)
template <int CAP, int WPL, typename T>
__global__ __launch_bounds__(256, CAP == 32 ? 5 : 4) void k_flag_num(const int* __restrict__ perm, const Control* __restrict__ ctl, int bin, const int64_t* __restrict__ a_rp,
                                                     const int32_t* __restrict__ a_col, const T* __restrict__ a_val, const int64_t* __restrict__ b_rp,
                                                     const int32_t* __restrict__ b_col, const T* __restrict__ b_val, int64_t b_nnz,
                                                     const int64_t* __restrict__ c_rp, int32_t* __restrict__ c_col, T* __restrict__ c_val) {
  constexpr int kPer = CAP / kFlagGroup;   // products per lane
  static_assert(CAP <= 256 && kFlagMaxCols <= 65536, "a place fits a byte, a column two");
  __shared__ __align__(16) unsigned s_flags[kFlagRows][WPL * kFlagGroup];
  __shared__ __align__(4) unsigned char s_rank[kFlagRows][WPL * kFlagGroup];   // place of a word's first column
  __shared__ double s_vals[kFlagRows][CAP];
  __shared__ unsigned short s_cols[kFlagRows][CAP];
  __shared__ FlagLds<CAP> s_lds[kFlagRows];
  __shared__ T s_av[kFlagRows][kFlagGroup];
  if (ctl->error) return;
  const unsigned first = ctl->offset[1][bin];
  const unsigned nrows = ctl->offset[1][bin + 1] - first;
  const int g = threadIdx.x / kFlagGroup, gl = threadIdx.x % kFlagGroup;
  unsigned* flags = s_flags[g];
  unsigned char* rank = s_rank[g];
  double* vals = s_vals[g];
  unsigned short* cols = s_cols[g];
  T* s_a = s_av[g];
  const unsigned ngroups = gridDim.x * kFlagRows;
  auto value = [&](int64_t a, int n) { return gl < n ? a_val[a + gl] : T(0); };
  auto position = [&](int row) { return row >= 0 ? c_rp[row] : 0; };
  RowChain<kFlagGroup> ch{perm + first, a_rp, a_col, b_rp, nullptr, nrows, ngroups};
  ch.start(blockIdx.x * kFlagRows + g);
  T av0 = value(ch.a0, ch.d), av1 = value(ch.a01, ch.d1);
  int64_t out0 = position(ch.row), out1 = position(ch.row1), out2 = position(ch.row2);
  FlagWalk<CAP> walk{&s_lds[g]};
  const unsigned rounds = (nrows + ngroups - 1) / ngroups;
  for (unsigned r = 0; r < rounds; ++r) {
    const RowChain<kFlagGroup>::Ahead nx = ch.fetch();
    const T av2 = value(ch.a02, ch.d2);
    const int64_t out3 = position(ch.row3);
    flags_clear<WPL>(flags, gl);
    s_a[gl] = av0;
    group_sync<kFlagGroup>();
    int filled = 0;
    for (int c = 0; __any(c < ch.d || c == 0); c += kFlagGroup) {
      if (c > 0) {
        ch.fetch_more(c);
        const T av = c + gl < ch.d ? a_val[ch.a0 + c + gl] : T(0);
        group_sync<kFlagGroup>();
        s_a[gl] = av;
        group_sync<kFlagGroup>();
      }
      const int len = (int)(ch.bounds.v[1] - ch.bounds.v[0]);
      const int incl = group_incl_scan<kFlagGroup>(len);
      walk.begin(ch.bounds.v[0], len, filled + incl - len);
      for (int t0 = 0; __any(t0 < walk.quads); t0 += kFlagGroup) {
        int src, pos, n, col[4];
        int64_t q;
        T b[4];
        walk.next(t0, src, pos, q, n);
        load_quad<int32_t>(b_col, q, n, b_nnz, col);
        load_quad<T>(b_val, q, n, b_nnz, b);
        const double a = (double)s_a[src];
        flags_mark<WPL>(flags, col, n);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u < n) {
            vals[(pos + u) & (CAP - 1)] = a * (double)b[u];
            cols[(pos + u) & (CAP - 1)] = (unsigned short)col[u];
          }
      }
      filled += group_last<kFlagGroup>(incl);
    }
    const int n = filled < CAP ? filled : CAP;
    group_sync<kFlagGroup>();
    int before = 0;   // places in the words before
#pragma unroll
    for (int j = 0; j < WPL / 4; ++j) {
      const uint4 v = reinterpret_cast<const uint4*>(flags)[j * kFlagGroup + gl];
      const int c0 = __popc(v.x), c1 = c0 + __popc(v.y), c2 = c1 + __popc(v.z), c3 = c2 + __popc(v.w);
      const int incl = group_incl_scan<kFlagGroup>(c3);
      const int e = before + incl - c3;
      reinterpret_cast<unsigned*>(rank)[j * kFlagGroup + gl] = (unsigned)e | ((unsigned)(e + c0) << 8) | ((unsigned)(e + c1) << 16) | ((unsigned)(e + c2) << 24);
      before += group_last<kFlagGroup>(incl);
    }
    before = before < CAP ? before : CAP;
    double v[kPer];
    int col[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (i == 0 || __any(i * kFlagGroup < n)) { v[i] = vals[i * kFlagGroup + gl]; col[i] = cols[i * kFlagGroup + gl]; }
    group_sync<kFlagGroup>();
    const bool twice = __any(before < n);   // (wave-uniform) some row has a column twice
    if (twice) {
      for (int t = gl; t < before; t += kFlagGroup) vals[t] = 0.0;
      group_sync<kFlagGroup>();
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (i * kFlagGroup + gl < n) {
        const int w = (col[i] >> 5) & (WPL * kFlagGroup - 1);
        const int at = (rank[w] + __popc(flags[w] & ((1u << (col[i] & 31)) - 1u))) & (CAP - 1);
        if (twice) __hip_atomic_fetch_add(&vals[at], v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else vals[at] = v[i];
        cols[at] = (unsigned short)col[i];
      }
    group_sync<kFlagGroup>();
    for (int t = gl; t < before; t += kFlagGroup) {
      c_col[out0 + t] = cols[t];
      c_val[out0 + t] = (T)vals[t];
    }
    group_sync<kFlagGroup>();
    ch.advance(nx);
    av0 = av1; av1 = av2;
    out0 = out1; out1 = out2; out2 = out3;
  }
}

}  // namespace spg
