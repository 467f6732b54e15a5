// The dense symbolic kernel's walk over the products of a row: the pieces of B's rows that the row's entries of A ask for,
// four consecutive elements (a quad) to a lane.  (Quads and lists of pieces are the numeric kernels' too.)
//
// A piece is cut into chunks of L = 1, 4 or 16 quads (the last one may be short); the chunks of all pieces are dealt to the waves in
// contiguous shares.  A wave finds where its next 64 chunks lie at once, a chunk to a lane: lane i looks at where the i-th
// piece behind the one in hand begins and pushes i + 1 to the lane whose chunk that is; a running maximum spreads it to the lanes behind.
// Then it walks them in L batches of 64 quads, and a lane fetches what it has to know of its chunk from the lane that found it.
// What bounds the pass is the vector instructions a wave spends beside its products (two thirds to nine tenths of the issue slots of
// k_sym_dense with a search for every batch): about 45 for the search and 10 for a batch, so long pieces take long chunks; short pieces
// leave lanes of long chunks empty.  piece_chunks weighs the two by the counts of the very pieces.  Symbolic kernel, search for every batch | for
// every 64 chunks: R-MAT squared scale 19 12.1 | 10.2 ms, deduplication sweep of 10 000 columns 735 | 520 us.
#pragma once
#include "common.hpp"

namespace spg {

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni64(long long v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(unsigned long long)v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// Exclusive scans of N ints over the workgroup, with totals.  Contains barriers.  red: N * WAVES ints.
// The wave totals are scanned by every wave itself: lane w reads the total of wave w, a DPP row
// scan adds them up, and the wave takes its own prefix and the grand total with readlane.
template <int WAVES, int N>
__device__ __forceinline__ void block_excl_scan(const int (&v)[N], int (&excl)[N], int (&total)[N], int* red) {
  static_assert(WAVES == 4 || WAVES == 8 || WAVES == 16, "one DPP row of wave totals, or the first lanes of one");
  const int wave = uni(threadIdx.x >> 6);
  int incl[N];
#pragma unroll
  for (int i = 0; i < N; ++i) incl[i] = wave_incl_scan(v[i]);
  __syncthreads();
  if (lane_id() == kWave - 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) red[i * WAVES + wave] = incl[i];
  }
  __syncthreads();
  const int l = lane_id() & (WAVES - 1);   // (the lanes behind WAVES repeat the totals: only the first ones are looked at)
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int s = group_incl_scan<16>(red[i * WAVES + l]);
    total[i] = __builtin_amdgcn_readlane(s, WAVES - 1);
    const int before = wave ? __builtin_amdgcn_readlane(s, wave - 1) : 0;
    excl[i] = before + incl[i] - v[i];
  }
}

// The non-empty pieces that a pass walks, in LDS: first B entry, exclusive prefix of the chunk counts (of the quad counts in quad_pass),
// length and (numeric) a_ik of every piece.
template <typename T>
struct PieceList {
  const long long* s;
  const int* cpre;
  const int* len;
  const T* av;
};

// Up to four consecutive elements of a piece.
template <typename T>
struct Quad {
  int n = 0;   // elements that are left in the piece from the quad's first on (0 or less: none; four or more: the quad is full)
  T a{};       // a_ik of the piece (numeric walks)
  Run<int32_t, 4> col{};
  Run<T, 4> b{};   // (numeric walks)
};

// How a workgroup's pieces are cut, a piece of len elements (0: none) a thread.  Contains barriers.  red: 4 * WAVES ints.
struct PieceCut {
  int idx;     // this thread's piece among the non-empty ones
  int first;   // its first chunk
  int pieces, chunks;
  int lanes;   // log2 of a chunk's quads
};
template <int WAVES>
__device__ __forceinline__ PieceCut piece_chunks(int len, int* red) {
  const int v[4] = {len > 0 ? 1 : 0, (len + 3) >> 2, (len + 15) >> 4, (len + 63) >> 6};
  int e[4], t[4];
  block_excl_scan<WAVES>(v, e, t, red);
  // vector instructions of a batch of 64 quads, search and all: 90, 56 and 48
  const int w1 = 2 * t[1], w4 = 5 * t[2], w16 = 17 * t[3];
  const int lanes = w16 <= w4 && w16 <= w1 ? 4 : (w4 <= w1 ? 2 : 0);
  return PieceCut{e[0], lanes == 4 ? e[3] : (lanes == 2 ? e[2] : e[1]), uni(t[0]), uni(lanes == 4 ? t[3] : (lanes == 2 ? t[2] : t[1])), uni(lanes)};
}

// Visits every element of np pieces (nch chunks of 2^lanes quads) once: g(quad, full) per lane and batch, full (a type) where all lanes' quads
// are; columns only.
template <int WAVES, class G>
__device__ __forceinline__ void piece_pass(int np, int nch, int lanes, const PieceList<int> pl, const int32_t* __restrict__ b_col, int64_t b_nnz,
                                           G g) {
  const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int cpb = kWave >> lanes;   // chunks of a batch
  const int nb = (nch + cpb - 1) >> (6 - lanes);
  const int per = (nb + WAVES - 1) / WAVES;
  int c = wave * per * cpb;
  const int cend = c + per * cpb < nch ? c + per * cpb : nch;
  if (c >= cend) return;
  int p;   // last piece whose first chunk is <= c: among every sixteenth piece first, then among the sixteen
  {
    static_assert(WAVES <= 16, "64 steps of sixteen pieces");
    const int i0 = lane * 16;
    const int hi = __popcll(__ballot(i0 < np && pl.cpre[i0 < np ? i0 : 0] <= c)) - 1;
    const int i1 = hi * 16 + lane;
    p = hi * 16 + __popcll(__ballot(lane < 16 && i1 < np && pl.cpre[i1 < np ? i1 : 0] <= c)) - 1;
  }
  const int in = (lane & ((1 << lanes) - 1)) * 4;   // where the lane's quad lies in its chunk
  Quad<int> now;
  bool have = false;
  auto visit = [&](const Quad<int>& q) {
    if (__all(q.n >= 4)) g(q, std::true_type{});
    else g(q, std::false_type{});
  };
  for (; c < cend; c += kWave) {
    // a chunk to a lane: where it begins and how much of its piece is left there
    const int ahead = p + 1 + lane;
    const int begins = (ahead < np ? pl.cpre[ahead] : 0x7fffffff) - c;   // (1 or more: piece p holds chunk c)
    int m = __builtin_amdgcn_ds_permute(begins < kWave ? begins * 4 : 0, lane + 1);   // (the others push to lane 0, which does not look)
    m = group_max_scan<kWave>(lane == 0 ? 0 : m);
    const int piece = p + m;
    const int off = (c + lane - pl.cpre[piece]) << (lanes + 2);
    const long long at0 = pl.s[piece] + off;
    const int left0 = c + lane < cend ? pl.len[piece] - off : 0;
    p += __popcll(__ballot(begins <= kWave));
    const int left_chunks = cend - c < kWave ? cend - c : kWave;
    const int batches = (left_chunks + cpb - 1) >> (6 - lanes);
    int src = (lane >> lanes) * 4;
    for (int b = 0; b < batches; ++b, src += cpb * 4) {
      Quad<int> q;
      const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(src, (int)(unsigned)(unsigned long long)at0);
      const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(src, (int)(unsigned)((unsigned long long)at0 >> 32));
      const long long at = (long long)(((unsigned long long)hi << 32) | lo) + in;
      q.n = __builtin_amdgcn_ds_bpermute(src, left0) - in;
      if (__all(q.n >= 4)) {
        q.col = load_run<int32_t, 4>(b_col + at);
      } else if (!__any(q.n > 0 && at + 4 > b_nnz)) {
        if (q.n > 0) q.col = load_run<int32_t, 4>(b_col + at);
      } else {   // (fewer than four elements behind some lane's position)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < q.n) q.col.v[i] = b_col[at + i];
      }
      if (have) visit(now);   // (the next batch is on its way while g works on this one)
      now = q;
      have = true;
    }
  }
  visit(now);
}

}  // namespace spg
