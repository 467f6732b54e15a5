// Per-row intermediate-product count, input checks, binning and the row-count scan.
#pragma once
#include "common.hpp"

namespace spg {

constexpr int kCountThreads = 1024;
constexpr int kCountMaxRows = 1024;   // rows of A in a chunk: at most
constexpr int kFineRows = 32, kFineProbe = 256, kHeavyChunk = 4;
constexpr int64_t kFineFrom = 65536;
inline bool fine_rows(int64_t m, int64_t nnz_a, int64_t b_rows, int64_t nnz_b) { return m >= kFineFrom && nnz_a >= 6 * m && nnz_b >= 6 * b_rows; }

// Clears the control block and says how many rows of A a workgroup of the row count takes at a time: chunk, or kCountMaxRows where
// there are enough rows for all workgroups, rows are short (a chunk of 256 rows of a few entries leaves most of the 1024 threads idle
// and costs six barriers) and no stretch of them is much heavier than what a workgroup gets anyway (two are resident on each of `cus`
// compute units; one that holds the hub rows of a graph keeps the whole count waiting).
// Where a stretch of 256 rows (of a thousandth of them) holds kHeavyChunk times what a workgroup gets on average, chunks are of kFineRows rows, or
// twice as many: the one with the hub rows of a graph took as long as the whole count.  fine: this is looked at, which takes 2 us, where rows are
// many and of some length.  Whole calls, us without | with, R-MAT squared: scale 16 1670 | 1681 (f64, 8 edges 1004 | 996), 17 4318 | 4262, 18 11 813 | 11 730, 19
// 34 178 | 34 034; 400 000 rows of 8 x 8 470 | 471; stencils no difference.  From 32 768 rows scale 15 gains nothing (790 | 790), from 131 072 scale 16 loses what
// it gains; with 3 entries a row in place of 6 scale 18 of 4 edges 2689 | 2709, scale 19 of 5 8744 | 8796; a kHeavyChunk of 2 or 8 makes no difference.
// us with chunks of 256 | 1024 rows: 4.2 M rows of 2 entries 329 | 241, of 16 entries 1368 | 1322, of 27 entries 2131 | 2200; 2 M rows of 2
// entries 121 | 67, of 16 entries 253 | 240, of 27 entries 385 | 383; R-MAT of 2^20 vertices, 4 edges each 248 | 398, of 2^21, 7 edges
// each 637 | 1061.
__global__ __launch_bounds__(kCountThreads) void k_init_control(Control* ctl, int64_t m, const int64_t* __restrict__ a_rp, int chunk, int cus, int fine) {
  __shared__ unsigned long long heaviest;
  __shared__ int heavy;
  // (a stretch of rows a thread, asked for before the block is cleared)
  const int64_t probe = m > (int64_t)kFineProbe * kCountThreads ? (m + kCountThreads - 1) / kCountThreads : kFineProbe, r0 = threadIdx.x * probe;
  int mine = 0;
  int64_t all = 0;
  if (fine) {
    const int64_t n = r0 < m ? a_rp[r0 + probe < m ? r0 + probe : m] - a_rp[r0] : 0;   // (nobody has checked these yet)
    mine = n < 0 ? 0 : (n < 0x7fffffff ? (int)n : 0x7fffffff);
    all = a_rp[m] - a_rp[0];
  }
  unsigned* w = reinterpret_cast<unsigned*>(ctl);
  for (int i = threadIdx.x; i < (int)(sizeof(Control) / sizeof(unsigned)); i += blockDim.x) w[i] = 0;
  if (threadIdx.x == 0) { heaviest = 0; heavy = 0; }
  __syncthreads();
  if (m >= (int64_t)kCountMaxRows * 2 * cus) {
    const int64_t nnz = a_rp[m] - a_rp[0];
    // (looked at are as many stretches of whole chunks as workgroups are resident, or up to twice as many: every chunk took 14 us more)
    const int64_t stretch = m / ((int64_t)kCountMaxRows * 2 * cus) * kCountMaxRows;
    unsigned long long most = 0;
    for (int64_t r = threadIdx.x * stretch; r < m; r += kCountThreads * stretch) {
      const unsigned long long n = (unsigned long long)(a_rp[r + stretch < m ? r + stretch : m] - a_rp[r]);
      most = n > most ? n : most;
    }
    for (int d = kWave / 2; d > 0; d >>= 1) { const unsigned long long o = __shfl_xor(most, d, kWave); most = o > most ? o : most; }
    if (lane_id() == 0) atomicMax(&heaviest, most);
    __syncthreads();
    // (a row pointer that descends gives a huge one)
    if (nnz <= 16 * m && heaviest <= (unsigned long long)nnz / (unsigned)cus) chunk = kCountMaxRows;
  }
  if (fine && chunk < kCountMaxRows) {
    const int most = group_max_scan<kWave>(mine);
    if (lane_id() == kWave - 1) atomicMax(&heavy, most);
    __syncthreads();
    if ((int64_t)(heavy - kCountThreads * 4) * (2 * cus) > kHeavyChunk * all) chunk = m <= (int64_t)kFineRows * 64 * cus ? kFineRows : 2 * kFineRows;
  }
  if (threadIdx.x == 0) ctl->chunk_rows = chunk;
}

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {   // 24-bit pieces: 64 of them stay below 2^31
  unsigned long long s = (unsigned)__builtin_amdgcn_readlane(wave_incl_scan((int)(v & 0xffffff)), kWave - 1);
  if (__any((v >> 24) != 0)) {
    s += (unsigned long long)(unsigned)__builtin_amdgcn_readlane(wave_incl_scan((int)((v >> 24) & 0xffffff)), kWave - 1) << 24;
    s += (unsigned long long)(unsigned)__builtin_amdgcn_readlane(wave_incl_scan((int)(v >> 48)), kWave - 1) << 48;
  }
  return s;
}

// Adds N rows per lane (bin < 0: none) to the bin populations in LDS, the lanes and rows of a bin together: atomics of 64 lanes on
// the same counter are executed one after the other.  hnz may be null.  (Four rows a lane at a time, and the bins by number instead of
// one after another as they come: k_classify_numeric for 16384 rows of a power-law graph 13.5 -> 6.7 us.)
template <int N>
__device__ __forceinline__ void add_to_bins(const int (&bin)[N], const unsigned long long (&ip)[N], const unsigned (&nnz)[N], unsigned* hist,
                                            unsigned long long* hip, unsigned long long* hnz) {
  unsigned mine = 0;   // bins of the lane's rows
#pragma unroll
  for (int u = 0; u < N; ++u) mine |= bin[u] >= 0 ? 1u << bin[u] : 0u;
#pragma unroll
  for (int v = 0; v < kNumBins; ++v) {
    if (!__any((mine >> v) & 1u)) continue;
    unsigned rows = 0;
    unsigned long long p = 0, z = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      rows += (unsigned)__popcll(__ballot(bin[u] == v));
      if (bin[u] == v) { p += ip[u]; z += nnz[u]; }
    }
    if (v == kEmptyBin) { p = 0; z = 0; }
    else {
      p = wave_sum64(p);
      if (hnz) z = wave_sum64(z);
    }
    if (lane_id() == 0) {
      atomicAdd(&hist[v], rows);
      if (p) atomicAdd(&hip[v], p);
      if (hnz && z) atomicAdd(&hnz[v], z);
    }
  }
}

// Checks B (workgroup `part` of `parts`): rowptr starts at 0, is non-decreasing, ends at nnz, no row of 2^31 or more
// entries; every column inside [0, cols).  Also counts descents (col[p] <= col[p-1]) over
// the flat column array and descents that straddle a row boundary: every row is strictly
// ascending exactly when the two counts agree (k_bin_scatter turns them into b_sorted).
__device__ __forceinline__ void validate_b(int part, int parts, int64_t rows, int64_t cols, int64_t nnz, const int64_t* __restrict__ rp,
                                           const int32_t* __restrict__ col, Control* ctl, int (*sums)[kCountThreads / kWave]) {
  const int64_t stride = (int64_t)parts * kCountThreads;
  const int64_t t0 = (int64_t)part * kCountThreads + threadIdx.x;
  bool bad = false;
  int flat = 0, bnd = 0;
  if (t0 == 0 && (rp[0] != 0 || rp[rows] != nnz)) bad = true;
  for (int64_t i = t0; i < rows; i += stride) {
    const int64_t a = rp[i], b = rp[i + 1];
    if (b < a || a < 0 || b > nnz || b - a > 0x7fffffff) { bad = true; continue; }
    if (b - a >= (1 << 21)) ctl->long_b_row = 1;
    if (b > a && a > 0 && col[a] <= col[a - 1]) ++bnd;
  }
  for (int64_t p = t0; p < nnz; p += stride) {
    const int c = col[p];
    if (c < 0 || c >= cols) bad = true;
    if (p > 0 && c <= col[p - 1]) ++flat;
  }
  if (bad) ctl->error = 1;
  // one pair of atomics per workgroup: nearly every wave has descents to report (the row boundaries)
  flat = wave_sum(flat);
  bnd = wave_sum(bnd);
  if (lane_id() == 0) { sums[0][threadIdx.x >> 6] = flat; sums[1][threadIdx.x >> 6] = bnd; }
  __syncthreads();
  if (threadIdx.x < 2) {
    unsigned long long t = 0;
    for (int w = 0; w < kCountThreads / kWave; ++w) t += (unsigned long long)sums[threadIdx.x][w];
    if (t) atomicAdd(threadIdx.x == 0 ? &ctl->desc_flat : &ctl->desc_bnd, t);
  }
}

// Are rows mostly the row before moved to other columns (as many entries, the first and the last moved by the same), as those of
// discretised operators are?  A pair of rows for every thread of one workgroup, spread over all rows.
__device__ __forceinline__ void sample_rows(int64_t m, int64_t nnz_a, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col,
    Control* ctl) {
  const int64_t r = (m - 1) * (int64_t)threadIdx.x / kCountThreads;
  bool looked = false, moved = false;
  if (r + 2 <= m) {
    const int64_t p0 = a_rp[r], p1 = a_rp[r + 1], p2 = a_rp[r + 2];
    looked = p0 >= 0 && p0 + 1 < p1 && p1 < p2 && p2 <= nnz_a;   // (nobody has checked them yet)
    if (looked) moved = p2 - p1 == p1 - p0 && (unsigned)a_col[p1] - (unsigned)a_col[p0] == (unsigned)a_col[p2 - 1] - (unsigned)a_col[p1 - 1];
  }
  const int all = __popcll(__ballot(looked)), some = __popcll(__ballot(moved));
  if (lane_id() == 0 && all) {
    atomicAdd(&ctl->looked, (unsigned)all);
    if (some) atomicAdd(&ctl->moved, (unsigned)some);
  }
}

// Starts and lengths of 12 rows of B in a load: B's row pointer in a sixth of its size, for the row count, which looks rows up in any order.
constexpr int kLensRows = 12;
struct __align__(16) RowLens {
  unsigned start;               // of the first row
  unsigned len[kLensRows / 4];  // a byte a row
};
static_assert(sizeof(RowLens) == 16, "one load");
constexpr unsigned kLensNear = 64;
constexpr int kLensThreads = 256;
constexpr int kLensGroup = kLensThreads / 4;   // of a workgroup, a thread writes a word

// Bound by reading the row pointer.  Rows that do not fit (more than 255 entries, a start beyond 32 bits, a row pointer that is not one) are
// reported, and nobody uses the table then.  Nor where most of 256 rows of A begin close to where the row before begins: their lookups share lines
// as it is, and taking the lengths out of the table costs more than it saves (27-point stencil of 110^3 rows, both phases, 2532 us without, 2569
// with).
__global__ __launch_bounds__(kLensThreads) void k_row_lens(int64_t b_rows, const int64_t* __restrict__ b_rp, int64_t m, int64_t nnz_a,
    const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, unsigned* __restrict__ out, Control* ctl) {
  if (blockIdx.x == 0) {
    const int64_t r = (m - 1) * (int64_t)threadIdx.x / kLensThreads;
    bool looked = false, close = false;
    if (r + 1 < m) {
      const int64_t p0 = a_rp[r], p1 = a_rp[r + 1];
      looked = p0 >= 0 && p0 < p1 && p1 < nnz_a;   // (nobody has checked them yet)
      if (looked) close = (unsigned)a_col[p1] - (unsigned)a_col[p0] + kLensNear <= 2 * kLensNear;
    }
    if (2 * __syncthreads_count(close) > __syncthreads_count(looked) && threadIdx.x == 0) ctl->no_lens = 1;
  }
  __shared__ unsigned words[kLensThreads];
  unsigned char* bytes = reinterpret_cast<unsigned char*>(words);
  const int64_t r0 = (int64_t)blockIdx.x * (kLensGroup * kLensRows);
  bool fits = true;
  for (int t = threadIdx.x; t < kLensGroup * kLensRows; t += kLensThreads) {
    const int64_t r = r0 + t;
    const int g = t / kLensRows, j = t - g * kLensRows;
    int64_t start = 0, len = 0;
    if (r < b_rows) {
      const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + r);
      start = bounds.v[0];
      len = bounds.v[1] - start;
      fits = fits && start >= 0 && start <= 0xffffffffLL && len >= 0 && len < 256;
    }
    bytes[g * 16 + 4 + j] = (unsigned char)len;
    if (j == 0) words[g * 4] = (unsigned)start;
  }
  if (__syncthreads_or(!fits)) {
    if (threadIdx.x == 0) ctl->no_lens = 1;
    return;
  }
  const int64_t g0 = (int64_t)blockIdx.x * kLensGroup + threadIdx.x / 4;
  if (g0 * kLensRows < b_rows) out[(int64_t)blockIdx.x * kLensThreads + threadIdx.x] = words[threadIdx.x];
}

// Start and length of row k.
__device__ __forceinline__ void lens_row(const RowLens& g, unsigned j, int64_t* start, long long* len) {
  unsigned before = 0, word = 0;
#pragma unroll
  for (unsigned w = 0; w < kLensRows / 4; ++w) {
    const unsigned bits = j > 4 * w ? (j - 4 * w) * 8 : 0;
    before = __builtin_amdgcn_sad_u8(bits >= 32 ? g.len[w] : g.len[w] & ((1u << bits) - 1), 0u, before);
    if (j >> 2 == w) word = g.len[w];
  }
  *start = (int64_t)g.start + before;
  *len = (word >> (j & 3) * 8) & 255;
}

// Bound: the gather of B's row pointer (a line per entry of A where it does not fit the L2 cache), a chain of three loads where there are few rows.
// COMPACT: out of the table of lens instead, unless it is not to be used (with the table and the descriptions written, 33.5 M entries, 4 M rows of B
// 0.71 | 0.45 ms, 16 M entries, 1 M rows 0.225 | 0.169; groups of 28 rows in 32 bytes 0.52 and 82 registers).
// Two workgroups on a compute unit, or nobody works while one waits at its barriers (the compiler took 7 waves a SIMD, one workgroup: 27-point
// stencil of 128^3 rows 391 | 274 us, 16 M entries in rows of 8 248 | 225; power-law graphs lose a tenth of the count, 2 in 1000 of their calls:
// R-MAT scale 17 131 | 142 us, scale 20 with 6 edges 337 | 392).  (Between events around all launches of the count; by themselves this kernel and
// that of the lengths take 228 + 8 us of the 274, and 380 + 13 us of the 0.45 ms.)
// The first `parts` workgroups check B.  The others count the products of A's rows: a workgroup takes chunks of `chunk_rows`
// consecutive rows (a chunk of hub rows holds a large share of all entries, hence the widest workgroup): the chunk's A
// entries are read coalesced, the lengths of their B rows are summed up over the workgroup, and a row takes the difference of the sums
// at its ends (an addition to the row's counter per entry, after a bisection for its row, was bound by LDS: 27-point
// stencil of 128^3 rows 494 -> 377 us, 10^7 entries in rows of 2.4 128 -> 95 us, R-MAT scale 14 27 -> 20 us, scale 19 442 -> 400 us).
// desc (optional): start and length of every A entry's B row, for the kernels of short rows.
// Writes ip (saturated to int32), the symbolic bin (with kCountLight kLightBin for rows of bin 4 of at most kDenseLight products), zero counts for
// rows without products.
// lens: of all rows of B, or reported as not to be used.  Both kernels are launched then, and the one that is not meant leaves at once (as two ways
// inside one kernel, 4 M rows of B take 0.50 instead of 0.45 ms and an R-MAT graph of scale 20, which has no use for the table, 0.42 instead of
// 0.40; the launch costs 10 us).
// modes: kCountBlock, A is a block of rows; kCountLight.  (One argument: with another one the scalar registers no longer suffice and the kernel takes
// scratch memory, 0.4 us a launch.)
constexpr int kCountBlock = 1, kCountLight = 2;
template <bool COMPACT>
__global__ __launch_bounds__(kCountThreads, 8) void k_count_rows(int parts, int64_t b_cols, int64_t b_nnz, const int32_t* __restrict__ b_col,
    int64_t m, int64_t nnz_a, int64_t b_rows, const int64_t* __restrict__ a_rp, const int32_t* __restrict__ a_col, const int64_t* __restrict__ b_rp,
    int* __restrict__ ip_out, unsigned char* __restrict__ bin_out, int* __restrict__ cnt_out, Control* ctl, int force, int modes,
    unsigned long long* __restrict__ desc, const RowLens* __restrict__ lens) {
  __shared__ long long rp[kCountMaxRows + 1];
  __shared__ unsigned long long ipl[kCountMaxRows];
  __shared__ __align__(16) unsigned pre[kCountThreads * 4 + 1];   // products before every entry of a round
  __shared__ unsigned hist[kNumBins];
  __shared__ unsigned long long hip[kNumBins];
  __shared__ int sums[2][kCountThreads / kWave];
  __shared__ int bad;
  __shared__ unsigned longs;
  if (lens && COMPACT == (ctl->no_lens != 0)) return;
  if ((int)blockIdx.x < parts) {
    if (blockIdx.x == 0) sample_rows(m, nnz_a, a_rp, a_col, ctl);
    validate_b(blockIdx.x, parts, b_rows, b_cols, b_nnz, b_rp, b_col, ctl, sums);
    return;
  }
  const int tid = threadIdx.x;
  const int chunk_rows = ctl->chunk_rows;
  if (tid < kNumBins) { hist[tid] = 0; hip[tid] = 0; }
  if (tid == 0) longs = 0;
  // a workgroup takes several chunks and reports its bin populations once (thousands of workgroups adding to
  // the same few counters cost more than the counting)
  __shared__ long long next_chunk;
  int64_t chunk = blockIdx.x - parts;
  while (chunk * chunk_rows < m) {
    // (the chunk after this one is drawn now and looked at when this one is done: chunks differ by orders of
    // magnitude in their entries, so they are handed out rather than dealt)
    long long drawn = 0;
    if (tid == 0) drawn = (long long)(gridDim.x - parts) + atomicAdd(&ctl->work[3], 1u);
    const int64_t r0 = chunk * chunk_rows;
    const int nr = (int)((m - r0) < chunk_rows ? (m - r0) : chunk_rows);
    __syncthreads();   // (the bin counters are initialised; the chunk before has left rp and ipl)
    if (tid == 0) bad = 0;
    for (int t = tid; t <= nr; t += kCountThreads) rp[t] = a_rp[r0 + t];
    if (tid < kCountMaxRows) ipl[tid] = 0;
    __syncthreads();
    if (tid < nr && rp[tid + 1] < rp[tid]) bad = 1;
    if (tid == 0) {
      if (rp[0] < 0 || rp[nr] > nnz_a) bad = 1;
      // (a block of rows of a larger matrix keeps that matrix's positions: it neither starts at 0 nor ends at nnz)
      if (!(modes & kCountBlock) && r0 == 0 && rp[0] != 0) bad = 1;
      if (!(modes & kCountBlock) && r0 + nr == m && rp[nr] != nnz_a) bad = 1;
    }
    __syncthreads();
    if (bad) {
      if (tid == 0) ctl->error = 1;
      return;
    }
    const long long lo = rp[0], hi = rp[nr];
    bool badcol = false;
    // row of entry p: the last t with rp[t] <= p
    auto row_of = [&](long long p) {
      int a = 0, b = nr;
      while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (rp[mid] <= p) a = mid; else b = mid;
      }
      return a;
    };
    const bool few = hi - lo <= kCountThreads;
    if (few) {
      // an entry to a thread, added to its row's counter, the lanes of a DPP row that hold the same row together: nobody waits for the
      // workgroup (with the sums below, 86 103 rows of 2 entries 27.4 us instead of 23.5, 1000 rows of 10 6.4 instead of 5.9)
      const long long p = lo + tid;
      long long len = 0;
      int a = -1;
      if (p < hi) {
        const int k = a_col[p];
        int64_t start = 0;
        if (k < 0 || k >= b_rows) badcol = true;
        else {
          const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k);
          start = bounds.v[0];
          len = bounds.v[1] - start;
          if (len < 0) { badcol = true; len = 0; }
        }
        if (desc) desc[p] = make_desc(start, len);
        a = row_of(p);
      }
      if (__any(len >= (1LL << 27))) {   // (sixteen of these need more than 32 bits)
        if (len > 0) atomicAdd(&ipl[a], (unsigned long long)len);
      } else {   // the entries of a row are neighbours: the last of them adds what all have
        unsigned sum = (unsigned)len;
        auto below = [&](auto step) {
          constexpr int kStep = decltype(step)::value;
          const int r = __builtin_amdgcn_update_dpp(-2, a, 0x110 + kStep, 0xf, 0xf, false);
          const unsigned l = (unsigned)__builtin_amdgcn_update_dpp(0, (int)sum, 0x110 + kStep, 0xf, 0xf, false);
          if (r == a) sum += l;
        };
        below(std::integral_constant<int, 1>{});
        below(std::integral_constant<int, 2>{});
        below(std::integral_constant<int, 4>{});
        below(std::integral_constant<int, 8>{});
        const int next = __builtin_amdgcn_update_dpp(-2, a, 0x101, 0xf, 0xf, false);
        if (next != a && sum > 0) atomicAdd(&ipl[a], (unsigned long long)sum);
      }
    }
    // four consecutive entries per thread and round, so that their (dependent) loads overlap
    for (long long q0 = few ? hi : lo; q0 < hi; q0 += kCountThreads * 4) {   // (all threads together)
      const long long p0 = q0 + tid * 4;
      int k[4];
      long long len[4];
      int64_t start[4];
      if (p0 + 4 <= hi) {
        const Run<int32_t, 4> r = load_run<int32_t, 4>(a_col + p0);
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = r.v[u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = p0 + u < hi ? a_col[p0 + u] : -1;
      }
      if constexpr (COMPACT) {
        RowLens g[4];
        unsigned at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {   // (an entry that is none, or not a row of B, reads the first)
          const bool row = k[u] >= 0 && k[u] < b_rows;
          if (p0 + u < hi && !row) badcol = true;
          const unsigned of = row ? (unsigned)k[u] : 0u;
          g[u] = lens[of / kLensRows];
          at[u] = of % kLensRows;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          lens_row(g[u], at[u], &start[u], &len[u]);
          if (k[u] < 0 || k[u] >= b_rows) { len[u] = 0; start[u] = 0; }
        }
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const long long p = p0 + u;
          len[u] = 0;
          start[u] = 0;
          if (p < hi) {
            if (k[u] < 0 || k[u] >= b_rows) { badcol = true; continue; }
            const Run<int64_t, 2> bounds = load_run<int64_t, 2>(b_rp + k[u]);   // (both ends of the row in one load)
            start[u] = bounds.v[0];
            len[u] = bounds.v[1] - bounds.v[0];
            if (len[u] < 0) { badcol = true; len[u] = 0; }
          }
        }
      }
      bool fits = true;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (desc && p0 + u < hi) desc[p0 + u] = make_desc(start[u], len[u]);
        fits = fits && len[u] < (1LL << 19);   // (4096 of these need less than 32 bits)
      }
      const int l0 = (int)len[0], l1 = l0 + (int)len[1], l2 = l1 + (int)len[2], l3 = l2 + (int)len[3];
      const int incl = wave_incl_scan(l3);
      const bool wave_fits = !__any(!fits);
      if (lane_id() == kWave - 1) sums[0][tid >> 6] = wave_fits ? incl : -1;
      __syncthreads();
      const int w = sums[0][lane_id() & 15];
      if (__any(w < 0)) {   // (all waves alike) some row of B is huge
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (p0 + u < hi && len[u] > 0) atomicAdd(&ipl[row_of(p0 + u)], (unsigned long long)len[u]);
      } else {
        const int tot = group_incl_scan<16>(w);
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const unsigned e = (unsigned)(incl - l3 + (wave ? __builtin_amdgcn_readlane(tot, wave - 1) : 0));
        *reinterpret_cast<uint4*>(&pre[tid * 4]) = make_uint4(e, e + l0, e + l1, e + l2);
        if (tid == kCountThreads - 1) pre[kCountThreads * 4] = e + l3;
        __syncthreads();
        if (tid < nr) {   // what the round holds of this thread's row
          const long long a = rp[tid] > q0 ? rp[tid] : q0, b = rp[tid + 1] < q0 + kCountThreads * 4 ? rp[tid + 1] : q0 + kCountThreads * 4;
          if (a < b) ipl[tid] += (unsigned long long)(pre[b - q0] - pre[a - q0]);
        }
      }
      if (q0 + kCountThreads * 4 < hi) __syncthreads();   // (the next round writes sums and pre)
    }
    if (badcol) ctl->error = 1;
    __syncthreads();
    {
      const unsigned long long mine = tid < nr ? ipl[tid] : 0ULL;
      const int bin = tid < nr ? classify_symbolic((long long)mine, force) : -1;
      if (tid < nr) {
        ip_out[r0 + tid] = mine > 0x7fffffffULL ? 0x7fffffff : (int)mine;
        bin_out[r0 + tid] = (unsigned char)(bin == 4 && (modes & kCountLight) && mine <= (unsigned long long)kDenseLight ? kLightBin : bin);
        if (bin == kEmptyBin) cnt_out[r0 + tid] = 0;
      }
      const int bins[1] = {bin};
      const unsigned long long ips[1] = {mine};
      const unsigned none[1] = {0};
      add_to_bins<1>(bins, ips, none, hist, hip, nullptr);
      const unsigned long long is_long = __ballot(bin == 2 && mine > (unsigned long long)kLongProducts);
      if (is_long && lane_id() == 0) atomicAdd(&longs, (unsigned)__popcll(is_long));
    }
    if (tid == 0) next_chunk = drawn;
    __syncthreads();
    chunk = next_chunk;
  }
  __syncthreads();
  if (tid < kNumBins && hist[tid]) {
    atomicAdd(&ctl->hist[0][tid], hist[tid]);
    if (hip[tid]) atomicAdd(&ctl->bin_ip[0][tid], hip[tid]);
  }
  if (tid == 0) {   // the products of all rows = the products of all bins
    unsigned long long tot = 0;
    for (int b = 0; b < kNumBins; ++b) tot += hip[b];
    if (tot) atomicAdd(&ctl->ip_total, tot);
    if (longs) atomicAdd(&ctl->long_rows, longs);
  }
}

// What the kernels below share.  A workgroup takes kScanTile rows, every wave kScanItems times 64 consecutive ones, so that the
// lists of a bin ascend and neighbouring groups of a kernel work on neighbouring rows.
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kScanWaves = kScanThreads / kWave;
constexpr int kScanDirect = 4096;   // up to this many tiles every workgroup adds up the sums of the tiles before its own

// Puts the rows of the tile into their bins: every wave ballots per bin and ranks its lanes inside the ballot masks (a
// wavefront-level prefix count); the waves of a workgroup add their counts up in LDS, so that a bin costs one global atomic
// per workgroup.  bin[u]: of row tile_row(u), -1 = none.  Also the bin offsets, by the first workgroup for
// the kernels that follow.
__device__ __forceinline__ int64_t tile_row(int u) {
  return (int64_t)blockIdx.x * kScanTile + (threadIdx.x >> 6) * (kScanItems * kWave) + u * kWave + lane_id();
}

struct ScatterLds {
  unsigned count[kNumBins + 1][kScanWaves], base[kNumBins + 1], offset[kNumBins + 1];
};
// hist: rows of every bin, of all tiles.  LIGHT: bin 4 is filled from both ends, its lighter rows (kLightBin) from the first place on, the others
// from the last one down (cursor[phase][kEmptyBin] counts these): k_sym_dense takes its rows from the end.
template <bool LIGHT>
__device__ __forceinline__ void scatter_bins(const int (&bin)[kScanItems], const unsigned* hist, int* __restrict__ perm, Control* ctl, int phase,
    ScatterLds* sl) {
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  if (tid == 0) {
    unsigned run = 0;
    for (int b = 0; b < kNumBins; ++b) { sl->offset[b] = run; run += hist[b]; }
    sl->offset[kNumBins] = run;
  }
  int rank[kScanItems];
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) rank[u] = 0;
  unsigned present = 0;   // bins that have rows
#pragma unroll
  for (int b = 0; b < kNumBins - 1; ++b) present |= hist[b] ? 1u << b : 0u;
  if (LIGHT && (present >> 4 & 1u)) present |= 1u << kLightBin;
  for (int v = 0; v <= kLightBin; ++v) {   // (rows with no work are not listed)
    if (!(present >> v & 1u)) continue;
    unsigned before = 0;
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
      const unsigned long long mask = __ballot(bin[u] == v);
      if (bin[u] == v) rank[u] = (int)before + lanes_below(mask);
      before += (unsigned)__popcll(mask);
    }
    if (lane == 0) sl->count[v][wave] = before;
  }
  __syncthreads();
  if (tid <= kLightBin && (present >> tid & 1u)) {
    unsigned run = 0;
    for (int w = 0; w < kScanWaves; ++w) { const unsigned c = sl->count[tid][w]; sl->count[tid][w] = run; run += c; }
    unsigned base = 0;
    if (run) {
      if (LIGHT && tid == 4) base = sl->offset[5] - run - atomicAdd(&ctl->cursor[phase][kEmptyBin], run);
      else base = sl->offset[tid == kLightBin ? 4 : tid] + atomicAdd(&ctl->cursor[phase][tid == kLightBin ? 4 : tid], run);
    }
    sl->base[tid] = base;
  }
  if (blockIdx.x == 0 && tid <= kNumBins) ctl->offset[phase][tid] = sl->offset[tid];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kScanItems; ++u)
    if (bin[u] >= 0 && bin[u] != kEmptyBin) perm[sl->base[bin[u]] + sl->count[bin[u]][wave] + rank[u]] = (int)tile_row(u);
}

// The control block to the host's copy (pinned memory), by one workgroup whose writes to it are done.
__device__ __forceinline__ void control_out(const Control* ctl, Control* host) {
  __threadfence();
  __syncthreads();
  const unsigned* from = reinterpret_cast<const unsigned*>(ctl);
  unsigned* to = reinterpret_cast<unsigned*>(host);
  for (int i = threadIdx.x; i < (int)(sizeof(Control) / 4); i += blockDim.x) to[i] = __hip_atomic_load(from + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Symbolic bins: lists of rows.
__global__ __launch_bounds__(kScanThreads) void k_bin_scatter(int64_t m, const unsigned char* __restrict__ bin_of, int* __restrict__ perm, Control* ctl,
                                                              Control* host) {
  __shared__ ScatterLds sl;
  int bin[kScanItems];
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    const int64_t i = tile_row(u);
    bin[u] = i < m ? bin_of[i] : -1;
  }
  // (an error of the count leaves rows without a bin; the one that is set below does not matter here, whoever sees it)
  if (ctl->error != 1) scatter_bins<true>(bin, ctl->hist[0], perm, ctl, 0, &sl);
  if (blockIdx.x == 0) {
    __syncthreads();
    if (threadIdx.x == 0) {
      const int sorted = ctl->desc_flat == ctl->desc_bnd ? 1 : 0;
      ctl->b_sorted = sorted;
      // the dense workspaces walk whole rows of an unsorted B per tile: 32-bit piece prefixes
      if (!sorted && ctl->long_b_row && !ctl->error) ctl->error = 2;
    }
    control_out(ctl, host);
  }
}

// Numeric classes of a tile's rows from ip and the symbolic counts; their numbers, products and entries are added to the workgroup's (all threads
// together; the barrier after it is the caller's).
struct ClassLds {
  unsigned hist[kNumBins];
  unsigned long long ip[kNumBins], nnz[kNumBins];
};
__device__ __forceinline__ void classify_tile(int64_t m, const int* __restrict__ ip, const int* __restrict__ cnt, unsigned char* __restrict__ bin_out,
                                              int force, int staged_cap, int (&bin)[kScanItems], unsigned (&c)[kScanItems], ClassLds* cl) {
  if (threadIdx.x < kNumBins) { cl->hist[threadIdx.x] = 0; cl->ip[threadIdx.x] = 0; cl->nnz[threadIdx.x] = 0; }
  unsigned long long p[kScanItems];
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    const int64_t i = tile_row(u);
    bin[u] = -1;
    p[u] = 0;
    c[u] = 0;
    if (i < m) {
      p[u] = (unsigned)ip[i];
      c[u] = (unsigned)cnt[i];
    }
  }
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    const int64_t i = tile_row(u);
    if (i < m) {
      bin[u] = classify_numeric((long long)p[u], (int)c[u], force, staged_cap);
      bin_out[i] = (unsigned char)bin[u];
    }
  }
  __syncthreads();
  add_to_bins<kScanItems>(bin, p, c, cl->hist, cl->ip, cl->nnz);
}

__device__ __forceinline__ void report_classes(const ClassLds* cl, Control* ctl) {
  if (threadIdx.x < kNumBins && cl->hist[threadIdx.x]) {
    atomicAdd(&ctl->hist[1][threadIdx.x], cl->hist[threadIdx.x]);
    atomicAdd(&ctl->bin_ip[1][threadIdx.x], cl->ip[threadIdx.x]);
    atomicAdd(&ctl->bin_nnz[threadIdx.x], cl->nnz[threadIdx.x]);
  }
}

// The classes, and the sum of the counts of every tile.
__global__ __launch_bounds__(kScanThreads) void k_classify_numeric(int64_t m, const int* __restrict__ ip, const int* __restrict__ cnt,
                                   unsigned char* __restrict__ bin_out, long long* __restrict__ partial, Control* ctl, int force, int staged_cap) {
  __shared__ ClassLds cl;
  __shared__ unsigned long long total;
  if (threadIdx.x == 0) total = 0;
  int bin[kScanItems];
  unsigned c[kScanItems];
  classify_tile(m, ip, cnt, bin_out, force, staged_cap, bin, c, &cl);
  unsigned long long sum = 0;
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) sum += c[u];
  const unsigned long long s = wave_sum64(sum);
  if (lane_id() == 0) atomicAdd(&total, s);
  __syncthreads();
  report_classes(&cl, ctl);
  if (threadIdx.x == 0) partial[blockIdx.x] = (long long)total;
}

// ---- exclusive scan of int32 row counts into the int64 row pointer -------------------
constexpr int kScanBlockThreads = 256;

__global__ __launch_bounds__(kScanBlockThreads) void k_scan_blocks(int64_t nblocks, long long* __restrict__ partial,
                                                              int64_t m, int64_t* __restrict__ rowptr, Control* ctl) {
  // single workgroup: exclusive scan of the per-tile sums, in place
  __shared__ long long tile[kScanBlockThreads];
  __shared__ long long carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nblocks; b0 += kScanBlockThreads) {
    const int64_t i = b0 + threadIdx.x;
    const long long v = i < nblocks ? partial[i] : 0;
    tile[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < kScanBlockThreads; d <<= 1) {
      long long t = threadIdx.x >= d ? tile[threadIdx.x - d] : 0;
      __syncthreads();
      tile[threadIdx.x] += t;
      __syncthreads();
    }
    if (i < nblocks) partial[i] = carry + tile[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += tile[kScanBlockThreads - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    rowptr[m] = carry;
    ctl->nnz_c = carry;
  }
}

// Six launches (classes, offsets, lists, three of the scan) took 19 us for 1000 rows and 57 us of colliding LDS atomics for
// 700 000; the two of now 14 and 25 us, and the control block reaches the host without a copy (two copies of 10 to 15 us each).
// The row pointer and the lists of the numeric bins.  direct: partial holds the sums of the tiles (at most kScanDirect), of
// which every workgroup adds up its own share; otherwise their exclusive prefix (k_scan_blocks).
// ONE: a single tile.  Its workgroup needs nobody else's numbers and classifies its rows itself: one launch instead of two (whole calls, us: 1000
// rows of 10 x 10 88.6 | 87.0, 4096 rows 90.9 | 88.1, R-MAT scale 12 197 | 195, 27-point stencil of 12^3 rows 109 | 106).
template <bool ONE>
__global__ __launch_bounds__(kScanThreads) void k_scan_final(int64_t m, int64_t tiles, int direct, const int* __restrict__ cnt, const long long* __restrict__ partial,
                                                             const int* __restrict__ ip, int force, int staged_cap,
                                                                 unsigned char* __restrict__ bin_of, int* __restrict__ perm,
                                                                 int64_t* __restrict__ rowptr, Control* ctl, Control* host) {
  __shared__ ScatterLds sl;
  __shared__ ClassLds cl;
  __shared__ unsigned long long before, all;
  __shared__ long long waves[kScanWaves];
  const int tid = threadIdx.x;
  if (tid == 0) { before = 0; all = 0; }
  int v[kScanItems], bin[kScanItems];
  long long excl[kScanItems], s = 0;   // entries of the wave's rows before a row, and of all its rows
  if (ONE) {
    unsigned c[kScanItems];
    classify_tile(m, ip, cnt, bin_of, force, staged_cap, bin, c, &cl);
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) v[u] = (int)c[u];
  } else {
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
      const int64_t i = tile_row(u);
      v[u] = i < m ? cnt[i] : 0;
      bin[u] = i < m ? bin_of[i] : -1;
    }
  }
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    int incl = wave_incl_scan(v[u] & 0xffffff);   // (24 bits at a time: 64 of them stay below 2^31)
    excl[u] = s + incl - (v[u] & 0xffffff);
    s += __builtin_amdgcn_readlane(incl, kWave - 1);
    if (__any(v[u] >> 24)) {
      incl = wave_incl_scan(v[u] >> 24);
      excl[u] += (long long)(incl - (v[u] >> 24)) << 24;
      s += (long long)__builtin_amdgcn_readlane(incl, kWave - 1) << 24;
    }
  }
  __syncthreads();
  if (ONE) {
    report_classes(&cl, ctl);
  } else if (direct) {
    unsigned long long b = 0, a = 0;
    for (int64_t t = tid; t < tiles; t += kScanThreads) {
      if (t >= (int64_t)blockIdx.x && blockIdx.x != 0) break;   // (the first workgroup wants the total)
      const unsigned long long x = (unsigned long long)partial[t];
      if (t < (int64_t)blockIdx.x) b += x;
      a += x;
    }
    b = wave_sum64(b);
    a = wave_sum64(a);
    if (lane_id() == 0 && b) atomicAdd(&before, b);
    if (lane_id() == 0 && a) atomicAdd(&all, a);
  } else if (tid == 0) {
    before = (unsigned long long)partial[blockIdx.x];
  }
  if (lane_id() == 0) waves[tid >> 6] = s;
  __syncthreads();
  long long run = (long long)before;
  for (int w = 0; w < (tid >> 6); ++w) run += waves[w];
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    const int64_t i = tile_row(u);
    if (i < m) rowptr[i] = run + excl[u];
  }
  scatter_bins<false>(bin, ONE ? cl.hist : ctl->hist[1], perm, ctl, 1, &sl);
  if (ONE && tid == kScanThreads - 1) { rowptr[m] = run + s; ctl->nnz_c = run + s; }
  if (blockIdx.x == 0) {
    if (!ONE && direct && tid == 0) { rowptr[m] = (int64_t)all; ctl->nnz_c = (long long)all; }
    control_out(ctl, host);
  }
}

// ---- row blocks of about equal work -----------------------------------------------------
// Sums of the tiles' weights: a row's products and one (rows without products still cost a little).
__global__ __launch_bounds__(kScanThreads) void k_weight_sums(int64_t m, const int* __restrict__ ip, unsigned long long* __restrict__ sums) {
  __shared__ unsigned long long part[kScanWaves];
  unsigned long long s = 0;
#pragma unroll
  for (int u = 0; u < kScanItems; ++u) {
    const int64_t i = tile_row(u);
    if (i < m) s += (unsigned)ip[i] + 1ULL;
  }
  s = wave_sum64(s);
  if (lane_id() == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kScanWaves; ++w) s += part[w];
    sums[blockIdx.x] = s;
  }
}

// first[t] = rows of the blocks before block t (t = 1 .. blocks - 1): the first boundary that has t / blocks of the whole weight in front of it;
// first[blocks + 1] = the whole weight.  sums: of the tiles, exclusive afterwards.  One workgroup; a wave a boundary.
// Bound by the chain of dependent loads.  (All rows' products copied to the host and added up there: an R-MAT graph of scale 17 in four blocks 6.30
// ms | with these kernels 6.16; scale 16 in eight, fp64, 3.79 | 3.72; scale 12 in two 0.544 | 0.535.)
__global__ __launch_bounds__(kScanThreads) void k_block_rows(int64_t m, int64_t tiles, int blocks, const int* __restrict__ ip,
    unsigned long long* __restrict__ sums, long long* __restrict__ first) {
  __shared__ unsigned long long all;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  if (wave == 0) {
    unsigned long long run = 0;
    for (int64_t t0 = 0; t0 < tiles; t0 += kWave) {
      const unsigned long long v = t0 + lane < tiles ? sums[t0 + lane] : 0ULL;
      unsigned long long incl = v;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const unsigned long long o = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += o;
      }
      if (t0 + lane < tiles) sums[t0 + lane] = run + incl - v;
      run += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) all = run;
  }
  __threadfence();
  __syncthreads();
  const double total = (double)all;
  if (threadIdx.x == 0) first[blocks + 1] = (long long)all;
  for (int t = 1 + wave; t < blocks; t += kScanWaves) {
    const double want = total * t / blocks;
    int64_t lo = 0, hi = tiles;   // the last tile with less in front of it
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if ((double)__hip_atomic_load(&sums[mid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) lo = mid; else hi = mid;
    }
    unsigned long long run = __hip_atomic_load(&sums[lo], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    long long at = m;
    for (int64_t i0 = lo * kScanTile; i0 < m; i0 += kWave) {   // (a step beyond the tile at most)
      const int64_t i = i0 + lane;
      unsigned long long incl = i < m ? (unsigned)ip[i] + 1ULL : 0ULL;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const unsigned long long o = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += o;
      }
      const unsigned long long there = __ballot(i < m && (double)(run + incl) >= want);
      if (there) {
        at = i0 + __ffsll((long long)there);
        break;
      }
      run += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) first[t] = at;
  }
}

}  // namespace spg
