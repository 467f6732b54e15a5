// C ABI of the SpGEMM library (see include/spgemm.h): argument checks, plan scratch,
// kernel launches.  All device work is in the *_kernels.hpp headers beside this file.
#include "../../include/spgemm.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "common.hpp"
#include "entry_order.hpp"
#include "plan_room.hpp"
#include "setup_kernels.hpp"
#include "esc_kernels.hpp"
#include "flag_kernels.hpp"
#include "record_kernels.hpp"
#include "hash_kernels.hpp"
#include "dense_kernels.hpp"
#include "tile_kernels.hpp"
#include "wide_kernels.hpp"
#include "short_kernels.hpp"
#include "staged_kernels.hpp"
#include "sort_kernels.hpp"
#include "tensor_kernels.hpp"
#include "outer_kernels.hpp"

using namespace spg;

// the LDS of a compute unit (160 KB) belongs to one workgroup of the big kernels, or to two
static_assert(num_wide_lds<double>() <= 160 * 1024, "numeric dense kernel exceeds LDS");
static_assert(sym_dense_lds<16, 1024>(kSymFlagWords) <= 160 * 1024, "symbolic dense kernel exceeds LDS");
static_assert(sym_dense_lds<16, 512>(kSymNarrowCols / 32) <= 80 * 1024 && sym_dense_lds<16, 1024>(kSymShortCols / 32) <= 80 * 1024 && num_tiles_lds<double>() <= 80 * 1024, "two workgroups on a compute unit");
static_assert(staged_lds<double>() <= 160 * 1024 && staged_lds<float>() <= 160 * 1024, "staged kernel exceeds LDS");

// Pinned host memory where kernels leave numbers for the host (the symbolic ones the control block).  Allocating and releasing it costs 50 to
// 300 us, so a few blocks wait for the next calls; a call holds its own from before its first kernel until its stream has been
// waited for, whatever handle, stream or thread it comes from: the lease itself waits where the call returns before it has (an
// allocation that is refused while kernels are on their way).
namespace {

class PinnedBlocks {
 public:
  Control* take() {
    {
      std::lock_guard<std::mutex> lock(mutex_);
      if (n_ > 0) return free_[--n_];
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, sizeof(Control), hipHostMallocPortable) == hipSuccess) return static_cast<Control*>(p);
    (void)hipGetLastError();
    return nullptr;
  }
  void give(Control* p) {
    {
      std::lock_guard<std::mutex> lock(mutex_);
      if (n_ < kKeep) { free_[n_++] = p; return; }
    }
    (void)hipHostFree(p);
  }

 private:
  static constexpr int kKeep = 16;
  std::mutex mutex_;
  Control* free_[kKeep] = {};
  int n_ = 0;
};
PinnedBlocks g_pinned;

struct PinnedLease {
  Control* p;
  explicit PinnedLease(hipStream_t stream) : p(g_pinned.take()), stream_(stream) {}
  ~PinnedLease() {
    if (!p) return;
    if (written_) (void)hipStreamSynchronize(stream_);
    g_pinned.give(p);
  }
  void written() { written_ = true; }   // kernels that write to the block are about to be launched
  void waited() { written_ = false; }   // and all of them are done
  PinnedLease(const PinnedLease&) = delete;
  PinnedLease& operator=(const PinnedLease&) = delete;

 private:
  hipStream_t stream_;
  bool written_ = false;
};

}  // namespace

struct TimedLaunch {
  int cls;
  hipEvent_t start, stop;
};

struct spgemm_context {
  hipStream_t stream = nullptr;
  spgemm_allocator alloc{};
  bool has_alloc = false;
  int timing = 0;
  int force = 0;
  int direct_min = kDirectMinDefault;
  int64_t col_list = 1;   // 0 off, 1 automatic size, larger: byte limit
  int block_table = 1;    // 0: never build the block-offset table of B (pieces are bisected)
  int64_t merge_limit = 0xffffffffLL;   // components of the outer product's all array and a batch together: fewer
  int search_ratio = 4;   // searched tiles for rows with at most this many products per entry (0: never)
  int row_block = 0;      // 1: A is a block of rows of a larger matrix (row pointer values are that matrix's positions)
  double whole_ip = 0;    // ... and the products of all its rows
  std::string err = "";
  bool device_ready = false;
  bool big_lds_ready = false;
  int num_cus = 0;
  std::vector<TimedLaunch> timed;        // launches of the phase in flight
  std::vector<hipEvent_t> event_pool;
  hipStream_t second = nullptr;   // of spgemm_pipelined, and the device it is on: made when first wanted, released with the handle
  int second_device = -1;
};

struct spgemm_plan_s {
  spgemm_context* h = nullptr;
  int64_t m = 0, k = 0, n = 0, nnz_a = 0, nnz_b = 0;
  int dtype = 0;
  void* scratch = nullptr;
  size_t scratch_bytes = 0, scratch2_bytes = 0;
  int* ip = nullptr;
  int* cnt = nullptr;
  int* perm_sym = nullptr;
  int* perm_num = nullptr;
  unsigned char* bin = nullptr;
  long long* partial = nullptr;
  unsigned long long* desc = nullptr;   // per entry of A: its B row (optional, an allocation of its own: given back when the rest needs the room)
  size_t desc_bytes = 0;
  void* scratch2 = nullptr;  // sized after the row classes are known: block offsets of B, tile and run lists
  int* blk_ptr = nullptr;    // rows(B) x blk_ptr_cols offsets, null when not needed or too large
  int blk_ptr_cols = 0;      // column blocks + 1
  TileRec* tiles = nullptr;
  RunRec* runs = nullptr;
  void* scratch3 = nullptr;  // optional, sized from what the device has free: what short rows leave for the numeric phase, then the column list of the ranked tiles
  int32_t* col_list = nullptr;
  unsigned long long col_list_cap = 0;
  size_t list_bytes = 0, short_bytes = 0;
  unsigned* esc_words[2] = {nullptr, nullptr};   // sorted words of the rows of symbolic bins 0 and 1
  unsigned* records = nullptr;   // rows of symbolic bin 2
  int* record_of = nullptr;      // per row of A: its record, -1 = none (written for the rows of symbolic bin 2)
  int* shift_of = nullptr;       // where rows are alike, per row of A: how far its columns are from the record's
  unsigned record_rows = 0;      // rows of the bin that have room for a record
  Control* ctl = nullptr;
  int64_t scan_blocks = 0;
  int64_t recorded = 0;          // rows that have a record
  int force = 0;                 // SPGEMM_OPT_FORCE_WORKSPACE of the symbolic phase
  bool alike = false;            // rows are mostly the row before moved to other columns
  bool flag_rows = false;        // classes 0 and 1 take the flag-list workspace
  bool all_listed = false;       // every row of the dense classes has its structure in the column list
  bool order_kept = false;       // the checksums of the order of the entries were taken
  bool tiles_ordered = false;    // rows were planned as tiles of an ascending B
  bool wide_tiles = false;       // the tiles are planned for a workgroup that has a compute unit to itself
  bool symbolic_done = false;
  bool numeric_pending = false;   // timed numeric launches not yet folded into stats
  bool numeric_in_flight = false; // numeric kernels were enqueued and the stream has not been waited for since
  spgemm_stats stats{};
};

namespace {

int fail(spgemm_context* h, int code, const std::string& msg) {
  if (h) h->err = msg;
  return code;
}

#define HIP_TRY(h, expr)                                                                 \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      return fail((h), SPGEMM_HIP_ERROR, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

int check_csr(spgemm_context* h, const spgemm_csr* M, const char* name) {
  if (!M) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + " is null");
  if (M->rows < 0 || M->cols < 0 || M->nnz < 0) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": negative size");
  if (M->dtype != SPGEMM_F32 && M->dtype != SPGEMM_F64) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": unknown dtype");
  if (!M->rowptr) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": rowptr is null");
  if (M->nnz > 0 && (!M->colidx || !M->values)) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": colidx/values null with nnz > 0");
  if (M->rows >= 0x7fffffffLL || M->cols >= 0x7fffffffLL)
    return fail(h, SPGEMM_UNSUPPORTED, std::string(name) + ": rows and cols must be below 2^31 - 1");
  return SPGEMM_OK;
}

int check_pair(spgemm_context* h, const spgemm_csr* A, const spgemm_csr* B) {
  int rc = check_csr(h, A, "A");
  if (rc) return rc;
  rc = check_csr(h, B, "B");
  if (rc) return rc;
  if (A->cols != B->rows) return fail(h, SPGEMM_DIM_MISMATCH, "A.cols != B.rows");
  if (A->dtype != B->dtype) return fail(h, SPGEMM_DTYPE_MISMATCH, "A and B value types differ");
  return SPGEMM_OK;
}

void* dev_alloc(spgemm_context* h, size_t bytes) {
  if (bytes == 0) bytes = 256;
  if (h->has_alloc) return h->alloc.alloc(h->alloc.ctx, bytes);
  void* p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();   // (the thread's last error stays until it is asked for: a call that goes on without would find it behind its kernels)
  return nullptr;
}

void dev_free(spgemm_context* h, void* p) {
  if (!p) return;
  if (h->has_alloc) h->alloc.free(h->alloc.ctx, p);
  else (void)hipFree(p);
}

template <typename K>
int allow_lds(spgemm_context* h, K kernel, size_t bytes) {
  HIP_TRY(h, hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  return SPGEMM_OK;
}

int ensure_device(spgemm_context* h) {
  if (h->device_ready) return SPGEMM_OK;
  int dev = 0;
  HIP_TRY(h, hipGetDevice(&dev));
  hipDeviceProp_t prop;
  HIP_TRY(h, hipGetDeviceProperties(&prop, dev));
  if (prop.warpSize != kWave) return fail(h, SPGEMM_UNSUPPORTED, "device is not wave64");
  h->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  h->device_ready = true;
  return SPGEMM_OK;
}

// The kernels that use more LDS than a kernel gets unasked are allowed it when a handle first has rows for them (a call each: for a handle
// that never has, that was 10 us of its first product).
int ensure_big_lds(spgemm_context* h) {
  if (h->big_lds_ready) return SPGEMM_OK;
  int rc;
  if ((rc = allow_lds(h, k_sym_dense<16, 8, 1024>, sym_dense_lds<16, 1024>(kSymShortCols / 32)))) return rc;
  if ((rc = allow_lds(h, k_sym_dense<16, 4, 1024>, sym_dense_lds<16, 1024>(kSymFlagWords)))) return rc;
  if ((rc = allow_lds(h, k_sym_dense<16, 8, 512>, sym_dense_lds<16, 512>(kSymNarrowCols / 32)))) return rc;
  if ((rc = allow_lds(h, k_sym_dense<8, 8, 512>, sym_dense_lds<8, 512>(kSymShortCols / 32)))) return rc;
  if ((rc = allow_lds(h, k_num_tiles<float>, num_tiles_lds<float>()))) return rc;
  if ((rc = allow_lds(h, k_num_tiles<double>, num_tiles_lds<double>()))) return rc;
  if ((rc = allow_lds(h, k_num_wide<float>, num_wide_lds<float>()))) return rc;
  if ((rc = allow_lds(h, k_num_wide<double>, num_wide_lds<double>()))) return rc;
  if ((rc = allow_lds(h, k_num_staged<float>, staged_lds<float>()))) return rc;
  if ((rc = allow_lds(h, k_num_staged<double>, staged_lds<double>()))) return rc;
  h->big_lds_ready = true;
  return SPGEMM_OK;
}

// The handle's second stream, on the device that is current.  (Made and released by every call: R-MAT scale 12 in two row blocks 432 | 384 us,
// scale 17 in four 5565 | 5520; finer chunks of rows in the row count are worth as much again there, 5571 | 5520.)
int ensure_second_stream(spgemm_context* h) {
  int dev = 0;
  HIP_TRY(h, hipGetDevice(&dev));
  if (h->second && h->second_device == dev) return SPGEMM_OK;
  if (h->second) (void)hipStreamDestroy(h->second);
  h->second = nullptr;
  HIP_TRY(h, hipStreamCreateWithFlags(&h->second, hipStreamNonBlocking));
  h->second_device = dev;
  return SPGEMM_OK;
}

hipEvent_t take_event(spgemm_context* h) {
  if (!h->event_pool.empty()) {
    hipEvent_t e = h->event_pool.back();
    h->event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}

struct Timer {
  spgemm_context* h;
  int cls;
  TimedLaunch t{};
  Timer(spgemm_context* h_, int cls_) : h(h_), cls(cls_) {
    if (h->timing) {
      t.cls = cls;
      t.start = take_event(h);
      t.stop = take_event(h);
      (void)hipEventRecord(t.start, h->stream);
    }
  }
  ~Timer() {
    if (h->timing) {
      (void)hipEventRecord(t.stop, h->stream);
      h->timed.push_back(t);
    }
  }
};

// After a stream synchronisation: fold event times into the plan's statistics.
void collect_times(spgemm_context* h, spgemm_stats* st) {
  for (auto& t : h->timed) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.start, t.stop) == hipSuccess) {
      st->kernel_ms[t.cls] += ms;
      st->kernel_launches[t.cls] += 1;
    }
    h->event_pool.push_back(t.start);
    h->event_pool.push_back(t.stop);
  }
  h->timed.clear();
}

// Forget the launches timed so far (their events go back to the pool).
void drop_timed(spgemm_context* h) {
  for (auto& t : h->timed) { h->event_pool.push_back(t.start); h->event_pool.push_back(t.stop); }
  h->timed.clear();
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

inline unsigned grid_for(int64_t items, int64_t per_block, int64_t cap) {
  int64_t g = ceil_div(items > 0 ? items : 1, per_block);
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Sorted-list keys can carry their list position when every column, shifted by the list's log2 capacity, stays below the padding key.
constexpr int64_t kEscPackCols0 = int64_t(1) << 25, kEscPackCols1 = int64_t(1) << 23;
// The numeric phase marks the columns again: where B is larger than a die's L2 cache that is a second line of memory per A entry,
// which pays when the entry brings eight products or more.  10^6 rows (fp64, us sorted list | flags, 4000 columns): 8 entries times
// rows of 4, B of 10^4 rows 576 | 515, 10^5 589 | 552, 5 10^5 739 | 819, 2 10^6 737 | 1032; 8 times 12: 1230 | 848, 1273 | 929, 1324 |
// 1152, 1465 | 1390; 3 times 16: 894 | 502, 927 | 525, 971 | 600, 1202 | 728.  Rows of fewer than four entries leave a lane's four places
// empty in both phases (whole calls, 8000 columns, near B): 16 times 2 1004 | 1128, 2 times 2 594 | 631, 4 times 3 683 | 697, but 6 times 4
// 472 | 464.
constexpr int64_t kFlagMaxNnz = int64_t(1) << 20;
// Few rows do not fill the card: then what counts is how long a row takes, and the numeric phase of 128 products takes longer.  Rows of 100
// products, both phases, us sorted list | flags: 500 rows 10.8 | 12.4, 2000 11.0 | 12.2, 4000 13.2 | 13.1, 8000 17.9 | 14.8, 32 000 44.8 | 26.6.
constexpr int64_t kFlagMinRows = 4096;
constexpr size_t kAskFreeAbove = (size_t)64 << 20;   // optional memory below this is taken without asking the device what it has free

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

// Whether the rows of classes 0 and 1 take the flag-list workspace (flag_kernels.hpp) instead of the sorted list, where there are
// kFlagMinRows of them.
bool flag_rows_ok(spgemm_context* h, const spgemm_csr* B) {
  return h->force != 1 && B->cols <= kFlagMaxCols && B->nnz >= (B->nnz <= kFlagMaxNnz ? 4 : 8) * B->rows;
}

// Whether the row count leaves start and length of every A entry's B row: 8 bytes an entry, written once and read twice, in place
// of a gather of B's row pointer in each of the two kernels of short rows.  It pays where those gathers miss the L2 cache (4 MB
// per XCD) and most rows are short.  4.2 M rows of 8 entries times 4.2 M rows of 4, both kernels and the count:
// 3.50 ms with the gathers, 2.51 ms without; with a cached B the words would cost what they save.
// (Part of a plan's optional memory.  A block of rows of a larger matrix goes without: its positions are those of the whole.)
bool wants_desc(spgemm_context* h, const spgemm_csr* A, const spgemm_csr* B) {   // (never with flag_rows_ok)
  if (flag_rows_ok(h, B) || !h->col_list || h->row_block || (h->col_list > 1 && A->nnz > h->col_list / 8)) return false;
  if (A->rows == 0 || B->rows * 8 <= ((int64_t)4 << 20) || B->nnz >= (int64_t(1) << 39) || A->nnz >= (int64_t(1) << 39)) return false;
  return (double)A->nnz / (double)A->rows * ((double)B->nnz / (double)B->rows) <= (double)kEscLargeCap;
}

void drop_desc(spgemm_context* h, spgemm_plan_s* p) {   // (no kernel that uses it is on its way)
  dev_free(h, p->desc);
  p->desc = nullptr;
  p->desc_bytes = 0;
}

// Rows of A that a workgroup of the row count takes at a time, where they are not so many that k_init_control may take more: fewer
// where there are too few rows to fill the card.  16384 rows of a power-law graph: 256 rows 57 us, 64 rows 27 us.
int count_chunk(spgemm_context* h, int64_t m) { return m >= (int64_t)256 * 2 * h->num_cus ? 256 : 64; }

// Whether rows of bin 4 of at most kDenseLight products are scheduled behind the others of their bin.  Where matrices are wide and rows many they
// lie as they come: the column list may be too short there, and with the rows that want flag words first the light ones, whose few columns save most of their
// tiles, found no room in it (R-MAT scale 20 squared, fp64, a list of three quarters of what all rows take: 3357 instead of 105 000 searched rows,
// k_num_wide 90.6 | 85.4 ms, the whole call 129.3 | 124.9; a shorter list 132.9 | 132.4), and light rows among heavy ones are
// what run_of is after anyway (fp32 113.2 | 113.0 ms, scale 21 with 6 edges 156.5 | 156.3).  With few rows the light ones fill the end (6000 rows of
// 60 x 400 products, 900 000 columns, 1503 | 1472 us).
bool light_last(spgemm_context* h, int64_t m, int64_t b_cols) { return b_cols <= kSymNarrowCols || m < (int64_t)kManyRuns * h->num_cus; }

// Lengths of B's rows in a byte each for the row count: where the row pointer is half as large again as a die's 4 MB of L2 cache (600 000 rows,
// 3 M lookups: no gain, and two launches of 10 us; 10^6 rows, 16 M lookups 225 | 169 us) and looked up more often than it has entries, and the table
// finds room where the lists of rows come to lie afterwards.  (Rows that do not fit a byte are found on the way: the row count looks into the row
// pointer then.)
bool row_lens_ok(const spgemm_csr* A, const spgemm_csr* B) {
  return B->rows * 8 > ((int64_t)6 << 20) && A->nnz >= 2 * B->rows && ceil_div(B->rows, kLensRows) * (int64_t)sizeof(RowLens) <= A->rows * 4;
}

// Symbolic phase, first part: count, check, bin.  Ends with the control block on the host
// (one synchronisation): the second part sizes its lists and launches from the bin populations.
int run_setup(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* A, const spgemm_csr* B, Control* pinned, Control* host) {
  hipStream_t s = h->stream;
  const int64_t m = p->m;
  {
    Timer t(h, SPGEMM_K_COUNT);
    const int chunk = count_chunk(h, m);
    const bool fine = fine_rows(m, A->nnz, B->rows, B->nnz);
    hipLaunchKernelGGL(k_init_control, dim3(1), dim3(kCountThreads), 0, s, p->ctl, m, A->rowptr, chunk, h->num_cus, fine ? 1 : 0);
    const unsigned parts = grid_for(B->nnz > B->rows ? B->nnz : B->rows, kCountThreads * 8, (int64_t)h->num_cus * 4);
    // (as many as run at a time; chunks are drawn: four times as many 500 000 rows 62 | 58 us)
    const unsigned groups = m > 0 ? grid_for(m, fine ? kFineRows : chunk, (int64_t)h->num_cus * 2) : 0;
    RowLens* lens = row_lens_ok(A, B) ? reinterpret_cast<RowLens*>(p->perm_sym) : nullptr;   // (perm_sym is written afterwards)
    if (lens)
      hipLaunchKernelGGL(k_row_lens, dim3((unsigned)ceil_div(B->rows, kLensGroup * kLensRows)), dim3(kLensThreads), 0, s, B->rows, B->rowptr, m,
                         A->nnz, A->rowptr, A->colidx, reinterpret_cast<unsigned*>(lens), p->ctl);
    for (int with = lens ? 1 : 0; with >= 0; --with)
      hipLaunchKernelGGL((with ? k_count_rows<true> : k_count_rows<false>), dim3(parts + groups), dim3(kCountThreads), 0, s, (int)parts, B->cols,
                         B->nnz, B->colidx, m, A->nnz, B->rows, A->rowptr, A->colidx, B->rowptr, p->ip, p->bin, p->cnt, p->ctl, h->force,
                         (h->row_block ? kCountBlock : 0) | (light_last(h, m, B->cols) ? kCountLight : 0), p->desc, lens);
  }
  {
    Timer t(h, SPGEMM_K_BIN);
    hipLaunchKernelGGL(k_bin_scatter, dim3(grid_for(m, kScanTile, (int64_t)1 << 30)), dim3(kScanThreads), 0, s, m, p->bin, p->perm_sym, p->ctl, pinned);
  }
  HIP_TRY(h, hipGetLastError());
  HIP_TRY(h, hipStreamSynchronize(s));
  std::memcpy(host, pinned, sizeof(Control));
  return SPGEMM_OK;
}

// Workgroups of the kernels of recorded rows.  Where rows are alike, as many as are resident together, the same number in both phases, so that a
// wave of the numeric one meets the rows that a wave of the symbolic one has given the same record; otherwise ten a compute unit, two or two and a half
// times as many as are resident in the symbolic phase, which evens out rows that differ (300 000 rows, symbolic us with 8 | 10 | 16 on a compute
// unit: 144 products 394 | 354 | 370, 256 294 | 282 | 287, 400 540 | 511 | 521, 756 1047 | 988 | 1006; 60 000 of 256 67 | 65 | 68; 100 000 ragged ones 247 |
// 254 | 263).
unsigned record_grid(spgemm_context* h, const spgemm_plan_s* p, int64_t rows) {
  const unsigned most = (unsigned)(ceil_div((int64_t)h->num_cus * (p->alike ? kRecordGroups : 10), kDies) * kDies);
  return (unsigned)(ceil_div(grid_for(rows, 4, most), kDies) * kDies);
}

// Workgroups of the sorted-list kernels, per_block rows at a time: each keeps the loads of several rows in flight and pays for their first ones, so
// it should have some twenty times as many; beyond 32 for a compute unit (what is resident, a few times over) they only even out the end.  Whole calls,
// us with 32 | 48 | 96 | 128 a compute unit: 4.2 M rows of 8 x 4 2460 | 2431 | 2434 | 2443, 3 M of 10 x 9 3645 | 3598 | 3555 | 3537, 2 M of 5 x 4 871 | 862 |
// 904 | 912, 400 000 of 8 x 8 461 | 467 | 488 | 504.
unsigned sorted_grid(spgemm_context* h, int64_t rows, int64_t per_block) {
  const int64_t least = (int64_t)h->num_cus * 32, most = (int64_t)h->num_cus * 128, twenty = ceil_div(rows, per_block) / 20;
  return grid_for(rows, per_block, twenty < least ? least : (twenty < most ? twenty : most));
}

// Whether the classes of shorter rows share a launch (short_kernels.hpp): where there are rows of two of them, and no more than fill the chip
// kShortRounds times (each class counted in the workgroups it would like).
constexpr int64_t kShortRounds = 16;
template <typename N>
bool short_rows_ok(spgemm_context* h, const N* hist) {
  int kinds = 0;
  for (int b = 0; b < 4; ++b) kinds += hist[b] > 0 ? 1 : 0;
  const int64_t wgs = (int64_t)hist[0] / 16 + (int64_t)hist[1] / 4 + (int64_t)hist[2] / 4 + (int64_t)hist[3];
  return !h->timing && kinds > 1 && wgs <= kShortRounds * kShortGroups * h->num_cus;   // (with timing every class has a time of its own)
}
unsigned short_grid(int64_t rows, int64_t per_block) { return rows > 0 ? (unsigned)(ceil_div(ceil_div(rows, per_block), kDies) * kDies) : 0; }

// The dense symbolic kernel's workgroups: waves of one, of a SIMD, and how many are resident on the card.
struct SymDense { int waves, per_simd, pieces; size_t lds; unsigned groups; };
SymDense sym_dense_shape(spgemm_context* h, int64_t rows, int64_t cols) {
  const int64_t words = sym_flag_words(cols);
  SymDense d{16, 8, 1024, 0, 0};
  if (cols > kSymNarrowCols) d.per_simd = 4;
  else if (cols > kSymShortCols) d.pieces = 512;
  else if (rows >= (int64_t)h->num_cus * 32) { d.waves = 8; d.pieces = 512; }
  d.lds = d.waves == 8 ? sym_dense_lds<8, 512>(words) : d.pieces == 512 ? sym_dense_lds<16, 512>(words) : sym_dense_lds<16, 1024>(words);
  int64_t per_cu = (int64_t)(160 * 1024 / d.lds);
  per_cu = per_cu < d.per_simd * 4 / d.waves ? per_cu : d.per_simd * 4 / d.waves;
  d.groups = grid_for(rows, 1, (int64_t)h->num_cus * per_cu);
  return d;
}

// Tiles of a row that a workgroup of the numeric kernel takes together: they share the set-up of the row's entries, but where
// rows are few the heavy ones should not be one workgroup's work (about 200 rows a block, us for seven blocks of scale 15: 675 | 486 by
// tile; 5266 rows of scale 14: 153 together, 161 by tile).
int run_tiles_of(spgemm_context* h, int64_t rows) { return rows <= (int64_t)h->num_cus * 8 ? 1 : kRunTiles; }

// Whether the tiles are planned for k_num_wide, one workgroup on a compute unit, from what is known before: the dense rows and their
// products, and the products of an entry of A.  (Later only whether the list holds all rows: run_symbolic.)
// k_num_tiles hides what a tile costs beside its products behind its neighbour's products, but has twice as many tiles.  It gains where a
// row's searched tiles or its only tile are few products, and where many products of an entry of A fall into a tile; it loses where
// these are few.  us for 3000 rows of uniform columns, wide | two workgroups: rows of B of 60 entries, 24 000 products a row, 20 000 columns
// 224 | 337 (3 small tiles a row), 150 000 columns 346 | 435 (4), 60 000 products 960 | 1574 (9), 150 000 products 2953 | 8108 (18);
// of 250 entries 285 | 298, 602 | 662, 1295 | 2143; of 1000 entries 281 | 291, 569 | 584, 1150 | 1318; one tile a row 114 | 107, 111 | 95, 111 |
// 97; direct tiles only (20 000 columns, 150 000 products) 1373 | 1270, 797 | 710, 715 | 596.  R-MAT squared, 16 edges: scale 14 204 | 169,
// scale 17 3311 | 2812, scale 19 25.9 | 23.4 ms; 4 edges, scale 18 1348 | 1210.  6000 products a row, 400 000 columns 293 | 186 us.
// Beyond 2^19 columns a row's flag words alone are four small tiles: 24 000 products, 10^6 columns 410 | 478 to 511 | 694 us, R-MAT scale 20
// 70.5 | 74.9 ms; but rows that are mostly searched 3.28 | 2.35 ms (600 000 columns, 4800 products).
bool wide_tiles_from(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* B, bool with_table, double rows_d, double ip_d, double ip_all) {
  if (!with_table || B->nnz >= kTileMaxNnz) return true;   // (k_num_tiles has no way without)
  const double ip_row = ip_d / rows_d, n = (double)B->cols, blocks = (double)ceil_div(B->cols, kBlkCols);
  if (ip_row <= (double)kSearchRow) return false;
  if (B->cols > kSymNarrowCols) return true;
  const double entries = n * -std::expm1(-ip_row / n);   // (of a row of C, were its columns drawn uniformly)
  const bool direct = entries >= h->direct_min * n / kBlkCols;
  const double per_tile = std::floor(kTileBudget / (kRankBlkBytes + kRankEntryBytes * entries / blocks));   // blocks
  const double tiles = direct || per_tile < 1.0 ? blocks : std::ceil(blocks / per_tile);
  const double per_entry = p->nnz_a > 0 ? ip_all / (double)p->nnz_a : 0.0;
  return tiles > 1.0 && per_entry < (direct ? 16.0 : 64.0) * tiles;
}

// Sizes and allocates what the dense kernels need beyond the per-row arrays: the tile and run
// lists (from an upper bound of the number of tiles) and the table of block offsets of B.
int alloc_dense_lists(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* B, const Control& host, unsigned* tile_cap,
                      unsigned* run_cap, double* list_want) {
  *tile_cap = 0; *run_cap = 0; *list_want = 0;
  double rows_d = 0, ip_d = 0;
  for (int b = 4; b <= 6; ++b) { rows_d += host.hist[0][b]; ip_d += (double)host.bin_ip[0][b]; }
  if (rows_d == 0) return SPGEMM_OK;
  const double n = (double)B->cols;
  const double blocks = (double)ceil_div(B->cols, kBlkCols);
  const double spans = (double)ceil_div(B->cols, (int64_t)kSymFlagWords * 32);
  // direct tiles hold at least direct_min entries each and there is at most one per block;
  // of two neighbouring ranked tiles at least one pair exceeds the tile budget together
  double direct = rows_d * blocks;
  if (ip_d / h->direct_min < direct) direct = ip_d / h->direct_min;
  const double entries = ip_d < rows_d * n ? ip_d : rows_d * n;
  const double weight = rows_d * blocks * kRankBlkBytes + (double)kRankEntryBytes * entries;
  // (+ a slab per workgroup of the symbolic kernel: what a workgroup has drawn and not used)
  p->blk_ptr_cols = (int)blocks + 1;
  const size_t bp_bytes = (size_t)B->rows * (size_t)p->blk_ptr_cols * 4;
  const bool with_bp = h->block_table && host.b_sorted && B->nnz > 0 && bp_bytes <= ((size_t)1 << 30);
  p->wide_tiles = wide_tiles_from(h, p, B, with_bp, rows_d, ip_d, h->row_block ? h->whole_ip : (double)host.ip_total);
  const double wgs = (double)sym_dense_shape(h, (int64_t)rows_d, B->cols).groups + 1.0;
  // (a row's tiles, at most kSpanBlocks a span, lie together: a slab may end with so many less one that its next row does not fit)
  const double planned = 2.0 * direct + 2.0 * weight / (p->wide_tiles ? kWideTileBudget : kTileBudget) + 4.0 * rows_d * spans + 16.0;
  const double tiles = planned * kTileSlab / (kTileSlab - kSpanBlocks + 1) + wgs * kTileSlab;
  const double runs = rows_d + planned / run_tiles_of(h, (int64_t)rows_d) + rows_d * spans + 16.0;
  if (tiles > 4.0e9) return fail(h, SPGEMM_UNSUPPORTED, "tile list of the dense workspace would exceed 2^32 records");
  *tile_cap = (unsigned)tiles;
  *run_cap = (unsigned)runs;
  size_t off = 0;
  const size_t o_tiles = off; off = align_up(off + (size_t)*tile_cap * sizeof(TileRec));
  const size_t o_runs = off; off = align_up(off + (size_t)*run_cap * sizeof(RunRec));
  const size_t o_bp = off; if (with_bp) off = align_up(off + bp_bytes);
  p->scratch2 = dev_alloc(h, off);
  p->scratch2_bytes = off;
  if (!p->scratch2) return fail(h, SPGEMM_ALLOC_FAILED, "device allocation of the dense workspace lists failed");
  unsigned char* base = static_cast<unsigned char*>(p->scratch2);
  p->tiles = reinterpret_cast<TileRec*>(base + o_tiles);
  p->runs = reinterpret_cast<RunRec*>(base + o_runs);
  p->blk_ptr = with_bp ? reinterpret_cast<int*>(base + o_bp) : nullptr;
  // Column list: the dense symbolic kernel leaves the columns of its ranked tiles there, which saves
  // the numeric kernel one pass over those tiles' products.  (Every row's share is rounded up to 16 bytes.)
  // On top of it what the workgroups of the symbolic kernel draw and leave unused: the first or last slab of each (a quarter of the list, at
  // most kListSlab entries each: list_slab_of) and the ends of the others.  Without room for that a quarter of the rows of a product with
  // few repeated columns lost their place in the list (300 rows of 3000 entries: 225 of them listed), and one such row sends all
  // tiles to the general numeric kernel.
  // (a row takes no more than the flag words of its spans, or the columns of a searched one)
  const double words = (double)(span_flag_words(B->cols, 0) + span_rank_slots(span_flag_words(B->cols, 0)));
  const double row_most = spans * (words > (double)kSearchRow ? words : (double)kSearchRow);
  const double entries_want = (entries < rows_d * row_most ? entries : rows_d * row_most) + 4.0 * rows_d * spans, slabs = wgs * kListSlab;
  *list_want = (1.15 * entries_want + (0.4 * entries_want < slabs ? 0.4 * entries_want : slabs) + 64.0) * 4.0;   // (+ 64: it is cut to whole 256 bytes)
  return SPGEMM_OK;
}

// The optional part of a plan, one allocation that the product does without when it fails: the column list of the dense rows, and
// what the symbolic kernels of short rows leave for the numeric ones (esc_kernels.hpp, record_kernels.hpp): sorted words for
// all rows of a bin or for none, records for as many rows as there is room for.  When it is refused, the list is asked for alone.
// The descriptions of A's entries, which the row count has left, go when there is no room for them.
// value_bytes: of an entry of C.  staged: the numeric phase takes all rows this short through the staged list, which reads neither.
// plan_leaves: the numeric phases on the plan look at the order of the entries first, which pays for sorted words alone from a million
// products on (numeric phase with words and check | without either, us: 0.1 M products 12 | 7, 0.75 M 14.6 | 10, 3 M 27 | 39).
constexpr unsigned long long kWordsWithCheck = 1ULL << 20;
void alloc_optional(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* B, const Control& host, double list_want, size_t value_bytes, bool staged,
                    bool plan_leaves) {
  if (!h->col_list) return;
  const int64_t max_cols[2] = {kEscPackCols0, kEscPackCols1};
  const size_t word_bytes[2] = {kEscSmallCap * 4, kEscLargeCap * 4};
  const size_t rec_rows = !staged && B->cols <= (int64_t(1) << kRecColBits) ? host.hist[0][2] : 0;
  const bool with_words = !staged && !p->flag_rows && (!plan_leaves || rec_rows || host.bin_ip[0][0] + host.bin_ip[0][1] >= kWordsWithCheck);
  size_t words[2], want = 0;
  for (int b = 0; b < 2; ++b) {
    words[b] = with_words && B->cols <= max_cols[b] ? align_up(host.hist[0][b] * word_bytes[b]) : 0;
    want += words[b];
  }
  const size_t rec_bytes = (size_t)kRecWords * 4, map = align_up((size_t)p->m * 4);
  if (rec_rows) want += map * (p->alike ? 2 : 1) + rec_rows * rec_bytes;
  const double asked = h->col_list > 1 ? (double)h->col_list : 1.0e30;
  size_t limit = asked - (double)p->desc_bytes < (double)want ? (size_t)(asked - (double)p->desc_bytes) : want;
  if ((double)(want + p->desc_bytes) + list_want > (double)kAskFreeAbove) {
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    double entries = 0;   // of C, at most
    for (int b = 0; b < kNumBins; ++b) {
      const double ip = (double)host.bin_ip[0][b], full = (double)host.hist[0][b] * (double)B->cols;
      entries += ip < full ? ip : full;
    }
    const PlanRoom room = plan_room((double)free_b, list_want, (double)want, (double)p->desc_bytes, entries * (double)(4 + value_bytes), asked);
    if (!room.desc) drop_desc(h, p);
    limit = (size_t)room.shorts;
    list_want = room.list;
  }
  if (list_want > asked) list_want = asked;
  size_t list_bytes = ((size_t)list_want) & ~(size_t)255;
  if (list_bytes < 4096) list_bytes = 0;
  size_t off = 0, o_words[2] = {0, 0};
  for (int b = 0; b < 2; ++b) {
    if (words[b] && off + words[b] <= limit) { o_words[b] = off; off += words[b]; }
    else words[b] = 0;
  }
  size_t rows = 0;
  const size_t o_map = off;
  if (rec_rows && off + map + rec_bytes <= limit && off + 2 * map + rec_bytes > limit) p->alike = false;   // (room for records, but not for shifts)
  const size_t maps = map * (p->alike ? 2 : 1);
  if (rec_rows && off + maps + rec_bytes <= limit) {
    rows = (limit - off - maps) / rec_bytes;
    if (rows > rec_rows) rows = rec_rows;
    off = align_up(off + maps + rows * rec_bytes);
  }
  if (off + list_bytes == 0) return;
  unsigned char* base = static_cast<unsigned char*>(dev_alloc(h, off + list_bytes));
  if (!base && off && list_bytes) {
    off = 0; rows = 0; words[0] = words[1] = 0;
    base = static_cast<unsigned char*>(dev_alloc(h, list_bytes));
  }
  if (!base) return;
  p->scratch3 = base;
  p->short_bytes = off;
  p->list_bytes = list_bytes;
  for (int b = 0; b < 2; ++b) if (words[b]) p->esc_words[b] = reinterpret_cast<unsigned*>(base + o_words[b]);
  if (rows) {
    p->record_of = reinterpret_cast<int*>(base + o_map);
    if (p->alike) p->shift_of = reinterpret_cast<int*>(base + o_map + map);
    p->records = reinterpret_cast<unsigned*>(base + o_map + maps);
    p->record_rows = (unsigned)rows;
  }
  if (list_bytes) {
    p->col_list = reinterpret_cast<int32_t*>(base + off);
    p->col_list_cap = list_bytes / 4;
  }
}

// Capacities of the dense workspace's lists, and their cursors behind the first slab of every workgroup of k_sym_dense (runs: behind a place
// for every row).
__global__ void k_set_caps(Control* ctl, unsigned tile_cap, unsigned run_cap, unsigned long long list_cap, int64_t rows, unsigned workgroups) {
  if (threadIdx.x == 0) {
    ctl->tile_cap = tile_cap; ctl->run_cap = run_cap; ctl->list_cap = list_cap;
    ctl->tile_cursor = workgroups * kTileSlab;
    ctl->run_cursor = (unsigned)rows;   // (a place for the first run of every row)
    ctl->list_cursor = workgroups * list_slab_of(list_cap, workgroups);
  }
}

bool same_columns(const spgemm_csr* A, const spgemm_csr* B) { return A->colidx == B->colidx && A->nnz == B->nnz; }

// The order of the operands' entries: kept with the plan (plan = 1), or compared with it.
void sum_order(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* A, const spgemm_csr* B, int plan) {
  const int64_t most = A->nnz > B->nnz ? A->nnz : B->nnz;
  hipLaunchKernelGGL(k_order_sum, dim3(grid_for(most, kOrderTile, kOrderParts)), dim3(kOrderThreads), 0, h->stream, A->nnz, A->colidx, B->nnz,
                     same_columns(A, B) ? (const int32_t*)nullptr : B->colidx, p->ctl, plan);
}

// launch(words of flags per lane, as a type)
template <class F>
void with_flag_words(int64_t cols, F launch) {
  switch (flag_words_per_lane(cols)) {
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    default: launch(std::integral_constant<int, 16>{});
  }
}

// plan_leaves: the plan goes to the caller, whose numeric phases may bring the entries in another order.
template <typename T>
int run_symbolic(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* A, const spgemm_csr* B, int64_t* c_rowptr,
                 const Control& host, Control* pinned, bool plan_leaves) {
  hipStream_t s = h->stream;
  const int64_t m = p->m;
  const int64_t cap_small = (int64_t)h->num_cus * 32;
  const int pack32 = B->cols <= kEscPackCols0 ? 1 : 0, pack128 = B->cols <= kEscPackCols1 ? 1 : 0;
  const size_t lds_hash_large = hash_lds_bytes<256, 12, false>();
  const unsigned* hist = host.hist[0];
  const int64_t rows_dense = (int64_t)hist[4] + hist[5] + hist[6];
  // rows of at most this many products never reach the dense numeric kernel (0: class unavailable)
  // (the staged class is taken only on request: short rows whose columns are in the plan's list
  // become searched tiles of the dense kernel, which costs them one global round trip less)
  const int staged = (h->force == 4 && ceil_div(B->cols, kStWinCols) <= kStMaxWindows) ? staged_cap<T>() : 0;
  unsigned tile_cap = 0, run_cap = 0;
  double list_want = 0;
  if (rows_dense > 0 || staged > 0) {
    const int lds = ensure_big_lds(h);
    if (lds) return lds;
  }
  p->alike = host.moved > 0 && host.moved * 2 >= host.looked;
  if (hist[0] + hist[1] == 0) drop_desc(h, p);   // (nobody reads it)
  if ((int64_t)hist[0] + hist[1] < kFlagMinRows) p->flag_rows = false;
  int rc = alloc_dense_lists(h, p, B, host, &tile_cap, &run_cap, &list_want);
  if (rc == SPGEMM_ALLOC_FAILED && p->desc) {
    drop_desc(h, p);
    rc = alloc_dense_lists(h, p, B, host, &tile_cap, &run_cap, &list_want);
  }
  if (rc) return rc;
  alloc_optional(h, p, B, host, list_want, sizeof(T), staged > 0, plan_leaves);
  if ((double)p->list_bytes + 256.0 <= list_want) p->wide_tiles = true;   // (some row may find no room in the list)
  p->tiles_ordered = rows_dense > 0 && host.b_sorted != 0;
  p->order_kept = plan_leaves && (p->records || p->esc_words[0] || p->esc_words[1] || (p->tiles_ordered && p->force != 2));
  if (p->order_kept) {
    Timer t(h, SPGEMM_K_COUNT);
    sum_order(h, p, A, B, 1);
  }
  if (rows_dense > 0) {
    hipLaunchKernelGGL(k_set_caps, dim3(1), dim3(64), 0, s, p->ctl, tile_cap, run_cap, p->col_list_cap, rows_dense, sym_dense_shape(h, rows_dense, B->cols).groups);
    if (p->blk_ptr) {
      Timer t(h, SPGEMM_K_BLOCK_PTR);
      const int64_t items = B->rows * (int64_t)p->blk_ptr_cols;
      hipLaunchKernelGGL(k_block_ptrs, dim3(grid_for(items, 256, (int64_t)h->num_cus * 64)), dim3(256), 0, s, B->rows,
                         p->blk_ptr_cols, B->rowptr, B->colidx, p->ctl, p->blk_ptr);
    }
  }
  // rows of bin 2 have few products and hardly any of them many, or none where they share a launch
  const bool few = !p->alike && host.bin_ip[0][2] <= (unsigned long long)kFewProducts * hist[2] && host.long_rows <= hist[2] / kFewLongShare;
  if (m > 0) {
    if (!p->flag_rows && !p->desc && short_rows_ok(h, hist)) {
      const SymShort sh{{short_grid(hist[3], 1), hist[2] ? record_grid(h, p, hist[2]) : 0u, short_grid(hist[1], 4), short_grid(hist[0], 16)},
          p->perm_sym, p->ip, A->rowptr, B->rowptr, A->colidx, B->colidx, B->nnz, B->cols, pack32, pack128, p->cnt, p->esc_words[0], p->esc_words[1],
          p->records, p->record_rows, p->record_of, p->shift_of};
      const bool slots_few = few && host.long_rows == 0;
      const size_t lds = slots_few ? sym_short_lds<kFewLogSlots>() : sym_short_lds<kSymLogSlots>();
      hipLaunchKernelGGL((p->alike ? k_sym_short<true, kSymLogSlots> : slots_few ? k_sym_short<false, kFewLogSlots> : k_sym_short<false, kSymLogSlots>),
                         dim3(sh.wgs[0] + sh.wgs[1] + sh.wgs[2] + sh.wgs[3]), dim3(256), lds, s, p->ctl, sh);
    } else {
      {
        Timer t(h, SPGEMM_K_SYM_ESC);
        if (p->flag_rows) {
          auto rows = [&](auto wpl) {
            constexpr int W = decltype(wpl)::value;
            if (hist[0])
              hipLaunchKernelGGL((k_flag_sym<32, W>), dim3(grid_for(hist[0], kFlagRows, cap_small)), dim3(256), 0, s, p->perm_sym, p->ctl, 0,
                                 A->rowptr, A->colidx, B->rowptr, B->colidx, B->nnz, p->cnt);
            if (hist[1])
              hipLaunchKernelGGL((k_flag_sym<128, W>), dim3(grid_for(hist[1], kFlagRows, cap_small)), dim3(256), 0, s, p->perm_sym, p->ctl, 1,
                                 A->rowptr, A->colidx, B->rowptr, B->colidx, B->nnz, p->cnt);
          };
          with_flag_words(B->cols, rows);
        }
        if (hist[0] && !p->flag_rows)
          hipLaunchKernelGGL((p->desc ? k_esc_sym<16, 32, true> : k_esc_sym<16, 32, false>), dim3(sorted_grid(h, hist[0], 16)), dim3(256), 0, s,
                             p->perm_sym, p->ctl, 0, A->rowptr, A->colidx, B->rowptr, p->desc, B->colidx, B->nnz, pack32, p->cnt, p->esc_words[0]);
        if (hist[1] && !p->flag_rows)
          hipLaunchKernelGGL((p->desc ? k_esc_sym<64, 128, true> : k_esc_sym<64, 128, false>), dim3(sorted_grid(h, hist[1], 4)), dim3(256), 0,
                             s, p->perm_sym, p->ctl, 1, A->rowptr, A->colidx, B->rowptr, p->desc, B->colidx, B->nnz, pack128, p->cnt,
                             p->esc_words[1]);
      }
      {
        Timer t(h, SPGEMM_K_SYM_HASH);
        if (hist[2]) {
          hipLaunchKernelGGL((p->alike ? k_sym_wave<true, kSymLogSlots> : few ? k_sym_wave<false, kFewLogSlots> : k_sym_wave<false, kSymLogSlots>),
                             dim3(record_grid(h, p, hist[2])), dim3(256), 0, s, p->perm_sym, p->ctl, 2, A->rowptr, A->colidx,
                             B->rowptr, B->colidx, B->nnz, p->cnt, p->records, p->record_rows, p->record_of, p->shift_of);
        }
        if (hist[3])
          hipLaunchKernelGGL((k_hash<256, 12, T, false>), dim3(grid_for(hist[3], 1, (int64_t)h->num_cus * 8)), dim3(256),
                             lds_hash_large, s, p->perm_sym, p->ctl, 0, 3, p->ip, A->rowptr, A->colidx,
                             (const T*)nullptr, B->rowptr, B->colidx, (const T*)nullptr, p->cnt, (const int64_t*)nullptr,
                             (int32_t*)nullptr, (T*)nullptr, B->cols, (const int*)nullptr, 0, kOrderNotLooked);
      }
    }
    if (rows_dense > 0) {
      Timer t(h, SPGEMM_K_SYM_DENSE);
      const SymDense d = sym_dense_shape(h, rows_dense, B->cols);
      hipLaunchKernelGGL((d.waves == 8 ? k_sym_dense<8, 8, 512> : d.per_simd == 4 ? k_sym_dense<16, 4, 1024> : d.pieces == 512 ? k_sym_dense<16, 8, 512> : k_sym_dense<16, 8, 1024>), dim3(d.groups), dim3(d.waves * kWave), d.lds, s, p->perm_sym, p->ctl, A->rowptr, A->colidx, B->rowptr, B->colidx, B->cols, p->ip, p->cnt, p->tiles, p->runs, p->col_list, h->direct_min,
                         staged, h->search_ratio, p->blk_ptr, p->blk_ptr_cols, B->nnz, run_tiles_of(h, rows_dense), p->wide_tiles ? 1 : 0);
    }
    if (p->scan_blocks > 1) {
      Timer t(h, SPGEMM_K_BIN);
      hipLaunchKernelGGL(k_classify_numeric, dim3((unsigned)p->scan_blocks), dim3(kScanThreads), 0, s, m, p->ip, p->cnt, p->bin, p->partial, p->ctl,
                         h->force, staged);
    }
  }
  {
    Timer t(h, SPGEMM_K_SCAN);
    const int direct = p->scan_blocks <= kScanDirect ? 1 : 0;
    if (!direct) hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(kScanBlockThreads), 0, s, p->scan_blocks, p->partial, m, c_rowptr, p->ctl);
    hipLaunchKernelGGL((p->scan_blocks == 1 ? k_scan_final<true> : k_scan_final<false>), dim3(p->scan_blocks > 0 ? (unsigned)p->scan_blocks : 1u),
                       dim3(kScanThreads), 0, s, m, p->scan_blocks, direct, p->cnt, p->partial, p->ip, h->force, staged, p->bin, p->perm_num,
                       c_rowptr, p->ctl, pinned);
  }
  HIP_TRY(h, hipGetLastError());
  return SPGEMM_OK;
}

__global__ void k_reset_numeric_work(Control* ctl) {
  if (threadIdx.x == 0) { ctl->work[1] = 0; ctl->work[2] = 0; }
  SPG_CLK(if (threadIdx.x < kClkSlots) ctl->clk[1][threadIdx.x] = 0;)
}

template <typename T>
int run_numeric(spgemm_context* h, spgemm_plan_s* p, const spgemm_csr* A, const spgemm_csr* B, const int64_t* c_rp,
                int32_t* c_col, void* c_val_v) {
  hipStream_t s = h->stream;
  const int64_t m = p->m;
  if (m == 0) return SPGEMM_OK;
  const int64_t cap_small = (int64_t)h->num_cus * 32;
  const int pack32 = B->cols <= kEscPackCols0 ? 1 : 0, pack128 = B->cols <= kEscPackCols1 ? 1 : 0;
  const T* a_val = static_cast<const T*>(A->values);
  const T* b_val = static_cast<const T*>(B->values);
  T* c_val = static_cast<T*>(c_val_v);
  const size_t lds_hash_small = hash_lds_bytes<64, 8, true>();
  const size_t lds_hash_large = hash_lds_bytes<256, 11, true>();
  const int64_t* hist = p->stats.num_bin_rows;
  // (rows of class 3 with more products than the symbolic hash takes have tiles: those do them, unless hashing is asked for)
  const bool tiles3 = p->force != 2;
  const bool run_tiles = hist[5] + hist[6] > 0 || (tiles3 && hist[3] > 0 && p->stats.dense_runs > 0);
  if (hist[4] > 0 || run_tiles) hipLaunchKernelGGL(k_reset_numeric_work, dim3(1), dim3(64), 0, s, p->ctl);
  // (the words were sorted for the rows of the symbolic bin: they serve when the numeric one holds the same rows)
  const bool words0 = hist[0] && p->esc_words[0] && hist[0] == p->stats.sym_bin_rows[0];
  const bool words1 = hist[1] && p->esc_words[1] && hist[1] == p->stats.sym_bin_rows[1];
  // On a plan that the caller holds: are the entries in the order of the plan?  If not, the kernels that need it end at once, and
  // k_other_order behind them, which ends at once otherwise (4 us), does their rows.
  const bool check = p->order_kept && (words0 || words1 || p->recorded);
  // (rows of class 3 with tiles, where no row is dense: in another order they are done without tiles)
  const bool check3 = p->order_kept && p->tiles_ordered && tiles3 && hist[3] > 0 && hist[5] + hist[6] == 0 && p->stats.dense_runs > 0;
  // (the kernel of recorded rows looks at the order beside its rows where the entries are few: the kernels that need the plan's
  // order then do their rows whatever it is)
  const bool same = same_columns(A, B);
  const bool inside = check && p->recorded && A->nnz + (same ? 0 : B->nnz) <= kOrderInside;
  const int looked3 = !check3 ? kOrderNotLooked : inside ? kOrderBeside : kOrderSummed;
  // (rows of class 3 that have no tiles; those too that have, in another order than the plan's)
  const bool rows3 = hist[3] && (!tiles3 || check3 || p->stats.sym_bin_rows[2] + p->stats.sym_bin_rows[3] > 0);
  const int most_ip = tiles3 ? kSymHashLarge : 0x7fffffff;
  const bool row_tiles = tiles3 && B->cols <= kRowTileMaxCols;
  auto other_order_rows = [&] {
    const unsigned w0 = words0 ? grid_for(hist[0], 16, cap_small) : 0, w1 = words1 ? grid_for(hist[1], 4, cap_small) : 0,
        w2 = p->recorded ? grid_for(hist[2], 4, cap_small) : 0;
    hipLaunchKernelGGL(k_other_order<T>, dim3(w0 + w1 + w2), dim3(256), other_order_lds_bytes<T>(), s, w0, w1, w2, p->perm_num, p->ctl, p->ip,
                       A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, c_rp, c_col, c_val, pack32, pack128, B->nnz, B->cols, inside ? 1
                       : 0);
  };
  if (!p->flag_rows && !p->desc && !inside && !check3 && short_rows_ok(h, hist)) {
    if (check) sum_order(h, p, A, B, 0);
    NumShort<T> sh{};
    sh.wgs[0] = rows3 ? short_grid(hist[3], 1) : 0;
    sh.wgs[1] = p->recorded ? record_grid(h, p, p->stats.sym_bin_rows[2]) : 0;
    sh.wgs[2] = hist[2] > p->recorded ? short_grid(hist[2], 4) : 0;
    sh.wgs[3] = short_grid(hist[1], 4);
    sh.wgs[4] = short_grid(hist[0], 16);
    sh.perm_sym = p->perm_sym; sh.perm_num = p->perm_num; sh.ip = p->ip;
    sh.a_rp = A->rowptr; sh.a_col = A->colidx; sh.a_val = a_val;
    sh.b_rp = B->rowptr; sh.b_col = B->colidx; sh.b_val = b_val; sh.b_nnz = B->nnz; sh.n_cols = B->cols;
    sh.pack32 = pack32; sh.pack128 = pack128;
    sh.words32 = words0 ? p->esc_words[0] : nullptr;
    sh.words128 = words1 ? p->esc_words[1] : nullptr;
    sh.records = p->records; sh.record_of = p->recorded ? p->record_of : nullptr; sh.shift_of = p->shift_of;
    sh.c_rp = c_rp; sh.c_col = c_col; sh.c_val = c_val;
    sh.tiles = row_tiles ? 1 : 0; sh.most_ip = most_ip; sh.looked = looked3;
    size_t lds = num_short_lds<T>();
    const size_t lds3 = rows3 ? (row_tiles ? row_tile_lds<T>(B->cols) : lds_hash_large) : 0;
    if (lds < lds3) lds = lds3;
    const unsigned wgs = sh.wgs[0] + sh.wgs[1] + sh.wgs[2] + sh.wgs[3] + sh.wgs[4];
    if (wgs) hipLaunchKernelGGL(k_num_short<T>, dim3(wgs), dim3(256), lds, s, p->ctl, sh);
    if (check) other_order_rows();
  } else {
    {
      Timer t(h, SPGEMM_K_NUM_ESC);
      if ((check || check3) && !inside) sum_order(h, p, A, B, 0);
      if (p->flag_rows) {
        auto rows = [&](auto wpl) {
          constexpr int W = decltype(wpl)::value;
          if (hist[0])
            hipLaunchKernelGGL((k_flag_num<32, W, T>), dim3(grid_for(hist[0], kFlagRows, cap_small)), dim3(256), 0, s, p->perm_num, p->ctl, 0,
                               A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, B->nnz, c_rp, c_col, c_val);
          if (hist[1])
            hipLaunchKernelGGL((k_flag_num<128, W, T>), dim3(grid_for(hist[1], kFlagRows, cap_small)), dim3(256), 0, s, p->perm_num, p->ctl, 1,
                               A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, B->nnz, c_rp, c_col, c_val);
        };
        with_flag_words(B->cols, rows);
      } else if (words0)
        hipLaunchKernelGGL((p->desc ? k_esc_num<16, 32, T, true> : k_esc_num<16, 32, T, false>), dim3(sorted_grid(h, hist[0], 16)), dim3(256),
                           0, s, p->perm_sym, p->ctl, 0, A->rowptr, A->colidx, a_val, B->rowptr, p->desc, b_val, B->nnz, p->esc_words[0], c_rp,
                           c_col, c_val);
      else if (hist[0])
        hipLaunchKernelGGL((k_esc<16, 32, T>), dim3(sorted_grid(h, hist[0], 16)), dim3(256), 0, s, p->perm_num, p->ctl, 1, 0,
                           A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, c_rp, c_col, c_val, pack32, B->nnz);
      if (p->flag_rows) {
      } else if (words1)
        hipLaunchKernelGGL((p->desc ? k_esc_num<64, 128, T, true> : k_esc_num<64, 128, T, false>), dim3(sorted_grid(h, hist[1], 4)), dim3(256),
                           0, s, p->perm_sym, p->ctl, 1, A->rowptr, A->colidx, a_val, B->rowptr, p->desc, b_val, B->nnz, p->esc_words[1], c_rp,
                           c_col, c_val);
      else if (hist[1])
        hipLaunchKernelGGL((k_esc<64, 128, T>), dim3(sorted_grid(h, hist[1], 4)), dim3(256), 0, s, p->perm_num, p->ctl, 1, 1,
                           A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, c_rp, c_col, c_val, pack128, B->nnz);
    }
    {
      Timer t(h, SPGEMM_K_NUM_HASH);
      // (rows of the bin with a record, then the ones without; a row that has a record is in this bin: it has more than
      // kEscLargeCap products, or hashing is forced, and at most kNumHashSmall entries)
      if (p->recorded) {
        const unsigned grid = record_grid(h, p, p->stats.sym_bin_rows[2]);
        if (inside) {
          const int64_t most = A->nnz > B->nnz ? A->nnz : B->nnz;
          const OrderOperands order{(int)grid_for(most, kOrderInsideTile, kOrderParts), A->nnz, B->nnz, A->colidx, same ? nullptr : B->colidx};
          hipLaunchKernelGGL((p->alike ? k_num_recorded<T, true, true> : k_num_recorded<T, true, false>), dim3(grid + order.parts), dim3(256), 0, s,
                             p->perm_sym, p->ctl, 2, p->records, p->record_of, p->shift_of, A->rowptr, A->colidx, a_val, B->rowptr, b_val, B->nnz,
                             c_rp, c_col, c_val, order);
        } else {
          hipLaunchKernelGGL((p->alike ? k_num_recorded<T, false, true> : k_num_recorded<T, false, false>), dim3(grid), dim3(256), 0, s, p->perm_sym,
                             p->ctl, 2, p->records, p->record_of, p->shift_of, A->rowptr, A->colidx, a_val, B->rowptr, b_val, B->nnz, c_rp, c_col,
                             c_val, OrderOperands{});
        }
      }
      if (hist[2] > p->recorded)
        hipLaunchKernelGGL((k_hash<64, 8, T, true>), dim3(grid_for(hist[2], 4, cap_small)), dim3(256), lds_hash_small, s,
                           p->perm_num, p->ctl, 1, 2, p->ip, A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, (int*)nullptr,
                           c_rp, c_col, c_val, B->cols, p->recorded ? p->record_of : nullptr, 0, kOrderNotLooked);
      if (check) other_order_rows();
      if (rows3) {
        if (row_tiles)
          hipLaunchKernelGGL(k_row_tiles<T>, dim3(grid_for(hist[3], 1, (int64_t)h->num_cus * 8)), dim3(kRowTileWaves * kWave),
                             row_tile_lds<T>(B->cols), s, p->perm_num, p->ctl, p->ip, most_ip, A->rowptr, A->colidx, a_val, B->rowptr, B->colidx,
                             b_val, B->nnz, B->cols, c_rp, c_col, c_val, looked3);
        else
          hipLaunchKernelGGL((k_hash<256, 11, T, true>), dim3(grid_for(hist[3], 1, (int64_t)h->num_cus * 8)), dim3(256),
                             lds_hash_large, s, p->perm_num, p->ctl, 1, 3, p->ip, A->rowptr, A->colidx, a_val, B->rowptr,
                             B->colidx, b_val, (int*)nullptr, c_rp, c_col, c_val, B->cols, (const int*)nullptr, most_ip, looked3);
      }
    }
  }
  if (hist[4]) {
    Timer t(h, SPGEMM_K_NUM_STAGED);
    hipLaunchKernelGGL(k_num_staged<T>, dim3(grid_for(hist[4], 1, h->num_cus)), dim3(kStThreads), staged_lds<T>(), s, p->perm_num,
                       p->ctl, A->rowptr, A->colidx, a_val, B->rowptr, B->colidx, b_val, B->cols, c_rp, c_col, c_val);
  }
  if (run_tiles) {
    Timer t(h, SPGEMM_K_NUM_DENSE);
    // (k_num_tiles has no way around the table, which is built for ascending rows only, or the list; k_num_wide takes tiles of any size)
    const bool wide = p->wide_tiles || !p->blk_ptr || !p->all_listed || B->nnz >= kTileMaxNnz;
    hipLaunchKernelGGL((wide ? k_num_wide<T> : k_num_tiles<T>), dim3(grid_for(p->stats.dense_runs, 1, (int64_t)h->num_cus * (wide ? 1 : 2))),
                       dim3(wide ? kWideThreads : kTileThreads), (wide ? num_wide_lds<T>() : num_tiles_lds<T>()), s, p->ctl, p->bin, p->tiles, p->runs, A->colidx,
                       a_val, B->rowptr, B->colidx, b_val, B->cols, p->blk_ptr, p->blk_ptr_cols, p->col_list, B->nnz, c_rp, c_col, c_val, tiles3 ? 1 : 0, looked3);
  }
  HIP_TRY(h, hipGetLastError());
  return SPGEMM_OK;
}

// plan_leaves: see run_symbolic.
int symbolic(spgemm_context* h, const spgemm_csr* A, const spgemm_csr* B, int64_t* c_rowptr, int64_t* nnz_c, spgemm_plan* plan, bool plan_leaves) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_pair(h, A, B);
  if (rc) return rc;
  if (!c_rowptr || !nnz_c || !plan) return fail(h, SPGEMM_INVALID_ARG, "c_rowptr, nnz_c and plan must not be null");
  *plan = nullptr;
  if ((rc = ensure_device(h))) return rc;
  drop_timed(h);   // (timed launches of an earlier plan that nobody asked about)
  PinnedLease pinned(h->stream);
  if (!pinned.p) return fail(h, SPGEMM_ALLOC_FAILED, "allocation of pinned host memory failed");

  spgemm_plan_s* p = new (std::nothrow) spgemm_plan_s();
  if (!p) return fail(h, SPGEMM_ALLOC_FAILED, "host allocation failed");
  p->h = h;
  p->m = A->rows; p->k = A->cols; p->n = B->cols; p->nnz_a = A->nnz; p->nnz_b = B->nnz; p->dtype = A->dtype;
  const int64_t m = p->m;
  p->force = h->force;
  p->flag_rows = flag_rows_ok(h, B);
  p->scan_blocks = m > 0 ? ceil_div(m, kScanTile) : 0;
  size_t off = 0;
  const size_t o_ctl = off; off = align_up(off + sizeof(Control));
  const size_t o_ip = off; off = align_up(off + (size_t)m * 4);
  const size_t o_cnt = off; off = align_up(off + (size_t)m * 4);
  const size_t o_ps = off; off = align_up(off + (size_t)m * 4);
  const size_t o_pn = off; off = align_up(off + (size_t)m * 4);
  const size_t o_bin = off; off = align_up(off + (size_t)m);
  const size_t o_part = off; off = align_up(off + (size_t)(p->scan_blocks + 1) * 8);
  p->scratch = dev_alloc(h, off);
  p->scratch_bytes = off;
  if (!p->scratch) {
    delete p;
    return fail(h, SPGEMM_ALLOC_FAILED, "device allocation of plan scratch failed");
  }
  if (wants_desc(h, A, B)) {
    p->desc = static_cast<unsigned long long*>(dev_alloc(h, (size_t)A->nnz * 8));
    p->desc_bytes = p->desc ? (size_t)A->nnz * 8 : 0;
  }
  unsigned char* base = static_cast<unsigned char*>(p->scratch);
  p->ctl = reinterpret_cast<Control*>(base + o_ctl);
  p->ip = reinterpret_cast<int*>(base + o_ip);
  p->cnt = reinterpret_cast<int*>(base + o_cnt);
  p->perm_sym = reinterpret_cast<int*>(base + o_ps);
  p->perm_num = reinterpret_cast<int*>(base + o_pn);
  p->bin = base + o_bin;
  p->partial = reinterpret_cast<long long*>(base + o_part);

  Control host{};
  pinned.written();
  rc = run_setup(h, p, A, B, pinned.p, &host);
  if (rc == SPGEMM_OK && !host.error)
    rc = (A->dtype == SPGEMM_F32) ? run_symbolic<float>(h, p, A, B, c_rowptr, host, pinned.p, plan_leaves)
                                 : run_symbolic<double>(h, p, A, B, c_rowptr, host, pinned.p, plan_leaves);
  if (rc == SPGEMM_OK && !host.error) {
    const hipError_t e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) rc = fail(h, SPGEMM_HIP_ERROR, std::string("symbolic phase: ") + hipGetErrorString(e));
    else std::memcpy(&host, pinned.p, sizeof(Control));
  }
  if (rc != SPGEMM_OK) (void)hipStreamSynchronize(h->stream);
  pinned.waited();
  if (rc != SPGEMM_OK) {
    drop_timed(h);
    spgemm_plan_destroy(p);
    return rc;
  }
  std::memset(&p->stats, 0, sizeof(p->stats));
  collect_times(h, &p->stats);
  if (host.error == 2 || host.error == 3) {
    spgemm_plan_destroy(p);
    return host.error == 2 ? fail(h, SPGEMM_UNSUPPORTED, "unsorted B with a row of 2^21 or more entries")
                           : fail(h, SPGEMM_HIP_ERROR, "internal: tile list overflow in the dense symbolic kernel");
  }
  if (host.error) {
    spgemm_plan_destroy(p);
    return fail(h, SPGEMM_INVALID_INPUT, "device-side input check failed (column out of range or rowptr not monotone)");
  }
  p->recorded = host.recorded;
  p->all_listed = !host.unlisted;
  p->stats.ip_total = (int64_t)host.ip_total;
  p->stats.nnz_c = host.nnz_c;
  for (int b = 0; b < kNumBins; ++b) {
    p->stats.sym_bin_rows[b] = host.hist[0][b];
    p->stats.num_bin_rows[b] = host.hist[1][b];
    p->stats.sym_bin_ip[b] = (int64_t)host.bin_ip[0][b];
    p->stats.num_bin_ip[b] = (int64_t)host.bin_ip[1][b];
    p->stats.num_bin_nnz[b] = (int64_t)host.bin_nnz[b];
  }
  p->stats.dense_tiles = host.tiles_used;
  p->stats.dense_direct_tiles = host.direct_tiles;
  p->stats.dense_runs = host.runs_used;
  p->stats.dense_search_tiles = host.search_tiles;
  p->stats.plan_bytes = (int64_t)(p->scratch_bytes + p->scratch2_bytes + p->desc_bytes + p->short_bytes + p->list_bytes);
  p->stats.plan_list_bytes = (int64_t)p->list_bytes;
  p->stats.plan_list_used = (int64_t)(host.list_used * 4ULL);
  p->symbolic_done = true;
  *nnz_c = host.nnz_c;
  *plan = p;
  return SPGEMM_OK;
}

}  // namespace

extern "C" {

int spgemm_version(void) { return 100; }

int spgemm_create(spgemm_handle* out, void* hip_stream, const spgemm_allocator* alloc) {
  if (!out) return SPGEMM_INVALID_ARG;
  if (alloc && (!alloc->alloc || !alloc->free)) return SPGEMM_INVALID_ARG;
  spgemm_context* h = new (std::nothrow) spgemm_context();
  if (!h) return SPGEMM_ALLOC_FAILED;
  h->stream = static_cast<hipStream_t>(hip_stream);
  if (alloc) {
    h->alloc = *alloc;
    h->has_alloc = true;
  }
  *out = h;
  return SPGEMM_OK;
}

int spgemm_destroy(spgemm_handle h) {
  if (!h) return SPGEMM_INVALID_ARG;
  for (auto e : h->event_pool) (void)hipEventDestroy(e);
  for (auto& t : h->timed) { (void)hipEventDestroy(t.start); (void)hipEventDestroy(t.stop); }
  if (h->second) (void)hipStreamDestroy(h->second);
  delete h;
  return SPGEMM_OK;
}

int spgemm_set_option(spgemm_handle h, int option, int64_t value) {
  if (!h) return SPGEMM_INVALID_ARG;
  switch (option) {
    case SPGEMM_OPT_TIMING:
      if (value != 0 && value != 1) return fail(h, SPGEMM_INVALID_ARG, "timing option takes 0 or 1");
      h->timing = (int)value;
      return SPGEMM_OK;
    case SPGEMM_OPT_FORCE_WORKSPACE:
      if (value < 0 || value > 4) return fail(h, SPGEMM_INVALID_ARG, "workspace option takes 0..4");
      h->force = (int)value;
      return SPGEMM_OK;
    case SPGEMM_OPT_DIRECT_MIN:
      // a direct block keeps its 256 flag words in the list space of its entries
      if (value < kBlkWords || value > 0x3fffffff) return fail(h, SPGEMM_INVALID_ARG, "direct-tile threshold takes 256..2^30-1");
      h->direct_min = (int)value;
      return SPGEMM_OK;
    case SPGEMM_OPT_SEARCH_RATIO:
      if (value < 0 || value > 1000000) return fail(h, SPGEMM_INVALID_ARG, "search-ratio option takes 0..1000000");
      h->search_ratio = (int)value;
      return SPGEMM_OK;
    case SPGEMM_OPT_MERGE_LIMIT:
      if (value < 2 || value > 0xffffffffLL) return fail(h, SPGEMM_INVALID_ARG, "merge-limit option takes 2..2^32-1");
      h->merge_limit = value;
      return SPGEMM_OK;
    case SPGEMM_OPT_BLOCK_TABLE:
      if (value != 0 && value != 1) return fail(h, SPGEMM_INVALID_ARG, "block-table option takes 0 or 1");
      h->block_table = (int)value;
      return SPGEMM_OK;
    case SPGEMM_OPT_COLUMN_LIST:
      if (value < 0 || (value > 1 && value < 4096)) return fail(h, SPGEMM_INVALID_ARG, "column-list option takes 0, 1 or a byte limit of 4096 or more");
      h->col_list = value;
      return SPGEMM_OK;
    default:
      return fail(h, SPGEMM_INVALID_ARG, "unknown option");
  }
}

const char* spgemm_last_error(spgemm_handle h) { return h ? h->err.c_str() : "null handle"; }

int spgemm_plan_destroy(spgemm_plan p) {
  if (!p) return SPGEMM_INVALID_ARG;
  // the numeric kernels read the plan's scratch: they must have finished before it is released
  if (p->numeric_in_flight) (void)hipStreamSynchronize(p->h->stream);
  dev_free(p->h, p->scratch);
  dev_free(p->h, p->scratch2);
  dev_free(p->h, p->scratch3);
  dev_free(p->h, p->desc);
  delete p;
  return SPGEMM_OK;
}

int spgemm_get_stats(spgemm_plan p, spgemm_stats* out) {
  if (!p || !out) return SPGEMM_INVALID_ARG;
  if (!p->symbolic_done) return fail(p->h, SPGEMM_BAD_STATE, "plan has no symbolic result");
  if (p->numeric_pending) {
    spgemm_context* h = p->h;
    if (!h->timed.empty()) HIP_TRY(h, hipEventSynchronize(h->timed.back().stop));
    p->numeric_in_flight = false;
    for (int c = SPGEMM_K_NUM_ESC; c <= SPGEMM_K_NUM_STAGED; ++c) { p->stats.kernel_ms[c] = 0; p->stats.kernel_launches[c] = 0; }
    collect_times(h, &p->stats);
    p->numeric_pending = false;
  }
  *out = p->stats;
  return SPGEMM_OK;
}

int spgemm_symbolic(spgemm_handle h, const spgemm_csr* A, const spgemm_csr* B, int64_t* c_rowptr, int64_t* nnz_c,
                    spgemm_plan* plan) {
  return symbolic(h, A, B, c_rowptr, nnz_c, plan, true);
}

int spgemm_numeric(spgemm_handle h, spgemm_plan p, const spgemm_csr* A, const spgemm_csr* B, const int64_t* c_rowptr,
                   int32_t* c_colidx, void* c_values) {
  if (!h) return SPGEMM_INVALID_ARG;
  if (!p) return fail(h, SPGEMM_INVALID_ARG, "plan is null");
  int rc = check_pair(h, A, B);
  if (rc) return rc;
  if (p->h != h || !p->symbolic_done) return fail(h, SPGEMM_BAD_STATE, "plan does not belong to this handle or has no symbolic result");
  if (A->rows != p->m || A->cols != p->k || B->cols != p->n || A->nnz != p->nnz_a || B->nnz != p->nnz_b)
    return fail(h, SPGEMM_DIM_MISMATCH, "operands differ from the ones the plan was built for");
  if (A->dtype != p->dtype) return fail(h, SPGEMM_DTYPE_MISMATCH, "value type differs from the plan's");
  if (!c_rowptr) return fail(h, SPGEMM_INVALID_ARG, "c_rowptr is null");
  if (p->stats.nnz_c > 0 && (!c_colidx || !c_values)) return fail(h, SPGEMM_INVALID_ARG, "c_colidx/c_values null with nnz_c > 0");
  if (p->stats.nnz_c == 0) return SPGEMM_OK;
  rc = (A->dtype == SPGEMM_F32) ? run_numeric<float>(h, p, A, B, c_rowptr, c_colidx, c_values)
                                : run_numeric<double>(h, p, A, B, c_rowptr, c_colidx, c_values);
  if (rc != SPGEMM_OK) return rc;
  p->numeric_pending = h->timing != 0;
  p->numeric_in_flight = true;
  return SPGEMM_OK;
}

#ifdef SPG_PHASE_CLOCKS
// Profiling builds only: shader clocks per phase of the dense kernels (2 x 32 values, host), summed
// over workgroups, of the plan's last symbolic and numeric runs.  Waits for the stream.
int spgemm_debug_phase_clocks(spgemm_plan p, unsigned long long* out) {
  if (!p || !out) return SPGEMM_INVALID_ARG;
  spgemm_context* h = p->h;
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  HIP_TRY(h, hipMemcpy(out, reinterpret_cast<unsigned char*>(p->ctl) + offsetof(Control, clk), sizeof(unsigned long long) * 2 * kClkSlots,
                       hipMemcpyDeviceToHost));
  return SPGEMM_OK;
}
#endif

int spgemm_free_device(spgemm_handle h, void* ptr) {
  if (!h) return SPGEMM_INVALID_ARG;
  dev_free(h, ptr);
  return SPGEMM_OK;
}

int spgemm(spgemm_handle h, const spgemm_csr* A, const spgemm_csr* B, spgemm_csr* C) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_pair(h, A, B);
  if (rc) return rc;
  if (!C) return fail(h, SPGEMM_INVALID_ARG, "C is null");
  std::memset(C, 0, sizeof(*C));
  int64_t* rp = static_cast<int64_t*>(dev_alloc(h, (size_t)(A->rows + 1) * sizeof(int64_t)));
  if (!rp) return fail(h, SPGEMM_ALLOC_FAILED, "allocation of C.rowptr failed");
  spgemm_plan plan = nullptr;
  int64_t nnz = 0;
  rc = symbolic(h, A, B, rp, &nnz, &plan, false);
  if (rc != SPGEMM_OK) {
    dev_free(h, rp);
    return rc;
  }
  const size_t vsz = A->dtype == SPGEMM_F32 ? 4 : 8;
  int32_t* col = nullptr;
  void* val = nullptr;
  if (nnz > 0) {
    col = static_cast<int32_t*>(dev_alloc(h, (size_t)nnz * 4));
    val = dev_alloc(h, (size_t)nnz * vsz);
    if ((!col || !val) && (plan->scratch3 || plan->desc)) {
      // the plan's optional memory may be what stands in the way: plan again without it
      dev_free(h, col); dev_free(h, val);
      spgemm_plan_destroy(plan);
      plan = nullptr;
      const int64_t keep = h->col_list;
      h->col_list = 0;
      rc = symbolic(h, A, B, rp, &nnz, &plan, false);
      h->col_list = keep;
      if (rc != SPGEMM_OK) { dev_free(h, rp); return rc; }
      col = static_cast<int32_t*>(dev_alloc(h, (size_t)nnz * 4));
      val = dev_alloc(h, (size_t)nnz * vsz);
    }
    if (!col || !val) {
      dev_free(h, col); dev_free(h, val); dev_free(h, rp);
      spgemm_plan_destroy(plan);
      return fail(h, SPGEMM_ALLOC_FAILED, "allocation of C.colidx/C.values failed");
    }
    rc = spgemm_numeric(h, plan, A, B, rp, col, val);
  }
  // the plan's scratch may be released only after the numeric kernels that read it finish
  if (hipStreamSynchronize(h->stream) != hipSuccess && rc == SPGEMM_OK) rc = fail(h, SPGEMM_HIP_ERROR, "numeric phase failed");
  spgemm_plan_destroy(plan);
  if (rc != SPGEMM_OK) {
    dev_free(h, col); dev_free(h, val); dev_free(h, rp);
    return rc;
  }
  C->rows = A->rows; C->cols = B->cols; C->nnz = nnz; C->dtype = A->dtype;
  C->rowptr = rp; C->colidx = col; C->values = val;
  return SPGEMM_OK;
}


}  // extern "C"

// ---- sparse tensor entry points ------------------------------------------------------------

namespace {

// The unfolding over `mode`: which coordinate arrays and extents play row-major, row-minor, column.
struct ModeView {
  const int32_t *xa, *xb, *xc;
  int64_t A, B, C;
};

bool mode_view(int mode, int64_t I, int64_t J, int64_t K, const int32_t* xi, const int32_t* xj, const int32_t* xk, ModeView* v) {
  switch (mode) {
    case 1: *v = ModeView{xj, xk, xi, J, K, I}; return true;
    case 2: *v = ModeView{xi, xk, xj, I, K, J}; return true;
    case 3: *v = ModeView{xi, xj, xk, I, J, K}; return true;
    default: return false;
  }
}

int check_tensor(spgemm_context* h, int mode, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj,
                 const int32_t* xk, const void* xval, int32_t dtype, ModeView* v) {
  if (!mode_view(mode, I, J, K, xi, xj, xk, v)) return fail(h, SPGEMM_INVALID_ARG, "mode must be 1, 2 or 3");
  if (I < 0 || J < 0 || K < 0 || nnz < 0) return fail(h, SPGEMM_INVALID_ARG, "negative size");
  if (dtype != SPGEMM_F32 && dtype != SPGEMM_F64) return fail(h, SPGEMM_INVALID_ARG, "unknown dtype");
  if (nnz > 0 && (!xi || !xj || !xk || !xval)) return fail(h, SPGEMM_INVALID_ARG, "coordinate or value array null with nnz > 0");
  if (v->C >= 0x7fffffffLL || (v->B > 0 && v->A > 0x7ffffffeLL / v->B) || nnz >= 0xffffffffLL)
    return fail(h, SPGEMM_UNSUPPORTED, "the folded row extent and the column extent must be below 2^31 - 1, nnz below 2^32 - 1");
  return SPGEMM_OK;
}

__global__ void k_clear_ints(int* p) {   // two of them
  if (threadIdx.x < 2 && blockIdx.x == 0) p[threadIdx.x] = 0;
}

int bits_of(int64_t n) {   // bits that hold 0 .. n-1
  int b = 0;
  while (n > 1 && (1LL << b) < n) ++b;
  return b;
}

// Stable radix sort of n (key, payload) pairs.  keys[0] holds the keys; the payloads start in pay_in and end in pay_a (pay_b is
// the other buffer; pay_in may be the one of the two that the first pass does not write).  first_counted: the first digit's
// counts are in `counters` already.  low: bits that the passes leave to k_sort_buckets, which may set *too_long: then the result is none, and the
// caller begins again without.  Returns which of the two key buffers holds the result.
template <typename K, typename P>
int sort_pairs(spgemm_context* h, int64_t n, const SortShape& sh, K* const keys[2], const P* pay_in, P* pay_a, P* pay_b, unsigned* counters,
               bool first_counted, int32_t* col_out, K col_mask, int low = 0, int* too_long = nullptr) {
  hipStream_t s = h->stream;
  unsigned* hist = counters + kSortBins;
  const int steps = sh.passes + (low > 0 ? 1 : 0);
  int cur = 0;
  for (int pass = 0; pass < sh.passes; ++pass) {
    const int shift = sh.first_bit + pass * sh.bits;
    const bool last = pass + 1 == steps;
    P* out = (steps - 1 - pass) % 2 == 0 ? pay_a : pay_b;
    if (pass > 0 || !first_counted)
      hipLaunchKernelGGL(k_sort_hist<K>, dim3(sh.ranges), dim3(kSortThreads), 0, s, n, sh.per_range, shift, sh.bits, keys[cur], hist);
    hipLaunchKernelGGL(k_sort_scan, dim3(1u << sh.bits), dim3(256), 0, s, sh.ranges, hist, counters);
    hipLaunchKernelGGL((sh.per_range <= kScatterThreads * kSortFewItems ? k_sort_scatter<K, P, kSortFewItems> : k_sort_scatter<K, P, kSortItems>), dim3(sh.ranges), dim3(kScatterThreads), 0, s, n, sh.per_range, shift, sh.bits, keys[cur], pay_in, hist,
                       counters, keys[1 - cur], out, last ? col_out : (int32_t*)nullptr, col_mask);
    pay_in = out;
    cur = 1 - cur;
  }
  if constexpr (sizeof(K) == 8) {   // (narrow keys have no buckets: buckets_pay)
    if (low > 0) {
      const int64_t buckets = (int64_t)1 << (sh.passes * sh.bits);   // (the passes may have sorted by a bit or two above the keys')
      hipLaunchKernelGGL((k_sort_buckets<K, P>), dim3((unsigned)ceil_div(buckets, 4)), dim3(256), 0, s, n, buckets, low, keys[cur], pay_in,
                         keys[1 - cur], pay_a, col_out, col_mask, too_long);
      cur = 1 - cur;
    }
  }
  return cur;
}

// Whether some bucket of a sort would be too long (k_sort_sample): asked for before the kernel that makes the keys, which the answer is then
// waited beside.  counts: room for 2^(upper bits) numbers and one, free until then.
class BucketSample {
 public:
  template <class KeyAt>
  BucketSample(spgemm_context* h, int64_t n, int nbits, bool wanted, const SortPlan& plan, const KeyAt& key_at, void* counts) : h_(h), block_(h->stream) {
    if (!wanted || plan.low == 0) return;
    asked_ = true;
    if (!block_.p) return;
    flag_ = reinterpret_cast<int*>(block_.p);
    *flag_ = 0;
    block_.written();
    const unsigned buckets = 1u << (nbits - plan.low);
    hipLaunchKernelGGL(k_sample_clear, dim3((unsigned)ceil_div(buckets + 1, kSampleThreads)), dim3(kSampleThreads), 0, h->stream, buckets,
                       static_cast<unsigned*>(counts));
    hipLaunchKernelGGL(k_sort_sample<KeyAt>, dim3((unsigned)ceil_div(ceil_div(n, kSampleStride), kSampleThreads * kSamplePer)), dim3(kSampleThreads),
                       0, h->stream, n, key_at, plan.low, buckets, static_cast<unsigned*>(counts), flag_);
    done_ = take_event(h);
    if (done_ && hipEventRecord(done_, h->stream) != hipSuccess) {
      (void)hipGetLastError();
      h->event_pool.push_back(done_);
      done_ = nullptr;
    }
  }
  ~BucketSample() { (void)crowded(); }
  BucketSample(const BucketSample&) = delete;
  BucketSample& operator=(const BucketSample&) = delete;
  bool crowded() {   // waits for the answer
    if (flag_) {
      const hipError_t e = done_ ? hipEventSynchronize(done_) : hipStreamSynchronize(h_->stream);
      crowded_ = e != hipSuccess || *static_cast<volatile int*>(flag_) != 0;
      if (e == hipSuccess) block_.waited();
      flag_ = nullptr;
      if (done_) h_->event_pool.push_back(done_);
    } else if (asked_ && !block_.p) {
      crowded_ = true;   // (no answer)
    }
    return crowded_;
  }

 private:
  spgemm_context* h_;
  PinnedLease block_;
  int* flag_ = nullptr;
  hipEvent_t done_ = nullptr;
  bool asked_ = false, crowded_ = false;
};

// Temporary memory of one unfolding: two key buffers, one value buffer (the output is the other), the sort's counters, one flag.
struct UnfoldTmp {
  size_t o_k0, o_k1, o_v, o_h, o_bad, bytes;
};

UnfoldTmp unfold_tmp_layout(int64_t nnz) {
  UnfoldTmp t{};
  size_t off = 0;
  t.o_k0 = off; off = align_up(off + (size_t)nnz * 8);
  t.o_k1 = off; off = align_up(off + (size_t)nnz * 8);
  t.o_v = off; off = align_up(off + (size_t)nnz * 8);
  t.o_h = off; off = align_up(off + sort_counter_bytes(nnz));
  t.o_bad = off; off = align_up(off + 8);   // (and whether a bucket of the sort was too long)
  t.bytes = off;
  return t;
}

template <typename K, typename T>
void unfold_launch(spgemm_context* h, const ModeView& v, int64_t nnz, const T* xval, unsigned char* tmp, const UnfoldTmp& lay, int col_bits,
                   int row_bits, bool plain, int64_t* rp, int32_t* col, T* val) {
  hipStream_t s = h->stream;
  const int64_t rows = v.A * v.B;
  K* keys[2] = {reinterpret_cast<K*>(tmp + lay.o_k0), reinterpret_cast<K*>(tmp + lay.o_k1)};
  unsigned* counters = reinterpret_cast<unsigned*>(tmp + lay.o_h);
  int cur = 0;
  if (nnz > 0) {
    SortPlan plan = sort_plan(nnz, col_bits + row_bits, plain || !buckets_pay(nnz, col_bits + row_bits));
    int* flags = reinterpret_cast<int*>(tmp + lay.o_bad);
    BucketSample sample(h, nnz, col_bits + row_bits, true, plan, TensorKey<unsigned long long>{v.A, v.B, v.C, col_bits, v.xa, v.xb, v.xc}, keys[1]);
    hipLaunchKernelGGL(k_tensor_keys<K>, dim3(plan.sh.ranges), dim3(kSortThreads), 0, s, nnz, plan.sh.per_range, v.A, v.B, v.C, col_bits,
                       plan.sh.first_bit, plan.sh.bits, v.xa, v.xb, v.xc, keys[0], counters + kSortBins, flags);
    const bool crowded = sample.crowded();
    if (crowded) plan = sort_plan(nnz, col_bits + row_bits, true);
    cur = sort_pairs<K, T>(h, nnz, plan.sh, keys, xval, val, reinterpret_cast<T*>(tmp + lay.o_v), counters, !crowded, col,
        (K)(((K)1 << col_bits) - 1), plan.low, flags + 1);
  }
  hipLaunchKernelGGL(k_key_ptr<K>, dim3((unsigned)ceil_div(rows + 1, kPtrRows)), dim3(256), 0, s, nnz, rows, col_bits, keys[cur], rp);
}

// Keys, stable radix sort, row pointer; everything it touches is given by the caller.
// Ends with one stream synchronisation (the out-of-range flag comes to the host).
int unfold_run(spgemm_context* h, const ModeView& v, int64_t nnz, const void* xval, int32_t dtype, unsigned char* tmp, const UnfoldTmp& lay,
               int64_t* rp, int32_t* col, void* val) {
  hipStream_t s = h->stream;
  int* bad = reinterpret_cast<int*>(tmp + lay.o_bad);
  const int col_bits = bits_of(v.C), row_bits = bits_of(v.A * v.B);
  const bool narrow = col_bits + row_bits <= 32;
  int flags[2] = {0, 0};   // a coordinate out of range; a bucket of the sort too long
  for (int plain = 0; plain < 2; ++plain) {
    hipLaunchKernelGGL(k_clear_ints, dim3(1), dim3(64), 0, s, bad);
    if (dtype == SPGEMM_F32) {
      if (narrow) unfold_launch<uint32_t>(h, v, nnz, static_cast<const float*>(xval), tmp, lay, col_bits, row_bits, plain != 0, rp, col,
          static_cast<float*>(val));
      else unfold_launch<unsigned long long>(h, v, nnz, static_cast<const float*>(xval), tmp, lay, col_bits, row_bits, plain != 0, rp, col,
          static_cast<float*>(val));
    } else {
      if (narrow) unfold_launch<uint32_t>(h, v, nnz, static_cast<const double*>(xval), tmp, lay, col_bits, row_bits, plain != 0, rp, col,
          static_cast<double*>(val));
      else unfold_launch<unsigned long long>(h, v, nnz, static_cast<const double*>(xval), tmp, lay, col_bits, row_bits, plain != 0, rp, col,
          static_cast<double*>(val));
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(flags, bad, 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(h, SPGEMM_HIP_ERROR, std::string("unfolding: ") + hipGetErrorString(e));
    if (flags[0]) return fail(h, SPGEMM_INVALID_INPUT, "a tensor coordinate is outside its mode's range");
    if (!flags[1]) break;
  }
  return SPGEMM_OK;
}

// Scratch of the entry point that allocates nothing: one array per device, held until the process ends.
constexpr int64_t kNoAllocMaxNnz = SPTENSOR_NOALLOC_MAX_NNZ;
constexpr size_t kNoAllocScratchBytes = (size_t)kNoAllocMaxNnz * 24 + sort_counter_bytes(kNoAllocMaxNnz) + 8 * 256;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each device, from hipGetSymbolAddress

}  // namespace

extern "C" {

int sptensor_unfold(spgemm_handle h, int mode, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj,
                    const int32_t* xk, const void* xval, int32_t dtype, spgemm_csr* out) {
  if (!h) return SPGEMM_INVALID_ARG;
  if (!out) return fail(h, SPGEMM_INVALID_ARG, "out is null");
  ModeView v{};
  int rc = check_tensor(h, mode, I, J, K, nnz, xi, xj, xk, xval, dtype, &v);
  if (rc) return rc;
  std::memset(out, 0, sizeof(*out));
  if ((rc = ensure_device(h))) return rc;
  const int64_t rows = v.A * v.B;
  const size_t vsz = dtype == SPGEMM_F32 ? 4 : 8;
  const UnfoldTmp lay = unfold_tmp_layout(nnz);
  int64_t* rp = static_cast<int64_t*>(dev_alloc(h, (size_t)(rows + 1) * 8));
  int32_t* col = nnz ? static_cast<int32_t*>(dev_alloc(h, (size_t)nnz * 4)) : nullptr;
  void* val = nnz ? dev_alloc(h, (size_t)nnz * vsz) : nullptr;
  unsigned char* tmp = static_cast<unsigned char*>(dev_alloc(h, lay.bytes));
  if (!rp || !tmp || (nnz && (!col || !val))) rc = fail(h, SPGEMM_ALLOC_FAILED, "allocation for the unfolding failed");
  if (rc == SPGEMM_OK) rc = unfold_run(h, v, nnz, xval, dtype, tmp, lay, rp, col, val);
  dev_free(h, tmp);
  if (rc != SPGEMM_OK) {
    dev_free(h, rp); dev_free(h, col); dev_free(h, val);
    return rc;
  }
  out->rows = rows; out->cols = v.C; out->nnz = nnz; out->dtype = dtype;
  out->rowptr = rp; out->colidx = col; out->values = val;
  return SPGEMM_OK;
}

int sptensor_unfold_noalloc(spgemm_handle h, int mode, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj,
                            const int32_t* xk, const void* xval, int32_t dtype, int64_t* out_rowptr, int32_t* out_colidx,
                            void* out_values) {
  if (!h) return SPGEMM_INVALID_ARG;
  ModeView v{};
  int rc = check_tensor(h, mode, I, J, K, nnz, xi, xj, xk, xval, dtype, &v);
  if (rc) return rc;
  if (!out_rowptr || (nnz > 0 && (!out_colidx || !out_values))) return fail(h, SPGEMM_INVALID_ARG, "output array null");
  if (nnz > kNoAllocMaxNnz)
    return fail(h, SPGEMM_UNSUPPORTED, "sptensor_unfold_noalloc takes at most " + std::to_string(kNoAllocMaxNnz) + " entries (fixed scratch)");
  if ((rc = ensure_device(h))) return rc;
  int dev = 0;
  HIP_TRY(h, hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(h, SPGEMM_UNSUPPORTED, "device ordinal beyond the scratch table");
  if (!g_scratch_ptr[dev]) {   // once per device, with that device current
    void* ptr = nullptr;
    HIP_TRY(h, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
  }
  const UnfoldTmp lay = unfold_tmp_layout(nnz);
  if (lay.bytes > kNoAllocScratchBytes) return fail(h, SPGEMM_UNSUPPORTED, "internal: scratch layout exceeds the fixed scratch");
  // (every buffer inside the scratch is written before it is read, the flag is cleared by a kernel:
  // what the previous call left behind does not matter)
  return unfold_run(h, v, nnz, xval, dtype, g_scratch_ptr[dev], lay, out_rowptr, out_colidx, out_values);
}

int sptensor_unfold_mode3(spgemm_handle h, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj,
                          const int32_t* xk, const void* xval, int32_t dtype, spgemm_csr* out) {
  return sptensor_unfold(h, 3, I, J, K, nnz, xi, xj, xk, xval, dtype, out);
}

int spttm(spgemm_handle h, int mode, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj, const int32_t* xk,
          const void* xval, int32_t dtype, const spgemm_csr* M, spgemm_csr* Y) {
  if (!h) return SPGEMM_INVALID_ARG;
  if (!Y) return fail(h, SPGEMM_INVALID_ARG, "Y is null");
  int rc = check_csr(h, M, "M");
  if (rc) return rc;
  ModeView v{};
  if (!mode_view(mode, I, J, K, xi, xj, xk, &v)) return fail(h, SPGEMM_INVALID_ARG, "mode must be 1, 2 or 3");
  if (M->rows != v.C) return fail(h, SPGEMM_DIM_MISMATCH, "M.rows differs from the extent of the contracted mode");
  if (M->dtype != dtype) return fail(h, SPGEMM_DTYPE_MISMATCH, "tensor and matrix value types differ");
  spgemm_csr X{};
  rc = sptensor_unfold(h, mode, I, J, K, nnz, xi, xj, xk, xval, dtype, &X);
  if (rc) return rc;
  rc = spgemm(h, &X, M, Y);
  dev_free(h, const_cast<int64_t*>(X.rowptr));
  dev_free(h, const_cast<int32_t*>(X.colidx));
  dev_free(h, const_cast<void*>(X.values));
  return rc;
}

int spttm_mode3(spgemm_handle h, int64_t I, int64_t J, int64_t K, int64_t nnz, const int32_t* xi, const int32_t* xj, const int32_t* xk,
                const void* xval, int32_t dtype, const spgemm_csr* M, spgemm_csr* Y) {
  return spttm(h, 3, I, J, K, nnz, xi, xj, xk, xval, dtype, M, Y);
}

int sptensor_fold(spgemm_handle h, int mode, int64_t I, int64_t J, int64_t K, const spgemm_csr* Y, int32_t* yi, int32_t* yj, int32_t* yk) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_csr(h, Y, "Y");
  if (rc) return rc;
  ModeView v{};
  if (!mode_view(mode, I, J, K, yi, yj, yk, &v)) return fail(h, SPGEMM_INVALID_ARG, "mode must be 1, 2 or 3");
  if (I < 0 || J < 0 || K < 0) return fail(h, SPGEMM_INVALID_ARG, "negative size");
  if (v.B <= 0 || Y->rows != v.A * v.B || Y->cols != v.C)
    return fail(h, SPGEMM_DIM_MISMATCH, "Y is not the unfolding of a tensor of these extents over this mode");
  if (Y->nnz > 0 && (!yi || !yj || !yk)) return fail(h, SPGEMM_INVALID_ARG, "coordinate arrays null with nnz > 0");
  if (Y->nnz == 0 || Y->rows == 0) return SPGEMM_OK;
  if ((rc = ensure_device(h))) return rc;
  // (the view was built over the output arrays: xa / xb take the row's two coordinates, xc the column)
  hipLaunchKernelGGL(k_tensor_fold, dim3(grid_for(Y->rows + Y->nnz, kFoldTile, (int64_t)h->num_cus * 256)), dim3(256), 0, h->stream, Y->rows, v.B, Y->rowptr,
                     Y->colidx, const_cast<int32_t*>(v.xa), const_cast<int32_t*>(v.xb), const_cast<int32_t*>(v.xc));
  HIP_TRY(h, hipGetLastError());
  return SPGEMM_OK;
}

int sptensor_fold_mode3(spgemm_handle h, int64_t J, const spgemm_csr* Y, int32_t* yi, int32_t* yj) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_csr(h, Y, "Y");
  if (rc) return rc;
  if (J <= 0 || Y->rows % J != 0) return fail(h, SPGEMM_INVALID_ARG, "Y.rows is not a multiple of J");
  if (Y->nnz > 0 && (!yi || !yj)) return fail(h, SPGEMM_INVALID_ARG, "coordinate arrays null with nnz > 0");
  if (Y->nnz == 0 || Y->rows == 0) return SPGEMM_OK;
  if ((rc = ensure_device(h))) return rc;
  hipLaunchKernelGGL(k_tensor_fold, dim3(grid_for(Y->rows + Y->nnz, kFoldTile, (int64_t)h->num_cus * 256)), dim3(256), 0, h->stream, Y->rows, J, Y->rowptr,
                     (const int32_t*)nullptr, yi, yj, (int32_t*)nullptr);
  HIP_TRY(h, hipGetLastError());
  return SPGEMM_OK;
}

// ---- row blocks in a pipeline ------------------------------------------------------------------

int spgemm_pipelined(spgemm_handle h, const spgemm_csr* A, const spgemm_csr* B, int nblocks, spgemm_csr* C_blocks, int64_t* block_rows) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_pair(h, A, B);
  if (rc) return rc;
  if (!C_blocks || !block_rows) return fail(h, SPGEMM_INVALID_ARG, "C_blocks and block_rows must not be null");
  if (nblocks < 1 || nblocks > 4096) return fail(h, SPGEMM_INVALID_ARG, "nblocks takes 1..4096");
  if ((rc = ensure_device(h))) return rc;
  const int64_t m = A->rows;
  for (int t = 0; t < nblocks; ++t) std::memset(&C_blocks[t], 0, sizeof(spgemm_csr));
  // 1. products per row of the whole A (the count kernel), block boundaries of equal work
  double total = 0;
  for (int t = 0; t <= nblocks; ++t) block_rows[t] = t == 0 ? 0 : m;
  if (m > 0) {
    const int64_t tiles = ceil_div(m, kScanTile);
    size_t off = 0;
    const size_t o_ctl = off; off = align_up(off + sizeof(Control));
    const size_t o_first = off; off = align_up(off + (size_t)(nblocks + 2) * 8);
    const size_t o_sums = off; off = align_up(off + (size_t)tiles * 8);
    const size_t o_ip = off; off = align_up(off + (size_t)m * 4);
    const size_t o_cnt = off; off = align_up(off + (size_t)m * 4);
    const size_t o_bin = off; off = align_up(off + (size_t)m);
    unsigned char* tmp = static_cast<unsigned char*>(dev_alloc(h, off));
    if (!tmp) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the row-block planning failed");
    Control* ctl = reinterpret_cast<Control*>(tmp + o_ctl);
    int* ip = reinterpret_cast<int*>(tmp + o_ip);
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(tmp + o_sums);
    Control host{};
    std::vector<long long> first((size_t)nblocks + 2);
    const int chunk = count_chunk(h, m);
    const bool fine = fine_rows(m, A->nnz, B->rows, B->nnz);
    hipLaunchKernelGGL(k_init_control, dim3(1), dim3(kCountThreads), 0, h->stream, ctl, m, A->rowptr, chunk, h->num_cus, fine ? 1 : 0);
    hipLaunchKernelGGL(k_count_rows<false>, dim3(grid_for(m, fine ? kFineRows : chunk, (int64_t)h->num_cus * 2)), dim3(kCountThreads), 0, h->stream, 0, B->cols, B->nnz,
                       B->colidx, m, A->nnz, B->rows, A->rowptr, A->colidx, B->rowptr, ip, tmp + o_bin, reinterpret_cast<int*>(tmp + o_cnt), ctl, 0,
                       0, (unsigned long long*)nullptr, (const RowLens*)nullptr);
    hipLaunchKernelGGL(k_weight_sums, dim3((unsigned)tiles), dim3(kScanThreads), 0, h->stream, m, ip, sums);
    hipLaunchKernelGGL(k_block_rows, dim3(1), dim3(kScanThreads), 0, h->stream, m, tiles, nblocks, ip, sums,
                       reinterpret_cast<long long*>(tmp + o_first));
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(first.data(), tmp + o_first, first.size() * 8, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(&host, ctl, sizeof(Control), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    dev_free(h, tmp);
    if (e != hipSuccess) return fail(h, SPGEMM_HIP_ERROR, std::string("row-block planning: ") + hipGetErrorString(e));
    if (host.error) return fail(h, SPGEMM_INVALID_INPUT, "device-side input check failed (column out of range or rowptr not monotone)");
    for (int t = 1; t < nblocks; ++t) block_rows[t] = first[(size_t)t];
    total = (double)first[(size_t)nblocks + 1];
  }
  if ((rc = ensure_big_lds(h))) return rc;   // (here, so that the copy below need not for every call)
  // 2. a second context on a stream of its own (same priority) for the symbolic phases
  if ((rc = ensure_second_stream(h))) return rc;
  const hipStream_t s2 = h->second;
  spgemm_context h2 = *h;
  h2.stream = s2;
  h2.row_block = 1;
  h2.whole_ip = total - (double)m;
  h2.timing = 0;
  h2.timed.clear();
  h2.event_pool.clear();
  h2.err.clear();
  struct Block { spgemm_plan plan = nullptr; int64_t* rp = nullptr; int32_t* col = nullptr; void* val = nullptr; int64_t nnz = 0; hipEvent_t done = nullptr; };
  std::vector<Block> blk((size_t)nblocks);
  const size_t vsz = A->dtype == SPGEMM_F32 ? 4 : 8;
  auto block_of_a = [&](int t) {
    spgemm_csr a = *A;
    a.rows = block_rows[t + 1] - block_rows[t];
    a.rowptr = A->rowptr + block_rows[t];
    return a;
  };
  auto release_plan = [&](int t) {
    Block& b = blk[(size_t)t];
    if (b.done) { (void)hipEventSynchronize(b.done); (void)hipEventDestroy(b.done); b.done = nullptr; }
    if (b.plan) { spgemm_plan_destroy(b.plan); b.plan = nullptr; }
  };
  auto symbolic_once = [&](int t) -> int {
    Block& b = blk[(size_t)t];
    const spgemm_csr a = block_of_a(t);
    if (!b.rp) b.rp = static_cast<int64_t*>(dev_alloc(h, (size_t)(a.rows + 1) * 8));
    if (!b.rp) return fail(h, SPGEMM_ALLOC_FAILED, "allocation of a block's row pointer failed");
    const int r = symbolic(&h2, &a, B, b.rp, &b.nnz, &b.plan, false);
    if (r != SPGEMM_OK) h->err = h2.err;
    return r;
  };
  // (when memory is short: once more with the plans before it gone, their numeric phases waited for, and without optional memory)
  auto symbolic_short = [&](int t) -> int {
    for (int before = t - 2 > 0 ? t - 2 : 0; before <= t; ++before) release_plan(before);
    h2.col_list = 0;
    const int r = symbolic_once(t);
    h2.col_list = h->col_list;
    return r;
  };
  auto symbolic_of = [&](int t) -> int {
    const int r = symbolic_once(t);
    return r == SPGEMM_ALLOC_FAILED ? symbolic_short(t) : r;
  };
  auto alloc_c = [&](int t) -> bool {
    Block& b = blk[(size_t)t];
    b.col = static_cast<int32_t*>(dev_alloc(h, (size_t)b.nnz * 4));
    b.val = b.col ? dev_alloc(h, (size_t)b.nnz * vsz) : nullptr;
    if (b.val) return true;
    dev_free(h, b.col);
    b.col = nullptr;
    return false;
  };
  rc = symbolic_of(0);
  for (int t = 0; t < nblocks && rc == SPGEMM_OK; ++t) {
    Block& b = blk[(size_t)t];
    const spgemm_csr a = block_of_a(t);
    // numeric of block t on the handle's stream (enqueued only) ...
    if (b.nnz > 0) {
      if (!alloc_c(t)) {
        rc = symbolic_short(t);
        if (rc == SPGEMM_OK && !alloc_c(t)) rc = fail(h, SPGEMM_ALLOC_FAILED, "allocation of a block of C failed");
        if (rc != SPGEMM_OK) break;
      }
      rc = A->dtype == SPGEMM_F32 ? run_numeric<float>(h, b.plan, &a, B, b.rp, b.col, b.val) : run_numeric<double>(h, b.plan, &a, B, b.rp, b.col, b.val);
      if (rc != SPGEMM_OK) break;
    }
    if (hipEventCreateWithFlags(&b.done, hipEventDisableTiming) != hipSuccess || hipEventRecord(b.done, h->stream) != hipSuccess) {
      rc = fail(h, SPGEMM_HIP_ERROR, "event for a block's numeric phase failed");
      break;
    }
    // ... while the symbolic phase of block t + 1 runs on the other stream (this call returns when it is done)
    if (t + 1 < nblocks) rc = symbolic_of(t + 1);
    if (t >= 1) release_plan(t - 1);   // (its numeric phase has been running for a whole symbolic phase: wait and release)
  }
  if (hipStreamSynchronize(h->stream) != hipSuccess && rc == SPGEMM_OK) rc = fail(h, SPGEMM_HIP_ERROR, "numeric phase failed");
  (void)hipStreamSynchronize(s2);
  for (int t = 0; t < nblocks; ++t) release_plan(t);
  for (auto e : h2.event_pool) (void)hipEventDestroy(e);
  drop_timed(h);   // (per-block times are not reported)
  if (rc != SPGEMM_OK) {
    for (auto& b : blk) { dev_free(h, b.rp); dev_free(h, b.col); dev_free(h, b.val); }
    return rc;
  }
  for (int t = 0; t < nblocks; ++t) {
    const Block& b = blk[(size_t)t];
    C_blocks[t].rows = block_rows[t + 1] - block_rows[t];
    C_blocks[t].cols = B->cols;
    C_blocks[t].nnz = b.nnz;
    C_blocks[t].dtype = A->dtype;
    C_blocks[t].rowptr = b.rp; C_blocks[t].colidx = b.col; C_blocks[t].values = b.val;
  }
  return SPGEMM_OK;
}

}  // extern "C"

// ---- outer-product route -------------------------------------------------------------------

namespace {

// In-place exclusive scan of n values, v[n] = their sum; sums: ceil(n / kScanTileN) + 1 slots of scratch.
// total: the sum in host memory too.
template <typename T>
void scan_values(spgemm_context* h, int64_t n, T* v, T* sums, T* total) {
  const int64_t tiles = ceil_div(n > 0 ? n : 1, kScanTileN);
  hipLaunchKernelGGL(k_scan_sums<T>, dim3((unsigned)tiles), dim3(256), 0, h->stream, n, v, sums);
  hipLaunchKernelGGL(k_scan_top<T>, dim3(1), dim3(256), 0, h->stream, tiles, sums, total);
  hipLaunchKernelGGL(k_scan_tiles<T>, dim3((unsigned)tiles), dim3(256), 0, h->stream, n, v, sums);
}

struct DevBufs {   // device buffers released together
  spgemm_context* h;
  std::vector<void*> v;
  explicit DevBufs(spgemm_context* h_) : h(h_) {}
  ~DevBufs() { for (void* p : v) dev_free(h, p); }
  template <typename P>
  P* get(size_t count) {
    void* p = dev_alloc(h, count * sizeof(P));
    if (p) v.push_back(p);
    return static_cast<P*>(p);
  }
  void release(void* p) {
    for (auto& q : v) if (q == p) { dev_free(h, q); q = nullptr; }
  }
  void keep(void* p) {   // ownership leaves
    for (auto& q : v) if (q == p) q = nullptr;
  }
};

// Keeps the non-empty vectors of a compressed matrix (ptr over n vectors): vec / out_ptr are allocated here.
int dcs_compress(spgemm_context* h, int64_t n, int64_t nnz, const int64_t* ptr, DevBufs& bufs, int32_t** vec, int64_t** out_ptr, int64_t* nvec) {
  hipStream_t s = h->stream;
  unsigned* pos = bufs.get<unsigned>((size_t)n + 1);
  if (!pos) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the doubly compressed format failed");
  const unsigned g = grid_for(n, 256, (int64_t)h->num_cus * 32);
  hipLaunchKernelGGL(k_dcs_flags, dim3(g), dim3(256), 0, s, n, ptr, pos);
  unsigned* sums = bufs.get<unsigned>((size_t)ceil_div(n > 0 ? n : 1, kScanTileN) + 1);
  if (!sums) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the doubly compressed format failed");
  PinnedLease pinned(s);
  if (!pinned.p) return fail(h, SPGEMM_ALLOC_FAILED, "allocation of pinned host memory failed");
  unsigned* host = reinterpret_cast<unsigned*>(pinned.p);
  pinned.written();
  scan_values(h, n, pos, sums, host);
  HIP_TRY(h, hipStreamSynchronize(s));
  pinned.waited();
  const unsigned total = *static_cast<volatile unsigned*>(host);
  *nvec = total;
  *vec = bufs.get<int32_t>((size_t)total + 1);
  *out_ptr = bufs.get<int64_t>((size_t)total + 1);
  if (!*vec || !*out_ptr) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the doubly compressed format failed");
  hipLaunchKernelGGL(k_dcs_fill, dim3(g), dim3(256), 0, s, n, ptr, pos, *vec, *out_ptr, nnz, (int64_t)total);
  HIP_TRY(h, hipGetLastError());
  return SPGEMM_OK;
}

// Accumulation arrays up to this long become the all array (1 GB, however many of its coordinates are equal).  Where memory is refused before the
// first merge is through, the call begins again without that.
constexpr int64_t kOuterKeepCap = (int64_t)1 << 26;

template <typename T>
int outer_run(spgemm_context* h, const spgemm_dcs* A, const spgemm_dcs* B, int64_t cap, spgemm_csr* C) {
  hipStream_t s = h->stream;
  const int64_t m = A->minor_dim, n = B->minor_dim, na = A->nvec, nb = B->nvec;
  DevBufs bufs(h);
  // numbers that come to the host: the products, components that stay, whether a bucket of a sort was too long.  (Sorts that may write the
  // last one are on their way whenever memory is refused.)
  PinnedLease pinned(s);
  if (!pinned.p) return fail(h, SPGEMM_ALLOC_FAILED, "allocation of pinned host memory failed");
  pinned.written();
  long long* host_total = reinterpret_cast<long long*>(pinned.p);
  unsigned* host_stay = reinterpret_cast<unsigned*>(host_total + 1);
  int* too_long = reinterpret_cast<int*>(host_total + 2);
  int64_t* rp = bufs.get<int64_t>((size_t)m + 1);
  long long* off = bufs.get<long long>((size_t)na + 1);
  int32_t* match = bufs.get<int32_t>((size_t)na + 1);
  if (!rp || !off || !match) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the outer product failed");
  long long total = 0;
  if (na > 0) {
    hipLaunchKernelGGL(k_outer_count, dim3(grid_for(na, 256, (int64_t)h->num_cus * 32)), dim3(256), 0, s, na, A->vec, A->ptr, nb, B->vec, B->ptr,
                       off, match);
    long long* sums = bufs.get<long long>((size_t)ceil_div(na, kScanTileN) + 1);
    if (!sums) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the outer product failed");
    scan_values(h, na, off, sums, host_total);
    HIP_TRY(h, hipStreamSynchronize(s));
    total = *static_cast<volatile long long*>(host_total);
  }
  if (cap <= 0) cap = (int64_t)1 << 24;
  if (cap > ((int64_t)1 << 30)) cap = (int64_t)1 << 30;
  if (cap > total) cap = total > 0 ? total : 1;
  // accumulation array: coordinates (row above the column's bits) and values, twice (the sort's two buffers)
  const int col_bits = bits_of(n);
  unsigned long long* keys[2] = {bufs.get<unsigned long long>((size_t)cap), bufs.get<unsigned long long>((size_t)cap)};
  double* vals[2] = {bufs.get<double>((size_t)cap), bufs.get<double>((size_t)cap)};
  unsigned* counters = bufs.get<unsigned>(sort_counter_bytes(cap) / 4);   // (the last batch is shorter and may take more ranges)
  if (!keys[0] || !keys[1] || !vals[0] || !vals[1] || !counters)
    return fail(h, SPGEMM_ALLOC_FAILED, "allocation of the accumulation array failed");
  // all array: sorted, unique coordinates with their sums
  unsigned long long* all_k = nullptr;
  double* all_v = nullptr;
  int64_t all_n = 0;
  uint32_t* all_row = nullptr;   // of C's entries
  int32_t* col = nullptr;
  T* val = nullptr;
  // Room for `uniq` components of the next all array; the last stage writes columns and values of C in place of sums.
  auto room = [&](unsigned uniq, bool last, OuterOut<T>* out) -> int {
    *out = OuterOut<T>{nullptr, nullptr, nullptr, nullptr, nullptr, col_bits};
    if (last) {
      out->row = all_row = bufs.get<uint32_t>((size_t)uniq);
      out->col = col = bufs.get<int32_t>((size_t)uniq);
      out->val = val = bufs.get<T>((size_t)uniq);
    } else {
      out->keys = bufs.get<unsigned long long>((size_t)uniq);
      out->vals = bufs.get<double>((size_t)uniq);
    }
    if (last ? out->row && out->col && out->val : out->keys && out->vals) return SPGEMM_OK;
    bufs.release(out->row); bufs.release(out->col); bufs.release(out->val); bufs.release(out->keys); bufs.release(out->vals);
    *out = OuterOut<T>{};
    return fail(h, SPGEMM_ALLOC_FAILED, "allocation of the all array failed");
  };
  // Scan of the tiles' counts; their sum comes to the host.
  auto total_of = [&](int64_t tiles, unsigned* sums, unsigned* uniq) -> int {
    hipLaunchKernelGGL(k_scan_top<unsigned>, dim3(1), dim3(256), 0, s, tiles, sums, host_stay);
    HIP_TRY(h, hipStreamSynchronize(s));
    *uniq = *static_cast<volatile unsigned*>(host_stay);
    return SPGEMM_OK;
  };
  // kept: the all array is the first batch as its sort has left it; all_raw: and nobody has waited for that
  bool plain_sorts = false, keep_first = cap <= kOuterKeepCap && 2 * cap < h->merge_limit, kept = false, all_raw = false;
  auto was_too_long = [&] { return *static_cast<volatile int*>(too_long) != 0; };
  *too_long = 0;
  for (long long t0 = 0; t0 < total; t0 += cap) {
    const int64_t cnt = total - t0 < cap ? total - t0 : cap;
    const bool last = t0 + cap >= total;
    double* sorted = nullptr;
    int cur = 0;
    auto insert_and_sort = [&](bool plain) {
      SortPlan plan = sort_plan(cnt, col_bits + bits_of(m), plain || !buckets_pay(cnt, col_bits + bits_of(m)));
      const SortShape& sh = plan.sh;
      // (the batches after the first are taken to be like it; one that is not is sorted again)
      const OuterKey key_at{(int64_t)t0, na, col_bits, off, match, A->ptr, B->ptr, A->idx, B->idx};
      BucketSample sample(h, cnt, col_bits + bits_of(m), t0 == 0, plan, key_at, keys[1]);
      // insert
      hipLaunchKernelGGL(k_outer_insert<T>, dim3(sh.ranges), dim3(kSortThreads), 0, s, (int64_t)t0, cnt, sh.per_range, sh.first_bit, sh.bits, na,
                         off, match, A->ptr, A->idx, static_cast<const T*>(A->values), B->ptr, B->idx, static_cast<const T*>(B->values), col_bits,
                         keys[0], vals[0], counters + kSortBins);
      // sort
      const bool crowded = sample.crowded();
      if (crowded) {
        plan = sort_plan(cnt, col_bits + bits_of(m), true);
        plain_sorts = true;
      }
      const int steps = sh.passes + (plan.low > 0 ? 1 : 0);
      sorted = vals[steps & 1];
      cur = sort_pairs<unsigned long long, double>(h, cnt, sh, keys, vals[0], sorted, vals[1 - (steps & 1)], counters, !crowded, nullptr, 0ULL,
          plan.low, too_long);
      return plan.low > 0;
    };
    const bool buckets = insert_and_sort(plain_sorts);
    int rc = SPGEMM_OK;
    auto sort_again = [&] {   // (and the batches after this one too, by passes alone)
      plain_sorts = true;
      *too_long = 0;
      (void)insert_and_sort(true);
    };
    OuterOut<T> batch{};
    unsigned uniq = 0;
    // Equal coordinates of the batch are added up; with to_c that gives C.
    auto add_up = [&](bool to_c) -> int {
      const int64_t tiles = ceil_div(cnt, kRunTile);
      unsigned* sums = bufs.get<unsigned>((size_t)tiles + 1);
      if (!sums) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the merge stage failed");
      hipLaunchKernelGGL(k_run_count, dim3((unsigned)tiles), dim3(256), 0, s, cnt, keys[cur], sums);
      int r = total_of(tiles, sums, &uniq);   // (waits)
      if (!r && buckets && was_too_long()) {
        sort_again();
        hipLaunchKernelGGL(k_run_count, dim3((unsigned)tiles), dim3(256), 0, s, cnt, keys[cur], sums);
        r = total_of(tiles, sums, &uniq);
      }
      if (!r) r = room(uniq, to_c, &batch);
      if (!r) hipLaunchKernelGGL(k_run_sum<T>, dim3((unsigned)tiles), dim3(256), 0, s, cnt, keys[cur], sorted, sums, batch);
      bufs.release(sums);
      return r;
    };
    // The batch into the all array.
    auto merge = [&](int64_t batch_n) -> int {
      const int64_t both = all_n + batch_n;
      if (both >= h->merge_limit)
        return fail(h, SPGEMM_UNSUPPORTED, "the all array of the outer product and a batch would reach " + std::to_string(h->merge_limit) + " components");
      const int64_t tiles = ceil_div(both, kMergeTile);
      int64_t* split = bufs.get<int64_t>((size_t)tiles + 1);
      unsigned* sums = bufs.get<unsigned>((size_t)tiles + 1);
      unsigned merged = 0;
      OuterOut<T> next{};
      int r = split && sums ? SPGEMM_OK : fail(h, SPGEMM_ALLOC_FAILED, "allocation for the merge stage failed");
      if (!r) {
        hipLaunchKernelGGL(k_merge_split, dim3((unsigned)ceil_div(tiles + 1, 256)), dim3(256), 0, s, all_n, all_k, batch_n, batch.keys, tiles, split);
        hipLaunchKernelGGL(k_merge_count, dim3((unsigned)tiles), dim3(256), 0, s, all_n, all_k, batch_n, batch.keys, split, sums);
        r = total_of(tiles, sums, &merged);
      }
      if (!r) r = room(merged, last, &next);
      if (!r) {
        hipLaunchKernelGGL(k_merge_put<T>, dim3((unsigned)tiles), dim3(256), 0, s, all_n, all_k, all_v, batch_n, batch.keys, batch.vals, split, sums, next);
        bufs.release(all_k); bufs.release(all_v);
        all_k = next.keys; all_v = next.vals; all_n = merged;
      }
      bufs.release(split); bufs.release(sums);
      return r;
    };
    auto from_start = [&] {   // the batches once more, from the first one on
      bufs.release(all_k); bufs.release(all_v);
      all_k = nullptr; all_v = nullptr; all_n = 0;
      kept = all_raw = false;
      *too_long = 0;
      t0 = -cap;
    };
    if (last && all_n == 0) {
      if ((rc = add_up(true))) return rc;
      all_n = uniq;
      continue;
    }
    // Of several batches none has to be added up by itself: the merge takes components that are there more than once.
    if (all_n == 0) {
      // the first one: its buffers become the all array, and the accumulation array gets others, where these are not large
      unsigned long long* next_keys = keep_first ? bufs.get<unsigned long long>((size_t)cap) : nullptr;
      double* next_vals = next_keys ? bufs.get<double>((size_t)cap) : nullptr;
      if (next_vals) {
        all_k = keys[cur]; all_v = sorted; all_n = cnt;
        kept = true;
        all_raw = buckets;
        keys[cur] = next_keys;
        vals[sorted == vals[0] ? 0 : 1] = next_vals;
      } else {
        bufs.release(next_keys);
        if ((rc = add_up(false))) return rc;
        all_k = batch.keys; all_v = batch.vals; all_n = uniq;
      }
      continue;
    }
    if (buckets || all_raw) {
      HIP_TRY(h, hipStreamSynchronize(s));
      if (was_too_long()) {
        if (all_raw) {   // (this batch or the first one: from the start, by passes alone)
          plain_sorts = true;
          from_start();
          continue;
        }
        sort_again();
      }
      all_raw = false;
    }
    const bool compact = all_n + cnt >= h->merge_limit;   // (too many, but perhaps not so many different ones)
    if (compact) {
      rc = add_up(false);
    } else {
      batch.keys = keys[cur];
      batch.vals = sorted;
    }
    if (!rc) rc = merge(compact ? uniq : cnt);
    if (compact) { bufs.release(batch.keys); bufs.release(batch.vals); }
    if (rc == SPGEMM_ALLOC_FAILED && kept) {
      // (the first batch, added up, may take less)
      keep_first = false;
      from_start();
      continue;
    }
    if (rc) return rc;
    HIP_TRY(h, hipGetLastError());
    kept = false;
  }
  // compress: columns and values are there, the row pointer comes from the coordinates
  hipLaunchKernelGGL(k_key_ptr<uint32_t>, dim3((unsigned)ceil_div(m + 1, kPtrRows)), dim3(256), 0, s, all_n, m, 0, all_row, rp);
  HIP_TRY(h, hipGetLastError());
  HIP_TRY(h, hipStreamSynchronize(s));
  pinned.waited();
  bufs.keep(rp); bufs.keep(col); bufs.keep(val);
  C->rows = m; C->cols = n; C->nnz = all_n; C->dtype = A->dtype;
  C->rowptr = rp; C->colidx = col; C->values = val;
  return SPGEMM_OK;
}

int check_dcs(spgemm_context* h, const spgemm_dcs* M, const char* name) {
  if (!M) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + " is null");
  if (M->major_dim < 0 || M->minor_dim < 0 || M->nvec < 0 || M->nnz < 0 || M->nvec > M->major_dim)
    return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": bad size");
  if (M->dtype != SPGEMM_F32 && M->dtype != SPGEMM_F64) return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": unknown dtype");
  if (!M->ptr || (M->nvec > 0 && !M->vec) || (M->nnz > 0 && (!M->idx || !M->values)))
    return fail(h, SPGEMM_INVALID_ARG, std::string(name) + ": array null");
  if (M->major_dim >= 0x7fffffffLL || M->minor_dim >= 0x7fffffffLL || M->nnz >= 0xffffffffLL)
    return fail(h, SPGEMM_UNSUPPORTED, std::string(name) + ": extents must be below 2^31 - 1, nnz below 2^32 - 1");
  return SPGEMM_OK;
}

}  // namespace

extern "C" {

int spgemm_dcs_free(spgemm_handle h, spgemm_dcs* M) {
  if (!h || !M) return SPGEMM_INVALID_ARG;
  dev_free(h, const_cast<int32_t*>(M->vec));
  dev_free(h, const_cast<int64_t*>(M->ptr));
  dev_free(h, const_cast<int32_t*>(M->idx));
  dev_free(h, const_cast<void*>(M->values));
  std::memset(M, 0, sizeof(*M));
  return SPGEMM_OK;
}

int spgemm_dcsr_from_csr(spgemm_handle h, const spgemm_csr* M, spgemm_dcs* out) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_csr(h, M, "M");
  if (rc) return rc;
  if (!out) return fail(h, SPGEMM_INVALID_ARG, "out is null");
  if (M->nnz >= 0xffffffffLL) return fail(h, SPGEMM_UNSUPPORTED, "nnz must be below 2^32 - 1");
  std::memset(out, 0, sizeof(*out));
  if ((rc = ensure_device(h))) return rc;
  DevBufs bufs(h);
  const size_t vsz = M->dtype == SPGEMM_F32 ? 4 : 8;
  int32_t* vec = nullptr;
  int64_t* ptr = nullptr;
  int64_t nvec = 0;
  if ((rc = dcs_compress(h, M->rows, M->nnz, M->rowptr, bufs, &vec, &ptr, &nvec))) return rc;
  int32_t* idx = bufs.get<int32_t>((size_t)M->nnz);
  void* val = bufs.get<unsigned char>((size_t)M->nnz * vsz);
  if (!idx || !val) return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the doubly compressed format failed");
  if (M->nnz > 0) {
    HIP_TRY(h, hipMemcpyAsync(idx, M->colidx, (size_t)M->nnz * 4, hipMemcpyDeviceToDevice, h->stream));
    HIP_TRY(h, hipMemcpyAsync(val, M->values, (size_t)M->nnz * vsz, hipMemcpyDeviceToDevice, h->stream));
  }
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  bufs.keep(vec); bufs.keep(ptr); bufs.keep(idx); bufs.keep(val);
  *out = spgemm_dcs{M->rows, M->cols, nvec, M->nnz, vec, ptr, idx, val, M->dtype};
  return SPGEMM_OK;
}

int spgemm_dcsc_from_csr(spgemm_handle h, const spgemm_csr* M, spgemm_dcs* out) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_csr(h, M, "M");
  if (rc) return rc;
  if (!out) return fail(h, SPGEMM_INVALID_ARG, "out is null");
  if (M->nnz >= 0xffffffffLL) return fail(h, SPGEMM_UNSUPPORTED, "nnz must be below 2^32 - 1");
  std::memset(out, 0, sizeof(*out));
  if ((rc = ensure_device(h))) return rc;
  hipStream_t s = h->stream;
  DevBufs bufs(h);
  const int64_t nnz = M->nnz;
  const size_t vsz = M->dtype == SPGEMM_F32 ? 4 : 8;
  // compressed sparse columns first: a stable sort by column alone (the entries are in row order; a sort by the row's bits as well
  // took five passes instead of three for 8 M entries of 10^6 columns)
  unsigned long long* keys[2] = {bufs.get<unsigned long long>((size_t)nnz), bufs.get<unsigned long long>((size_t)nnz)};
  void* tmp = bufs.get<unsigned char>((size_t)nnz * vsz);
  unsigned* counters = bufs.get<unsigned>(sort_counter_bytes(nnz) / 4);
  int64_t* colptr = bufs.get<int64_t>((size_t)M->cols + 1);
  int32_t* idx = bufs.get<int32_t>((size_t)nnz);
  void* val = bufs.get<unsigned char>((size_t)nnz * vsz);
  if (!keys[0] || !keys[1] || !tmp || !counters || !colptr || !idx || !val)
    return fail(h, SPGEMM_ALLOC_FAILED, "allocation for the doubly compressed format failed");
  int cur = 0;
  const int64_t cap_grid = (int64_t)h->num_cus * 32;
  const int row_bits = bits_of(M->rows);
  if (nnz > 0) {
    const SortShape sh = sort_shape(nnz, bits_of(M->cols), row_bits);
    const unsigned long long row_mask = (1ULL << row_bits) - 1;
    hipLaunchKernelGGL(k_column_keys, dim3(grid_for(M->rows, 16, cap_grid)), dim3(256), 0, s, M->rows, row_bits, M->rowptr, M->colidx, keys[0]);
    if (M->dtype == SPGEMM_F32)
      cur = sort_pairs<unsigned long long, float>(h, nnz, sh, keys, static_cast<const float*>(M->values), static_cast<float*>(val),
                                                  static_cast<float*>(tmp), counters, false, idx, row_mask);
    else
      cur = sort_pairs<unsigned long long, double>(h, nnz, sh, keys, static_cast<const double*>(M->values), static_cast<double*>(val),
                                                   static_cast<double*>(tmp), counters, false, idx, row_mask);
  }
  hipLaunchKernelGGL(k_key_ptr<unsigned long long>, dim3((unsigned)ceil_div(M->cols + 1, kPtrRows)), dim3(256), 0, s, nnz, M->cols, row_bits, keys[cur],
                     colptr);
  HIP_TRY(h, hipGetLastError());
  int32_t* vec = nullptr;
  int64_t* ptr = nullptr;
  int64_t nvec = 0;
  if ((rc = dcs_compress(h, M->cols, nnz, colptr, bufs, &vec, &ptr, &nvec))) return rc;
  HIP_TRY(h, hipStreamSynchronize(s));
  bufs.keep(vec); bufs.keep(ptr); bufs.keep(idx); bufs.keep(val);
  *out = spgemm_dcs{M->cols, M->rows, nvec, nnz, vec, ptr, idx, val, M->dtype};
  return SPGEMM_OK;
}

int spgemm_outer(spgemm_handle h, const spgemm_dcs* A, const spgemm_dcs* B, int64_t acc_capacity, spgemm_csr* C) {
  if (!h) return SPGEMM_INVALID_ARG;
  int rc = check_dcs(h, A, "A");
  if (rc) return rc;
  if ((rc = check_dcs(h, B, "B"))) return rc;
  if (!C) return fail(h, SPGEMM_INVALID_ARG, "C is null");
  if (acc_capacity < 0) return fail(h, SPGEMM_INVALID_ARG, "negative accumulation capacity");
  if (A->major_dim != B->major_dim) return fail(h, SPGEMM_DIM_MISMATCH, "A's columns and B's rows differ in extent");
  if (A->dtype != B->dtype) return fail(h, SPGEMM_DTYPE_MISMATCH, "A and B value types differ");
  std::memset(C, 0, sizeof(*C));
  if ((rc = ensure_device(h))) return rc;
  return A->dtype == SPGEMM_F32 ? outer_run<float>(h, A, B, acc_capacity, C) : outer_run<double>(h, A, B, acc_capacity, C);
}

}  // extern "C"
