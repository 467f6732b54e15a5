// The classes of shorter rows (0 to 3) in one launch, a stretch of workgroups for each, where they are few: the kernel of a class takes as long as
// its slowest row (a chain of dependent loads and LDS steps: 5 us for 128 products, 25 us for 768, 35 before their set had 2048 slots), whether it has ten rows
// or a thousand, and so do four of them one after the other, with a launch each.
// Bound: the slowest row.  Registers and LDS are those of the hungriest class, 16 waves on a compute unit, so where the rows fill the
// chip several times over the kernels of the classes follow each other as before (short_rows_ok).
// 5003 x 3001 x 7777, rows of 40 and 25 entries on average in any order (fp32): symbolic 59 -> 48 us, numeric 37 -> 29 us and five launches fewer,
// the whole call 287 -> 254 us.  Whole calls, us a kernel for each class | one launch where the rows fill the chip up to 4 | 16 times: R-MAT squared
// (fp32), 16 edges, scale 10 200 | 159 | 158, 13 390 | 359 | 357, 14 547 | 532 | 521, 16 1933 | 1951 (not reached) | 1897; ragged rows of 40 and 25
// entries (fp64), 400 rows 194 | 156 | 154, 8000 361 | 340 | 328, 30 000 1027 | 1049 (not reached) | 1028.  (The dense kernels beside
// it on a second stream: what the events that order the streams cost is what it gains, 282 and 543 us where it is 254 and 530.)
#pragma once
#include "esc_kernels.hpp"
#include "hash_kernels.hpp"
#include "record_kernels.hpp"
#include "tile_kernels.hpp"

namespace spg {

constexpr int kShortGroups = 4;   // workgroups on a compute unit

struct SymShort {
  unsigned wgs[4];   // workgroups of the classes 3, 2, 1, 0 (whole multiples of kDies)
  const int *perm, *ip;
  const int64_t *a_rp, *b_rp;
  const int32_t *a_col, *b_col;
  int64_t b_nnz, n_cols;
  int pack32, pack128;
  int* cnt;
  unsigned *words32, *words128, *records;
  unsigned record_rows;
  int *record_of, *shift_of;
};

template <int LOG_SLOTS>
constexpr size_t sym_short_lds() {
  size_t n = hash_lds_bytes<256, 12, false>();
  if (n < sizeof(SymWaveLds<LOG_SLOTS>)) n = sizeof(SymWaveLds<LOG_SLOTS>);
  if (n < sizeof(EscSymLds<64, 128>)) n = sizeof(EscSymLds<64, 128>);
  if (n < sizeof(EscSymLds<16, 32>)) n = sizeof(EscSymLds<16, 32>);
  return n;
}

template <bool ALIKE, int LOG_SLOTS>
__global__ __launch_bounds__(256, kShortGroups) void k_sym_short(Control* __restrict__ ctl, const SymShort s) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (ctl->error) return;
  unsigned wg = blockIdx.x;
  if (wg < s.wgs[0]) {
    hash_rows<256, 12, float, false>(smem, wg, s.wgs[0], s.perm, ctl, 0, 3, s.ip, s.a_rp, s.a_col, (const float*)nullptr, s.b_rp, s.b_col,
        (const float*)nullptr, s.cnt, (const int64_t*)nullptr, (int32_t*)nullptr, (float*)nullptr, s.n_cols, (const int*)nullptr, 0);
    return;
  }
  wg -= s.wgs[0];
  if (wg < s.wgs[1]) {
    sym_wave_rows<ALIKE, LOG_SLOTS>(reinterpret_cast<SymWaveLds<LOG_SLOTS>*>(smem), wg, s.wgs[1], s.perm, ctl, 2, s.a_rp, s.a_col, s.b_rp, s.b_col, s.b_nnz, s.cnt,
        s.records, s.record_rows, s.record_of, s.shift_of);
    return;
  }
  wg -= s.wgs[1];
  if (wg < s.wgs[2]) {
    esc_sym_rows<64, 128, false>(reinterpret_cast<EscSymLds<64, 128>*>(smem), wg, s.wgs[2], s.perm, ctl, 1, s.a_rp, s.a_col, s.b_rp, nullptr,
        s.b_col, s.b_nnz, s.pack128, s.cnt, s.words128);
    return;
  }
  wg -= s.wgs[2];
  esc_sym_rows<16, 32, false>(reinterpret_cast<EscSymLds<16, 32>*>(smem), wg, s.wgs[3], s.perm, ctl, 0, s.a_rp, s.a_col, s.b_rp, nullptr, s.b_col,
      s.b_nnz, s.pack32, s.cnt, s.words32);
}

template <typename T>
struct NumShort {
  // workgroups of class 3, of the recorded rows, of the rows of class 2 without a record, of the classes 1, 0 (whole multiples of kDies)
  unsigned wgs[5];
  const int *perm_sym, *perm_num, *ip;
  const int64_t *a_rp, *b_rp, *c_rp;
  const int32_t *a_col, *b_col;
  const T *a_val, *b_val;
  int64_t b_nnz, n_cols;
  int pack32, pack128;
  const unsigned *words32, *words128, *records;   // (no words: the rows are sorted here)
  const int *record_of, *shift_of;   // (no shifts: all are none)
  int32_t* c_col;
  T* c_val;
  int tiles, most_ip, looked;   // rows of class 3: as a tile without structure, or hashed; see run_numeric
};

template <typename T>
constexpr size_t num_short_lds() {   // (class 3 beside it)
  size_t n = sizeof(NumRecordedLds<T>);
  if (n < hash_lds_bytes<64, 8, true>()) n = hash_lds_bytes<64, 8, true>();
  if (n < sizeof(EscNumLds<64, 128>)) n = sizeof(EscNumLds<64, 128>);
  if (n < sizeof(EscNumLds<16, 32>)) n = sizeof(EscNumLds<16, 32>);
  if (n < sizeof(EscRowsLds<64, 128, T>)) n = sizeof(EscRowsLds<64, 128, T>);
  if (n < sizeof(EscRowsLds<16, 32, T>)) n = sizeof(EscRowsLds<16, 32, T>);
  return n;
}

template <typename T>
__global__ __launch_bounds__(256, kShortGroups) void k_num_short(const Control* __restrict__ ctl, const NumShort<T> s) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (ctl->error) return;
  unsigned wg = blockIdx.x;
  if (wg < s.wgs[0]) {
    if (s.tiles) {
      row_tiles_rows<T>(smem, wg, s.wgs[0], s.perm_num, ctl, s.ip, s.most_ip, s.a_rp, s.a_col, s.a_val, s.b_rp, s.b_col, s.b_val, s.b_nnz, s.n_cols,
          s.c_rp, s.c_col, s.c_val, s.looked);
    } else {
      const int most_ip = other_order(ctl, s.looked) ? 0x7fffffff : s.most_ip;
      hash_rows<256, 11, T, true>(smem, wg, s.wgs[0], s.perm_num, ctl, 1, 3, s.ip, s.a_rp, s.a_col, s.a_val, s.b_rp, s.b_col, s.b_val, (int*)nullptr,
          s.c_rp, s.c_col, s.c_val, s.n_cols, (const int*)nullptr, most_ip);
    }
    return;
  }
  wg -= s.wgs[0];
  // (the form for rows alike also where they differ: the launch has its registers anyway; with either form 5003 ragged rows 256 us, 8000 177, R-MAT
  // scale 14 521)
  if (wg < s.wgs[1]) {
    if (ctl->order_differs) return;
    num_recorded_rows<true, T>(reinterpret_cast<NumRecordedLds<T>*>(smem), wg, s.wgs[1], s.perm_sym, ctl, 2, s.records, s.record_of, s.shift_of,
        s.a_rp, s.a_col, s.a_val, s.b_rp, s.b_val, s.b_nnz, s.c_rp, s.c_col, s.c_val);
    return;
  }
  wg -= s.wgs[1];
  if (wg < s.wgs[2]) {
    hash_rows<64, 8, T, true>(smem, wg, s.wgs[2], s.perm_num, ctl, 1, 2, s.ip, s.a_rp, s.a_col, s.a_val, s.b_rp, s.b_col, s.b_val, (int*)nullptr,
        s.c_rp, s.c_col, s.c_val, s.n_cols, s.record_of, 0);
    return;
  }
  wg -= s.wgs[2];
  if (wg < s.wgs[3]) {
    if (!s.words128) {
      esc_rows<64, 128, T>(reinterpret_cast<EscRowsLds<64, 128, T>*>(smem), wg, s.wgs[3], s.perm_num, ctl, 1, 1, s.a_rp, s.a_col, s.a_val, s.b_rp,
          s.b_col, s.b_val, s.c_rp, s.c_col, s.c_val, s.pack128, s.b_nnz);
    } else if (!ctl->order_differs) {
      esc_num_rows<64, 128, T, false>(reinterpret_cast<EscNumLds<64, 128>*>(smem), wg, s.wgs[3], s.perm_sym, ctl, 1, s.a_rp, s.a_col, s.a_val,
          s.b_rp, nullptr, s.b_val, s.b_nnz, s.words128, s.c_rp, s.c_col, s.c_val);
    }
    return;
  }
  wg -= s.wgs[3];
  if (!s.words32) {
    esc_rows<16, 32, T>(reinterpret_cast<EscRowsLds<16, 32, T>*>(smem), wg, s.wgs[4], s.perm_num, ctl, 1, 0, s.a_rp, s.a_col, s.a_val, s.b_rp,
        s.b_col, s.b_val, s.c_rp, s.c_col, s.c_val, s.pack32, s.b_nnz);
  } else if (!ctl->order_differs) {
    esc_num_rows<16, 32, T, false>(reinterpret_cast<EscNumLds<16, 32>*>(smem), wg, s.wgs[4], s.perm_sym, ctl, 0, s.a_rp, s.a_col, s.a_val, s.b_rp,
        nullptr, s.b_val, s.b_nnz, s.words32, s.c_rp, s.c_col, s.c_val);
  }
}

}  // namespace spg
