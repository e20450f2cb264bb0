// Host-side helpers shared by the HIP translation units.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace spg {

int hip_fail(hipError_t e);
int read_header(WsHeader *dev, hipStream_t st, WsHeader *out);  // synchronizes st
int device_cus();
// keep_tag: the zero_region_tag of the caller's accumulator region (the
// header's clean_tag survives only if it equals it), 0, or kKeepAnyTag
int launch_init_header(WsHeader *h, uint64_t keep_tag, hipStream_t st);
int launch_set_tag(WsHeader *h, uint64_t tag, hipStream_t st);
// Row sort of C's columns into (ro, vo) with column lists in `lists`
// (3 * C->ncols int32) and counters in hdr's sort_count and sort_cursor (zero
// on entry unless init is given, which sets the header up).  Columns that esc_class(skip_flops[j], nnz_j, skip_cf) places in
// an expand-sort-compress kernel are skipped (skip_flops NULL: none).
// Kernels for columns longer than max_len are not launched.
int sort_column_lists(const spgemm_csc *C, int32_t *ro, void *vo, int32_t *lists, WsHeader *hdr,
                      const int64_t *skip_flops, double skip_cf, hipStream_t st, int64_t max_len,
                      bool init = false);
int g_min_bin_value();  // the spgemm_debug_min_bin setting
// thresholds of numeric, merge and masked products over columns of up to m rows:
// those in force, but where the largest table holds every column it takes those
// above its threshold too (no workspace is set aside for heavier ones then)
BinCaps num_caps(int64_t m);
// colptr_out[0] = 0, colptr_out[i+1] = counts[0] + ... + counts[i]; bsum holds n / 8192 + 2 int64
// (hdr, if given, is initialised as by launch_init_header(hdr, 0, st))
int launch_colptr_scan(const int64_t *counts, int64_t n, int64_t *colptr_out, int64_t *bsum, hipStream_t st,
                       WsHeader *hdr = nullptr);

// Bins of whose columns those that fill at most half of what the bin holds take
// tables of half the slots (bit 0: bin 2, bit 1: bin 3), for a call over ncol
// columns.  Half tables let more columns run at once and are fuller, so searches
// in them are longer: they pay once the columns do not all run at once in full
// ones anyway.  Masked products, columns of 130-256 rows (bin 2), half against
// full: 0.77 to 1.1 times as fast at 50 to 2000 columns, 1.25 to 1.75 at 4000;
// of 520-1024 rows (bin 3), 0.73 to 1.1 at 50 to 500 columns, 1.0 to 2.4 at 1000
// (numeric pass 0.88 to 1.0 and 1.9 to 2.2; 0.95 to 1.0 and 1.2 to 1.7).
inline int half_tables(int64_t ncol) {
  return (ncol > 12 * (int64_t)device_cus() ? 1 : 0) | (ncol > 3 * (int64_t)device_cus() ? 2 : 0);
}

// What launch_init_header does, for kernels that do it beside their own work.
__device__ __forceinline__ void init_header(WsHeader *h, uint64_t keep_tag, int keep_status, int keep_left) {
  if (!keep_status) h->status = 0;
  if (!keep_left) h->left_tag = 0;  // every other operation may overwrite the slabbed copy
  h->left_new = 0;
  for (int b = 0; b < kNumBins; b++) h->bin_count[b] = 0;
  for (int b = 0; b < kNumBins; b++) h->cursor[b] = 0;
  for (int b = 0; b < 4; b++) h->esc_count[b] = 0;
  for (int b = 0; b < 4; b++) h->sort_count[b] = 0;
  h->sort_cursor = 0;
  h->half_count[0] = h->half_count[1] = 0;
  h->split_cursor = 0;
  h->items = 0;
  h->item_cursor = 0;
  h->nwide = 0;
  h->wide_cursor = 0;
  if (keep_tag != kKeepAnyTag && h->clean_tag != keep_tag) h->clean_tag = 0;
}

inline unsigned grid_of(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }

#define HIPCHK(x)                              \
  do {                                         \
    hipError_t e_ = (x);                       \
    if (e_ != hipSuccess) return hip_fail(e_); \
  } while (0)
#define LAUNCHCHK()                            \
  do {                                         \
    hipError_t e_ = hipGetLastError();         \
    if (e_ != hipSuccess) return hip_fail(e_); \
  } while (0)

}  // namespace spg
