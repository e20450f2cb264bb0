// Row-sorted output columns.  The paper keeps the final output of its
// column-wise merge (Merge-Fiber) sorted within each column (Sec. IV-D),
// while the sort-free hash kernels of this library write rows in table
// order; this pass turns any such output into row-sorted columns, so a
// caller that needs sorted columns pays for the ordering once, after the
// product (or after the merge), instead of inside every accumulation.
//
// Each column is sorted by row, values moving with their rows, from the
// input arrays into separate output arrays (the column pointers stay the
// same).  Rows must be unique within a column, as in every output of the
// library.  Columns are binned by length:
//   up to 64 entries  : one wave, a bitonic network across the lanes;
//   up to 512         : one wave, ranked in LDS by distribution;
//   up to 4096        : one workgroup, likewise;
//   longer            : one workgroup, row windows of up to 2^19 rows: the
//                       window's rows are marked in an LDS bitmap, a prefix
//                       count over the bitmap words gives every row its
//                       rank, and each entry is written straight to its
//                       sorted position (no data movement between passes; a
//                       window with no entry is skipped).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.hpp"
#include "hip_host.hpp"
#include "internal.hpp"
#include "profile.hpp"
#include "rank_sort.hpp"

namespace spg {
namespace {

constexpr int kSortWaveLen = 64;
constexpr int kSortWave512Len = 512;
constexpr int kSortBlockLen = 4096;
constexpr int kSortBlockThreads = 512;
constexpr int kSortWinWords = (1 << 19) / 32;  // bitmap words of the largest row window
constexpr int kSortDupCode = 11;  // status code: a row twice in one column, or a row outside [0, m)

// Column lists per length class, counts in the header: up to 64 entries from
// the front of the first array (sort_count[0]), up to 512 from its end
// (sort_count[3]), up to 4096 in the second (sort_count[1]), longer ones in the
// third (sort_count[2]).
__device__ __forceinline__ int sort_class(int64_t len) {
  return len <= 0 ? -1 : (len <= kSortWaveLen ? 0 : (len <= kSortWave512Len ? 3 : (len <= kSortBlockLen ? 1 : 2)));
}

// Lists this wave's columns (column j of class cls per lane; cls < 0: none);
// counts: one counter per class, in LDS or in memory.
__device__ __forceinline__ void sort_append(int64_t j, int cls, int64_t n, int32_t *lists, int32_t *counts) {
  for (int c = 0; c < 4; c++) {
    const uint64_t mask = __ballot(cls == c);
    if (!mask) continue;
    int base = 0;
    if (lane() == 0) base = atomicAdd(&counts[c], __popcll(mask));
    base = readlane(base, 0);
    const int64_t p = base + mbcnt(mask);
    if (cls == c) lists[c == 3 ? n - 1 - p : (int64_t)c * n + p] = (int32_t)j;
  }
}

// Columns formed in row order by expand-sort-compress (skip_flops given) are
// left out.
__global__ __launch_bounds__(256) void k_sort_bin(const int64_t *cp, int64_t n, int32_t *lists, WsHeader *hdr,
                                                  const int64_t *skip_flops, double skip_cf, int64_t max_len) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int cls = -1;
  if (j < n) {
    const int64_t len = cp[j + 1] - cp[j];
    if (len > max_len) flag_error(&hdr->status, kSortDupCode);  // its class may not be launched
    cls = sort_class(len);
    if (skip_flops && esc_class(skip_flops[j], len, skip_cf) >= 0) cls = -1;
  }
  sort_append(j, cls, n, lists, hdr->sort_count);
}

// Few columns: one workgroup lists them all and sets the header up, which saves
// a launch (10 columns of 4500 entries: 27 -> 24.5 us).
constexpr int64_t kSortFewCols = 4096;
__global__ __launch_bounds__(1024) void k_sort_bin_few(const int64_t *cp, int64_t n, int32_t *lists, WsHeader *hdr,
                                                       int64_t max_len) {
  __shared__ int32_t s_cnt[4];
  __shared__ int s_bad;
  if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  for (int64_t j0 = 0; j0 < n; j0 += 1024) {
    const int64_t j = j0 + threadIdx.x;
    const int64_t len = j < n ? cp[j + 1] - cp[j] : 0;
    if (len > max_len) s_bad = 1;
    sort_append(j, sort_class(len), n, lists, s_cnt);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    init_header(hdr, 0, 0, 0);
    for (int c = 0; c < 4; c++) hdr->sort_count[c] = s_cnt[c];
    if (s_bad) hdr->status = kSortDupCode;
  }
}

template <class VT>
__device__ __forceinline__ VT shfl_xor_v(VT v, int m) {
  return __shfl_xor(v, m, kWave);
}

template <class VT>
__global__ __launch_bounds__(256) void k_sort_wave(const int64_t *cp, const int32_t *ri, const VT *v, int64_t m,
                                                   const int32_t *list, const int32_t *count_p, int32_t *ro, VT *vo,
                                                   int32_t *status) {
  const int count = *count_p;
  const int w = threadIdx.x / kWave, l = lane();
  for (int64_t i = (int64_t)blockIdx.x * 4 + w; i < count; i += (int64_t)gridDim.x * 4) {
    const int64_t j = list[i];
    const int64_t b = cp[j];
    const int len = (int)(cp[j + 1] - b);
    int32_t key = INT32_MAX;  // padding sorts last (rows are below INT32_MAX)
    VT val = VT(0);
    if (l < len) {
      key = ri[b + l];
      val = v[b + l];
    }
#pragma unroll
    for (int k = 2; k <= kWave; k <<= 1) {
#pragma unroll
      for (int s = k >> 1; s > 0; s >>= 1) {
        const int32_t ok = __shfl_xor(key, s, kWave);
        const VT ov = shfl_xor_v(val, s);
        const bool up = (l & k) == 0;     // this block of k lanes sorts ascending
        const bool low = (l & s) == 0;    // the lower lane of the pair keeps the smaller key when ascending
        if (low == up ? ok < key : ok > key) {
          key = ok;
          val = ov;
        }
      }
    }
    if (l < len) {
      ro[b + l] = key;
      vo[b + l] = val;
    }
    // sorted: a repeated row sits next to its twin
    const int32_t nxt = __shfl_down(key, 1, kWave);
    if (__ballot(l < len && ((l + 1 < len && nxt == key) || key < 0 || (int64_t)key >= m)) && l == 0)
      flag_error(status, kSortDupCode);
  }
}

// 65 to 512 entries: one wave per column.  The column's loads are issued
// together, the sorted order is formed in LDS (rank_sort.hpp) and written out
// in order, so both sides of the copy are coalesced.  2.1e6 entries in 18,900
// columns of 65-512: 19 us (a workgroup's bitonic network in LDS took 135).
template <class VT>
__global__ __launch_bounds__(256) void k_sort_wave512(const int64_t *cp, const int32_t *ri, const VT *v, int64_t m,
                                                      const int32_t *list, const int32_t *count_p, int32_t *ro,
                                                      VT *vo, int32_t *status) {
  constexpr int E = kSortWave512Len / kWave;
  __shared__ RankLds<kSortWave512Len, VT> s_r[4];
  const int count = *count_p;
  const int w = threadIdx.x / kWave, l = lane();
  auto &L = s_r[w];
  for (int64_t i = (int64_t)blockIdx.x * 4 + w; i < count; i += (int64_t)gridDim.x * 4) {
    const int64_t j = list[-i];  // listed from the end of the array
    const int64_t b = cp[j];
    const int len = (int)(cp[j + 1] - b);
    int32_t row[E];
    VT val[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
      row[e] = 0;
      val[e] = VT(0);
      if (l + e * kWave < len) {
        row[e] = ri[b + l + e * kWave];
        val[e] = v[b + l + e * kWave];
      }
    }
    int rank[E];
    rank_rows<kWave, E, Ties::kRare>(row, len, l, L, (uint32_t *)nullptr, rank);
#pragma unroll
    for (int e = 0; e < E; e++)
      if (l + e * kWave < len) {
        L.u.s.key[rank[e]] = row[e];
        L.u.s.val[rank[e]] = val[e];
      }
    wave_sync();
    bool bad = false;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int t = l + e * kWave;
      if (t < len) {
        const int32_t k = L.u.s.key[t];
        ro[b + t] = k;
        vo[b + t] = L.u.s.val[t];
        bad |= k < 0 || (int64_t)k >= m;
        bad |= t + 1 < len && L.u.s.key[t + 1] <= k;  // a repeated row sits next to its twin
      }
    }
    if (__ballot(bad) && l == 0) flag_error(status, kSortDupCode);
    wave_sync();  // the next column overwrites the LDS
  }
}

// 513 to 4096 entries: one workgroup per column, likewise.  9e6 entries
// (float64) in columns of 513-4096: 39 us against 424 by the bitonic network.
template <class VT>
__global__ __launch_bounds__(kSortBlockThreads) void k_sort_block(const int64_t *cp, const int32_t *ri, const VT *v,
                                                                  int64_t m, const int32_t *list,
                                                                  const int32_t *count_p, int32_t *ro, VT *vo,
                                                                  int32_t *status) {
  constexpr int E = kSortBlockLen / kSortBlockThreads;
  __shared__ RankLds<kSortBlockLen, VT> L;
  __shared__ uint32_t s_red[4 * kSortBlockThreads / kWave];
  const int count = *count_p;
  const int t = threadIdx.x;
  for (int64_t i = blockIdx.x; i < count; i += gridDim.x) {
    const int64_t j = list[i];
    const int64_t b = cp[j];
    const int len = (int)(cp[j + 1] - b);
    int32_t row[E];
    VT val[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int q = t + e * kSortBlockThreads;
      row[e] = 0;
      val[e] = VT(0);
      if (q < len) {
        row[e] = ri[b + q];
        val[e] = v[b + q];
      }
    }
    int rank[E];
    rank_rows<kSortBlockThreads, E, Ties::kRare>(row, len, t, L, s_red, rank);
#pragma unroll
    for (int e = 0; e < E; e++)
      if (t + e * kSortBlockThreads < len) {
        L.u.s.key[rank[e]] = row[e];
        L.u.s.val[rank[e]] = val[e];
      }
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int q = t + e * kSortBlockThreads;
      if (q < len) {
        const int32_t k = L.u.s.key[q];
        ro[b + q] = k;
        vo[b + q] = L.u.s.val[q];
        bad |= k < 0 || (int64_t)k >= m || (q + 1 < len && L.u.s.key[q + 1] <= k);
      }
    }
    if (__ballot(bad) && lane() == 0) flag_error(status, kSortDupCode);
    __syncthreads();  // the next column overwrites the LDS
  }
}

// Longer columns: windows of rows (the launch sizes the window: every row up
// to 2^19, so one window where m allows).  s_dyn holds the window's bitmap
// and, per word, the entries of the window in words before it.  Columns come
// from a work queue.  A window no larger than m leaves room for two to four
// workgroups per CU, and one that covers m saves the pass for the row range:
// 3.1e8 float32 entries at m = 65,536 take 1.58 ms (3.25 with one workgroup
// and a 2^19-row window each; the copy itself 1.04 at 4.77 TB/s).
template <int THREADS, class VT>
__global__ __launch_bounds__(THREADS) void k_sort_heavy(const int64_t *cp, const int32_t *ri, const VT *v, int64_t m,
                                                        const int32_t *list, const int32_t *count_p, int *cursor,
                                                        int words, int32_t *ro, VT *vo, int32_t *status) {
  constexpr int NW = THREADS / kWave;
  constexpr int U = 8;
  constexpr int kOwn = 16;
  extern __shared__ __align__(16) uint32_t s_dyn[];
  uint32_t *s_bits = s_dyn;
  int32_t *s_pref = (int32_t *)(s_dyn + words);
  __shared__ int s_wtot[NW];
  __shared__ uint32_t s_lo[NW], s_hi[NW];
  __shared__ int s_item;
  const int w = threadIdx.x / kWave, l = lane();
  const int count = *count_p;
  if (blockIdx.x >= count) return;  // the other workgroups empty the queue
  const int64_t win = (int64_t)words * 32;
  const int per = words / NW;  // a multiple of 64
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(cursor, 1);
    __syncthreads();
    const int64_t i = s_item;
    if (i >= count) break;
    const int64_t j = list[i];
    const int64_t b = cp[j], e = cp[j + 1];
    int64_t rlo = 0, rhi = m - 1;
    if (m > win) {  // the column's row range: windows that hold no entry are skipped
      uint32_t hi = 0, nlo = 0;
      for (int64_t p = b + threadIdx.x; p < e; p += THREADS) {
        const int32_t r = ri[p];
        hi = max(hi, (uint32_t)max(r, 0));
        nlo = max(nlo, ~(uint32_t)max(r, 0));
      }
      hi = wave_umax(hi);
      nlo = wave_umax(nlo);
      if (l == 0) {
        s_hi[w] = hi;
        s_lo[w] = nlo;
      }
      __syncthreads();
#pragma unroll
      for (int z = 0; z < NW; z++) {
        hi = max(hi, s_hi[z]);
        nlo = max(nlo, s_lo[z]);
      }
      rlo = (int64_t)~nlo;
      rhi = min((int64_t)hi, m - 1);
    }
    int64_t done = 0;
    for (int64_t w0 = rlo / win * win; w0 <= rhi; w0 += win) {
      const int64_t lim = min(win, m - w0);
      for (int q = threadIdx.x; q < words; q += THREADS) s_bits[q] = 0u;
      __syncthreads();
      for (int64_t p0 = b + threadIdx.x; p0 < e; p0 += U * THREADS) {
        int32_t row[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int64_t p = p0 + u * THREADS;
          row[u] = p < e ? ri[p] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int64_t r = (int64_t)opaque(row[u]) - w0;
          if (row[u] >= 0 && r >= 0 && r < lim) atomicOr(&s_bits[r >> 5], 1u << (r & 31));
        }
      }
      __syncthreads();
      // exclusive prefix of the word counts
      int run = 0, before = 0, tot = 0;
      if (words == kOwn * THREADS) {
        // the largest window: kOwn consecutive words per thread, in registers.
        // (Columns of 4500 entries over the 39 windows of 2.0e7 rows: 1.50 ms for
        // 2000, 1.99 with the loop below, whose scans wait for each other.)
        const uint4 *mine = reinterpret_cast<const uint4 *>(s_bits) + threadIdx.x * (kOwn / 4);
        int c[kOwn];
#pragma unroll
        for (int q = 0; q < kOwn / 4; q++) {
          const uint4 x = mine[q];
          c[4 * q] = __popc(x.x);
          c[4 * q + 1] = __popc(x.y);
          c[4 * q + 2] = __popc(x.z);
          c[4 * q + 3] = __popc(x.w);
        }
#pragma unroll
        for (int q = 0; q < kOwn; q++) run += c[q];
        const int incl = wave_incl_add(run);
        if (l == kWave - 1) s_wtot[w] = incl;
        __syncthreads();
#pragma unroll
        for (int z = 0; z < NW; z++) {
          if (z < w) before += s_wtot[z];
          tot += s_wtot[z];
        }
        int at = before + incl - run;
        int4 *out = reinterpret_cast<int4 *>(s_pref) + threadIdx.x * (kOwn / 4);
#pragma unroll
        for (int q = 0; q < kOwn / 4; q++) {
          const int4 x = make_int4(at, at + c[4 * q], at + c[4 * q] + c[4 * q + 1],
                                   at + c[4 * q] + c[4 * q + 1] + c[4 * q + 2]);
          out[q] = x;
          at = x.w + c[4 * q + 3];
        }
      } else {
        // wave w takes its share of the words, 64 at a time; then the waves'
        // totals are added
        for (int q = w * per; q < (w + 1) * per; q += kWave) {
          const int c = __popc(s_bits[q + l]);
          const int incl = wave_incl_add(c);
          s_pref[q + l] = run + incl - c;
          run += readlane(incl, kWave - 1);
        }
        if (l == 0) s_wtot[w] = run;
        __syncthreads();
#pragma unroll
        for (int z = 0; z < NW; z++) {
          if (z < w) before += s_wtot[z];
          tot += s_wtot[z];
        }
        for (int q = w * per; q < (w + 1) * per; q += kWave) s_pref[q + l] += before;
      }
      __syncthreads();
      for (int64_t p0 = b + threadIdx.x; p0 < e; p0 += U * THREADS) {
        int32_t row[U];
        VT val[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int64_t p = p0 + u * THREADS;
          row[u] = p < e ? ri[p] : -1;
          val[u] = p < e ? v[p] : VT(0);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
          const int64_t r = (int64_t)opaque(row[u]) - w0;
          if (row[u] >= 0 && r >= 0 && r < lim) {
            const int q = (int)(r >> 5);
            const int64_t dst = b + done + s_pref[q] + __popc(s_bits[q] & ((1u << (r & 31)) - 1u));
            if (dst < e) {
              ro[dst] = row[u];
              vo[dst] = opaque(val[u]);
            }
          }
        }
      }
      done += tot;
      __syncthreads();  // the next window clears s_bits, s_pref, s_wtot
    }
    if (threadIdx.x == 0 && done != e - b) flag_error(status, kSortDupCode);
  }
}

template <class VT>
int sort_typed(const spgemm_csc *C, int32_t *ro, void *vo, int32_t *lists, WsHeader *hdr,
               const int64_t *skip_flops, double skip_cf, hipStream_t st, int64_t max_len, bool init) {
  const int64_t n = C->ncols;
  const bool few = init && !skip_flops && n <= kSortFewCols;
  if (init && !few) {
    const int rc = launch_init_header(hdr, (uint64_t)0, st);
    if (rc) return rc;
  }
  ProfScope prof("sort_columns", st);
  if (few)
    hipLaunchKernelGGL(k_sort_bin_few, dim3(1), dim3(1024), 0, st, C->colptr, n, lists, hdr, max_len);
  else
    hipLaunchKernelGGL(k_sort_bin, dim3(grid_of(n, 256)), dim3(256), 0, st, C->colptr, n, lists, hdr, skip_flops,
                       skip_cf, max_len);
  LAUNCHCHK();
  const VT *v = (const VT *)C->values;
  const int cus = device_cus();
  hipLaunchKernelGGL(k_sort_wave<VT>, dim3(8 * cus), dim3(256), 0, st, C->colptr, C->rowidx, v, C->nrows, lists,
                     (const int32_t *)&hdr->sort_count[0], ro, (VT *)vo, &hdr->status);
  LAUNCHCHK();
  if (max_len > kSortWaveLen) {
    hipLaunchKernelGGL(k_sort_wave512<VT>, dim3(8 * cus), dim3(256), 0, st, C->colptr, C->rowidx, v, C->nrows,
                       lists + n - 1, (const int32_t *)&hdr->sort_count[3], ro, (VT *)vo, &hdr->status);
    LAUNCHCHK();
  }
  if (max_len > kSortWave512Len) {
    hipLaunchKernelGGL(k_sort_block<VT>, dim3(4 * cus), dim3(kSortBlockThreads), 0, st, C->colptr, C->rowidx, v,
                       C->nrows, lists + n, (const int32_t *)&hdr->sort_count[1], ro, (VT *)vo, &hdr->status);
    LAUNCHCHK();
  }
  if (max_len <= kSortBlockLen) return SPGEMM_OK;
  // a window as large as m asks for, so that several workgroups fit a CU
  int words = 1024;
  while (words < kSortWinWords && (int64_t)words * 32 < C->nrows) words *= 2;
  const size_t lds = (size_t)words * 8;
  const int32_t *hl = lists + 2 * n, *hc = (const int32_t *)&hdr->sort_count[2];
  if (words <= 4096)
    hipLaunchKernelGGL((k_sort_heavy<512, VT>), dim3(4 * cus), dim3(512), lds, st, C->colptr, C->rowidx, v, C->nrows,
                       hl, hc, &hdr->sort_cursor, words, ro, (VT *)vo, &hdr->status);
  else
    hipLaunchKernelGGL((k_sort_heavy<1024, VT>), dim3((words <= 8192 ? 2 : 1) * cus), dim3(1024), lds, st, C->colptr,
                       C->rowidx, v, C->nrows, hl, hc, &hdr->sort_cursor, words, ro, (VT *)vo, &hdr->status);
  LAUNCHCHK();
  return SPGEMM_OK;
}

}  // namespace

int sort_column_lists(const spgemm_csc *C, int32_t *ro, void *vo, int32_t *lists, WsHeader *hdr,
                      const int64_t *skip_flops, double skip_cf, hipStream_t st, int64_t max_len, bool init) {
  if (C->dtype == SPGEMM_F32) return sort_typed<float>(C, ro, vo, lists, hdr, skip_flops, skip_cf, st, max_len, init);
  return sort_typed<double>(C, ro, vo, lists, hdr, skip_flops, skip_cf, st, max_len, init);
}

}  // namespace spg

using namespace spg;

extern "C" {

int spgemm_sort_columns(const spgemm_csc *C, int32_t *rowidx_out, void *values_out, void *ws, size_t ws_bytes,
                        void *stream) {
  int st = check_csc(C, true);
  if (st) return st;
  if (C->ncols > INT32_MAX) return SPGEMM_E_OVERFLOW;
  if (C->nnz > 0 && (!rowidx_out || !values_out)) return SPGEMM_E_INVAL;
  if (C->nnz > 0 && ((const void *)rowidx_out == (const void *)C->rowidx || values_out == C->values))
    return SPGEMM_E_INVAL;  // out of place only
  WsLayout L;
  st = ws_layout(SPGEMM_OP_SORT, C, nullptr, 0, 0, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  if (C->ncols == 0) return launch_init_header((WsHeader *)ws, (uint64_t)0, (hipStream_t)stream);
  hipStream_t s = (hipStream_t)stream;
  return sort_column_lists(C, rowidx_out, values_out, (int32_t *)((char *)ws + L.bins), (WsHeader *)ws, nullptr, 0.0,
                           s, C->nnz, true);
}

}  // extern "C"
