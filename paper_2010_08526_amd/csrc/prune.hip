// Per-column pruning of one output batch: the step an application applies
// to each batch of C before it moves on to the next (Sec. I and Sec. IV-B:
// Markov clustering keeps the k largest entries of every column; Sec. V-C:
// HipMCL prunes column by column).
//
// Candidates are the entries with value >= threshold, compared in float64
// (NaN is never a candidate).  With k >= 0 at most the k largest candidates
// are kept, equal values going to the smaller row; kept entries stay in
// their input order, so the hash-table order of the numeric pass carries
// over unchanged.
//
// For small k against the columns' lengths (see read_once), k_prune_top
// reads every column once (see there).  Otherwise, and for columns with too
// many equal values for it:
//
// One workgroup per column.  Every entry gets a composite key that orders
// it as the selection does: the value mapped onto an unsigned integer in
// numeric order (-0 folded onto +0), then the row mapped so that a smaller
// row ranks higher.  Rows are unique inside a column, so keys are too, and
// a most-significant-digit radix select ends with a cut key: an entry is
// kept iff it is a candidate and its key is at least the cut.  The first
// digit is wide (12 bits, a 4096-bucket LDS histogram that skips entries
// below a lower bound on the k-th largest key's digit) and its chosen bucket
// is usually settled by sorting its candidates in LDS; otherwise 8-bit
// digits (256-bucket histograms) follow.  A scan of the per-column counts
// gives the output column pointers, and a second kernel compacts the kept
// entries in order with one exchange of per-wave counts per 2048 entries
// that keep any (one flag per wave for those that keep none).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "device.hpp"
#include "hip_host.hpp"
#include "internal.hpp"
#include "profile.hpp"
#include "rank_sort.hpp"

namespace spg {
namespace {

constexpr int kPrThreads = 256;
constexpr int kPrWaves = kPrThreads / kWave;
constexpr int kPrMaxGrid = 65536;
constexpr int kSelUnroll = 8;    // select: coalesced loads per thread per step
constexpr int kFillUnroll = 8;   // compaction: coalesced slots per thread per step
constexpr int kPrDupRows = 10;  // status code: a row twice in one column

// Values of cutv for the columns that k_prune_top has seen; neither is the key
// of a candidate (float keys are below 2^32, a double's would be a NaN).
constexpr uint64_t kTopDone = ~0ull;      // settled
constexpr uint64_t kTopLeft = ~0ull - 1;  // left to the kernels that follow

__device__ __forceinline__ uint64_t order_key(float v) {
  uint32_t b = __float_as_uint(v);
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? (uint64_t)(~b) : (uint64_t)(b | 0x80000000u);
}
__device__ __forceinline__ uint64_t order_key(double v) {
  uint64_t b = (uint64_t)__double_as_longlong(v);
  if (b == 0x8000000000000000ull) b = 0ull;
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
// rows in [0, 2^31 - 1] map onto [2^31 - 1, 0]: the smaller row, the larger key
__device__ __forceinline__ uint32_t row_key(int32_t r) { return 0x7FFFFFFFu - (uint32_t)r; }

// Digit d of the composite key, most significant first: VD digits of the
// value key, then 4 of the row key.
template <int VD>
__device__ __forceinline__ int key_digit(int d, uint64_t vk, uint32_t rk) {
  return d < VD ? (int)((vk >> (8 * (VD - 1 - d))) & 255u) : (int)((rk >> (8 * (3 - (d - VD)))) & 255u);
}
// Masks of the digits above d.
template <int VD>
__device__ __forceinline__ uint64_t value_mask(int d) {
  return d >= VD ? ~0ull : (d == 0 ? 0ull : (~0ull << (8 * (VD - d))));
}
template <int VD>
__device__ __forceinline__ uint32_t row_mask(int d) {
  return d <= VD ? 0u : (~0u << (8 * (4 - (d - VD))));
}

template <typename VT>
__device__ __forceinline__ bool candidate(VT v, double thr) {
  return (double)v >= thr;
}

// Adds one to s_hist[dig] for every lane with `act`.  The digit of the first
// such lane is added once for all lanes that share it (one LDS atomic
// instead of up to 64 serialized on one address: the leading digits of a
// column's keys fall mostly into one or two buckets); the other lanes add
// their own.  Called by the whole wave.
__device__ __forceinline__ void hist_add(int *s_hist, bool act, int dig) {
  const uint64_t m = __ballot(act);
  if (m == 0) return;
  const int src = __builtin_ctzll(m);
  const int lead = __builtin_amdgcn_readlane(dig, src);
  const bool same = act && dig == lead;
  const uint64_t ms = __ballot(same);
  if (lane() == src) atomicAdd(&s_hist[lead], __popcll(ms));
  if (act && !same) atomicAdd(&s_hist[dig], 1);
}

// Wide first digit: the top kWideBits of the value key (sign, exponent and
// the top mantissa bits of a float32), a 4096-bucket histogram; the bucket
// holding the k-th largest key is then resolved in LDS when it holds at most
// kStage candidates (gathered by a second pass, sorted by key), so most
// columns are read twice whatever their length.
constexpr int kWideBits = 12;
constexpr int kWideBuckets = 1 << kWideBits;
constexpr int kStage = 2048;

// Bitonic sort of s_v / s_r (n a power of two), descending by (value key,
// row key).  Contains barriers.
__device__ __forceinline__ void stage_sort_desc(uint64_t *s_v, uint32_t *s_r, int n) {
  for (int k = 2; k <= n; k <<= 1) {
    for (int s = k >> 1; s > 0; s >>= 1) {
      for (int t = threadIdx.x; t < n / 2; t += kPrThreads) {
        const int a = ((t & ~(s - 1)) << 1) | (t & (s - 1));  // lower element of pair t at distance s
        const int c = a + s;
        const bool down = (a & k) == 0;  // this block of k sorts descending
        const uint64_t va = s_v[a], vc = s_v[c];
        const uint32_t ra = s_r[a], rc = s_r[c];
        const bool lt = va < vc || (va == vc && ra < rc);  // key a below key c
        if (lt == down) {
          s_v[a] = vc;
          s_v[c] = va;
          s_r[a] = rc;
          s_r[c] = ra;
        }
      }
      __syncthreads();
    }
  }
}

// Which of the columns j0 ... j0 + per a workgroup has to work on (bit i: column
// j0 + i): its one or, with LEFT, those that k_prune_top has not settled, found
// one per lane (looked at one by one, 100,000 settled columns took 25 us).
template <bool LEFT>
__device__ __forceinline__ uint64_t prune_columns(int64_t j0, int64_t per, int64_t ncols, const uint64_t *cutv) {
  if constexpr (!LEFT) return 1ull;
  const int64_t j = j0 + lane();
  const uint64_t m = __ballot(lane() < per && j < ncols && cutv[j] != kTopDone);
  __syncthreads();  // cutv is written below
  return m;
}

// cnt[j]: entries column j keeps; (cutv[j], cutr[j]): the smallest kept key
// ((0, 0) keeps every candidate).  The histogram of the first digit also
// counts the candidates, so a column that keeps all of them is read once.
template <bool LEFT, typename VT>
__global__ __launch_bounds__(kPrThreads) void k_prune_select(const int64_t *__restrict__ colptr,
                                                             const int32_t *__restrict__ rowidx,
                                                             const VT *__restrict__ vals, int64_t ncols, double thr,
                                                             int64_t nnz, int64_t k, int64_t *__restrict__ cnt,
                                                             uint64_t *__restrict__ cutv, uint32_t *__restrict__ cutr,
                                                             int32_t *status) {
  constexpr int VD = (int)sizeof(VT), ND = VD + 4;
  constexpr int kShift = 8 * VD - kWideBits;  // value key bits below the wide digit
  __shared__ int s_hist[256];
  __shared__ int s_sel[4];  // chosen digit, entries still needed inside it, selection complete, candidates
  // the wide histogram, then (same memory) the staged value keys of its chosen bucket
  __shared__ __align__(16) uint64_t s_wide[kWideBuckets / 2];
  __shared__ uint32_t s_srow[kStage];
  __shared__ int s_n;
  __shared__ int s_ncw[kPrWaves];  // candidates counted by each wave
  int *s_whist = reinterpret_cast<int *>(s_wide);
  const int t = threadIdx.x;
  const int64_t per = LEFT ? min((int64_t)kWave, (ncols + gridDim.x - 1) / gridDim.x) : 1;
  for (int64_t j0 = (int64_t)blockIdx.x * per; j0 < ncols; j0 += (int64_t)gridDim.x * per)
  for (uint64_t todo = prune_columns<LEFT>(j0, per, ncols, cutv); todo; todo &= todo - 1) {
    const int64_t j = LEFT ? j0 + __builtin_ctzll(todo) : j0;
    int64_t b = colptr[j], e = colptr[j + 1];
    if (b < 0 || e < b || e > nnz) {  // pointers outside the arrays: the column counts as empty
      if (t == 0) flag_error(status, 5);
      b = e = 0;
    }
    // need: entries still to keep among those matching the prefix; until the
    // first digit has counted the candidates it stands for "all of them"
    int need = k >= 0 && k < INT32_MAX ? (int)k : INT32_MAX, above = 0, last = 0, kept = -1;
    uint64_t pv = 0;
    uint32_t pr = 0;
    bool fast = k > 0 && k < INT32_MAX;  // the wide digit first; cleared when the digit loop must run
    if (fast) {
      // A lower bound on the wide digit of the k-th largest key of a column
      // longer than one step: the k-th largest of the per-thread maxima of
      // the first step (k distinct entries at or above it), rounded down to
      // its bucket.  Buckets below it cannot hold one of the k largest keys
      // and are not counted (the candidates are counted apart).
      int lo_dig = 0;
      if (e - b > kSelUnroll * kPrThreads && k <= kPrThreads) {
        uint64_t mk = 0;
        bool has = false;
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          // (an opaque index: these loads stay apart from the histogram loop's)
          const VT v = vals[opaque(b + q * kPrThreads + t)];
          if (candidate(v, thr)) {
            const uint64_t vk = order_key(v);
            mk = vk > mk ? vk : mk;
            has = true;
          }
        }
        for (int i = t; i < kWideBuckets; i += kPrThreads) s_whist[i] = 0;
        __syncthreads();
        if (has) atomicAdd(&s_whist[(int)(mk >> kShift)], 1);
        __syncthreads();
        if (t < kWave) {
          constexpr int PER = kWideBuckets / kWave;
          int sum = 0;
#pragma unroll 1
          for (int q = 0; q < PER; q++) sum += s_whist[kWideBuckets - 1 - PER * t - q];
          const int incl = wave_incl_add(sum);
          if (t == kWave - 1 && incl < need) s_sel[0] = 0;  // fewer maxima than k: no bound
          int acc = incl - sum;
          if (acc < need && need <= incl) {
#pragma unroll 1
            for (int q = 0; q < PER; q++) {
              acc += s_whist[kWideBuckets - 1 - PER * t - q];
              if (acc >= need) {
                s_sel[0] = kWideBuckets - 1 - PER * t - q;
                break;
              }
            }
          }
        }
        __syncthreads();
        lo_dig = s_sel[0];
      }
      for (int i = t; i < kWideBuckets; i += kPrThreads) s_whist[i] = 0;
      __syncthreads();
      int nc = 0;  // this thread's candidates
      for (int64_t c0 = b; c0 < e; c0 += kSelUnroll * kPrThreads) {
        VT vq[kSelUnroll];
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          const int64_t p = c0 + q * kPrThreads + t;
          vq[q] = p < e ? vals[p] : VT(0);
        }
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          const int64_t p = c0 + q * kPrThreads + t;
          const bool cand = p < e && candidate(vq[q], thr);
          const int dig = cand ? (int)(order_key(vq[q]) >> kShift) : 0;
          nc += cand ? 1 : 0;
          hist_add(s_whist, cand && dig >= lo_dig, dig);
        }
      }
      nc = wave_sum_i32(nc);
      if (lane() == 0) s_ncw[t / kWave] = nc;
      __syncthreads();
      if (t < kWave) {
        // lane l owns buckets 4095 - 64l ... 4032 - 64l, scanned from the top
        constexpr int PER = kWideBuckets / kWave;
        int sum = 0;
        for (int q = 0; q < PER; q++) sum += s_whist[kWideBuckets - 1 - PER * t - q];
        const int incl = wave_incl_add(sum);
        if (t == kWave - 1) {
          int tot = 0;
#pragma unroll
          for (int z = 0; z < kPrWaves; z++) tot += s_ncw[z];
          s_sel[3] = tot;
        }
        int acc = incl - sum;
        if (acc < need && need <= incl) {
          for (int q = 0; q < PER; q++) {
            const int h = s_whist[kWideBuckets - 1 - PER * t - q];
            if (acc + h >= need) {
              s_sel[0] = kWideBuckets - 1 - PER * t - q;
              s_sel[1] = need - acc;
              s_sel[2] = h;
              break;
            }
            acc += h;
          }
        }
      }
      __syncthreads();
      const int ncand = s_sel[3];
      if (ncand <= need) {  // every candidate is kept
        kept = ncand;
      } else if (s_sel[2] <= kStage) {
        // gather the chosen bucket's candidates, sort them, take the need-th largest
        const uint64_t bucket = (uint64_t)s_sel[0];
        const int rest = s_sel[1], nb = s_sel[2];
        __syncthreads();  // s_sel and the histogram are read; the stage reuses its memory
        if (t == 0) s_n = 0;
        __syncthreads();
        for (int64_t c0 = b; c0 < e; c0 += kSelUnroll * kPrThreads) {
          VT vq[kSelUnroll];
#pragma unroll
          for (int q = 0; q < kSelUnroll; q++) {
            const int64_t p = c0 + q * kPrThreads + t;
            vq[q] = p < e ? vals[p] : VT(0);
          }
#pragma unroll
          for (int q = 0; q < kSelUnroll; q++) {
            const int64_t p = c0 + q * kPrThreads + t;
            const uint64_t vk = order_key(vq[q]);
            const bool in = p < e && candidate(vq[q], thr) && (vk >> kShift) == bucket;
            const uint64_t m = __ballot(in);
            if (m == 0) continue;  // uniform
            int base = 0;
            if (lane() == 0) base = atomicAdd(&s_n, __popcll(m));
            base = readlane(base, 0);
            const int pos = base + mbcnt(m);
            if (in && pos < kStage) {
              s_wide[pos] = vk;
              s_srow[pos] = row_key(rowidx[p]);
            }
          }
        }
        __syncthreads();
        int n2 = kWave;
        while (n2 < nb) n2 <<= 1;
        for (int i = nb + t; i < n2; i += kPrThreads) {  // padding sorts last
          s_wide[i] = 0ull;
          s_srow[i] = 0u;
        }
        __syncthreads();
        stage_sort_desc(s_wide, s_srow, n2);
        above = need - rest;
        need = rest;
        pv = s_wide[rest - 1];
        pr = s_srow[rest - 1];
        kept = (int)k;
        __syncthreads();  // the stage is rewritten by the next column
      } else {
        fast = false;  // the bucket is too full to stage: the digit loop decides
        __syncthreads();
      }
    }
    for (int d = 0; d < ND && !fast; d++) {
      for (int i = t; i < 256; i += kPrThreads) s_hist[i] = 0;
      if (t == 0) {
        s_sel[0] = 0;
        s_sel[1] = need;
        s_sel[2] = 1;
      }
      __syncthreads();
      const uint64_t vm = value_mask<VD>(d);
      const uint32_t rm = row_mask<VD>(d);
      // kSelUnroll coalesced loads per thread in flight, then their digits;
      // the same trip count for every lane
      for (int64_t c0 = b; c0 < e; c0 += kSelUnroll * kPrThreads) {
        VT vq[kSelUnroll];
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          const int64_t p = c0 + q * kPrThreads + t;
          vq[q] = p < e ? vals[p] : VT(0);
        }
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          const int64_t p = c0 + q * kPrThreads + t;
          bool act = false;
          int dig = 0;
          if (p < e) {
            const VT v = vq[q];
            if (candidate(v, thr)) {
              const uint64_t vk = order_key(v);
              if (d < VD) {  // value digits: the row is not read
                act = (vk & vm) == pv;
                dig = key_digit<VD>(d, vk, 0u);
              } else if (vk == pv) {  // row digits, among entries of the chosen value
                const uint32_t rk = row_key(rowidx[p]);
                act = (rk & rm) == pr;
                dig = key_digit<VD>(d, vk, rk);
              }
            }
          }
          hist_add(s_hist, act, dig);
        }
      }
      __syncthreads();
      if (t < kWave) {
        // lane l owns buckets 255 - 4l ... 252 - 4l, scanned from the top
        int h[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          h[q] = s_hist[255 - 4 * t - q];
          sum += h[q];
        }
        const int incl = wave_incl_add(sum);
        if (d == 0 && t == kWave - 1) s_sel[3] = incl;
        int acc = incl - sum;
        if (acc < need && need <= incl) {
#pragma unroll
          for (int q = 0; q < 4; q++) {
            if (acc + h[q] >= need) {
              s_sel[0] = 255 - 4 * t - q;
              s_sel[1] = need - acc;
              s_sel[2] = h[q] == need - acc ? 1 : 0;
              break;
            }
            acc += h[q];
          }
        }
      }
      __syncthreads();
      if (d == 0) {
        const int ncand = s_sel[3];
        if (k < 0 || (int64_t)ncand <= k) {  // every candidate is kept
          kept = ncand;
          pv = 0;
          pr = 0;
          __syncthreads();
          break;
        }
        if (k == 0) {
          kept = 0;
          pv = ~0ull;
          pr = ~0u;
          __syncthreads();
          break;
        }
      }
      // 0 < k < candidates: the scan found the bucket of the k-th largest key
      const int dig = s_sel[0], rest = s_sel[1], done = s_sel[2];
      above += need - rest;
      need = rest;
      last = s_hist[dig];
      if (d < VD)
        pv |= (uint64_t)dig << (8 * (VD - 1 - d));
      else
        pr |= (uint32_t)dig << (8 * (3 - (d - VD)));
      __syncthreads();  // s_hist and s_sel are rewritten by the next digit or column
      if (done) break;
    }
    if (t == 0) {
      // selection: every key with the chosen prefix is kept; `above` outrank it, `last` share it
      if (kept < 0) {
        const int64_t all = (int64_t)above + last;
        kept = (int)(all < k ? all : k);
      }
      cnt[j] = kept;
      cutv[j] = pv;
      cutr[j] = pr;
    }
  }
}

// Compacts the kept entries of every column, in input order, to
// out_colptr[j] ... out_colptr[j + 1].  A column that holds more keys at the
// cut than its count (a row twice) writes only its count and flags status.
template <bool LEFT, typename VT>
__global__ __launch_bounds__(kPrThreads) void k_prune_fill(
    const int64_t *__restrict__ colptr, const int32_t *__restrict__ rowidx, const VT *__restrict__ vals,
    int64_t ncols, int64_t nnz, double thr, const uint64_t *__restrict__ cutv, const uint32_t *__restrict__ cutr,
    const int64_t *__restrict__ out_colptr, int32_t *__restrict__ out_rowidx, VT *__restrict__ out_vals,
    int32_t *status) {
  __shared__ int s_cnt[kFillUnroll][kPrWaves];
  __shared__ int s_any[2][kPrWaves];
  const int t = threadIdx.x, w = t / kWave;
  int par = 0;
  const int64_t per = LEFT ? min((int64_t)kWave, (ncols + gridDim.x - 1) / gridDim.x) : 1;
  for (int64_t j0 = (int64_t)blockIdx.x * per; j0 < ncols; j0 += (int64_t)gridDim.x * per)
  for (uint64_t todo = prune_columns<LEFT>(j0, per, ncols, cutv); todo; todo &= todo - 1) {
    const int64_t j = LEFT ? j0 + __builtin_ctzll(todo) : j0;
    int64_t b = colptr[j], e = colptr[j + 1];
    if (b < 0 || e < b || e > nnz) b = e = 0;  // flagged by the select kernel
    const int64_t o = out_colptr[j], lim = out_colptr[j + 1];
    const uint64_t cv = cutv[j];
    const uint32_t cr = cutr[j];
    int64_t run = 0;
    // kFillUnroll coalesced slots per thread per step (entry c0 + q * 256 + t
    // in slot q); an entry's place in input order is the kept count of the
    // earlier slots, then of earlier waves in its slot, then of lower lanes,
    // so one exchange of per-wave counts orders the whole step.  The row is
    // read only for an entry that is kept or ties the cut's value.
    for (int64_t c0 = b; c0 < e; c0 += kFillUnroll * kPrThreads) {
      VT v[kFillUnroll];
#pragma unroll
      for (int q = 0; q < kFillUnroll; q++) {
        const int64_t p = c0 + q * kPrThreads + t;
        v[q] = p < e ? vals[p] : VT(0);
      }
      uint32_t keep = 0;
#pragma unroll
      for (int q = 0; q < kFillUnroll; q++) {
        const int64_t p = c0 + q * kPrThreads + t;
        if (p < e && candidate(v[q], thr)) {
          const uint64_t vk = order_key(v[q]);
          if (vk > cv || (vk == cv && row_key(rowidx[p]) >= cr)) keep |= 1u << q;
        }
      }
      // a step in which no wave keeps an entry (the common case: k is
      // small against the column) only exchanges one flag per wave, through
      // two alternating flag sets (a set is rewritten two steps later, after
      // every wave has passed the barrier between)
      const bool wkeep = __ballot(keep != 0u) != 0ull;
      int *any_w = s_any[par];
      par ^= 1;
      if (lane() == 0) any_w[w] = wkeep ? 1 : 0;
      __syncthreads();
      bool any = false;
#pragma unroll
      for (int z = 0; z < kPrWaves; z++) any |= any_w[z] != 0;
      if (!any) continue;
      int below[kFillUnroll];
#pragma unroll
      for (int q = 0; q < kFillUnroll; q++) {
        const uint64_t m = __ballot((keep >> q) & 1u);
        below[q] = mbcnt(m);
        if (lane() == 0) s_cnt[q][w] = __popcll(m);
      }
      __syncthreads();
      int64_t base = o + run;
#pragma unroll
      for (int q = 0; q < kFillUnroll; q++) {
        int before = 0, tot = 0;
#pragma unroll
        for (int z = 0; z < kPrWaves; z++) {
          const int c = s_cnt[q][z];
          before += z < w ? c : 0;
          tot += c;
        }
        if ((keep >> q) & 1u) {
          const int64_t pos = base + before + below[q];
          if (pos < lim) {
            out_rowidx[pos] = rowidx[c0 + q * kPrThreads + t];
            out_vals[pos] = v[q];
          }
        }
        base += tot;
      }
      run = base - o;
      __syncthreads();  // s_cnt is written again by the next step
    }
    if (t == 0 && o + run != lim) flag_error(status, kPrDupRows);
  }
}

// ----------------------------------------------------------------------------
// One reading of a column, for 1 <= k <= kTopMaxK: entries at or above a bound
// are appended to a list in LDS (value key and position); whenever the list
// holds more than kTopLimit of them, the bound rises to its k-th largest value
// and the list shrinks to the entries at or above it.  The k largest entries
// are always in the list, an entry below the bound costs one comparison, and
// after N entries about one in N / k passes.  The kept positions, in input
// order, go to stage[j * k ...]; cutv / cutr are set to kTopDone.  A column
// with more equal values at its bound than the list can hold is left to the
// kernels above (kTopLeft).
//
// Values are read once, the next step's while one is worked on, where the
// digit histogram read them twice and worked on each, and the fill kernel a
// third time.  2.0e8 float32 entries in 20,011 columns, k = 100: 349 us (2.3
// TB/s; digit passes for the bounds, two or three per column, take most of the
// rest) and 100 us for the entries kept, against 973 and 394 us; 2.96e9 entries
// of a scale 18 R-MAT square in four batches: 6.3 + 0.9 against 15.2 + 8.4 ms.
// ----------------------------------------------------------------------------
constexpr int kTopMaxK = 1024;
constexpr int kTopStep = kSelUnroll * kPrThreads;

template <typename VT>
struct TopKey;
template <>
struct TopKey<float> {
  using T = uint32_t;
};
template <>
struct TopKey<double> {
  using T = uint64_t;
};

__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k);
}
__device__ __forceinline__ double key_value(uint64_t k) {
  return __longlong_as_double((long long)((k >> 63) ? k & 0x7fffffffffffffffull : ~k));
}

// The need-th largest of the keys key[e] with bit e of `have` set, over the
// workgroup (1 <= need <= their number), by 8-bit digits, most significant
// first.  Digits stop once no more than `stop` keys are at or above the chosen
// bucket: returned is its lower edge (the key itself after the last digit).
// above / equal: the keys above the bucket, and in it.  With TIGHT (32-bit keys
// whose high digits are alike: rows) the digits that all keys share are passed
// over: 50,000 columns of 300 entries of 8 values, k = 10, 611 -> 569 us.  (The
// same for the low digits of float64 values takes registers that cost more.)
// s_hist: kKthWords words; a digit uses one of two histograms while the other is
// cleared.  Contains barriers.
constexpr int kKthWords = 2 * 256 + 4 + 2 * kPrWaves;
template <bool TIGHT, int E, typename KT>
__device__ __forceinline__ KT block_kth(const KT (&key)[E], uint32_t have, int need, int stop, int *s_hist, int &above,
                                        int &equal) {
  constexpr int ND = (int)sizeof(KT);
  static_assert(!TIGHT || ND == 4, "32-bit keys");
  int *s_sel = s_hist + 512;
  uint32_t *s_key = reinterpret_cast<uint32_t *>(s_hist + 516);  // each wave's largest key and largest complement
  const int t = threadIdx.x;
  KT prefix = 0;
  above = 0;
  equal = 0;
  s_hist[t] = 0;  // (256 threads)
  __syncthreads();
  int top = ND - 1, par = 0;
  if constexpr (TIGHT) {
    // the highest digit in which the keys differ; those above it are the prefix
    uint32_t hi = 0, nlo = 0;
#pragma unroll
    for (int e = 0; e < E; e++) {
      hi = max(hi, (have >> e) & 1u ? key[e] : 0u);
      nlo = max(nlo, (have >> e) & 1u ? ~key[e] : 0u);
    }
    hi = wave_umax(hi);
    nlo = wave_umax(nlo);
    if (lane() == 0) {
      s_key[t / kWave] = hi;
      s_key[kPrWaves + t / kWave] = nlo;
    }
    __syncthreads();
#pragma unroll
    for (int z = 0; z < kPrWaves; z++) {
      hi = max(hi, s_key[z]);
      nlo = max(nlo, s_key[kPrWaves + z]);
    }
    const uint32_t diff = hi ^ ~nlo;
    top = diff == 0 ? 0 : (31 - __clz((int)diff)) / 8;  // (alike: the last digit counts them)
    if (top < 3) prefix = hi & (~0u << (8 * (top + 1)));
  }
#pragma unroll 1
  for (int d = top; d >= 0; d--) {
    int *h_cur = s_hist + 256 * par, *h_next = s_hist + 256 * (par ^ 1);
    par ^= 1;
    const KT mask = d == ND - 1 ? KT(0) : (KT)(~KT(0) << (8 * (d + 1)));
#pragma unroll
    for (int e = 0; e < E; e++)
      hist_add(h_cur, ((have >> e) & 1u) && (key[e] & mask) == prefix, (int)((key[e] >> (8 * d)) & 255u));
    __syncthreads();
    h_next[t] = 0;
    if (t < kWave) {
      int h[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        h[q] = h_cur[255 - 4 * t - q];
        sum += h[q];
      }
      const int incl = wave_incl_add(sum);
      int acc = incl - sum;
      const int want = need - above;
      if (acc < want && want <= incl) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
          if (acc + h[q] >= want) {
            s_sel[0] = 255 - 4 * t - q;
            s_sel[1] = acc;
            s_sel[2] = h[q];
            break;
          }
          acc += h[q];
        }
      }
    }
    __syncthreads();
    prefix |= (KT)s_sel[0] << (8 * d);
    above += s_sel[1];
    equal = s_sel[2];
    if (above + equal <= stop) break;  // uniform
  }
  __syncthreads();  // s_hist and s_sel may be written again
  return prefix;
}

// One step's values from entry c0 on; past e a value that no bound lets pass.
template <typename VT>
__device__ __forceinline__ void top_load(const VT *__restrict__ vals, int64_t c0, int64_t e, int t,
                                         VT (&v)[kSelUnroll]) {
  if (c0 + kTopStep <= e) {
#pragma unroll
    for (int q = 0; q < kSelUnroll; q++) v[q] = vals[c0 + q * kPrThreads + t];
  } else {
#pragma unroll
    for (int q = 0; q < kSelUnroll; q++) {
      const int64_t p = c0 + q * kPrThreads + t;
      v[q] = p < e ? vals[p] : VT(NAN);
    }
  }
}

template <int CAP, typename VT>
__global__ __launch_bounds__(kPrThreads) void k_prune_top(const int64_t *__restrict__ colptr,
                                                          const int32_t *__restrict__ rowidx,
                                                          const VT *__restrict__ vals, int64_t ncols, VT thr,
                                                          int64_t nnz, int k, int64_t *__restrict__ cnt,
                                                          uint64_t *__restrict__ cutv, int32_t *__restrict__ stage,
                                                          int32_t *status) {
  using KT = typename TopKey<VT>::T;
  constexpr int E = CAP / kPrThreads;      // list entries per thread
  constexpr int kLimit = CAP - kTopStep;   // a step fits on top of this many
  constexpr int KE = kTopMaxK / kPrThreads;
  static_assert(CAP % kPrThreads == 0 && kLimit >= 512, "a whole step fits the list");
  union Lds {
    struct {
      KT key[CAP];
      int32_t pos[CAP];
    } list;
    RankLds<kTopMaxK, int32_t> rank;
  };
  __shared__ Lds s;
  __shared__ int s_hist[kKthWords];
  __shared__ uint32_t s_red[4 * kPrWaves];
  __shared__ int s_add[3];  // entries appended by the steps t, t + 1, t + 2 (mod 3)
  __shared__ int s_n;
  const int t = threadIdx.x, l = lane();
  for (int64_t j = blockIdx.x; j < ncols; j += gridDim.x) {
    int64_t b = colptr[j], e = colptr[j + 1];
    if (b < 0 || e < b || e > nnz) {  // pointers outside the arrays: the column counts as empty
      if (t == 0) flag_error(status, 5);
      b = e = 0;
    }
    if (t < 3) s_add[t] = 0;
    __syncthreads();  // also: the previous column's LDS is free
    VT lo = thr;
    int n = 0;        // list length (uniform)
    bool left = false;
    int step = 0;
    VT nv[kSelUnroll];
    top_load(vals, b, e, t, nv);
    for (int64_t c0 = b; c0 < e; c0 += kTopStep, step = step == 2 ? 0 : step + 1) {
      // the next step's values are loaded before this one's are worked on
      VT v[kSelUnroll];
#pragma unroll
      for (int q = 0; q < kSelUnroll; q++) v[q] = nv[q];
      if (c0 + kTopStep < e) top_load(vals, c0 + kTopStep, e, t, nv);
      if (c0 == b && k <= kPrThreads && e - b > kTopStep) {
        // A first bound from the first step: the k-th largest of the threads'
        // largest values has k entries at or above it.  (The list then holds
        // little more than k entries after the step, not all of its 2048.)
        KT mk[1] = {0};
        bool has = false;
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          if (v[q] >= lo) {
            const KT key = (KT)order_key(v[q]);
            mk[0] = has && mk[0] > key ? mk[0] : key;
            has = true;
          }
        }
        if (__syncthreads_count(has ? 1 : 0) >= k) {  // uniform
          int above, equal;
          const KT kth = block_kth<false, 1>(mk, has ? 1u : 0u, k, (k + kPrThreads) / 2, s_hist, above, equal);
          const KT least = (KT)order_key(VT(-INFINITY));
          const VT edge = key_value(kth < least ? least : kth);
          lo = edge > lo ? edge : lo;
        }
      }
      // the counter of the next step was last read before the previous barrier
      if (t == 0) s_add[step == 2 ? 0 : step + 1] = 0;
      uint64_t any = 0;
#pragma unroll
      for (int q = 0; q < kSelUnroll; q++) any |= __ballot(v[q] >= lo);
      if (any) {  // uniform
#pragma unroll
        for (int q = 0; q < kSelUnroll; q++) {
          const bool in = v[q] >= lo;
          const uint64_t m = __ballot(in);
          if (m == 0) continue;
          int at = 0;
          if (l == 0) at = atomicAdd(&s_add[step], __popcll(m));
          at = n + readlane(at, 0) + mbcnt(m);
          if (in) {  // at < n + kTopStep <= CAP
            s.list.key[at] = (KT)order_key(v[q]);
            s.list.pos[at] = (int32_t)(c0 - b) + q * kPrThreads + t;
          }
        }
      }
      __syncthreads();
      n += s_add[step];
      if (n > kLimit) {  // uniform: raise the bound (n > kLimit >= k)
        KT key[E];
        int32_t pos[E];
        uint32_t have = 0;
#pragma unroll
        for (int i = 0; i < E; i++) {
          const int x = t + i * kPrThreads;
          key[i] = 0;
          pos[i] = 0;
          if (x < n) {
            key[i] = s.list.key[x];
            pos[i] = s.list.pos[x];
            have |= 1u << i;
          }
        }
        int above, equal;
        // (the lower edge of the k-th largest key's bucket will do, unless
        // the bucket is crowded; no value is below -infinity)
        KT kth = block_kth<false, E>(key, have, k, (k + kLimit) / 2, s_hist, above, equal);
        const KT least = (KT)order_key(VT(-INFINITY));
        kth = kth < least ? least : kth;
        if (t == 0) s_n = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < E; i++) {
          const bool in = ((have >> i) & 1u) && key[i] >= kth;
          const uint64_t m = __ballot(in);
          if (m == 0) continue;
          int at = 0;
          if (l == 0) at = atomicAdd(&s_n, __popcll(m));
          at = readlane(at, 0) + mbcnt(m);
          if (in) {
            s.list.key[at] = key[i];
            s.list.pos[at] = pos[i];
          }
        }
        n = above + equal;
        lo = key_value(kth);
        left = n > kLimit;
        __syncthreads();
        if (left) break;  // uniform
      }
    }
    int kept = n;
    if (!left && n > 0) {
      // the list holds every candidate, or at least the k largest
      KT key[E];
      int32_t pos[E];
      uint32_t have = 0;
#pragma unroll
      for (int i = 0; i < E; i++) {
        const int x = t + i * kPrThreads;
        key[i] = 0;
        pos[i] = 0;
        if (x < n) {
          key[i] = s.list.key[x];
          pos[i] = s.list.pos[x];
          have |= 1u << i;
        }
      }
      if (n > k) {
        int above, equal;
        const KT kth = block_kth<false, E>(key, have, k, k, s_hist, above, equal);
        uint32_t keep = 0, tie = 0;
#pragma unroll
        for (int i = 0; i < E; i++) {
          if (!((have >> i) & 1u)) continue;
          if (key[i] >= kth) {
            // exactly k at or above the edge, or kth is the k-th largest key
            if (above + equal == k || key[i] > kth) keep |= 1u << i;
            else tie |= 1u << i;
          }
        }
        if (above + equal > k) {  // uniform: among equal values the smaller rows
          uint32_t rk[E];
#pragma unroll
          for (int i = 0; i < E; i++) rk[i] = (tie >> i) & 1u ? row_key(rowidx[b + pos[i]]) : 0u;
          int ra, re;
          const uint32_t rth = block_kth<true, E>(rk, tie, k - above, k - above, s_hist, ra, re);
#pragma unroll
          for (int i = 0; i < E; i++)
            if (((tie >> i) & 1u) && rk[i] < rth) tie &= ~(1u << i);
          left = above + ra + re != k;  // a row twice: the kernels that follow report it and keep the first k
        }
        have = keep | tie;
        kept = k;
      }
      if (!left) {  // uniform
        // the kept positions, one list again, in input order
        if (t == 0) s_n = 0;
        __syncthreads();  // also: the list is in registers
#pragma unroll
        for (int i = 0; i < E; i++) {
          const bool in = (have >> i) & 1u;
          const uint64_t m = __ballot(in);
          if (m == 0) continue;
          int at = 0;
          if (l == 0) at = atomicAdd(&s_n, __popcll(m));
          at = readlane(at, 0) + mbcnt(m);
          if (in) s.list.pos[at] = pos[i];
        }
        __syncthreads();
        int32_t row[KE];
        int rank[KE];
#pragma unroll
        for (int i = 0; i < KE; i++) row[i] = t + i * kPrThreads < kept ? s.list.pos[t + i * kPrThreads] : 0;
        __syncthreads();
        rank_rows<kPrThreads, KE, Ties::kNone>(row, kept, t, s.rank, s_red, rank);
        int32_t *dst = stage + j * (int64_t)k;
#pragma unroll
        for (int i = 0; i < KE; i++)
          if (t + i * kPrThreads < kept) dst[rank[i]] = row[i];
      }
    }
    if (t == 0) {
      cnt[j] = left ? 0 : kept;
      cutv[j] = left ? kTopLeft : kTopDone;
    }
    __syncthreads();  // s_add is reset for the next column
  }
}

// The staged positions of the columns that k_prune_top settled, moved to the
// columns' places in the output (one wave per column) ...
__global__ __launch_bounds__(kPrThreads) void k_prune_place(const int64_t *__restrict__ out_colptr, int64_t ncols,
                                                            int64_t k, const uint64_t *__restrict__ cutv,
                                                            const int32_t *__restrict__ stage,
                                                            int32_t *__restrict__ out_rowidx) {
  for (int64_t j = (int64_t)blockIdx.x * kPrWaves + threadIdx.x / kWave; j < ncols; j += (int64_t)gridDim.x * kPrWaves) {
    if (cutv[j] != kTopDone) continue;
    const int64_t o = out_colptr[j], n = out_colptr[j + 1] - o;
    for (int64_t i = lane(); i < n; i += kWave) out_rowidx[o + i] = stage[j * k + i];
  }
}

// ... and replaced by the entries they name (the stage, which shares its
// memory with out_vals, is no longer needed).
template <typename VT>
__global__ __launch_bounds__(kPrThreads) void k_prune_take(const int64_t *__restrict__ colptr,
                                                           const int32_t *__restrict__ rowidx,
                                                           const VT *__restrict__ vals, int64_t ncols,
                                                           const uint64_t *__restrict__ cutv,
                                                           const int64_t *__restrict__ out_colptr,
                                                           int32_t *__restrict__ out_rowidx,
                                                           VT *__restrict__ out_vals) {
  for (int64_t j = (int64_t)blockIdx.x * kPrWaves + threadIdx.x / kWave; j < ncols; j += (int64_t)gridDim.x * kPrWaves) {
    if (cutv[j] != kTopDone) continue;
    const int64_t b = colptr[j], o = out_colptr[j], n = out_colptr[j + 1] - o;
    for (int64_t i = lane(); i < n; i += kWave) {
      const int64_t p = b + out_rowidx[o + i];
      out_rowidx[o + i] = rowidx[p];
      out_vals[o + i] = vals[p];
    }
  }
}

// The smallest value of type VT that a candidate can have.
inline double threshold_of(double thr, double) { return thr; }
inline float threshold_of(double thr, float) {
  const float f = (float)thr;
  return (double)f < thr ? std::nextafterf(f, INFINITY) : f;
}

// Whether columns are read by k_prune_top.  It stages k positions per column in
// out_values, which holds that many where columns hold k entries or more on
// average; three more launches (25 us) have to be won back, and a large k against
// the column means that the bound rises slowly and lists are sorted through.  Two
// kernels against it, us, uniform values:
//   float32, k = 10:  n x 100: 62 90 (n = 1000), 143 131 (10,000), 475 348 (50,000)
//                     n x 1200: 105 109 (4000), 204 192 (12,000); n x 1000: 113 119
//                     (5000), 289 264 (20,000)
//                     n x 3000: 78 83 (400), 96 83 (1500); n x 8000: 103 83 (4)
//   float64, k = 10:  n x 1200: 81 84 (400), 115 85 (1500); n x 2048: 100 83 (4)
//   float32, k / length 1/16, 1/10, 1/8 at 4000 x 5000: 200 171, 200 191, 201 204;
//                     k = 100, 256, 600 at 20,000 x 1000: 283 283, 287 298, 282 328
// (Values of few kinds, whose ties have to be broken by row, can take up to 1.2
// times as long as by the two kernels, in short float64 columns 1.4.)
inline bool read_once(int vbytes, int64_t nnz, int64_t n, int64_t k) {
  const int64_t mean = nnz / n;
  if (k < 1 || k > mean || k > kTopMaxK - kTopMaxK / 16) return false;
  if (k > (mean >= 2048 ? mean / 16 : 256)) return false;
  if (vbytes == 8) return mean >= 2048 || n >= 8192 || nnz >= (1 << 20);
  if (mean >= 8192) return true;
  if (mean >= 2048) return nnz >= (1 << 22);
  return mean < 512 ? n >= 8192 : nnz >= (1 << 24);
}

template <typename VT>
int prune_typed(const spgemm_csc *C, double thr, int64_t k, int64_t *out_colptr, int32_t *out_rowidx,
                void *out_values, const WsLayout &L, char *ws, hipStream_t st) {
  WsHeader *hdr = (WsHeader *)ws;
  int rc = launch_init_header(hdr, (uint64_t)0, st);
  if (rc) return rc;
  const int64_t n = C->ncols;
  int64_t *cnt = (int64_t *)(ws + L.pr_cnt);
  uint64_t *cutv = (uint64_t *)(ws + L.pr_cutv);
  uint32_t *cutr = (uint32_t *)(ws + L.pr_cutr);
  const unsigned grid = (unsigned)(n < kPrMaxGrid ? n : kPrMaxGrid);
  const bool top = n > 0 && read_once((int)sizeof(VT), C->nnz, n, k);
  int32_t *stage = (int32_t *)out_values;
  if (top) {
    ProfScope prof("prune_select", st);
    const VT t = threshold_of(thr, VT(0));
    if (3 * k <= 2 * (2560 - kTopStep))  // the list can grow by half before the bound rises
      hipLaunchKernelGGL((k_prune_top<2560, VT>), dim3(grid), dim3(kPrThreads), 0, st, C->colptr, C->rowidx,
                         (const VT *)C->values, n, t, C->nnz, (int)k, cnt, cutv, stage, &hdr->status);
    else
      hipLaunchKernelGGL((k_prune_top<3072, VT>), dim3(grid), dim3(kPrThreads), 0, st, C->colptr, C->rowidx,
                         (const VT *)C->values, n, t, C->nnz, (int)k, cnt, cutv, stage, &hdr->status);
    LAUNCHCHK();
  }
  if (n > 0) {
    ProfScope prof("prune_select", st);
    if (top)
      hipLaunchKernelGGL((k_prune_select<true, VT>), dim3(std::min(grid, 4096u)), dim3(kPrThreads), 0, st, C->colptr,
                         C->rowidx, (const VT *)C->values, n, thr, C->nnz, k, cnt, cutv, cutr, &hdr->status);
    else
      hipLaunchKernelGGL((k_prune_select<false, VT>), dim3(grid), dim3(kPrThreads), 0, st, C->colptr, C->rowidx,
                         (const VT *)C->values, n, thr, C->nnz, k, cnt, cutv, cutr, &hdr->status);
    LAUNCHCHK();
  }
  rc = launch_colptr_scan(cnt, n, out_colptr, (int64_t *)(ws + L.scan), st);
  if (rc || n == 0) return rc;
  if (top) {
    ProfScope prof("prune_fill", st);
    const unsigned gw = std::min(grid_of(n, kPrWaves), 8u * (unsigned)device_cus());
    hipLaunchKernelGGL(k_prune_place, dim3(gw), dim3(kPrThreads), 0, st, (const int64_t *)out_colptr, n, k,
                       (const uint64_t *)cutv, (const int32_t *)stage, out_rowidx);
    LAUNCHCHK();
    hipLaunchKernelGGL(k_prune_take<VT>, dim3(gw), dim3(kPrThreads), 0, st, C->colptr, C->rowidx,
                       (const VT *)C->values, n, (const uint64_t *)cutv, (const int64_t *)out_colptr, out_rowidx,
                       (VT *)out_values);
    LAUNCHCHK();
  }
  ProfScope prof("prune_fill", st);
  if (top)
    hipLaunchKernelGGL((k_prune_fill<true, VT>), dim3(std::min(grid, 4096u)), dim3(kPrThreads), 0, st, C->colptr,
                       C->rowidx, (const VT *)C->values, n, C->nnz, thr, (const uint64_t *)cutv, (const uint32_t *)cutr,
                       (const int64_t *)out_colptr, out_rowidx, (VT *)out_values, &hdr->status);
  else
    hipLaunchKernelGGL((k_prune_fill<false, VT>), dim3(grid), dim3(kPrThreads), 0, st, C->colptr, C->rowidx,
                       (const VT *)C->values, n, C->nnz, thr, (const uint64_t *)cutv, (const uint32_t *)cutr,
                       (const int64_t *)out_colptr, out_rowidx, (VT *)out_values, &hdr->status);
  LAUNCHCHK();
  return SPGEMM_OK;
}

}  // namespace
}  // namespace spg

using namespace spg;

extern "C" {

int spgemm_prune_topk(const spgemm_csc *C, double threshold, int64_t k, int64_t *out_colptr, int32_t *out_rowidx,
                      void *out_values, int64_t out_cap, void *ws, size_t ws_bytes, void *stream) {
  int st = check_csc(C, true);
  if (st) return st;
  if (!out_colptr || out_cap < 0) return SPGEMM_E_INVAL;
  // the output never holds more than min(nnz, k * ncols) entries
  int64_t bound = C->nnz;
  if (k >= 0 && (C->ncols == 0 || k <= bound / C->ncols) && k * C->ncols < bound) bound = k * C->ncols;
  if (out_cap < bound) return SPGEMM_E_INVAL;
  if (bound > 0 && (!out_rowidx || !out_values)) return SPGEMM_E_INVAL;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_PRUNE, C, nullptr, 0, 0, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  if (C->dtype == SPGEMM_F32)
    return prune_typed<float>(C, threshold, k, out_colptr, out_rowidx, out_values, L, (char *)ws, s);
  return prune_typed<double>(C, threshold, k, out_colptr, out_rowidx, out_values, L, (char *)ws, s);
}

}  // extern "C"
