// Sorted positions of the rows of one short column, in LDS: the rows are
// distributed over about as many buckets as entries by the high bits of their
// distance to the smallest row, the bucket counts are scanned, and each entry
// ranks itself among its bucket's entries.  A bitonic network over n entries
// takes log2(n) (log2(n) + 1) / 2 dependent exchange steps (78 at 4096), each
// with a barrier between the waves of a workgroup; this takes a handful of
// LDS accesses per entry and a fixed number of barriers.  Rows that crowd into
// few buckets (more than kRankCrowd entries in one) are ranked by a bitonic
// sort of (row, entry number) instead, so no input costs more than that.
//
// Equal rows are ordered by entry number (a stable sort).  Where none are
// expected (Ties::kRare) an entry is ranked without its number, and columns
// found to hold a row twice are ranked by the bitonic sort: keeping the numbers
// costs 2.4 of 196 us of a captured product of 64 instances and its sort.
#pragma once

#include "device.hpp"

namespace spg {

constexpr int kRankCrowd = 64;

// Equal rows in a column: usual, rare, or none (equal rows would get one rank).
enum class Ties { kUsual, kRare, kNone };

// Largest value over the wave (unsigned).
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
  v = max(v, (uint32_t)dpp0<0x111>((int)v));
  v = max(v, (uint32_t)dpp0<0x112>((int)v));
  v = max(v, (uint32_t)dpp0<0x114>((int)v));
  v = max(v, (uint32_t)dpp0<0x118>((int)v));
  v = max(v, (uint32_t)dpp0<0x142, 0xa>((int)v));
  v = max(v, (uint32_t)dpp0<0x143, 0xc>((int)v));
  return (uint32_t)readlane((int)v, kWave - 1);
}

// Power of two at least n and at least 64.
__device__ __forceinline__ int log2_ceil64(int n) { return max(6, 32 - __clz(max(n, 1) - 1)); }

// Shift that maps [0, range] onto fewer than 2^log_nb buckets.
__device__ __forceinline__ int bucket_shift(uint32_t range, int log_nb) { return max(0, 32 - __clz((int)range) - log_nb); }

// LDS of one column of up to N entries: rows (and, for the caller, values of
// type VT) in sorted order at the end, bucketed rows in between.
template <int N, class VT>
struct RankLds {
  union {
    struct {
      VT val[N];      // the caller's, free during the ranking
      int32_t key[N];
    } s;
    uint64_t comp[N];  // crowded buckets: row << 16 | entry number
  } u;
  int cnt[N + 1];
  uint16_t ord[N];
};

// Bitonic sort of comp[0, n2), ascending, by THREADS threads (a wave if 64).
template <int THREADS>
__device__ __forceinline__ void bitonic_u64(uint64_t *comp, int n2, int t) {
  const auto sync = [] {
    if constexpr (THREADS == kWave)
      wave_sync();
    else
      __syncthreads();
  };
  for (int k = 2; k <= n2; k <<= 1) {
    for (int s = k >> 1; s > 0; s >>= 1) {
      for (int i = t; i < n2 / 2; i += THREADS) {
        const int a = ((i & ~(s - 1)) << 1) | (i & (s - 1));  // lower element of pair i at distance s
        const uint64_t x = comp[a], y = comp[a + s];
        if ((x > y) == ((a & k) == 0)) {
          comp[a] = y;
          comp[a + s] = x;
        }
      }
      sync();
    }
  }
}

// Ranks the n <= N entries held by THREADS threads (entry t + e * THREADS in
// row[e] of thread t): rank[e] is the entry's sorted position.  s_red: 4 *
// THREADS / 64 words of LDS (unused by a single wave).  All threads call it
// (a wave: THREADS = 64); LDS contents written before must be past a barrier.
// On return every thread has its ranks and the LDS may be rewritten.
template <int THREADS, int E, Ties TIES, int N, class VT>
__device__ __forceinline__ void rank_rows(const int32_t (&row)[E], int n, int t, RankLds<N, VT> &L, uint32_t *s_red,
                                          int (&rank)[E]) {
  static_assert(N == THREADS * E, "one register per entry");
  constexpr int NW = THREADS / kWave;
  constexpr bool kOne = NW == 1;
  const int l = lane(), w = t / kWave;
  const auto sync = [] {
    if constexpr (kOne)
      wave_sync();
    else
      __syncthreads();
  };
  uint32_t hi = 0, nlo = 0;
#pragma unroll
  for (int e = 0; e < E; e++)
    if (t + e * THREADS < n) {
      hi = max(hi, (uint32_t)row[e]);
      nlo = max(nlo, ~(uint32_t)row[e]);
    }
  hi = wave_umax(hi);
  nlo = wave_umax(nlo);
  const int log_nb = min(log2_ceil64(n), 31 - __clz(N));
  const int nb = 1 << log_nb;
  for (int i = t; i < nb; i += THREADS) L.cnt[i] = 0;
  if constexpr (!kOne) {
    if (l == 0) {
      s_red[w] = hi;
      s_red[NW + w] = nlo;
    }
  }
  sync();
  if constexpr (!kOne) {
#pragma unroll
    for (int z = 0; z < NW; z++) {
      hi = max(hi, s_red[z]);
      nlo = max(nlo, s_red[NW + z]);
    }
  }
  const uint32_t lo = ~nlo;
  const int sh = bucket_shift(hi - lo, log_nb);
  int old[E];
#pragma unroll
  for (int e = 0; e < E; e++) {
    old[e] = 0;
    if (t + e * THREADS < n) old[e] = atomicAdd(&L.cnt[((uint32_t)row[e] - lo) >> sh], 1);
  }
  sync();
  // exclusive scan of the counts: wave w takes its share of the buckets, 64 at
  // a time; then the waves' totals are added
  const int per = nb / NW < kWave ? kWave : nb / NW;
  int run = 0, big = 0;
  for (int i = w * per; i < min((w + 1) * per, nb); i += kWave) {
    const int v = L.cnt[i + l];
    const int incl = wave_incl_add(v);
    L.cnt[i + l] = run + incl - v;
    run += readlane(incl, kWave - 1);
    big = max(big, v);
  }
  big = (int)wave_umax((uint32_t)big);
  if constexpr (kOne) {
    if (t == 0) L.cnt[nb] = n;
  } else {
    if (l == 0) {
      s_red[2 * NW + w] = (uint32_t)run;
      s_red[3 * NW + w] = (uint32_t)big;
    }
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int z = 0; z < NW; z++) {
      if (z < w) before += (int)s_red[2 * NW + z];
      big = max(big, (int)s_red[3 * NW + z]);
    }
    for (int i = w * per; i < min((w + 1) * per, nb); i += kWave) L.cnt[i + l] += before;
    if (t == 0) L.cnt[nb] = n;
  }
  sync();
  bool by_number = big > kRankCrowd;  // uniform
  if (!by_number) {
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int i = t + e * THREADS;
      if (i < n) {
        const int p = L.cnt[((uint32_t)row[e] - lo) >> sh] + old[e];
        L.u.s.key[p] = row[e];
        if (TIES == Ties::kUsual) L.ord[p] = (uint16_t)i;
      }
    }
    sync();
    bool twice = false;
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int i = t + e * THREADS;
      rank[e] = 0;
      if (i < n) {
        const uint32_t b = ((uint32_t)row[e] - lo) >> sh;
        const int c0 = L.cnt[b], c1 = L.cnt[b + 1];
        int r = c0;
        if (c1 - c0 > 1) {
          int same = 0;
          for (int q = c0; q < c1; q++) {
            const uint32_t k = (uint32_t)L.u.s.key[q];
            r += k < (uint32_t)row[e] || (TIES == Ties::kUsual && k == (uint32_t)row[e] && L.ord[q] < i) ? 1 : 0;
            if (TIES == Ties::kRare) same += k == (uint32_t)row[e] ? 1 : 0;
          }
          twice |= same > 1;
        }
        rank[e] = r;
      }
    }
    if constexpr (TIES == Ties::kRare) {
      if constexpr (kOne)
        by_number = __ballot(twice) != 0;
      else
        by_number = __syncthreads_or(twice ? 1 : 0) != 0;
    }
  }
  if (by_number) {  // uniform
    sync();  // the ranking above has read the keys
    const int n2 = 1 << log2_ceil64(n);
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int i = t + e * THREADS;
      if (i < n2) L.u.comp[i] = i < n ? ((uint64_t)(uint32_t)row[e] << 16) | (uint64_t)i : ~0ull;
    }
    sync();
    bitonic_u64<THREADS>(L.u.comp, n2, t);
    for (int i = t; i < n; i += THREADS) L.ord[(uint16_t)L.u.comp[i]] = (uint16_t)i;
    sync();
#pragma unroll
    for (int e = 0; e < E; e++) {
      const int i = t + e * THREADS;
      rank[e] = i < n ? (int)L.ord[i] : 0;
    }
  }
  sync();
}

}  // namespace spg
