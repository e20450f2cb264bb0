// Kernels for the gradient of C = A*B with respect to the stored values of A
// and B, for a loss defined on the pattern of C (not part of the paper; the
// product itself follows Gustavson's column formula, Sec. II-C).
//
//   dB(k,j) = sum over i in A(:,k) of A(i,k) * dC(i,j),   (k,j) in P(B)
//   dA(i,k) = sum over j in B(k,:) of dC(i,j) * B(k,j),   (i,k) in P(A)
//
// Both are masked products out = (X^T Y) restricted to a pattern M:
//   dB  = masked_xty(X = A,   Y = dC,   M = P(B))
//   dA^T = masked_xty(X = B^T, Y = dC^T, M = P(A^T))
// Every dC(i,j) they need lies in P(C), so no term is lost by the mask.
// For each output column j the kernel loads Y(:,j) into an LDS hash table
// (row -> value) and forms one dot product per requested entry (k,j) of M
// against X(:,k); the work equals the forward flops plus nnz(Y).
//
// The transposes are sort-free: a row histogram that also ranks the entries of
// a row, a scan, and a scatter (entry order inside each output column is
// arbitrary).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "device.hpp"
#include "hip_host.hpp"
#include "internal.hpp"
#include "lds_hash.hpp"
#include "profile.hpp"

namespace spg {

// ============================================================================
// Transpose
// ============================================================================
__global__ void k_tr_zero(unsigned long long *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// Row counts and, with RANK, each entry's place among its row's entries (as
// counted).
template <bool RANK>
__global__ __launch_bounds__(256) void k_tr_count(const int32_t *ri, int64_t nnz, int64_t m, unsigned long long *cnt,
                                                  int32_t *rank, int32_t *status) {
  constexpr int U = 4;  // entries a thread has in flight
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p0 < nnz; p0 += U * step) {
    int32_t r_[U];
    unsigned long long c_[U];
#pragma unroll
    for (int u = 0; u < U; u++) r_[u] = p0 + u * step < nnz ? ri[p0 + u * step] : 0;
#pragma unroll
    for (int u = 0; u < U; u++) {
      c_[u] = 0;
      if (p0 + u * step < nnz) {
        const int32_t r = opaque(r_[u]);
        if ((uint32_t)r < (uint32_t)m) {
          if constexpr (RANK)
            c_[u] = atomicAdd(&cnt[r], 1ull);
          else
            atomicAdd(&cnt[r], 1ull);
        } else {
          flag_error(status, 3);
        }
      }
    }
    if constexpr (RANK) {
#pragma unroll
      for (int u = 0; u < U; u++)
        if (p0 + u * step < nnz) rank[p0 + u * step] = (int32_t)c_[u];
    }
  }
}

// The last column in [lo, hi) that starts at or before p (cp[lo] <= p < cp[hi]),
// found by a whole wave, 64 probes a step.
__device__ __forceinline__ int64_t column_of(const int64_t *cp, int64_t lo, int64_t hi, int64_t p) {
  while (hi - lo > 1) {
    const int64_t d = (hi - lo + kWave - 1) / kWave;
    const int64_t j = min(lo + (int64_t)lane() * d, hi);
    const uint64_t le = __ballot(j < hi && cp[j] <= p);  // lane 0 always
    const int c = 63 - __clzll((long long)le);
    const int64_t nlo = lo + (int64_t)c * d;
    hi = min(hi, nlo + d);
    lo = nlo;
  }
  return lo;
}

// Entries in tiles of kTrTile consecutive ones, whatever the columns' lengths:
// the tile's columns mark where they start in LDS, a prefix maximum gives
// every entry its column, and an entry goes to its row's column pointer plus
// its rank.  Random atomics (23e9 a second) and random writes bound a
// transpose, so each entry pays for one of each: 1.0e7 entries, two per
// column: 1.87 ms with a wave per column and a second atomic, 0.81 now.
// A tile that spans more than kTrSpan columns, nearly all of them empty, has its
// entries look their columns up instead (a binary search each, kTrPer in
// flight): 4000 entries in 5,000,000 columns 12.1 ms -> 0.10, 1,000,000 entries in
// as many 149 -> 140 us; at 8000 columns a tile both take 48 us.
// The entries' places are formed first and each output is then written by
// itself: random writes to three arrays at a time (1.0e7 entries in columns of
// 10 or more, values and permutation both wanted) 1.25 ms, one at a time 1.18.
// (A second atomic in place of the rank takes 1.0 to 1.1 there in float32, but
// 1.4 in float64, and 1.4 against 0.8 where one of the two is wanted.)
constexpr int64_t kTrSpan = 8192;
constexpr int kTrPer = 16;
constexpr int kTrTile = 256 * kTrPer;
template <class VT>
__global__ __launch_bounds__(256) void k_tr_scatter(const int64_t *cp, const int32_t *ri, const VT *v, int64_t ncols,
                                                    int64_t m, int64_t nnz, const int64_t *t_colptr,
                                                    const int32_t *rank, int32_t *t_ri, VT *t_v, int64_t *perm) {
  __shared__ int s_own[kTrTile];
  __shared__ int s_w[4];
  const int t = threadIdx.x, l = lane(), w = t / kWave;
  const int64_t first = max(cp[0], (int64_t)0), end = min(cp[ncols], nnz);
  for (int64_t p0 = first + (int64_t)blockIdx.x * kTrTile; p0 < end; p0 += (int64_t)gridDim.x * kTrTile) {
    const int64_t p1 = min(end, p0 + kTrTile);
    const int64_t lo = column_of(cp, 0, ncols, p0);
    if (ncols - lo > kTrSpan && cp[lo + kTrSpan] < p1) {  // uniform
      // the entries' columns, each from lo up: cp[a] <= p < cp[b]
      const int64_t hi = column_of(cp, lo + kTrSpan, ncols, p1 - 1) + 1;
      int64_t a[kTrPer], b[kTrPer];
#pragma unroll
      for (int i = 0; i < kTrPer; i++) {
        a[i] = lo;
        b[i] = hi;
      }
      for (int64_t left = hi - lo; left > 1; left = (left + 1) / 2) {
        int64_t c[kTrPer];
#pragma unroll
        for (int i = 0; i < kTrPer; i++) c[i] = cp[(a[i] + b[i]) / 2];
#pragma unroll
        for (int i = 0; i < kTrPer; i++) {
          const int64_t mid = (a[i] + b[i]) / 2;
          if (c[i] <= p0 + t + i * 256)
            a[i] = mid;
          else
            b[i] = mid;
        }
      }
#pragma unroll
      for (int i = 0; i < kTrPer; i++) s_own[t + i * 256] = (int)(a[i] - lo);
    } else {
#pragma unroll
      for (int i = 0; i < kTrPer; i++) s_own[t + i * 256] = 0;
      __syncthreads();
      for (int64_t j0 = lo + 1;; j0 += 256) {
        const int64_t j = j0 + t;
        const int64_t c = j < ncols ? cp[j] : p1;
        if (c > p0 && c < p1) atomicMax(&s_own[c - p0], (int)(j - lo));
        if (!__syncthreads_or(t == 255 && c < p1)) break;
      }
      // prefix maximum, kTrPer consecutive entries per thread
      int x[kTrPer], top = 0;
#pragma unroll
      for (int i = 0; i < kTrPer; i++) {
        top = max(top, s_own[t * kTrPer + i]);
        x[i] = top;
      }
      const int incl = wave_incl_max(top);
      if (l == kWave - 1) s_w[w] = incl;
      __syncthreads();
      int before = wave_prev(incl);
#pragma unroll
      for (int z = 0; z < 4; z++)
        if (z < w) before = max(before, s_w[z]);
#pragma unroll
      for (int i = 0; i < kTrPer; i++) s_own[t * kTrPer + i] = max(x[i], before);
      __syncthreads();
    }
    int64_t pos[kTrPer];
#pragma unroll
    for (int i = 0; i < kTrPer; i++) {
      const int64_t p = p0 + t + i * 256;
      pos[i] = -1;
      if (p < p1) {
        const int32_t r = ri[p];
        if ((uint32_t)r < (uint32_t)m) pos[i] = t_colptr[r] + rank[p];  // (counted as an error otherwise)
      }
    }
#pragma unroll
    for (int i = 0; i < kTrPer; i++)
      if (pos[i] >= 0) t_ri[pos[i]] = (int32_t)(lo + s_own[t + i * 256]);
    if (t_v) {
#pragma unroll
      for (int i = 0; i < kTrPer; i++)
        if (pos[i] >= 0) t_v[pos[i]] = v[p0 + t + i * 256];
    }
    if (perm) {
#pragma unroll
      for (int i = 0; i < kTrPer; i++)
        if (pos[i] >= 0) perm[pos[i]] = p0 + t + i * 256;
    }
    __syncthreads();  // the next tile clears s_own
  }
}

// ============================================================================
// Permute
// ============================================================================
template <class T>
__global__ void k_permute(const T *src, const int64_t *perm, int64_t n, T *dst, int scatter) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = perm[i];
    if ((uint64_t)q >= (uint64_t)n) continue;
    if (scatter)
      dst[q] = src[i];
    else
      dst[i] = src[q];
  }
}

// ============================================================================
// Masked X^T Y
// ============================================================================
// Operands of a masked product out = (X^T Y) on the pattern of M, and of the
// fused backward (X = A, Y = dC, M = B), which also adds M(k,j) Y(i,j) to
// acc at X(i,k).
template <class VT>
struct DotArgs {
  const int64_t *Xcp;
  const int32_t *Xri;
  const VT *Xv;
  const int64_t *Ycp;
  const int32_t *Yri;
  const VT *Yv;
  const int64_t *Mcp;
  const int32_t *Mri;
  const VT *Mv;  // fused backward only
  VT *out;
  double *acc;  // fused backward only: one float64 per entry of X
  int64_t m, kdim, nnzX;
};

// Binning by nnz(Y(:,j)) with the numeric bins' capacities; columns of M
// with no entry need no work.  Columns that fill at most half of what bins 2
// and 3 hold take tables of half the slots (two more lists): LDS, and with it
// the waves in flight, is what bounds these kernels.
// heavy_code: the status of a column above the largest table (0: none, the
// caller forms those itself).
__global__ __launch_bounds__(256) void k_mxty_bin(const int64_t *Ycp, const int64_t *Mcp, int64_t ncol, int min_bin,
                                                  BinCaps caps, int32_t *bins, WsHeader *hdr, int heavy_code,
                                                  int halves) {
  constexpr int NL = kNumBins + 2;
  __shared__ int s_cnt[NL];
  __shared__ int s_base[NL];
  __shared__ int s_bin[256];
  __shared__ int s_pos[256];
  const int t = threadIdx.x;
  if (t < NL) s_cnt[t] = 0;
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * 256 + t;
  int bin = -1;
  if (j < ncol && Mcp[j + 1] > Mcp[j]) {
    const int64_t u = Ycp[j + 1] - Ycp[j];
    bin = kNumBins - 1;
#pragma unroll
    for (int b = kNumBins - 2; b >= 0; b--)
      if (u <= caps.cap[b]) bin = b;
    bin = max(bin, min_bin);
    if (bin == kNumBins - 1 && heavy_code) flag_error(&hdr->status, heavy_code);
    // half tables: listed from the end of their bin's array
    if ((bin == 2 || bin == 3) && (halves >> (bin - 2)) & 1 && 2 * u <= kNumTableCap[bin]) bin += kNumBins - 2;
  }
  s_bin[t] = bin;
  s_pos[t] = bin >= 0 ? atomicAdd(&s_cnt[bin], 1) : 0;
  __syncthreads();
  if (t < NL)
    s_base[t] = s_cnt[t] ? atomicAdd(t < kNumBins ? &hdr->bin_count[t] : &hdr->half_count[t - kNumBins], s_cnt[t]) : 0;
  __syncthreads();
  if (bin >= 0) {
    const int64_t p = s_base[bin] + s_pos[t];
    bins[bin < kNumBins ? (int64_t)bin * ncol + p : (int64_t)(bin - kNumBins + 3) * ncol - 1 - p] = (int32_t)j;
  }
}

constexpr int kLongDot = 64;
constexpr int kDotPipe = 4;  // rounds whose gathers are in flight together
constexpr int kDotIns = 4;   // entries of Y(:,j) a thread has in flight when the table is filled

// Scratch of one wave: the nonempty short segments (columns of X) of a chunk
// of up to 64 entries of M(:,j), flattened into rounds of 64 products.
struct DotScratch {
  uint64_t rmask[kWave];  // one bit per product of a round that starts a segment
  struct {
    int64_t off;   // first X entry of the segment minus its exclusive prefix
    double scale;  // M(k,j) (fused backward)
  } seg[kWave];
  double db[kWave];  // the segment's dot product, summed by LDS atomics
};

// Entries a wave takes at once when nw waves share a column of n entries: 64,
// or fewer where that would leave waves without any.
__device__ __forceinline__ int chunk_width(int64_t n, int nw) {
  return (int)max((int64_t)1, min((int64_t)kWave, (n + nw - 1) / nw));
}

template <int CTRL>
__device__ __forceinline__ double dpp_quad(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)dpp0<CTRL>((int)(uint32_t)b), hi = (uint32_t)dpp0<CTRL>((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sums t over lanes of a pair, then a quad, that share an owner (own < 0: no
// product); returns whether this lane holds a sum to be added.  A segment's
// products sit in consecutive lanes, and LDS atomics of many lanes on one
// address are served one after another.  Called by the whole wave.
__device__ __forceinline__ bool quad_sum(int own, double &t) {
  const int l = lane();
  const int o1 = dpp0<0xB1>(own);  // quad_perm [1,0,3,2]
  const bool pair = o1 == own;
  const double t1 = dpp_quad<0xB1>(t);
  if (pair) t += t1;
  const int c = pair ? own : -2 - l;  // pairs that are not uniform match nothing
  const int c2 = dpp0<0x4E>(c);  // quad_perm [2,3,0,1]; every lane active
  const double t2 = dpp_quad<0x4E>(t);
  const bool quad = pair && c2 == c;
  if (quad) t += t2;
  return own >= 0 && (quad ? (l & 3) == 0 : (!pair || (l & 1) == 0));
}

// A column and a wave's first chunk of its M entries, loaded ahead in
// dependent steps placed where the current column has other work: the
// pointers, the entries, X's column pointers.
template <class VT>
struct DotPre {
  int64_t y0, y1, m0, m1;
  int32_t k;
  VT mv;
  int64_t x0, x1;
};

template <class VT>
__device__ __forceinline__ void dot_pre_ptr(const DotArgs<VT> &a, int64_t j, DotPre<VT> &pre) {
  const int64_t z = opaque((int64_t)0);  // per-lane addresses: vector loads do not hold up LDS waits
  pre.y0 = ld_global(a.Ycp + j + z);
  pre.y1 = ld_global(a.Ycp + j + 1 + z);
  pre.m0 = ld_global(a.Mcp + j + z);
  pre.m1 = ld_global(a.Mcp + j + 1 + z);
}

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  return (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
         ((int64_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)v >> 32)) << 32);
}

template <bool FUSED, class VT>
__device__ __forceinline__ void dot_pre_m(const DotArgs<VT> &a, int w, int nw, DotPre<VT> &pre) {
  pre.y0 = uniform64(pre.y0);
  pre.y1 = uniform64(pre.y1);
  pre.m0 = uniform64(pre.m0);
  pre.m1 = uniform64(pre.m1);
  const int cw = chunk_width(pre.m1 - pre.m0, nw);
  const int64_t p = pre.m0 + (int64_t)w * cw + lane();
  pre.k = -1;
  pre.mv = VT(0);
  if (lane() < cw && p < pre.m1) {
    pre.k = a.Mri[p];
    if (FUSED) pre.mv = a.Mv[p];
  }
}

template <class VT>
__device__ __forceinline__ void dot_pre_x(const DotArgs<VT> &a, DotPre<VT> &pre) {
  pre.x0 = pre.x1 = 0;
  if ((uint32_t)pre.k < (uint32_t)a.kdim) {
    pre.x0 = a.Xcp[pre.k];
    pre.x1 = a.Xcp[pre.k + 1];
  }
}

// Entries [pb, end) of M(:,j) in chunks of chunk_width (chunk c by the wave
// with c % c_stride == c_rank): each entry's dot product of X(:,k) with
// Y(:,j), look(row) giving Y(row, j).  Columns of X shorter than kLongDot are
// flattened into rounds of 64 products, one per lane, so a column with few
// entries of M still fills the wave; one 64-bit word per round marks where
// segments start, so a product's owner is (segments starting before the
// round) + (starts in the round at or below it) - 1.  Sums are gathered by
// LDS atomics; FUSED products also add to acc (float64 global atomics).  Long
// columns are walked by the whole wave with a wave reduction.
// pre: the first chunk loaded ahead (or nullptr).
template <bool FUSED, class VT, class Look>
__device__ __forceinline__ void dot_entries(const DotArgs<VT> &a, int64_t pb, int64_t end, int c_rank, int c_stride,
                                            int32_t *status, DotScratch &sc, const DotPre<VT> *pre, Look &&look) {
  const int l = lane();
  const int cw = chunk_width(end - pb, c_stride);
  for (int64_t base = pb + (int64_t)c_rank * cw; base < end; base += (int64_t)c_stride * cw) {
    const int64_t p = base + l;
    const int64_t pe = min(end, base + cw);  // this chunk's entries
    const bool ahead = pre && base == pb + (int64_t)c_rank * cw;  // uniform
    int64_t x0 = 0, x1 = 0;
    double mkj = 0.0;
    if (p < pe) {
      const int32_t k = ahead ? pre->k : a.Mri[p];
      if ((uint32_t)k >= (uint32_t)a.kdim) {
        flag_error(status, 1);
      } else {
        x0 = ahead ? pre->x0 : a.Xcp[k];
        x1 = ahead ? pre->x1 : a.Xcp[k + 1];
        if (FUSED) mkj = (double)(ahead ? pre->mv : a.Mv[p]);
        if (x0 < 0 || x1 < x0 || x1 > a.nnzX) {
          flag_error(status, 5);
          x0 = x1 = 0;
        }
      }
    }
    const bool lg = x1 - x0 >= kLongDot;
    const int ls = lg ? 0 : (int)(x1 - x0);
    const int incl = wave_incl_add(ls);
    const int excl = incl - ls;
    const int total = readlane(incl, kWave - 1);
    const uint64_t nz = __ballot(ls > 0);
    const int ord = mbcnt(nz);
    if (ls > 0) {  // the nonempty short segments in lane order
      sc.seg[ord].off = x0 - excl;
      if (FUSED) sc.seg[ord].scale = mkj;
    }
    sc.db[l] = 0.0;
    sc.rmask[l] = 0ull;  // at most 64 segments of 63 products: 63 rounds
    wave_sync();
    if (ls > 0) atomicOr((unsigned long long *)&sc.rmask[excl >> 6], 1ull << (excl & 63));
    wave_sync();
    const int nround = (total + kWave - 1) / kWave;
    for (int r = 0; r < nround; r += kDotPipe) {
      int own_[kDotPipe];
      int64_t q_[kDotPipe];
      double sc_[kDotPipe];
#pragma unroll
      for (int u = 0; u < kDotPipe; u++) {
        own_[u] = -1;
        if (r + u < nround) {
          const int fb = (r + u) * kWave;
          const uint64_t mm = sc.rmask[r + u];
          const int carry = __popcll(__ballot(ls > 0 && excl < fb));
          if (fb + l < total) own_[u] = carry + mbcnt(mm) + (int)((mm >> l) & 1ull) - 1;
        }
      }
#pragma unroll
      for (int u = 0; u < kDotPipe; u++) {
        const int o = max(own_[u], 0);
        q_[u] = sc.seg[o].off + (r + u) * kWave + l;
        if (FUSED) sc_[u] = sc.seg[o].scale;
      }
      int32_t row_[kDotPipe];
      VT xv_[kDotPipe];
#pragma unroll
      for (int u = 0; u < kDotPipe; u++) {
        row_[u] = -1;
        xv_[u] = VT(0);
        if (own_[u] >= 0) {
          row_[u] = a.Xri[q_[u]];
          xv_[u] = a.Xv[q_[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < kDotPipe; u++) {
        if (r + u >= nround) break;  // uniform
        double t = 0.0;
        if (own_[u] >= 0) {
          const int32_t rt = opaque(row_[u]);
          if ((uint32_t)rt < (uint32_t)a.m) {
            const double g = look(rt);
            if (FUSED) atomicAdd(&a.acc[q_[u]], sc_[u] * g);
            t = (double)opaque(xv_[u]) * g;
          } else {
            flag_error(status, 3);
          }
        }
        if (quad_sum(own_[u], t)) atomicAdd(&sc.db[own_[u]], t);
      }
    }
    wave_sync();
    if (p < pe && !lg) a.out[p] = ls > 0 ? (VT)sc.db[ord] : VT(0);
    uint64_t lm = __ballot(lg);
    while (lm) {
      const int L = __builtin_ctzll(lm);
      lm &= lm - 1;
      const int64_t lx0 = readlane64(x0, L), lx1 = readlane64(x1, L);
      const double lb = FUSED ? readlane_f64(mkj, L) : 0.0;
      double s = 0.0;
      for (int64_t q0 = lx0 + l; q0 < lx1; q0 += 4 * kWave) {
        int32_t r[4];
        VT xv[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
          const int64_t q = q0 + t * kWave;
          r[t] = 0;
          xv[t] = VT(0);
          if (q < lx1) {
            r[t] = a.Xri[q];
            xv[t] = a.Xv[q];
          }
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
          if (q0 + t * kWave < lx1) {
            const int32_t rt = opaque(r[t]);
            if ((uint32_t)rt < (uint32_t)a.m) {
              const double g = look(rt);
              s += (double)opaque(xv[t]) * g;
              if (FUSED) atomicAdd(&a.acc[q0 + t * kWave], lb * g);
            } else {
              flag_error(status, 3);
            }
          }
        }
      }
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
      if (l == 0) a.out[base + L] = (VT)s;
    }
    wave_sync();  // sc is rewritten by the next chunk
  }
}

// Fills the table with Y(:,j) (entries [y0, y1)), kDotIns loads in flight
// per thread.
template <int TBL, int THREADS, class VT>
__device__ __forceinline__ void dot_fill(const DotArgs<VT> &a, int64_t y0, int64_t y1, int t, int32_t *keys, VT *vals,
                                         int32_t *status) {
  for (int64_t p0 = y0 + t; p0 < y1; p0 += kDotIns * THREADS) {
    int32_t row[kDotIns];
    VT v[kDotIns];
#pragma unroll
    for (int u = 0; u < kDotIns; u++) {
      const int64_t p = p0 + u * THREADS;
      row[u] = 0;
      v[u] = VT(0);
      if (p < y1) {
        row[u] = a.Yri[p];
        v[u] = a.Yv[p];
      }
    }
#pragma unroll
    for (int u = 0; u < kDotIns; u++) {
      if (p0 + u * THREADS < y1) {
        const int32_t r = opaque(row[u]);
        if ((uint32_t)r < (uint32_t)a.m)
          ht_put(keys, vals, TBL, r, opaque(v[u]));
        else
          flag_error(status, 3);
      }
    }
  }
}

template <int TBL, int THREADS>
__device__ __forceinline__ void dot_clear(int t, int32_t *keys) {
  static_assert(TBL % 4 == 0, "tables cleared 16 bytes at a time");
  for (int s = t; s < TBL / 4; s += THREADS)
    reinterpret_cast<int4 *>(keys)[s] = make_int4(kEmpty, kEmpty, kEmpty, kEmpty);
}

// Both kernels are bound by LDS atomics (57% of the LDS cycles at first) and
// by the latency of the dependent loads.  Fused backward of 256 products,
// 1.0e9 terms: 18.8 ms with a marker and max-scan per round and one LDS atomic
// per product; 17.0 with loads ahead and start words; 13.0 with the products
// of a quad summed first and values put without a read.
// The kernels below: the next column's pointers, first chunk of M and X's
// column pointers are loaded while a column is processed, and a table's
// entries are loaded kDotIns at a time, so that a column does not wait for
// each of its dependent loads in turn.  list[dir * i]: half tables are listed
// from the end of their array.
// One wavefront per column, TBL-slot table of Y(:,j) private to the wave.
template <int TBL, bool FUSED, class VT>
__global__ __launch_bounds__(256) void k_dot_wave(DotArgs<VT> a, const int32_t *list, int dir, const int32_t *count_p,
                                                  int32_t *status) {
  __shared__ __align__(16) int32_t s_keys[4][TBL];
  __shared__ __align__(16) VT s_vals[4][TBL];
  __shared__ DotScratch s_sc[4];
  const int w = threadIdx.x / kWave, l = lane();
  const int count = *count_p;
  int32_t *keys = s_keys[w];
  VT *vals = s_vals[w];
  const int64_t stride = (int64_t)gridDim.x * 4;
  int64_t idx = (int64_t)blockIdx.x * 4 + w;
  const int64_t z = opaque((int64_t)0);
  DotPre<VT> pre;
  int32_t jn2 = 0;
  if (idx < count) {
    dot_pre_ptr(a, (int64_t)list[dir * idx], pre);
    dot_pre_m<FUSED>(a, 0, 1, pre);
    dot_pre_x(a, pre);
    if (idx + stride < count) jn2 = ld_global(list + dir * (idx + stride) + z);
  }
  for (; idx < count; idx += stride) {
    const DotPre<VT> cur = pre;
    const bool more = idx + stride < count;  // uniform
    if (more) {
      dot_pre_ptr(a, (int64_t)__builtin_amdgcn_readfirstlane(jn2), pre);
      if (idx + 2 * stride < count) jn2 = ld_global(list + dir * (idx + 2 * stride) + z);
    }
    dot_clear<TBL, kWave>(l, keys);
    wave_sync();
    dot_fill<TBL, kWave>(a, cur.y0, cur.y1, l, keys, vals, status);
    if (more) dot_pre_m<FUSED>(a, 0, 1, pre);
    wave_sync();
    dot_entries<FUSED>(a, cur.m0, cur.m1, 0, 1, status, s_sc[w], &cur,
                       [&](int32_t r) { return ht_lookup(keys, vals, TBL, r); });
    if (more) dot_pre_x(a, pre);
    wave_sync();
  }
}

// One workgroup per column, shared table.
template <int TBL, int THREADS, bool FUSED, class VT>
__global__ __launch_bounds__(THREADS) void k_dot_block(DotArgs<VT> a, const int32_t *list, int dir,
                                                       const int32_t *count_p, int32_t *status) {
  constexpr int NW = THREADS / kWave;
  __shared__ __align__(16) int32_t s_keys[TBL];
  __shared__ __align__(16) VT s_vals[TBL];
  __shared__ DotScratch s_sc[NW];
  const int w = threadIdx.x / kWave;
  const int count = *count_p;
  int64_t item = blockIdx.x;
  const int64_t z = opaque((int64_t)0);
  DotPre<VT> pre;
  int32_t jn2 = 0;
  if (item < count) {
    dot_pre_ptr(a, (int64_t)list[dir * item], pre);
    dot_pre_m<FUSED>(a, w, NW, pre);
    dot_pre_x(a, pre);
    if (item + gridDim.x < count) jn2 = ld_global(list + dir * (item + gridDim.x) + z);
  }
  for (; item < count; item += gridDim.x) {
    const DotPre<VT> cur = pre;
    const bool more = item + gridDim.x < count;  // uniform
    if (more) {
      dot_pre_ptr(a, (int64_t)__builtin_amdgcn_readfirstlane(jn2), pre);
      if (item + 2 * (int64_t)gridDim.x < count) jn2 = ld_global(list + dir * (item + 2 * (int64_t)gridDim.x) + z);
    }
    dot_clear<TBL, THREADS>(threadIdx.x, s_keys);
    __syncthreads();
    dot_fill<TBL, THREADS>(a, cur.y0, cur.y1, threadIdx.x, s_keys, s_vals, status);
    if (more) dot_pre_m<FUSED>(a, w, NW, pre);
    __syncthreads();
    dot_entries<FUSED>(a, cur.m0, cur.m1, w, NW, status, s_sc[w], &cur,
                       [&](int32_t r) { return ht_lookup(s_keys, s_vals, TBL, r); });
    if (more) dot_pre_x(a, pre);
    __syncthreads();
  }
}

// Heavy columns: Y(:,j) scattered into a dense float64 column of the
// workspace (zero outside Y's rows), dots read it, then it is cleared.
template <class VT>
__global__ __launch_bounds__(256) void k_mxty_heavy_fill(DotArgs<VT> a, const int32_t *list, int first, int ns,
                                                         double *dense, int clear) {
  const int slot = blockIdx.y;
  if (slot >= ns) return;
  const int32_t j = list[first + slot];
  double *d = dense + (int64_t)slot * a.m;
  for (int64_t p = a.Ycp[j] + (int64_t)blockIdx.x * 256 + threadIdx.x; p < a.Ycp[j + 1];
       p += (int64_t)gridDim.x * 256) {
    const int32_t r = a.Yri[p];
    if ((uint32_t)r < (uint32_t)a.m) d[r] = clear ? 0.0 : (double)a.Yv[p];
  }
}

template <class VT>
__global__ __launch_bounds__(256) void k_mxty_heavy_dot(DotArgs<VT> a, const int32_t *list, int first, int ns,
                                                        const double *dense, int parts, int32_t *status) {
  __shared__ DotScratch s_sc[4];
  const int slot = blockIdx.x / parts, part = blockIdx.x % parts;
  if (slot >= ns) return;
  const int32_t j = list[first + slot];
  const double *d = dense + (int64_t)slot * a.m;
  const int w = threadIdx.x / kWave;
  dot_entries<false>(a, a.Mcp[j], a.Mcp[j + 1], part * 4 + w, parts * 4, status, s_sc[w],
                     (const DotPre<VT> *)nullptr, [&](int32_t r) { return d[r]; });
}

static unsigned mx_grid(int cnt, bool wave_kernel, int blocks_per_cu) {
  const unsigned full = (unsigned)(blocks_per_cu * device_cus());
  if (cnt < 0) return full;
  const unsigned need = wave_kernel ? grid_of(cnt, 4) : (unsigned)cnt;
  return std::max(1u, std::min(need, full));
}

template <class VT>
static int mxty_typed(const spgemm_csc *X, const spgemm_csc *Y, const spgemm_csc *M, void *out, const WsLayout &L,
                      char *ws, hipStream_t st, bool sync) {
  WsHeader *hdr = (WsHeader *)ws;
  int32_t *bins = (int32_t *)(ws + L.bins);
  const int64_t n = Y->ncols;
  int rc = launch_init_header(hdr, zero_region_tag(kTagMasked, L), st);
  if (rc) return rc;
  hipLaunchKernelGGL(k_mxty_bin, dim3(grid_of(n, 256)), dim3(256), 0, st, Y->colptr, M->colptr, n, g_min_bin_value(),
                     num_caps(Y->nrows), bins, hdr, sync ? 0 : 7, half_tables(n));
  LAUNCHCHK();
  WsHeader h;
  int cnt[kNumBins];
  if (sync) {
    rc = read_header(hdr, st, &h);
    if (rc) return rc;
    for (int b = 0; b < kNumBins; b++) cnt[b] = h.bin_count[b];
  } else {
    for (int b = 0; b < kNumBins; b++) cnt[b] = -1;
    memset(&h, 0, sizeof(h));
  }
  DotArgs<VT> a{X->colptr, X->rowidx, (const VT *)X->values, Y->colptr, Y->rowidx, (const VT *)Y->values,
                 M->colptr, M->rowidx, (const VT *)nullptr, (VT *)out, (double *)nullptr, Y->nrows, X->ncols, X->nnz};
  int32_t *status = &hdr->status;
  for (int b = 0; b < kNumBins + 1; b++) {
    const int half = b - (kNumBins - 1);  // 0, 1: the half tables of bins 2 and 3
    const int c = half < 0 ? cnt[b] : (sync ? h.half_count[half] : ((half_tables(n) >> half) & 1 ? -1 : 0));
    if (c == 0) continue;
    ProfScope prof("masked_xty", st);
    const int32_t *list = half < 0 ? bins + (int64_t)b * n : bins + (int64_t)(half + 3) * n - 1;
    const int32_t *cp = half < 0 ? &hdr->bin_count[b] : &hdr->half_count[half];
    const int dir = half < 0 ? 1 : -1;
    switch (b) {
      case 0: hipLaunchKernelGGL((k_dot_wave<64, false, VT>), dim3(mx_grid(c, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 1: hipLaunchKernelGGL((k_dot_wave<256, false, VT>), dim3(mx_grid(c, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 2: hipLaunchKernelGGL((k_dot_wave<1024, false, VT>), dim3(mx_grid(c, true, 4)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 3: hipLaunchKernelGGL((k_dot_block<4096, 256, false, VT>), dim3(mx_grid(c, false, 4)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 4: hipLaunchKernelGGL((k_dot_block<10240, 1024, false, VT>), dim3(mx_grid(c, false, 1)), dim3(1024), 0, st, a, list, dir, cp, status); break;
      case 5: hipLaunchKernelGGL((k_dot_wave<512, false, VT>), dim3(mx_grid(c, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      default: hipLaunchKernelGGL((k_dot_block<2048, 256, false, VT>), dim3(mx_grid(c, false, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
    }
    LAUNCHCHK();
  }
  const int heavy = cnt[kNumBins - 1];
  if (heavy < 0) return SPGEMM_OK;  // no host count: heavy columns cannot be scheduled here (reported by the binning)
  if (heavy > 0) {
    if (L.slots <= 0) return SPGEMM_E_INVAL;
    double *dense = (double *)(ws + L.heavy_vals);
    const uint64_t tag = zero_region_tag(kTagMasked, L);
    if (h.clean_tag != tag) {
      hipLaunchKernelGGL(k_tr_zero, dim3(4 * device_cus()), dim3(256), 0, st, (unsigned long long *)dense,
                         L.slots * L.m);
      LAUNCHCHK();
      rc = launch_set_tag(hdr, tag, st);
      if (rc) return rc;
    }
    const int32_t *list = bins + (int64_t)(kNumBins - 1) * n;
    for (int first = 0; first < heavy; first += (int)L.slots) {
      const int ns = (int)std::min<int64_t>(L.slots, heavy - first);
      hipLaunchKernelGGL(k_mxty_heavy_fill<VT>, dim3(64, ns), dim3(256), 0, st, a, list, first, ns, dense, 0);
      LAUNCHCHK();
      const int parts = (int)std::max<int64_t>(1, std::min<int64_t>(64, (4 * device_cus() + ns - 1) / ns));
      hipLaunchKernelGGL(k_mxty_heavy_dot<VT>, dim3(ns * parts), dim3(256), 0, st, a, list, first, ns, dense, parts,
                         status);
      LAUNCHCHK();
      hipLaunchKernelGGL(k_mxty_heavy_fill<VT>, dim3(64, ns), dim3(256), 0, st, a, list, first, ns, dense, 1);
      LAUNCHCHK();
    }
  }
  return SPGEMM_OK;
}

// ============================================================================
// Fused gradient (graph-capturable): for each output column j, dC(:,j) goes
// into an LDS hash table; every entry (k,j) of B then gives
//   dB(k,j)  = sum over i in A(:,k) of A(i,k) * dC(i,j)     (a dot product)
//   dA(i,k) += B(k,j) * dC(i,j)  for i in A(:,k)           (float64 atomics)
// in one traversal of the product's terms, with no transpose.  dA is
// accumulated in a float64 workspace array and rounded once.
// ============================================================================
__global__ void k_fbwd_init(WsHeader *hdr, double *p, int64_t n) {
  if (blockIdx.x == 0 && threadIdx.x == 0) init_header(hdr, 0, 0, 0);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0.0;
}

template <class VT>
__global__ void k_round(const double *src, int64_t n, VT *dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = (VT)src[i];
}

template <class VT>
static int fbwd_typed(const spgemm_csc *A, const spgemm_csc *B, const spgemm_csc *C, const void *dC, void *dA,
                      void *dB, const WsLayout &L, char *ws, hipStream_t st) {
  WsHeader *hdr = (WsHeader *)ws;
  int32_t *bins = (int32_t *)(ws + L.bins);
  // float64 gradients are summed where they are wanted (unless that is over
  // an input, which the terms still read), float32 ones in the workspace
  const auto over = [&](const void *p, int64_t count) {
    const uintptr_t a = (uintptr_t)dA, b = (uintptr_t)p;
    return b < a + sizeof(VT) * (uintptr_t)A->nnz && a < b + sizeof(VT) * (uintptr_t)count;
  };
  const bool in_place = sizeof(VT) == sizeof(double) && !over(A->values, A->nnz) && !over(B->values, B->nnz) &&
                        !over(dC, C->nnz);
  double *acc = in_place ? (double *)dA : (double *)(ws + L.heavy_vals);
  const int64_t n = C->ncols;
  const unsigned gz = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid_of(A->nnz, 256), 8 * device_cus()));
  // (launches count for small batches: the header, the sums' zeros and the
  // report of columns above the tables take none of their own; gradients of 64
  // products of 256: 50.7 -> 40.1 us)
  hipLaunchKernelGGL(k_fbwd_init, dim3(gz), dim3(256), 0, st, hdr, acc, A->nnz);
  LAUNCHCHK();
  BinCaps caps = num_caps(C->nrows);
  caps.cap[kNumBins - 2] = kNumTableCap[kNumBins - 2];  // whatever fits the largest table is formed
  if (n > 0) {
    hipLaunchKernelGGL(k_mxty_bin, dim3(grid_of(n, 256)), dim3(256), 0, st, C->colptr, B->colptr, n,
                       std::min(g_min_bin_value(), kNumBins - 2), caps, bins, hdr, 7, half_tables(n));
    LAUNCHCHK();
  }
  DotArgs<VT> a{A->colptr, A->rowidx, (const VT *)A->values, C->colptr, C->rowidx, (const VT *)dC,
                B->colptr, B->rowidx, (const VT *)B->values, (VT *)dB, acc, C->nrows, A->ncols, A->nnz};
  int32_t *status = &hdr->status;
  for (int b = 0; n > 0 && b < kNumBins + 1; b++) {  // (no columns: dA is zero)
    const int half = b - (kNumBins - 1);  // 0, 1: the half tables of bins 2 and 3
    static const char *kNames[kNumBins + 1] = {"fbwd_wave64", "fbwd_wave256", "fbwd_wave1024", "fbwd_block4096",
                                               "fbwd_block10240", "fbwd_wave512", "fbwd_block2048"};
    if (half >= 0 && !((half_tables(n) >> half) & 1)) continue;
    ProfScope prof(kNames[b], st);
    const int32_t *list = half < 0 ? bins + (int64_t)b * n : bins + (int64_t)(half + 3) * n - 1;
    const int32_t *cp = half < 0 ? &hdr->bin_count[b] : &hdr->half_count[half];
    const int dir = half < 0 ? 1 : -1;
    switch (b) {
      case 0: hipLaunchKernelGGL((k_dot_wave<64, true, VT>), dim3(mx_grid(-1, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 1: hipLaunchKernelGGL((k_dot_wave<256, true, VT>), dim3(mx_grid(-1, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 2: hipLaunchKernelGGL((k_dot_wave<1024, true, VT>), dim3(mx_grid(-1, true, 4)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 3: hipLaunchKernelGGL((k_dot_block<4096, 256, true, VT>), dim3(mx_grid(-1, false, 4)), dim3(256), 0, st, a, list, dir, cp, status); break;
      case 4: hipLaunchKernelGGL((k_dot_block<10240, 1024, true, VT>), dim3(mx_grid(-1, false, 1)), dim3(1024), 0, st, a, list, dir, cp, status); break;
      case 5: hipLaunchKernelGGL((k_dot_wave<512, true, VT>), dim3(mx_grid(-1, true, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
      default: hipLaunchKernelGGL((k_dot_block<2048, 256, true, VT>), dim3(mx_grid(-1, false, 8)), dim3(256), 0, st, a, list, dir, cp, status); break;
    }
    LAUNCHCHK();
  }
  if (!in_place) {
    hipLaunchKernelGGL(k_round<VT>, dim3(gz), dim3(256), 0, st, acc, A->nnz, (VT *)dA);
    LAUNCHCHK();
  }
  return SPGEMM_OK;
}

template <class VT>
static int transpose_typed(const spgemm_csc *X, int64_t *t_colptr, int32_t *t_rowidx, void *t_values, int64_t *perm,
                           const WsLayout &L, char *ws, hipStream_t st) {
  WsHeader *hdr = (WsHeader *)ws;
  int rc = launch_init_header(hdr, (uint64_t)0, st);
  if (rc) return rc;
  ProfScope prof("transpose", st);
  const int64_t m = X->nrows;
  unsigned long long *cnt = (unsigned long long *)(ws + L.bins);
  int32_t *rank = (int32_t *)(ws + L.slab_ri);
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid_of(std::max(m, X->nnz), 256), 8 * device_cus()));
  hipLaunchKernelGGL(k_tr_zero, dim3(g), dim3(256), 0, st, cnt, m);
  LAUNCHCHK();
  if (X->nnz > 0) {
    hipLaunchKernelGGL(k_tr_count<true>, dim3(g), dim3(256), 0, st, X->rowidx, X->nnz, m, cnt, rank, &hdr->status);
    LAUNCHCHK();
  }
  rc = launch_colptr_scan((const int64_t *)cnt, m, t_colptr, (int64_t *)(ws + L.scan), st);
  if (rc) return rc;
  if (X->nnz > 0) {
    const unsigned gs = (unsigned)std::min<int64_t>((X->nnz + kTrTile - 1) / kTrTile, 8 * device_cus());
    hipLaunchKernelGGL(k_tr_scatter<VT>, dim3(gs), dim3(256), 0, st, X->colptr, X->rowidx,
                       t_values ? (const VT *)X->values : (const VT *)nullptr, X->ncols, m, X->nnz,
                       (const int64_t *)t_colptr, (const int32_t *)rank, t_rowidx, (VT *)t_values, perm);
    LAUNCHCHK();
  }
  return SPGEMM_OK;
}

}  // namespace spg

using namespace spg;

extern "C" {

int spgemm_transpose(const spgemm_csc *X, int64_t *t_colptr, int32_t *t_rowidx, void *t_values, int64_t *perm,
                     void *ws, size_t ws_bytes, void *stream) {
  int st = check_csc(X, t_values != nullptr);
  if (st) return st;
  if (!t_colptr || (X->nnz > 0 && !t_rowidx)) return SPGEMM_E_INVAL;
  if (X->ncols > INT32_MAX) return SPGEMM_E_OVERFLOW;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_TRANSPOSE, X, nullptr, 0, 0, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  if (t_values && X->dtype == SPGEMM_F64)
    return transpose_typed<double>(X, t_colptr, t_rowidx, t_values, perm, L, (char *)ws, s);
  return transpose_typed<float>(X, t_colptr, t_rowidx, t_values, perm, L, (char *)ws, s);
}

int spgemm_longest_row(const spgemm_csc *X, int64_t *longest_host, void *ws, size_t ws_bytes, void *stream) {
  int st = check_csc(X, false);
  if (st) return st;
  if (!longest_host) return SPGEMM_E_INVAL;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_TRANSPOSE, X, nullptr, 0, 0, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  WsHeader *hdr = (WsHeader *)ws;
  st = launch_init_header(hdr, (uint64_t)0, s);
  if (st) return st;
  unsigned long long *cnt = (unsigned long long *)((char *)ws + L.bins);
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid_of(std::max(X->nrows, X->nnz), 256), 8 * device_cus()));
  hipLaunchKernelGGL(k_tr_zero, dim3(g), dim3(256), 0, s, cnt, X->nrows);
  LAUNCHCHK();
  if (X->nnz > 0) {
    hipLaunchKernelGGL(k_tr_count<false>, dim3(g), dim3(256), 0, s, X->rowidx, X->nnz, X->nrows, cnt,
                       (int32_t *)nullptr, &hdr->status);
    LAUNCHCHK();
  }
  int64_t sum;
  return spgemm_count_sums((const int64_t *)cnt, X->nrows, 1, &sum, longest_host, ws, ws_bytes, stream);
}

int spgemm_masked_xty(const spgemm_csc *X, const spgemm_csc *Y, const spgemm_csc *M, void *out_values, void *ws,
                      size_t ws_bytes, void *stream) {
  int st = check_csc(X, true);
  if (!st) st = check_csc(Y, true);
  if (!st) st = check_csc(M, false);
  if (st) return st;
  if (X->dtype != Y->dtype) return SPGEMM_E_DTYPE;
  if (X->nrows != Y->nrows || M->nrows != X->ncols || M->ncols != Y->ncols) return SPGEMM_E_SHAPE;
  if (M->nnz > 0 && !out_values) return SPGEMM_E_INVAL;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_MASKED_XTY, X, Y, 0, Y->ncols, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  if (Y->ncols == 0 || M->nnz == 0) return launch_init_header((WsHeader *)ws, kKeepAnyTag, s);
  if (X->dtype == SPGEMM_F64) return mxty_typed<double>(X, Y, M, out_values, L, (char *)ws, s, true);
  return mxty_typed<float>(X, Y, M, out_values, L, (char *)ws, s, true);
}

int spgemm_batched_masked_xty(const spgemm_csc *X, const spgemm_csc *Y, const spgemm_csc *M, void *out_values,
                              void *ws, size_t ws_bytes, void *stream) {
  int st = check_csc(X, true);
  if (!st) st = check_csc(Y, true);
  if (!st) st = check_csc(M, false);
  if (st) return st;
  if (X->dtype != Y->dtype) return SPGEMM_E_DTYPE;
  if (X->nrows != Y->nrows || M->nrows != X->ncols || M->ncols != Y->ncols) return SPGEMM_E_SHAPE;
  if (M->nnz > 0 && !out_values) return SPGEMM_E_INVAL;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_MASKED_XTY, X, Y, 0, Y->ncols, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  if (Y->ncols == 0 || M->nnz == 0) return launch_init_header((WsHeader *)ws, kKeepAnyTag, s);
  if (X->dtype == SPGEMM_F64) return mxty_typed<double>(X, Y, M, out_values, L, (char *)ws, s, false);
  return mxty_typed<float>(X, Y, M, out_values, L, (char *)ws, s, false);
}

int spgemm_batched_backward(const spgemm_csc *A, const spgemm_csc *B, const spgemm_csc *C, const void *dC_values,
                            void *dA_out, void *dB_out, void *ws, size_t ws_bytes, void *stream) {
  int st = check_csc(A, true);
  if (!st) st = check_csc(B, true);
  if (!st) st = check_csc(C, false);
  if (st) return st;
  if (A->dtype != B->dtype) return SPGEMM_E_DTYPE;
  if (A->ncols != B->nrows || C->nrows != A->nrows || C->ncols != B->ncols) return SPGEMM_E_SHAPE;
  if ((C->nnz > 0 && !dC_values) || (A->nnz > 0 && !dA_out) || (B->nnz > 0 && !dB_out)) return SPGEMM_E_INVAL;
  WsLayout L;
  st = ws_layout(SPGEMM_OP_BATCHED_BACKWARD, A, B, 0, B->ncols, 1, &L);
  if (st) return st;
  st = check_ws(ws, ws_bytes, L.total);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  if (A->dtype == SPGEMM_F64) return fbwd_typed<double>(A, B, C, dC_values, dA_out, dB_out, L, (char *)ws, s);
  return fbwd_typed<float>(A, B, C, dC_values, dA_out, dB_out, L, (char *)ws, s);
}

int spgemm_permute(const void *src, const int64_t *perm, int64_t n, int32_t dtype, int32_t scatter, void *dst,
                   void *stream) {
  if (n < 0 || (n > 0 && (!src || !perm || !dst))) return SPGEMM_E_INVAL;
  const int vb = dtype_bytes(dtype);
  if (!vb) return SPGEMM_E_DTYPE;
  if (n == 0) return SPGEMM_OK;
  hipStream_t s = (hipStream_t)stream;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid_of(n, 256), 8 * device_cus()));
  if (vb == 8)
    hipLaunchKernelGGL(k_permute<double>, dim3(g), dim3(256), 0, s, (const double *)src, perm, n, (double *)dst,
                       (int)scatter);
  else
    hipLaunchKernelGGL(k_permute<float>, dim3(g), dim3(256), 0, s, (const float *)src, perm, n, (float *)dst,
                       (int)scatter);
  LAUNCHCHK();
  return SPGEMM_OK;
}

}  // extern "C"
