// Device-side structural analysis (sd_analyze_device): the statistics of
// sd_analyze for a CSR matrix whose arrays live in device memory.
//
// The kernels compute only exact integer aggregates (counts, sums, maxima,
// histograms, order statistics); the host turns them into sd_stats_t with the
// same finishing step as the host analysis, so both give bit-identical
// statistics.  Nothing is read back before the end: a pass that indexes by
// what an earlier one checks tests the device-side `bad` flag and leaves.
//
//  * rows      512 rows per workgroup and turn: length, squares, span, column
//              gaps, SELL slot counts, row-pointer checks, and a histogram of
//              lengths in LDS (quartiles and log2 bins come from it);
//  * strips    b consecutive rows (b = 4, 8, 16) hold one row of b x b blocks.
//              Short strips (up to kSmall entries): one wave each, the block
//              columns counted in an LDS hash table; middling ones (up to
//              kMid): one workgroup each, the same; long ones: one workgroup
//              per window of kWindow columns, each block column a bit (or a
//              counter) of the window.  At b = 16 the same passes check the
//              column range and order, and count the diagonal;
//  * columns   degrees by integer atomics, then their maximum and squares;
//  * medians   radix selection, three passes over 32-bit keys with the chosen
//              bins kept on the device.
//
// A plan needs only the row statistics, the 16x16 block count and the widest
// block-row (kPlanStats); sd_analyze_device runs everything (kAllStats).
//
// Shared counters are added up per workgroup in registers and LDS, one atomic
// per workgroup: device-wide atomics are slow here (62 M adds to counters spread
// over 2.4 M addresses took 2.3 ms, 27 G/s, and 4.1 ms over 4,096 addresses).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>

#include "kernels.h"
#include "sd_internal.h"

namespace {

typedef unsigned long long u64;

constexpr int32_t kLenBins = 4096;        // row lengths counted exactly below kLenBins - 1
constexpr int32_t kSmall = 512;           // entries of a strip that one wave takes
constexpr int32_t kMid = 4096;            // entries of a strip that one workgroup takes
constexpr int32_t kWindow = 128 * 1024;   // columns per window of a longer strip

struct DevAgg {
  u64 row_sumsq, col_sumsq, span_sum, nonempty, gap_num, gap_den, diag;
  u64 nnzb[3], dense_tiles, dense_nnz, sell_slots[3];
  u64 row_hist[33], fill16_hist[8];
  int32_t quart[3];                       // row lengths at the quartile ranks (-1: kLenBins - 1 or more)
  int32_t rmax, rmin_c, dmax, width16;    // rmin_c = INT32_MAX - the shortest row, so every counter starts at 0
  int32_t bad_rows, bad;                  // row pointers / columns break a rule
  uint32_t n_mid[3], n_big[3];            // strips in the lists, per block size
  // radix selection: the bits chosen so far, the rank left inside them, the keys seen
  uint32_t sel_prefix, sel_n;
  u64 sel_rank;
};

__device__ __forceinline__ int log2_bin_dev(int64_t r) {
  return r == 0 ? 0 : 64 - __builtin_clzll((u64)r);
}

// smallest p in [lo, hi) with col[p] >= v (hi if none)
__device__ __forceinline__ int32_t lower_bound_dev(const int32_t *__restrict__ col, int32_t lo, int32_t hi, int64_t v) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (col[mid] < v) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Wave-wide reductions (every lane of the wave must call them).
__device__ __forceinline__ u64 wave_sum(u64 v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ int32_t wave_max(int32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Adds (or maxes, v >= 0) each thread's v over the workgroup into *dst: one atomic.
// Called by every thread; `part` holds one value per wave.
__device__ __forceinline__ void block_add(u64 *dst, u64 v, u64 *part) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    u64 t = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += part[w];
    if (t) atomicAdd(dst, t);
  }
}
__device__ __forceinline__ void block_max(int32_t *dst, int32_t v, u64 *part) {
  v = wave_max(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[wave] = (u64)(uint32_t)v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = (int32_t)part[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t = max(t, (int32_t)part[w]);
    if (t > 0) atomicMax(dst, t);
  }
}

__global__ __launch_bounds__(256) void k_an_zero(uint32_t *__restrict__ x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x[i] = 0;
}

// Rows in turns of 512 (two per thread), so the SELL slices of 16, 32 and 512
// rows lie inside one turn.  Lengths from kLenBins - 1 on share the last bin.
// spans: the spans of non-empty rows, UINT32_MAX for empty ones (null: not kept).
__global__ __launch_bounds__(256) void k_an_rows(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                                                 int32_t m, int64_t nnz, uint32_t *__restrict__ len_hist,
                                                 uint32_t *__restrict__ spans, DevAgg *__restrict__ agg) {
  __shared__ uint32_t hist[kLenBins];
  __shared__ u64 part[4];
  __shared__ int32_t turn_max[4];
  for (int t = threadIdx.x; t < kLenBins; t += 256) hist[t] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  u64 sumsq = 0, nonempty = 0, span_sum = 0, gap_num = 0, gap_den = 0, slots[3] = {0, 0, 0};
  int32_t rmax = 0, rmin = INT32_MAX, bad = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0 && (rowptr[0] != 0 || (int64_t)rowptr[m] != nnz)) bad = 1;
  for (int64_t r0 = (int64_t)blockIdx.x * 512; r0 < m; r0 += (int64_t)gridDim.x * 512) {
    int32_t mx = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t i = r0 + h * 256 + threadIdx.x;
      int32_t len = 0;
      if (i < m) {
        const int32_t p0 = rowptr[i], p1 = rowptr[i + 1];
        uint32_t key = UINT32_MAX;
        if (p1 < p0 || p0 < 0 || (int64_t)p1 > nnz) {
          bad = 1;
        } else {
          len = p1 - p0;
          atomicAdd(&hist[min(len, kLenBins - 1)], 1u);
          if (len >= kLenBins - 1) atomicAdd(&agg->row_hist[log2_bin_dev(len)], 1ull);
          sumsq += (u64)((int64_t)len * len);
          rmax = max(rmax, len);
          rmin = min(rmin, len);
          if (len > 0) {
            const int64_t span = (int64_t)colidx[p1 - 1] - colidx[p0] + 1;
            key = (uint32_t)span;
            ++nonempty;
            span_sum += (u64)span;
            if (len >= 2) {
              gap_num += (u64)(span - 1);
              gap_den += (u64)(len - 1);
            }
          }
        }
        if (spans) spans[i] = key;
      }
      // slices: the longest of 16, then of 32 rows
      int32_t x = len;
      for (int o = 1; o < 16; o <<= 1) x = max(x, __shfl_xor(x, o, 64));
      const int64_t s16 = i & ~(int64_t)15, s32 = i & ~(int64_t)31;
      if ((lane & 15) == 0 && s16 < m) slots[0] += (u64)(min((int64_t)16, m - s16) * x);
      x = max(x, __shfl_xor(x, 16, 64));
      if ((lane & 31) == 0 && s32 < m) slots[1] += (u64)(min((int64_t)32, m - s32) * x);
      mx = max(mx, max(x, __shfl_xor(x, 32, 64)));
    }
    __syncthreads();
    if (lane == 0) turn_max[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      mx = max(max(turn_max[0], turn_max[1]), max(turn_max[2], turn_max[3]));
      slots[2] += (u64)(min((int64_t)512, m - r0) * mx);
    }
  }
  block_add(&agg->row_sumsq, sumsq, part);
  block_add(&agg->nonempty, nonempty, part);
  block_add(&agg->span_sum, span_sum, part);
  block_add(&agg->gap_num, gap_num, part);
  block_add(&agg->gap_den, gap_den, part);
  for (int t = 0; t < 3; ++t) block_add(&agg->sell_slots[t], slots[t], part);
  block_max(&agg->rmax, rmax, part);
  block_max(&agg->rmin_c, INT32_MAX - rmin, part);
  block_max(&agg->bad_rows, bad, part);
  for (int t = threadIdx.x; t < kLenBins; t += 256)
    if (hist[t]) atomicAdd(&len_hist[t], hist[t]);
}

// Quartiles (lower nearest rank) and log2 bins from the length histogram, and
// the widest block-row among the long strips.  One workgroup of 256 threads.
__global__ __launch_bounds__(256) void k_an_finish(const uint32_t *__restrict__ len_hist, int32_t m,
                                                   const int32_t *__restrict__ big_blocks, DevAgg *__restrict__ agg) {
  __shared__ uint32_t sum[256];
  __shared__ u64 part[4];
  constexpr int kEach = kLenBins / 256;
  uint32_t h[kEach], mine = 0;
  for (int t = 0; t < kEach; ++t) {
    h[t] = len_hist[threadIdx.x * kEach + t];
    mine += h[t];
  }
  sum[threadIdx.x] = mine;
  __syncthreads();
  uint32_t before = 0;
  for (int t = 0; t < (int)threadIdx.x; ++t) before += sum[t];
  if (m > 0) {
    for (int q = 0; q < 3; ++q) {
      const uint32_t rank = (uint32_t)(q == 2 ? 3 * (int64_t)(m - 1) / 4 : q == 1 ? (m - 1) / 2 : (m - 1) / 4);
      if (rank >= before && rank - before < mine) {
        uint32_t left = rank - before;
        int t = 0;
        while (left >= h[t]) left -= h[t++];
        const int32_t len = (int32_t)threadIdx.x * kEach + t;
        agg->quart[q] = len < kLenBins - 1 ? len : -1;
      }
    }
  }
  for (int t = 0; t < kEach; ++t) {
    const int32_t len = (int32_t)threadIdx.x * kEach + t;
    if (h[t] && len < kLenBins - 1) atomicAdd(&agg->row_hist[log2_bin_dev(len)], (u64)h[t]);
  }
  int32_t w = 0;
  for (uint32_t t = threadIdx.x; t < agg->n_big[2]; t += 256) w = max(w, big_blocks[t]);
  block_max(&agg->width16, w, part);
}

// ---- strips of b = 2^LB rows
// Finds (or opens) the slot of key in an open-addressing table of mask + 1
// slots, at least twice the keys it can hold; sets fresh if it opened it.
__device__ __forceinline__ uint32_t table_slot(uint32_t *__restrict__ tab, uint32_t mask, int lg, uint32_t key,
                                               bool &fresh) {
  uint32_t h = (key * 2654435761u) >> (32 - lg);
  for (;;) {
    const uint32_t old = atomicCAS(&tab[h], UINT32_MAX, key);
    if (old == UINT32_MAX || old == key) {
      fresh = old == UINT32_MAX;
      return h;
    }
    h = (h + 1) & mask;
  }
}

// What a thread has counted; added to the totals once per workgroup.
struct StripSums {
  u64 blocks = 0, diag = 0, dense_tiles = 0, dense_nnz = 0, fh[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int32_t width = 0, bad = 0;
  __device__ __forceinline__ void tile(int32_t f, int32_t dense_threshold) {
    if (f < 1) return;
    if (f > 256) {  // only a matrix with repeated columns (invalid) gets here
      bad = 1;
      return;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) fh[t] += (f - 1) / 32 == t;
    if (f >= dense_threshold) {
      ++dense_tiles;
      dense_nnz += (u64)f;
    }
  }
  template <int LB, bool ALL>
  __device__ __forceinline__ void flush(DevAgg *__restrict__ agg, u64 *part) {
    block_add(&agg->nnzb[LB - 2], blocks, part);
    if constexpr (LB == 4) {
      block_add(&agg->diag, diag, part);
      block_max(&agg->width16, width, part);
      block_max(&agg->bad, bad, part);
      if constexpr (ALL) {
        block_add(&agg->dense_tiles, dense_tiles, part);
        block_add(&agg->dense_nnz, dense_nnz, part);
        for (int t = 0; t < 8; ++t) block_add(&agg->fill16_hist[t], fh[t], part);
      }
    }
  }
};

// prev: the column of entry p - 1 (any value at a row's start)
__device__ __forceinline__ bool entry_bad(int32_t p, int32_t row_start, int32_t c, int32_t prev, int32_t k) {
  return c < 0 || c >= k || (p > row_start && prev >= c);
}

// Short strips, one wave each: an LDS table of at least twice the entries.
// The others go to the list of middling strips.
template <int LB, bool ALL>
__global__ __launch_bounds__(256) void k_an_strips(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx, int32_t m, int32_t k,
                                                   int32_t dense_threshold, int32_t *__restrict__ mid,
                                                   DevAgg *__restrict__ agg) {
  constexpr bool kFill = LB == 4 && ALL;
  constexpr int B = 1 << LB;
  __shared__ uint32_t tabs[4][2 * kSmall];
  __shared__ uint32_t cnts[kFill ? 4 : 1][kFill ? 2 * kSmall : 1];
  __shared__ u64 part[4];
  if (agg->bad_rows) return;  // the row pointers are not usable
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  volatile uint32_t *vtab = tabs[wave];
  uint32_t *tab = tabs[wave];
  const int64_t ns = ((int64_t)m + B - 1) / B;
  StripSums sum;
  for (int64_t s = (int64_t)blockIdx.x * 4 + wave; s < ns; s += (int64_t)gridDim.x * 4) {
    const int32_t rp = rowptr[min(s * B + min(lane, B), (int64_t)m)];
    const int32_t p0 = __shfl(rp, 0, 64), p1 = __shfl(rp, B, 64), E = p1 - p0;
    if (E == 0) continue;  // wave-uniform
    if (E > kSmall) {
      if (lane == 0) mid[atomicAdd(&agg->n_mid[LB - 2], 1u)] = (int32_t)s;
      continue;
    }
    const int lg = max(6, 33 - __builtin_clz(((uint32_t)E - 1u) | 1u));  // 2^lg >= 2 E
    const uint32_t mask = (1u << lg) - 1;
    for (uint32_t t = lane; t <= mask; t += 64) {
      vtab[t] = UINT32_MAX;
      if constexpr (kFill) ((volatile uint32_t *)cnts[wave])[t] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // positions are unsigned: those past a strip that ends near entry 2^31 pass INT32_MAX
    const uint32_t end = (uint32_t)p1;
    int32_t fresh_here = 0, next = lane < E ? colidx[p0 + lane] : 0, last = 0;
    for (uint32_t q = (uint32_t)p0; q < end; q += 64) {  // wave-uniform
      const uint32_t p = q + lane;
      const bool in = p < end;
      const int32_t c = next;
      if (p + 64 < end) next = colidx[p + 64];  // behind this turn's work
      if constexpr (LB == 4) {
        int32_t prev = __shfl_up(c, 1, 64);
        if (lane == 0) prev = last;
        last = __shfl(c, 63, 64);
        int r = 0;  // the last row starting at or before p
#pragma unroll
        for (int st = B / 2; st >= 1; st >>= 1) r += (uint32_t)__shfl(rp, r + st, 64) <= p ? st : 0;
        const int32_t rs = __shfl(rp, r, 64);
        if (in) {
          sum.bad |= entry_bad((int32_t)p, rs, c, prev, k);
          sum.diag += c == s * B + r;
        }
      }
      if (in) {
        bool fresh;
        const uint32_t h = table_slot(tab, mask, lg, (uint32_t)c >> LB, fresh);
        fresh_here += fresh;
        if constexpr (kFill) atomicAdd(&cnts[wave][h], 1u);
        (void)h;
      }
    }
    const int32_t blocks = (int32_t)wave_sum((u64)fresh_here);
    if (lane == 0) sum.blocks += (u64)blocks;
    sum.width = max(sum.width, blocks);
    if constexpr (kFill) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (uint32_t t = lane; t <= mask; t += 64)
        sum.tile((int32_t)((volatile uint32_t *)cnts[wave])[t], dense_threshold);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  sum.template flush<LB, ALL>(agg, part);
}

// Middling strips, one workgroup of 512 threads each; longer ones go to the
// list of long strips.
template <int LB, bool ALL>
__global__ __launch_bounds__(512) void k_an_strips_mid(const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ colidx, int32_t m, int32_t k,
                                                       int32_t dense_threshold, const int32_t *__restrict__ mid,
                                                       int32_t *__restrict__ big, DevAgg *__restrict__ agg) {
  constexpr bool kFill = LB == 4 && ALL;
  constexpr int B = 1 << LB;
  __shared__ uint32_t tab[2 * kMid];
  __shared__ uint32_t cnt[kFill ? kMid : 1];  // 16-bit counters: at most kMid entries
  __shared__ int32_t rps[B + 1];
  __shared__ u64 part[8];
  __shared__ int32_t found;
  if (agg->bad_rows) return;
  StripSums sum;
  const uint32_t n = agg->n_mid[LB - 2];
  for (uint32_t t = blockIdx.x; t < n; t += gridDim.x) {
    const int64_t s = mid[t];
    __syncthreads();
    if (threadIdx.x <= B) rps[threadIdx.x] = rowptr[min(s * B + threadIdx.x, (int64_t)m)];
    if (threadIdx.x == 0) found = 0;
    __syncthreads();
    const int32_t p0 = rps[0], p1 = rps[B];
    if (p1 - p0 > kMid) {  // workgroup-uniform
      if (threadIdx.x == 0) big[atomicAdd(&agg->n_big[LB - 2], 1u)] = (int32_t)s;
      continue;
    }
    const int lg = 33 - __builtin_clz((uint32_t)(p1 - p0) - 1u);  // more than kSmall entries: 2^lg at least twice them
    for (uint32_t i = threadIdx.x; i < (1u << lg); i += 512) tab[i] = UINT32_MAX;
    if constexpr (kFill)
      for (uint32_t i = threadIdx.x; i < (1u << lg) / 2; i += 512) cnt[i] = 0;
    __syncthreads();
    int32_t fresh_here = 0;
    for (int64_t pp = (int64_t)p0 + threadIdx.x; pp < p1; pp += 512) {
      const int32_t p = (int32_t)pp;
      const int32_t c = colidx[p];
      if constexpr (LB == 4) {
        int r = 0;
#pragma unroll
        for (int st = B / 2; st >= 1; st >>= 1) r += rps[r + st] <= p ? st : 0;
        sum.bad |= entry_bad(p, rps[r], c, p > p0 ? colidx[p - 1] : 0, k);
        sum.diag += c == s * B + r;
      }
      bool fresh;
      const uint32_t h = table_slot(tab, (1u << lg) - 1, lg, (uint32_t)c >> LB, fresh);
      fresh_here += fresh;
      if constexpr (kFill) atomicAdd(&cnt[h >> 1], 1u << (16 * (h & 1)));
      (void)h;
    }
    sum.blocks += (u64)fresh_here;
    if constexpr (LB == 4) {
      const u64 w = wave_sum((u64)fresh_here);
      if ((threadIdx.x & 63) == 0) atomicAdd(&found, (int32_t)w);
      __syncthreads();
      sum.width = max(sum.width, found);
      if constexpr (ALL)
        for (uint32_t i = threadIdx.x; i < (1u << lg) / 2; i += 512) {
          sum.tile((int32_t)(cnt[i] & 0xffffu), dense_threshold);
          sum.tile((int32_t)(cnt[i] >> 16), dense_threshold);
        }
    }
  }
  sum.template flush<LB, ALL>(agg, part);
}

// Long strips, one workgroup of 1,024 threads per window of kWindow columns: each
// row's entries of the window by binary search, each block column one bit (with
// fill counts: one 16-bit counter).  big_blocks[t]: blocks of strip t.
//
// The windows take every entry of a row exactly once whether the row is sorted
// or not, so the checks at b = 16 see every entry: the search for a smaller
// column never ends further right (its test col[mid] < v holds for every larger
// v too), one window's end is the next one's start by the same search, and the
// first and last windows are widened to the row's ends.
template <int LB, bool ALL>
__global__ __launch_bounds__(1024) void k_an_strips_big(const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ colidx, int32_t m, int32_t k,
                                                       int32_t dense_threshold, const int32_t *__restrict__ big,
                                                       int32_t *__restrict__ big_blocks, DevAgg *__restrict__ agg) {
  constexpr bool kFill = LB == 4 && ALL;
  constexpr int B = 1 << LB;
  constexpr int kBlocks = kWindow >> LB;
  constexpr int kWords = kFill ? kBlocks / 2 : kBlocks / 32;
  __shared__ uint32_t words[kWords];
  __shared__ int32_t lo[2 * B], rs[B], before[B + 1];
  __shared__ u64 part[16];
  __shared__ int32_t found;
  if (agg->bad_rows) return;
  StripSums sum;
  const int64_t nw = ((int64_t)k + kWindow - 1) / kWindow, n = (int64_t)agg->n_big[LB - 2] * nw;
  for (int64_t t = blockIdx.x; t < n; t += gridDim.x) {
    const int64_t s = big[t / nw], base = t % nw * kWindow;
    __syncthreads();
    if (threadIdx.x < 2 * B) {  // the window's first entry in each row, and the next window's
      const int r = threadIdx.x % B, side = threadIdx.x / B;
      const int64_t i = s * B + r;
      int32_t a = 0;
      if (i < m) {
        const int32_t p0 = rowptr[i], p1 = rowptr[i + 1];
        if (side == 0) rs[r] = p0;
        a = side == 0 && base == 0            ? p0
            : side == 1 && base + kWindow >= k ? p1
                                               : lower_bound_dev(colidx, p0, p1, base + side * kWindow);
      }
      lo[threadIdx.x] = a;
    }
    if (threadIdx.x == 0) found = 0;
    for (int i = threadIdx.x; i < kWords; i += 1024) words[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
      before[0] = 0;
      for (int i = 0; i < B; ++i) before[i + 1] = before[i] + lo[B + i] - lo[i];
    }
    __syncthreads();
    const int32_t total = before[B];
    if (total == 0) continue;  // workgroup-uniform
    for (int64_t ii = threadIdx.x; ii < total; ii += 1024) {  // rows in no order: up to all entries
      const int32_t i = (int32_t)ii;
      int r = 0;
#pragma unroll
      for (int st = B / 2; st >= 1; st >>= 1) r += before[r + st] <= i ? st : 0;
      const int32_t p = lo[r] + (i - before[r]), c = colidx[p];
      if constexpr (LB == 4) {
        sum.bad |= entry_bad(p, rs[r], c, p > rs[r] ? colidx[p - 1] : 0, k);
        sum.diag += c == s * B + r;
      }
      const int64_t d = (int64_t)c - base;
      if (d < 0 || d >= kWindow) continue;  // an unsorted row
      const uint32_t blk = (uint32_t)d >> LB;
      if constexpr (kFill) atomicAdd(&words[blk >> 1], 1u << (16 * (blk & 1)));
      else atomicOr(&words[blk >> 5], 1u << (blk & 31));
    }
    __syncthreads();
    int32_t here = 0;
    for (int i = threadIdx.x; i < kWords; i += 1024) {
      const uint32_t w = words[i];
      if constexpr (kFill) {
        here += ((w & 0xffffu) != 0) + ((w >> 16) != 0);
        sum.tile((int32_t)(w & 0xffffu), dense_threshold);
        sum.tile((int32_t)(w >> 16), dense_threshold);
      } else {
        here += __popc(w);
      }
    }
    sum.blocks += (u64)here;
    if constexpr (LB == 4) {
      const u64 w = wave_sum((u64)here);
      if ((threadIdx.x & 63) == 0 && w) atomicAdd(&found, (int32_t)w);
      __syncthreads();
      if (threadIdx.x == 0 && found) atomicAdd(&big_blocks[t / nw], found);
    }
  }
  sum.template flush<LB, ALL>(agg, part);
}

// ---- columns
__global__ __launch_bounds__(256) void k_an_degrees(const int32_t *__restrict__ colidx, int64_t nnz,
                                                    int32_t *__restrict__ deg, const DevAgg *__restrict__ agg) {
  if (agg->bad || agg->bad_rows) return;
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p < nnz) atomicAdd(&deg[colidx[p]], 1);  // columns are in range: checked
}

__global__ __launch_bounds__(256) void k_an_cols(const int32_t *__restrict__ deg, int32_t k, DevAgg *__restrict__ agg) {
  __shared__ u64 part[4];
  u64 sq = 0;
  int32_t mx = 0;
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < k; j += (int64_t)gridDim.x * 256) {
    const int64_t d = deg[j];
    sq += (u64)(d * d);
    mx = max(mx, (int32_t)d);
  }
  block_add(&agg->col_sumsq, sq, part);
  block_max(&agg->dmax, mx, part);
}

// ---- radix selection: 11, 11 and 10 bits from the top
// Keys of UINT32_MAX are left out.  hist: 2048 counters, zero on entry and
// zeroed again by k_sel_pick.
constexpr int kSelBins = 2048;
__device__ __forceinline__ int sel_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }

// keys, or (keys null) the row lengths
__global__ __launch_bounds__(256) void k_sel_hist(const uint32_t *__restrict__ keys,
                                                  const int32_t *__restrict__ rowptr, int64_t n, int pass,
                                                  const DevAgg *__restrict__ agg, uint32_t *__restrict__ hist) {
  __shared__ uint32_t h[kSelBins];
  for (int t = threadIdx.x; t < kSelBins; t += 256) h[t] = 0;
  __syncthreads();
  const int shift = sel_shift(pass), bits = pass == 2 ? 10 : 11;
  const uint32_t prefix = agg->sel_prefix;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const uint32_t key = keys ? keys[i] : (uint32_t)(rowptr[i + 1] - rowptr[i]);
    if (key == UINT32_MAX || (pass > 0 && (key >> (shift + bits)) != prefix)) continue;
    atomicAdd(&h[(key >> shift) & ((1u << bits) - 1)], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kSelBins; t += 256)
    if (h[t]) atomicAdd(&hist[t], h[t]);
}

// Picks the bin holding the rank (pass 0: `rank`, or the lower median of the
// keys counted when rank < 0).  One workgroup of 256 threads.
__global__ __launch_bounds__(256) void k_sel_pick(int pass, int64_t rank, uint32_t *__restrict__ hist,
                                                  DevAgg *__restrict__ agg) {
  __shared__ uint32_t sum[256];
  constexpr int kEach = kSelBins / 256;
  uint32_t h[kEach], mine = 0;
  for (int t = 0; t < kEach; ++t) {
    h[t] = hist[threadIdx.x * kEach + t];
    mine += h[t];
    hist[threadIdx.x * kEach + t] = 0;
  }
  sum[threadIdx.x] = mine;
  const u64 left0 = agg->sel_rank;
  const uint32_t prefix = pass > 0 ? agg->sel_prefix : 0;
  __syncthreads();
  u64 before = 0, total = 0;
  for (int t = 0; t < 256; ++t) {
    before += t < (int)threadIdx.x ? sum[t] : 0;
    total += sum[t];
  }
  const u64 want = pass > 0 ? left0 : rank >= 0 ? (u64)rank : total ? (total - 1) / 2 : 0;
  if (pass == 0 && threadIdx.x == 0) agg->sel_n = (uint32_t)total;
  if (want >= before && want - before < mine) {
    u64 left = want - before;
    int t = 0;
    while (left >= h[t]) left -= h[t++];
    agg->sel_rank = left;
    agg->sel_prefix = prefix << (pass == 2 ? 10 : 11) | (uint32_t)(threadIdx.x * kEach + t);
  }
}

// max(|first column - row|, |last column - row|), UINT32_MAX for an empty row
__global__ __launch_bounds__(256) void k_row_reach(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx, int32_t m,
                                                   uint32_t *__restrict__ reach) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  const int32_t p0 = rowptr[i], p1 = rowptr[i + 1];
  uint32_t v = UINT32_MAX;
  if (p1 > p0) {
    const int64_t a = colidx[p0] - i, b = colidx[p1 - 1] - i;
    v = (uint32_t)max(a < 0 ? -a : a, b < 0 ? -b : b);
  }
  reach[i] = v;
}

uint32_t grid_for(int64_t items, int64_t most = INT64_MAX) {
  return (uint32_t)std::max<int64_t>(1, std::min((items + 255) / 256, most));
}

// Three passes of histogram and pick; the value ends in agg->sel_prefix.
hipError_t launch_select(const uint32_t *keys, const int32_t *rowptr, int64_t n, int64_t rank, uint32_t *hist,
                         DevAgg *agg, hipStream_t s) {
  for (int pass = 0; pass < 3; ++pass) {
    hipLaunchKernelGGL(k_sel_hist, dim3(grid_for(n, 512)), dim3(256), 0, s, keys, rowptr, n, pass, agg, hist);
    hipLaunchKernelGGL(k_sel_pick, dim3(1), dim3(256), 0, s, pass, rank, hist, agg);
  }
  return hipGetLastError();
}

// The three passes over strips of 2^LB rows.  Persistent grids: the lists'
// lengths are known on the device only.
template <int LB, bool ALL>
hipError_t launch_strips(const sd_csr_t *A, int32_t dense_threshold, int32_t *mid, int32_t *big, int32_t *big_blocks,
                         DevAgg *agg, hipStream_t s) {
  const int64_t ns = ((int64_t)A->m + (1 << LB) - 1) >> LB;
  const uint32_t g = (uint32_t)std::max<int64_t>(1, std::min<int64_t>((ns + 3) / 4, 2048));
  hipLaunchKernelGGL((k_an_strips<LB, ALL>), dim3(g), dim3(256), 0, s, A->rowptr, A->colidx, A->m, A->k,
                     dense_threshold, mid, agg);
  if (A->nnz > kSmall) {
    const uint32_t gm = (uint32_t)std::min<int64_t>(A->nnz / kSmall + 1, 768);
    hipLaunchKernelGGL((k_an_strips_mid<LB, ALL>), dim3(gm), dim3(512), 0, s, A->rowptr, A->colidx, A->m, A->k,
                       dense_threshold, mid, big, agg);
  }
  if (A->nnz > kMid) {
    const int64_t nw = ((int64_t)A->k + kWindow - 1) / kWindow;
    const uint32_t gb = (uint32_t)std::min<int64_t>((A->nnz / kMid + 1) * nw, 1024);
    hipLaunchKernelGGL((k_an_strips_big<LB, ALL>), dim3(gb), dim3(1024), 0, s, A->rowptr, A->colidx, A->m, A->k,
                       dense_threshold, big, big_blocks, agg);
  }
  return hipGetLastError();
}

// Device scratch, given back once the stream has drained (an early error
// return may leave kernels that use it in flight).
struct DevBuf {
  hipStream_t s;
  void *p = nullptr;
  ~DevBuf() {
    if (p) sd::pool_free(p, hipStreamSynchronize(s) == hipSuccess ? sd::kIdle : sd::kUnknown);
  }
};

int hip_status(hipError_t e) {
  if (e == hipSuccess) return SD_OK;
  return e == hipErrorOutOfMemory ? SD_ERR_OUT_OF_MEMORY : SD_ERR_HIP;
}

// Offsets of the scratch arrays in one allocation.  The first n_zero words
// start at zero.
struct Layout {
  size_t words = 0;
  size_t take(size_t n) {  // 256-byte steps
    const size_t at = words;
    words += (n + 63) & ~(size_t)63;
    return at;
  }
};

}  // namespace

namespace sd {

int analyze_device(const sd_csr_t *A, int32_t dense_threshold, sd_stats_t *out, hipStream_t s, DeviceStats what) {
  if (!A || !out) return SD_ERR_INVALID_VALUE;
  if (dense_threshold == 0) dense_threshold = 128;
  if (dense_threshold < 1 || dense_threshold > 256) return SD_ERR_INVALID_VALUE;
  const int32_t m = A->m, k = A->k;
  const int64_t nnz = A->nnz;
  if (m < 0 || k < 0 || nnz < 0) return SD_ERR_INVALID_CSR;
  if (nnz >= ((int64_t)1 << 31)) return SD_ERR_OVERFLOW;
  if (!A->rowptr || (nnz > 0 && (!A->colidx || !A->values))) return SD_ERR_INVALID_VALUE;
  if (nnz > 0 && (m == 0 || k == 0)) return SD_ERR_INVALID_CSR;
  const bool all = what == kAllStats;

  const size_t n_big = (size_t)(nnz / kMid + 1);
  Layout L;
  const size_t at_agg = L.take((sizeof(DevAgg) + 3) / 4), at_len = L.take(kLenBins), at_blocks = L.take(n_big);
  const size_t at_sel = L.take(all ? kSelBins : 0), at_deg = L.take(all ? (size_t)k : 0);
  const size_t n_zero = L.words;
  const size_t at_mid = L.take(((size_t)m + 3) / 4), at_big = L.take(n_big), at_span = L.take(all ? (size_t)m : 0);
  DevBuf buf{s};
  hipError_t e;
  if ((e = sd::pool_alloc(&buf.p, 4 * L.words)) != hipSuccess) return hip_status(e);
  uint32_t *w = static_cast<uint32_t *>(buf.p);
  DevAgg *agg = reinterpret_cast<DevAgg *>(w + at_agg);
  uint32_t *len_hist = w + at_len, *sel_hist = w + at_sel, *spans = all ? w + at_span : nullptr;
  int32_t *deg = reinterpret_cast<int32_t *>(w + at_deg), *mid = reinterpret_cast<int32_t *>(w + at_mid);
  int32_t *big = reinterpret_cast<int32_t *>(w + at_big), *big_blocks = reinterpret_cast<int32_t *>(w + at_blocks);
  hipLaunchKernelGGL(k_an_zero, dim3(grid_for((int64_t)n_zero, 1024)), dim3(256), 0, s, w, (int64_t)n_zero);
  // one workgroup at least: it checks the ends of the row pointers
  hipLaunchKernelGGL(k_an_rows, dim3((uint32_t)std::max<int64_t>(1, std::min<int64_t>(((int64_t)m + 511) / 512, 512))),
                     dim3(256), 0, s, A->rowptr, A->colidx, m, nnz, len_hist, spans, agg);
  if ((e = hipGetLastError()) != hipSuccess) return hip_status(e);
  if (nnz > 0) {
    if (all) {
      if ((e = launch_strips<4, true>(A, dense_threshold, mid, big, big_blocks, agg, s)) != hipSuccess ||
          (e = launch_strips<3, true>(A, dense_threshold, mid, big, big_blocks, agg, s)) != hipSuccess ||
          (e = launch_strips<2, true>(A, dense_threshold, mid, big, big_blocks, agg, s)) != hipSuccess)
        return hip_status(e);
      hipLaunchKernelGGL(k_an_degrees, dim3(grid_for(nnz)), dim3(256), 0, s, A->colidx, nnz, deg, agg);
      hipLaunchKernelGGL(k_an_cols, dim3(grid_for(k, 1024)), dim3(256), 0, s, deg, k, agg);
      if ((e = launch_select(spans, nullptr, m, -1, sel_hist, agg, s)) != hipSuccess) return hip_status(e);
    } else if ((e = launch_strips<4, false>(A, dense_threshold, mid, big, big_blocks, agg, s)) != hipSuccess) {
      return hip_status(e);
    }
  }
  hipLaunchKernelGGL(k_an_finish, dim3(1), dim3(256), 0, s, len_hist, m, big_blocks, agg);
  DevAgg h;
  if ((e = hipGetLastError()) != hipSuccess ||
      (e = hipMemcpyAsync(&h, agg, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return hip_status(e);
  if (h.bad || h.bad_rows) return SD_ERR_INVALID_CSR;
  const uint32_t span_median = h.sel_prefix;

  // a quartile in the last length bin (a matrix of very long rows): selected among the row lengths
  for (int q = 0; q < 3 && m > 0; ++q) {
    if (h.quart[q] >= 0) continue;
    const int64_t rank = q == 2 ? 3 * (int64_t)(m - 1) / 4 : q == 1 ? (m - 1) / 2 : (m - 1) / 4;
    // the length histogram is done with: its first bins, zeroed, serve the selection
    hipLaunchKernelGGL(k_an_zero, dim3(8), dim3(256), 0, s, len_hist, (int64_t)kSelBins);
    uint32_t len = 0;
    if ((e = launch_select(nullptr, A->rowptr, m, rank, len_hist, agg, s)) != hipSuccess ||
        (e = hipMemcpyAsync(&len, &agg->sel_prefix, sizeof(len), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
      return hip_status(e);
    h.quart[q] = (int32_t)len;
  }

  sd_stats_t st;
  std::memset(&st, 0, sizeof(st));
  st.m = m;
  st.k = k;
  st.nnz = nnz;
  st.dense_threshold = dense_threshold;
  st.row_min = m > 0 ? INT32_MAX - h.rmin_c : 0;
  st.row_max = h.rmax;
  st.empty_rows = (int64_t)m - (int64_t)h.nonempty;
  for (int t = 0; t < 33; ++t) st.row_hist[t] = (int64_t)h.row_hist[t];
  if (m > 0) {
    st.row_q25 = h.quart[0];
    st.row_q50 = h.quart[1];
    st.row_q75 = h.quart[2];
  }
  if (all && h.nonempty > 0) st.row_span_median = (int64_t)span_median;
  st.col_deg_max = h.dmax;
  st.diag_nnz = (int64_t)h.diag;
  st.nnzb4 = (int64_t)h.nnzb[0];
  st.nnzb8 = (int64_t)h.nnzb[1];
  st.nnzb16 = (int64_t)h.nnzb[2];
  st.dense_tiles16 = (int64_t)h.dense_tiles;
  st.dense_tile_nnz16 = (int64_t)h.dense_nnz;
  st.bell16_width = h.width16;
  for (int t = 0; t < 8; ++t) st.fill16_hist[t] = (int64_t)h.fill16_hist[t];
  st.sell16_slots = (int64_t)h.sell_slots[0];
  st.sell32_slots = (int64_t)h.sell_slots[1];
  st.sell512_slots = (int64_t)h.sell_slots[2];
  StatsSums sum;
  sum.row_sumsq = (int64_t)h.row_sumsq;
  sum.col_sumsq = (int64_t)h.col_sumsq;
  sum.span_sum = (int64_t)h.span_sum;
  sum.nonempty = (int64_t)h.nonempty;
  sum.gap_num = (int64_t)h.gap_num;
  sum.gap_den = (int64_t)h.gap_den;
  finish_stats(sum, &st);
  *out = st;
  return SD_OK;
}

hipError_t dev_median_reach(const int32_t *rowptr, const int32_t *colidx, int32_t m, hipStream_t s, int64_t *out) {
  *out = 0;
  if (m == 0) return hipSuccess;
  Layout L;
  const size_t at_agg = L.take((sizeof(DevAgg) + 3) / 4), at_sel = L.take(kSelBins), n_zero = L.words;
  const size_t at_key = L.take((size_t)m);
  DevBuf buf{s};
  hipError_t e;
  if ((e = sd::pool_alloc(&buf.p, 4 * L.words)) != hipSuccess) return e;
  uint32_t *w = static_cast<uint32_t *>(buf.p);
  DevAgg *agg = reinterpret_cast<DevAgg *>(w + at_agg);
  hipLaunchKernelGGL(k_an_zero, dim3(8), dim3(256), 0, s, w, (int64_t)n_zero);
  hipLaunchKernelGGL(k_row_reach, dim3(grid_for(m)), dim3(256), 0, s, rowptr, colidx, m, w + at_key);
  uint32_t got[2] = {0, 0};  // the median, the number of non-empty rows
  static_assert(offsetof(DevAgg, sel_n) == offsetof(DevAgg, sel_prefix) + 4, "read together");
  if ((e = launch_select(w + at_key, nullptr, m, -1, w + at_sel, agg, s)) != hipSuccess ||
      (e = hipMemcpyAsync(got, &agg->sel_prefix, sizeof(got), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  if (got[1]) *out = (int64_t)got[0];
  return hipSuccess;
}

}  // namespace sd
