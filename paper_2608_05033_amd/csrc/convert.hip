// Device-side conversions and partitions for plans built from a CSR matrix
// already in device memory (sd_plan_device).  Each produces exactly the
// arrays of its host counterpart in host_plan.cpp:
//
//  * ELL        rows padded to W slots, column -1 / value +0.0f padding;
//  * merge path U + 1 split coordinates (rows, nonzeros consumed), one binary
//               search per coordinate on the merged sequence of row ends and
//               nonzero indices;
//  * heavy split light rows (r < T), by the column of their last nonzero or in
//               row order; heavy rows and the first chunk of each (plus the
//               total); chunks (row, begin, end) of at most c nonzeros in row
//               and chunk order and their processing order; the entries in that
//               layout.  Places come from running sums over the rows;
//  * transpose  the CSR of A^T: a stable radix sort (hipCUB) of the nonzeros'
//               (row, value) pairs by column keeps each column's rows ascending,
//               as the host's counting sort does; row pointers by binary search
//               in the sorted keys;
//  * 16x16 BSR / Blocked-ELL  one workgroup per block-row: its block columns are
//               bits in LDS, a bit's rank is its block's place; counts, a scan,
//               then columns and values (row-major inside the block);
//  * SELL-C-sigma  a stable radix sort of the rows by (sort window, longest
//               first) gives the permutation; slice widths, slice offsets by
//               an exclusive sum, then one thread per sorted row copies its
//               entries into the padded slice;
//  * windows    a stable radix sort of the nonzeros by (window, column): a
//               run of two or more equal keys is a staged column of that
//               window; scans number the runs and the staged columns, window
//               pointers by binary search, then one thread per nonzero writes
//               its code (staged position or column) and value;
//  * cold tags  column degrees by integer atomics; the hot threshold is taken
//               on the host from the degrees exactly as the host conversion
//               takes it; then one thread per nonzero sets bit 31 of a cold
//               column;
//  * pattern hash  the sum, modulo 2^64, of a mixed (array, position, value)
//               term per row pointer and column index: the same on the host
//               (pattern_hash in runtime.hip) and, being a sum, computed in any
//               order on the device.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cstdint>
#include <functional>
#include <vector>

#include "kernels.h"

namespace sd {
namespace {

__global__ __launch_bounds__(256) void k_ell_fill(const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ colidx,
                                                  const float *__restrict__ vals, int32_t m, int32_t W,
                                                  int32_t *__restrict__ ecol, float *__restrict__ eval) {
  const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (slot >= (int64_t)m * W) return;
  const int64_t i = slot / W, t = slot - i * W;
  const int32_t p0 = rowptr[i], r = rowptr[i + 1] - p0;
  if (t < r) {
    ecol[slot] = colidx[p0 + t];
    eval[slot] = vals[p0 + t];  // a bit copy: loads and stores move the pattern unchanged
  } else {
    ecol[slot] = -1;
    eval[slot] = 0.0f;
  }
}

__global__ __launch_bounds__(256) void k_merge_coords(const int32_t *__restrict__ rowptr, int32_t m, int64_t nnz,
                                                      int32_t U, int64_t L, int32_t *__restrict__ coords) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u > U) return;
  const int64_t total = (int64_t)m + nnz;
  const int64_t d = min(u * L, total);
  int64_t lo = max((int64_t)0, d - nnz), hi = min(d, (int64_t)m);
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if ((int64_t)rowptr[mid + 1] + mid >= d) hi = mid;
    else lo = mid + 1;
  }
  coords[2 * u] = (int32_t)lo;
  coords[2 * u + 1] = (int32_t)(d - lo);
}

// the row holding nonzero p of a valid CSR (m >= 1): the last row starting at
// or before p
__device__ inline int32_t row_of(const int32_t *__restrict__ rowptr, int32_t m, int64_t p) {
  int32_t lo = 0, hi = m - 1;
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if (rowptr[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// t_rowptr[j] = number of sorted keys below j, for j in [0, k]
__global__ __launch_bounds__(256) void k_transpose_rowptr(const uint32_t *__restrict__ keys, int64_t nnz, int32_t k,
                                                          int32_t *__restrict__ t_rowptr) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j > k) return;
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if ((int64_t)keys[mid] < j) lo = mid + 1;
    else hi = mid;
  }
  t_rowptr[j] = (int32_t)lo;
}

// (row, value bits) of nonzero p, what the sort by column carries along
__global__ __launch_bounds__(256) void k_transpose_pack(const int32_t *__restrict__ rowptr, int32_t m,
                                                        const float *__restrict__ vals, int64_t nnz,
                                                        uint64_t *__restrict__ packed) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= nnz) return;
  packed[p] = (uint64_t)(uint32_t)row_of(rowptr, m, p) << 32 | __float_as_uint(vals[p]);
}

__global__ __launch_bounds__(256) void k_transpose_unpack(const uint64_t *__restrict__ packed, int64_t nnz,
                                                          int32_t *__restrict__ t_colidx,
                                                          float *__restrict__ t_vals) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= nnz) return;
  const uint64_t x = packed[q];
  t_colidx[q] = (int32_t)(x >> 32);
  t_vals[q] = __uint_as_float((uint32_t)x);
}

// ---- 16x16 blocks
// One workgroup per block-row.  Its block columns are bits of a window of
// kBlkWindow blocks in LDS (windows in turn where the row reaches further), set
// by its entries: a bit's rank is its block's place, in ascending block-column
// order.  A pass counts, a scan places the block-rows, a second pass sets the
// bits again and writes columns and values, zeros first.  The writes bound it: 8192
// block-rows of 32 blocks, 60 M nonzeros, plan in 1.05 ms, against 7.2 ms with a
// sort of all nonzeros by (block-row, block column), run lengths and a search for
// each nonzero's block.
constexpr int kBlkWindow = 65536, kBlkWords = kBlkWindow / 32;

struct BlkLds {
  uint32_t words[kBlkWords];
  int32_t prefix[kBlkWords];
  int32_t rps[17];
  int32_t lo, hi, waves[4];
};

// Row starts, and the first and last block column (hi < lo: no entries).
__device__ __forceinline__ void blk_row(BlkLds &l, const int32_t *__restrict__ rowptr,
                                        const int32_t *__restrict__ colidx, int64_t br, int32_t m) {
  __syncthreads();  // the previous block-row is done with
  if (threadIdx.x == 0) {
    l.lo = INT32_MAX;
    l.hi = -1;
  }
  if (threadIdx.x <= 16) l.rps[threadIdx.x] = rowptr[min(br * 16 + threadIdx.x, (int64_t)m)];
  __syncthreads();
  if (threadIdx.x < 16) {
    const int32_t p0 = l.rps[threadIdx.x], p1 = l.rps[threadIdx.x + 1];
    if (p1 > p0) {
      atomicMin(&l.lo, colidx[p0] / 16);
      atomicMax(&l.hi, colidx[p1 - 1] / 16);
    }
  }
  __syncthreads();
}

// Sets the bits of the window starting at block column base; returns the words in use.
__device__ __forceinline__ int blk_bits(BlkLds &l, const int32_t *__restrict__ colidx, int32_t base) {
  const int words = min(kBlkWords, (l.hi - base) / 32 + 1);
  for (int i = threadIdx.x; i < words; i += 256) l.words[i] = 0;
  __syncthreads();
  for (int64_t p = (int64_t)l.rps[0] + threadIdx.x; p < l.rps[16]; p += 256) {
    const int32_t d = colidx[p] / 16 - base;
    if (d >= 0 && d < kBlkWindow) atomicOr(&l.words[d >> 5], 1u << (d & 31));
  }
  __syncthreads();
  return words;
}

__global__ __launch_bounds__(256) void k_blk_count(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx, int32_t m, int64_t mb,
                                                   int32_t *__restrict__ count) {
  __shared__ BlkLds l;
  if (blockIdx.x == 0 && threadIdx.x == 0) count[mb] = 0;
  for (int64_t br = blockIdx.x; br < mb; br += gridDim.x) {
    blk_row(l, rowptr, colidx, br, m);
    int32_t n = 0;
    for (int64_t base = l.lo; base <= l.hi; base += kBlkWindow) {  // workgroup-uniform
      const int words = blk_bits(l, colidx, (int32_t)base);
      for (int i = threadIdx.x; i < words; i += 256) n += __popc(l.words[i]);
      __syncthreads();
    }
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    if ((threadIdx.x & 63) == 0) l.waves[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) count[br] = l.waves[0] + l.waves[1] + l.waves[2] + l.waves[3];
  }
}

// The longest block-row of ptr [mb + 1]; *out starts at 0.
__global__ __launch_bounds__(256) void k_blk_width(const int32_t *__restrict__ ptr, int64_t mb,
                                                   int32_t *__restrict__ out) {
  int32_t w = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < mb; i += (int64_t)gridDim.x * 256)
    w = max(w, ptr[i + 1] - ptr[i]);
  for (int o = 32; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, 64));
  if ((threadIdx.x & 63) == 0 && w) atomicMax(out, w);
}

// ell_width < 0: block-row br's blocks at ptr[br] ..; else at br * ell_width .., the
// rest of its slots padding (column -1, zero values).  The last workgroup (br = mb)
// writes the zero block after the stored ones.
__global__ __launch_bounds__(256) void k_blk_fill(const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ colidx,
                                                  const float *__restrict__ vals, int32_t m, int64_t mb,
                                                  const int32_t *__restrict__ ptr, int32_t ell_width, int64_t slots,
                                                  int32_t *__restrict__ bcol, float *__restrict__ bval) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  __shared__ BlkLds l;
  auto zero = [&](int64_t first, int64_t n) {  // blocks [first, first + n)
    f4 *z = reinterpret_cast<f4 *>(bval + first * 256);
    for (int64_t i = threadIdx.x; i < n * 64; i += 256) z[i] = (f4)(0.0f);
  };
  for (int64_t br = blockIdx.x; br <= mb; br += gridDim.x) {  // workgroup-uniform
    if (br == mb) {
      zero(slots, 1);
      if (threadIdx.x == 0) bcol[slots] = -1;
      continue;
    }
    blk_row(l, rowptr, colidx, br, m);
    const int64_t first = ell_width < 0 ? (int64_t)ptr[br] : br * ell_width;
    const int32_t total = ptr[br + 1] - ptr[br];
    zero(first, ell_width < 0 ? total : ell_width);
    for (int32_t i = total + (int32_t)threadIdx.x; i < ell_width; i += 256) bcol[first + i] = -1;
    int64_t slot0 = first;  // of the window's first block
    for (int64_t base = l.lo; base <= l.hi; base += kBlkWindow) {  // workgroup-uniform
      const int words = blk_bits(l, colidx, (int32_t)base);
      // exclusive prefix of the words' bit counts: 8 consecutive words per thread
      constexpr int kEach = kBlkWords / 256;
      const int w0 = threadIdx.x * kEach, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
      int32_t mine = 0;
      for (int i = w0; i < min(words, w0 + kEach); ++i) mine += __popc(l.words[i]);
      int32_t x = mine;
      for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
      }
      if (lane == 63) l.waves[wave] = x;
      __syncthreads();
      int32_t at = x - mine, all = 0;
      for (int i = 0; i < 4; ++i) {
        if (i < wave) at += l.waves[i];
        all += l.waves[i];
      }
      for (int i = w0; i < min(words, w0 + kEach); ++i) {
        l.prefix[i] = at;
        for (uint32_t w = l.words[i]; w; w &= w - 1) bcol[slot0 + at++] = (int32_t)base + i * 32 + __ffs(w) - 1;
      }
      __syncthreads();  // prefixes, and the zeros under this block-row's values
      for (int64_t pp = (int64_t)l.rps[0] + threadIdx.x; pp < l.rps[16]; pp += 256) {
        const int32_t p = (int32_t)pp, c = colidx[p];
        const int32_t d = c / 16 - (int32_t)base;
        if (d < 0 || d >= kBlkWindow) continue;
        int r = 0;  // the last row starting at or before p
#pragma unroll
        for (int st = 8; st >= 1; st >>= 1) r += l.rps[r + st] <= p ? st : 0;
        const int64_t slot = slot0 + l.prefix[d >> 5] + __popc(l.words[d >> 5] & ((1u << (d & 31)) - 1u));
        bval[slot * 256 + r * 16 + c % 16] = vals[p];
      }
      slot0 += all;
      __syncthreads();  // before the words are cleared for the next window
    }
  }
}

// ---- SELL-C-sigma
__global__ __launch_bounds__(256) void k_sell_keys(const int32_t *__restrict__ rowptr, int32_t m, int32_t sigma,
                                                   int32_t row_max, uint64_t *__restrict__ keys,
                                                   int32_t *__restrict__ rows) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  const int32_t len = rowptr[i + 1] - rowptr[i];
  keys[i] = (uint64_t)(i / sigma) * (uint64_t)(row_max + 1) + (uint64_t)(row_max - len);
  rows[i] = (int32_t)i;
}

__global__ __launch_bounds__(256) void k_sell_sizes(const int32_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ perm, int32_t m, int32_t C,
                                                    int64_t ns, int64_t *__restrict__ size) {
  const int64_t sl = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (sl >= ns) return;
  const int64_t r0 = sl * C, r1 = min((int64_t)m, r0 + C);
  int32_t w = 0;
  for (int64_t i = r0; i < r1; ++i) {
    const int32_t r = perm[i];
    w = max(w, rowptr[r + 1] - rowptr[r]);
  }
  size[sl] = (r1 - r0) * w;
}

__global__ __launch_bounds__(256) void k_sell_fill(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx,
                                                   const float *__restrict__ vals, const int32_t *__restrict__ perm,
                                                   const int64_t *__restrict__ sptr, int32_t m, int32_t C,
                                                   int32_t *__restrict__ scol, float *__restrict__ sval) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  const int64_t sl = i / C, r0 = sl * C, rows = min((int64_t)m, r0 + C) - r0;
  const int64_t w = (sptr[sl + 1] - sptr[sl]) / rows;
  const int32_t r = perm[i], p0 = rowptr[r], len = rowptr[r + 1] - p0;
  const int64_t base = sptr[sl] + (i - r0) * w;
  for (int32_t t = 0; t < len; ++t) {
    scol[base + t] = colidx[p0 + t];
    sval[base + t] = vals[p0 + t];
  }
}

__global__ __launch_bounds__(256) void k_col_degree(const int32_t *__restrict__ colidx, int64_t nnz,
                                                    int32_t *__restrict__ deg) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p < nnz) atomicAdd(&deg[colidx[p]], 1);
}

__global__ __launch_bounds__(256) void k_tag_cold(const int32_t *__restrict__ colidx, int64_t nnz,
                                                  const int32_t *__restrict__ deg, int32_t D,
                                                  int32_t *__restrict__ tagged) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= nnz) return;
  const int32_t c = colidx[p];
  tagged[p] = deg[c] >= D ? c : (int32_t)((uint32_t)c | 0x80000000u);
}

// splitmix64's finaliser
__device__ __host__ inline uint64_t mix64(uint64_t x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

__global__ __launch_bounds__(256) void k_pattern_hash(const int32_t *__restrict__ a, int64_t len, uint64_t salt,
                                                      unsigned long long *__restrict__ sum) {
  uint64_t acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (int64_t)gridDim.x * 256)
    acc += mix64(salt ^ ((uint64_t)i << 32 | (uint32_t)a[i]));
  atomicAdd(sum, (unsigned long long)acc);  // a sum: the same total in any order
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *__restrict__ x, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) x[i] = v;
}

uint32_t grid_for(int64_t items) { return (uint32_t)((items + 255) / 256); }

// Device scratch of one conversion.  Given back on return, after the stream has
// drained: an early error return may leave kernels that use it in flight.
struct Scratch {
  hipStream_t s;
  void *p[12] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                 nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  explicit Scratch(hipStream_t stream) : s(stream) {}
  ~Scratch() {
    bool any = false;
    for (void *q : p) any = any || q;
    const bool drained = !any || hipStreamSynchronize(s) == hipSuccess;
    for (void *q : p)
      pool_free(q, drained ? kIdle : kUnknown);
  }
};

}  // namespace

hipError_t dev_ell(const int32_t *rowptr, const int32_t *colidx, const float *vals, int32_t m, int32_t W,
                   int32_t *ecol, float *eval, hipStream_t s) {
  const int64_t slots = (int64_t)m * W;
  if (slots == 0) return hipSuccess;
  hipLaunchKernelGGL(k_ell_fill, dim3(grid_for(slots)), dim3(256), 0, s, rowptr, colidx, vals, m, W, ecol, eval);
  return hipGetLastError();
}

hipError_t dev_merge_coords(const int32_t *rowptr, int32_t m, int64_t nnz, int32_t U, int64_t L, int32_t *coords,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_merge_coords, dim3(grid_for((int64_t)U + 1)), dim3(256), 0, s, rowptr, m, nnz, U, L, coords);
  return hipGetLastError();
}

namespace {

// ---- heavy split
// Rows are taken 1,024 per workgroup, four consecutive ones per thread.  Three
// running sums place everything: heavy rows (light rows are the others), their
// chunks, and their nonzeros.  One pass adds them per workgroup, one workgroup
// scans those sums (the host reads the three totals to size the arrays), and a
// second pass writes.  Chunks are then cut in the split layout's coordinates by
// one thread each, and the entries moved by 16 lanes per light row and a wave per
// chunk, so a row of any length is spread over the chip.
constexpr int kSplitRows = 1024;

struct SplitSums {
  uint32_t heavy, chunks, nnz;
};
__device__ __forceinline__ SplitSums operator+(SplitSums a, SplitSums b) {
  return {a.heavy + b.heavy, a.chunks + b.chunks, a.nnz + b.nnz};
}
__device__ __forceinline__ SplitSums shfl_up(SplitSums a, int d) {
  return {(uint32_t)__shfl_up((int)a.heavy, d, 64), (uint32_t)__shfl_up((int)a.chunks, d, 64),
          (uint32_t)__shfl_up((int)a.nnz, d, 64)};
}
__device__ __forceinline__ SplitSums split_row(const int32_t *__restrict__ rowptr, int64_t i, int32_t m, int32_t T,
                                               int32_t c, int32_t &p0, int32_t &len) {
  if (i >= m) return {0, 0, 0};
  p0 = rowptr[i];
  len = rowptr[i + 1] - p0;
  if (len < T) return {0, 0, 0};
  return {1, (uint32_t)(((int64_t)len + c - 1) / c), (uint32_t)len};
}

// Exclusive prefix of v over the workgroup (N waves), and the total.
template <int N>
__device__ __forceinline__ SplitSums block_prefix(SplitSums v, SplitSums *__restrict__ waves, SplitSums &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  SplitSums x = v;
  for (int d = 1; d < 64; d <<= 1) {
    const SplitSums y = shfl_up(x, d);
    if (lane >= d) x = x + y;
  }
  __syncthreads();
  if (lane == 63) waves[wave] = x;
  __syncthreads();
  SplitSums before{0, 0, 0};
  total = {0, 0, 0};
  for (int w = 0; w < N; ++w) {
    if (w < wave) before = before + waves[w];
    total = total + waves[w];
  }
  return {before.heavy + x.heavy - v.heavy, before.chunks + x.chunks - v.chunks, before.nnz + x.nnz - v.nnz};
}

__global__ __launch_bounds__(256) void k_split_sums(const int32_t *__restrict__ rowptr, int32_t m, int32_t T,
                                                    int32_t c, SplitSums *__restrict__ sums) {
  __shared__ SplitSums waves[4];
  SplitSums v{0, 0, 0}, total;
  int32_t p0, len;
  for (int t = 0; t < 4; ++t)
    v = v + split_row(rowptr, (int64_t)blockIdx.x * kSplitRows + threadIdx.x * 4 + t, m, T, c, p0, len);
  block_prefix<4>(v, waves, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// In place: sums[b] = the sum before workgroup b, sums[nb] = the total.
__global__ __launch_bounds__(1024) void k_split_scan(SplitSums *__restrict__ sums, int32_t nb) {
  __shared__ SplitSums waves[16];
  SplitSums carry{0, 0, 0};
  for (int32_t b0 = 0; b0 < nb; b0 += 1024) {  // the same trip count for every thread
    const int32_t b = b0 + (int32_t)threadIdx.x;
    SplitSums v{0, 0, 0}, total;
    if (b < nb) v = sums[b];
    const SplitSums before = block_prefix<16>(v, waves, total);
    if (b < nb) sums[b] = carry + before;
    carry = carry + total;
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(256) void k_split_fill(const int32_t *__restrict__ rowptr, int32_t m, int32_t T,
                                                    int32_t c, const SplitSums *__restrict__ sums, int32_t nb,
                                                    int32_t *__restrict__ light, int32_t *__restrict__ heavy_rows,
                                                    int32_t *__restrict__ heavy_ptr,
                                                    uint32_t *__restrict__ heavy_start) {
  __shared__ SplitSums waves[4];
  const int64_t i0 = (int64_t)blockIdx.x * kSplitRows + threadIdx.x * 4;
  SplitSums r[4], v{0, 0, 0}, total;
  int32_t p0, len;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    r[t] = split_row(rowptr, i0 + t, m, T, c, p0, len);
    v = v + r[t];
  }
  SplitSums at = sums[blockIdx.x] + block_prefix<4>(v, waves, total);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t i = i0 + t;
    if (i < m) {
      if (r[t].heavy) {
        heavy_rows[at.heavy] = (int32_t)i;
        heavy_ptr[at.heavy] = (int32_t)at.chunks;
        heavy_start[at.heavy] = at.nnz;
      } else {
        light[i - at.heavy] = (int32_t)i;
      }
    }
    at = at + r[t];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) heavy_ptr[sums[nb].heavy] = (int32_t)sums[nb].chunks;
}

// Chunk q: (row, begin, end) in the split layout, where the heavy rows' entries
// follow the light_nnz entries of the light rows; its middle column as sort key
// and, for the move, where its entries lie in the input.
__global__ __launch_bounds__(256) void k_split_chunks(const int32_t *__restrict__ rowptr,
                                                      const int32_t *__restrict__ colidx,
                                                      const int32_t *__restrict__ heavy_rows,
                                                      const int32_t *__restrict__ heavy_ptr,
                                                      const uint32_t *__restrict__ heavy_start, int32_t n_heavy,
                                                      int32_t n_chunks, int32_t c, uint32_t light_nnz,
                                                      int32_t *__restrict__ chunks, int32_t *__restrict__ from,
                                                      int32_t *__restrict__ keys, int32_t *__restrict__ idx) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= n_chunks) return;
  int32_t lo = 0, hi = n_heavy - 1;  // the last heavy row whose chunks start at or before q
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if (heavy_ptr[mid] <= q) lo = mid;
    else hi = mid - 1;
  }
  const int32_t row = heavy_rows[lo], p0 = rowptr[row], len = rowptr[row + 1] - p0;
  const int64_t off = (q - heavy_ptr[lo]) * c;
  const int32_t take = (int32_t)min((int64_t)c, len - off);
  const int64_t begin = (int64_t)light_nnz + heavy_start[lo] + off;
  chunks[3 * q] = row;
  chunks[3 * q + 1] = (int32_t)begin;
  chunks[3 * q + 2] = (int32_t)(begin + take);
  from[q] = (int32_t)(p0 + off);
  keys[q] = colidx[p0 + off + take / 2];  // the entry at (begin + end) / 2 of the split layout
  idx[q] = (int32_t)q;
}

__global__ __launch_bounds__(256) void k_last_col_keys(const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ colidx, int32_t k,
                                                       const int32_t *__restrict__ light, int64_t n,
                                                       int32_t *__restrict__ keys) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int32_t r = light[i], p1 = rowptr[r + 1];
  keys[i] = p1 > rowptr[r] ? colidx[p1 - 1] : k;
}

// Lengths of the light rows in list order, and a last 0 (their exclusive sum is
// the row pointers and the total).
__global__ __launch_bounds__(256) void k_light_lengths(const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ light, int64_t n,
                                                       int32_t *__restrict__ len) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) len[i] = rowptr[light[i] + 1] - rowptr[light[i]];
  else if (i == n) len[i] = 0;
}

// W lanes per light row.
template <int W>
__global__ __launch_bounds__(256) void k_move_light(const int32_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ colidx,
                                                    const float *__restrict__ vals,
                                                    const int32_t *__restrict__ light, int64_t n,
                                                    const int32_t *__restrict__ lptr,
                                                    int32_t *__restrict__ colidx_out, float *__restrict__ vals_out) {
  const int64_t i = (int64_t)blockIdx.x * (256 / W) + threadIdx.x / W;
  if (i >= n) return;
  const int32_t p0 = rowptr[light[i]], q0 = lptr[i], len = lptr[i + 1] - q0;
  for (int32_t t = threadIdx.x & (W - 1); t < len; t += W) {
    colidx_out[q0 + t] = colidx[p0 + t];
    vals_out[q0 + t] = vals[p0 + t];
  }
}

// A wave per chunk.
__global__ __launch_bounds__(256) void k_move_chunks(const int32_t *__restrict__ colidx,
                                                     const float *__restrict__ vals,
                                                     const int32_t *__restrict__ chunks,
                                                     const int32_t *__restrict__ from, int64_t n,
                                                     int32_t *__restrict__ colidx_out, float *__restrict__ vals_out) {
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= n) return;
  const int32_t p0 = from[q], b = chunks[3 * q + 1], len = chunks[3 * q + 2] - b;
  for (int32_t t = threadIdx.x & 63; t < len; t += 64) {
    colidx_out[b + t] = colidx[p0 + t];
    vals_out[b + t] = vals[p0 + t];
  }
}

// ---- stable sort of up to two lists of (key, value) pairs, keys below 2^bits
// A radix sort of 10 bits a pass, three launches a pass for both lists together:
// digits counted per tile, one wave per digit scans the tiles, and each tile's waves
// rank their pairs by ballots and write them.  Launches bound it at these sizes:
// analysis, plan and one product of a graph with 486 k light rows and 87 k chunks
// take 663 us, against 781 with hipCUB's sort, which merges up to 1 M pairs in 24
// launches for the two lists; a plan with 1.03 M light rows 0.70 ms against 0.82.
// Longer lists go to hipCUB's single-sweep passes: a plan with 2.2 M light rows
// takes 2.1 ms either way.
constexpr int kSortTile = 4096, kSortBits = 10, kSortDigits = 1 << kSortBits;
constexpr int64_t kSortMax = 1 << 20;

struct SortJob {
  const int32_t *key, *val;
  int32_t *key_out, *val_out;
  int32_t *count;  // [digits][tiles], then [digits] totals
  int32_t n, tiles;
};
struct SortJobs {
  SortJob j[2];
};

__global__ __launch_bounds__(256) void k_sort_count(SortJobs jobs, int shift, int digits) {
  __shared__ int32_t cnt[kSortDigits];
  const SortJob j = jobs.j[blockIdx.y];
  const int32_t tile = (int32_t)blockIdx.x;
  if (tile >= j.tiles) return;  // the whole workgroup
  for (int d = threadIdx.x; d < digits; d += 256) cnt[d] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)tile * kSortTile;
#pragma unroll
  for (int t = 0; t < kSortTile / 256; ++t) {
    const int64_t i = i0 + t * 256 + threadIdx.x;
    if (i < j.n) atomicAdd(&cnt[((uint32_t)j.key[i] >> shift) & (uint32_t)(digits - 1)], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < digits; d += 256) j.count[(int64_t)d * j.tiles + tile] = cnt[d];
}

// A wave per digit: its tiles' counts to the sums before them, and its total.
__global__ __launch_bounds__(256) void k_sort_scan(SortJobs jobs, int digits) {
  const SortJob j = jobs.j[blockIdx.y];
  const int d = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (d >= digits) return;
  int32_t *c = j.count + (int64_t)d * j.tiles;
  int32_t run = 0;
  for (int32_t t0 = 0; t0 < j.tiles; t0 += 64) {
    const int32_t t = t0 + lane, v = t < j.tiles ? c[t] : 0;
    int32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (t < j.tiles) c[t] = run + x - v;
    run += __shfl(x, 63, 64);
  }
  if (lane == 0) j.count[(int64_t)digits * j.tiles + d] = run;
}

__global__ __launch_bounds__(256) void k_sort_place(SortJobs jobs, int shift, int bits) {
  __shared__ int32_t at[4][kSortDigits];  // per wave: its pairs of a digit, then where the next one goes
  __shared__ int32_t wsum[4];
  const SortJob j = jobs.j[blockIdx.y];
  const int32_t tile = (int32_t)blockIdx.x;
  if (tile >= j.tiles) return;  // the whole workgroup
  const int digits = 1 << bits, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kRounds = kSortTile / 256;
  const int64_t i0 = (int64_t)tile * kSortTile + wave * (kSortTile / 4) + lane;
  int32_t key[kRounds], val[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool in = i0 + r * 64 < j.n;
    key[r] = in ? j.key[i0 + r * 64] : 0;
    val[r] = in ? j.val[i0 + r * 64] : 0;
  }
  for (int d = threadIdx.x; d < kSortDigits; d += 256) at[0][d] = at[1][d] = at[2][d] = at[3][d] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    if (i0 + r * 64 < j.n) atomicAdd(&at[wave][((uint32_t)key[r] >> shift) & (uint32_t)(digits - 1)], 1);
  // the digits' starts: a thread sums four digits' totals
  int32_t tot[4], mine = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int d = (int)threadIdx.x * 4 + t;
    tot[t] = d < digits ? j.count[(int64_t)digits * j.tiles + d] : 0;
    mine += tot[t];
  }
  int32_t x = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  int32_t start = x - mine;
  for (int w = 0; w < wave; ++w) start += wsum[w];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int d = (int)threadIdx.x * 4 + t;
    if (d < digits) {
      int32_t b = start + j.count[(int64_t)d * j.tiles + tile];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int32_t c = at[w][d];
        at[w][d] = b;
        b += c;
      }
    }
    start += tot[t];
  }
  __syncthreads();
  // a wave's rounds in turn: lanes of one digit take consecutive places in lane order
  const uint64_t below = ((uint64_t)1 << lane) - 1;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool in = i0 + r * 64 < j.n;
    const uint32_t dg = ((uint32_t)key[r] >> shift) & (uint32_t)(digits - 1);
    uint64_t same = __ballot(in);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (dg >> b) & 1;
      const uint64_t ones = __ballot(bit);
      same &= bit ? ones : ~ones;
    }
    const int leader = in ? __ffsll((unsigned long long)same) - 1 : lane;
    int32_t first = 0;
    if (in && lane == leader) first = atomicAdd(&at[wave][dg], __popcll(same));
    first = __shfl(first, leader, 64);
    if (in) {
      const int32_t to = first + __popcll(same & below);
      j.key_out[to] = key[r];
      j.val_out[to] = val[r];
    }
  }
}

// Sorts each job's (key, val) into (key_out, val_out); jobs with n = 0 are skipped.
// Scratch in sc.p[slot], sc.p[slot + 1].
hipError_t sort_pairs(Scratch &sc, int slot, const SortJob *job, int bits, hipStream_t s) {
  hipError_t e;
  SortJobs own{};
  int n_own = 0;
  size_t words = 0;
  const int passes = (bits + kSortBits - 1) / kSortBits, per = (bits + passes - 1) / passes;
  const int digits = 1 << per;
  for (int q = 0; q < 2; ++q) {
    if (job[q].n == 0) continue;
    if (job[q].n > kSortMax) {
      size_t tmp = 0;
      if ((e = hipcub::DeviceRadixSort::SortPairs(nullptr, tmp, job[q].key, job[q].key_out, job[q].val,
                                                  job[q].val_out, job[q].n, 0, bits, s)) != hipSuccess ||
          (e = pool_alloc(&sc.p[slot + 1 + q], std::max<size_t>(tmp, 1))) != hipSuccess ||
          (e = hipcub::DeviceRadixSort::SortPairs(sc.p[slot + 1 + q], tmp, job[q].key, job[q].key_out, job[q].val,
                                                  job[q].val_out, job[q].n, 0, bits, s)) != hipSuccess)
        return e;
      continue;
    }
    SortJob &o = own.j[n_own++] = job[q];
    o.tiles = (o.n + kSortTile - 1) / kSortTile;
    words += (size_t)digits * (o.tiles + 1) + 2 * (size_t)o.n;
  }
  if (n_own == 0) return hipSuccess;
  if ((e = pool_alloc(&sc.p[slot], sizeof(int32_t) * words)) != hipSuccess) return e;
  int32_t *w = static_cast<int32_t *>(sc.p[slot]);
  int32_t *other[2][2];  // the pairs that the passes write in turn with the outputs
  int32_t tiles = 0;
  for (int q = 0; q < n_own; ++q) {
    SortJob &o = own.j[q];
    o.count = w;
    other[q][0] = w + (size_t)digits * (o.tiles + 1);
    other[q][1] = other[q][0] + o.n;
    w = other[q][1] + o.n;
    tiles = std::max(tiles, o.tiles);
  }
  for (int p = 0; p < passes; ++p) {
    SortJobs now = own;
    for (int q = 0; q < n_own; ++q) {
      SortJob &o = now.j[q];
      if ((passes - 1 - p) % 2) {  // the last pass writes the outputs
        o.key_out = other[q][0];
        o.val_out = other[q][1];
      }
      own.j[q].key = o.key_out;  // the next pass reads them
      own.j[q].val = o.val_out;
    }
    hipLaunchKernelGGL(k_sort_count, dim3((uint32_t)tiles, (uint32_t)n_own), dim3(256), 0, s, now, p * per, digits);
    hipLaunchKernelGGL(k_sort_scan, dim3((uint32_t)((digits + 3) / 4), (uint32_t)n_own), dim3(256), 0, s, now, digits);
    hipLaunchKernelGGL(k_sort_place, dim3((uint32_t)tiles, (uint32_t)n_own), dim3(256), 0, s, now, p * per, per);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t dev_split(const int32_t *rowptr, const int32_t *colidx, const float *vals, int32_t m, int32_t k, int64_t nnz,
                     int32_t T, int32_t c, int32_t light_order, int32_t chunk_order,
                     const std::function<void *(size_t)> &alloc, hipStream_t s, DeviceSplit *out) {
  hipError_t e;
  const int32_t nb = (int32_t)(((int64_t)m + kSplitRows - 1) / kSplitRows);
  Scratch sc(s);
  if ((e = pool_alloc(&sc.p[0], sizeof(SplitSums) * ((size_t)nb + 1))) != hipSuccess) return e;
  SplitSums *sums = static_cast<SplitSums *>(sc.p[0]);
  if (nb > 0)
    hipLaunchKernelGGL(k_split_sums, dim3((uint32_t)nb), dim3(256), 0, s, rowptr, m, T, c, sums);
  hipLaunchKernelGGL(k_split_scan, dim3(1), dim3(1024), 0, s, sums, nb);
  SplitSums tot{0, 0, 0};
  if ((e = hipGetLastError()) != hipSuccess ||
      (e = hipMemcpyAsync(&tot, sums + nb, sizeof(tot), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  const int64_t n_heavy = tot.heavy, n_chunks = tot.chunks, n_light = (int64_t)m - n_heavy;
  const uint32_t light_nnz = (uint32_t)(nnz - (int64_t)tot.nnz);
  if (n_chunks > INT32_MAX) return hipErrorInvalidValue;
  auto ints = [&](int64_t n) { return static_cast<int32_t *>(alloc(sizeof(int32_t) * (size_t)std::max<int64_t>(1, n))); };
  out->n_light = n_light;
  out->n_heavy = n_heavy;
  out->n_chunks = n_chunks;
  out->light = ints(n_light);
  out->lptr = ints(n_light + 1);
  out->colidx = ints(nnz);
  out->vals = reinterpret_cast<float *>(ints(nnz));
  out->chunks = ints(3 * n_chunks);
  out->corder = ints(n_chunks);
  out->heavy_rows = ints(n_heavy);
  out->heavy_ptr = ints(n_heavy + 1);
  if (!out->light || !out->lptr || !out->colidx || !out->vals || !out->chunks || !out->corder || !out->heavy_rows ||
      !out->heavy_ptr)
    return hipErrorOutOfMemory;
  // heavy starts; chunk sources, keys in and out, indices; light keys in and out, rows before the sort
  const size_t nh = (size_t)n_heavy, nc = (size_t)n_chunks, nl = (size_t)n_light;
  if ((e = pool_alloc(&sc.p[1], sizeof(int32_t) * (nh + 4 * nc + 3 * nl + 1))) != hipSuccess) return e;
  int32_t *w = static_cast<int32_t *>(sc.p[1]);
  uint32_t *hstart = reinterpret_cast<uint32_t *>(w);
  int32_t *from = w + nh, *ckey = from + nc, *ckey2 = ckey + nc, *cidx = ckey2 + nc;
  int32_t *lkey = cidx + nc, *lkey2 = lkey + nl + 1, *lraw = lkey2 + nl;  // lkey also holds n_light + 1 lengths
  const bool by_last = light_order == 2 && n_light > 1, by_mid = chunk_order == 2 && n_chunks > 1;
  int bits = 1;
  while (bits < 31 && ((int64_t)1 << bits) <= (int64_t)k) ++bits;  // light keys lie in [0, k], chunk keys below k
  if (nb > 0)
    hipLaunchKernelGGL(k_split_fill, dim3((uint32_t)nb), dim3(256), 0, s, rowptr, m, T, c, sums, nb,
                       by_last ? lraw : out->light, out->heavy_rows, out->heavy_ptr, hstart);
  else
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, s, out->heavy_ptr, (int64_t)1, 0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (n_chunks > 0) {
    hipLaunchKernelGGL(k_split_chunks, dim3(grid_for(n_chunks)), dim3(256), 0, s, rowptr, colidx, out->heavy_rows,
                       out->heavy_ptr, hstart, (int32_t)n_heavy, (int32_t)n_chunks, c, light_nnz, out->chunks, from,
                       ckey, by_mid ? cidx : out->corder);
    hipLaunchKernelGGL(k_move_chunks, dim3((uint32_t)((n_chunks + 3) / 4)), dim3(256), 0, s, colidx, vals,
                       out->chunks, from, n_chunks, out->colidx, out->vals);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (by_last)
    hipLaunchKernelGGL(k_last_col_keys, dim3(grid_for(n_light)), dim3(256), 0, s, rowptr, colidx, k, lraw, n_light,
                       lkey);
  const SortJob jobs[2] = {{ckey, cidx, ckey2, out->corder, nullptr, by_mid ? (int32_t)n_chunks : 0, 0},
                           {lkey, lraw, lkey2, out->light, nullptr, by_last ? (int32_t)n_light : 0, 0}};
  if ((e = hipGetLastError()) != hipSuccess || (e = sort_pairs(sc, 5, jobs, bits, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_light_lengths, dim3(grid_for(n_light + 1)), dim3(256), 0, s, rowptr, out->light, n_light, lkey);
  size_t tmp = 0;
  if ((e = hipGetLastError()) != hipSuccess ||
      (e = hipcub::DeviceScan::ExclusiveSum(nullptr, tmp, lkey, out->lptr, (size_t)n_light + 1, s)) != hipSuccess ||
      (e = pool_alloc(&sc.p[4], std::max<size_t>(tmp, 1))) != hipSuccess ||
      (e = hipcub::DeviceScan::ExclusiveSum(sc.p[4], tmp, lkey, out->lptr, (size_t)n_light + 1, s)) != hipSuccess)
    return e;
  if (n_light > 0) {
    // 8 lanes for short rows on average, else 16
    if ((int64_t)light_nnz <= 8 * n_light)
      hipLaunchKernelGGL((k_move_light<8>), dim3((uint32_t)((n_light + 31) / 32)), dim3(256), 0, s, rowptr, colidx,
                         vals, out->light, n_light, out->lptr, out->colidx, out->vals);
    else
      hipLaunchKernelGGL((k_move_light<16>), dim3((uint32_t)((n_light + 15) / 16)), dim3(256), 0, s, rowptr, colidx,
                         vals, out->light, n_light, out->lptr, out->colidx, out->vals);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipStreamSynchronize(s);  // the scratch arrays are given back on return
}

namespace {

// ---- packed column windows over the split layout
// Light entry p belongs to the light row t with lptr[t] <= p < lptr[t + 1]
// (the last such t when empty rows share a pointer) and to window t / R; its
// key is (window << 32) | column.
__global__ __launch_bounds__(256) void k_win_entry_keys(const int32_t *__restrict__ lptr, int64_t n_light,
                                                        const int32_t *__restrict__ colidx, int64_t E, int32_t R,
                                                        uint64_t *__restrict__ keys) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= E) return;
  int64_t lo = 0, hi = n_light - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) / 2;
    if (lptr[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  keys[p] = ((uint64_t)(lo / R) << 32) | (uint32_t)colidx[p];
}

// Runs of equal (window, column) keys: a run of two or more is a candidate,
// keyed (window, uses descending, column) so that a window's most used come
// first; the rest sort to the end.
__global__ __launch_bounds__(256) void k_win_candidates(const uint64_t *__restrict__ run_key,
                                                        const int32_t *__restrict__ run_len,
                                                        const int32_t *__restrict__ n_runs, int32_t cbits,
                                                        uint64_t *__restrict__ key2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= *n_runs) return;
  const uint64_t w = run_key[i] >> 32, col = run_key[i] & 0xffffffffull;
  const uint64_t inv = ((1ull << cbits) - 1) - (uint64_t)run_len[i];
  key2[i] = run_len[i] >= 2 ? (w << (cbits + 32)) | (inv << 32) | col : ~0ull;
}

// Candidate i (sorted) is kept when fewer than cap candidates of its window
// precede it; kept ones are re-keyed (window, column), the others sort last.
__global__ __launch_bounds__(256) void k_win_keep(const uint64_t *__restrict__ key2, const int32_t *__restrict__ n_runs,
                                                  int32_t cbits, int32_t cap, uint64_t *__restrict__ key3,
                                                  int32_t *__restrict__ kept) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= *n_runs) return;
  const uint64_t k = key2[i];
  kept[i] = 0;
  if (k == ~0ull) {
    key3[i] = ~0ull;
    return;
  }
  const uint64_t w = k >> (cbits + 32);
  const uint64_t first_key = w << (cbits + 32);
  int64_t lo = 0, hi = i;  // first index whose key is >= first_key
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (key2[mid] < first_key) lo = mid + 1;
    else hi = mid;
  }
  key3[i] = (i - lo < cap) ? (w << 32) | (k & 0xffffffffull) : ~0ull;
  kept[i] = (i - lo < cap) ? 1 : 0;
}

// wptr[w] = first staged key of window w (keys sorted, kept ones first).
__global__ __launch_bounds__(256) void k_win_ptr_cols(const uint64_t *__restrict__ key3, int64_t n_kept, int64_t nw,
                                                      int32_t *__restrict__ wptr, int32_t *__restrict__ wcols) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n_kept) wcols[i] = (int32_t)(key3[i] & 0xffffffffull);
  if (i > nw) return;
  const uint64_t target = (uint64_t)i << 32;
  int64_t lo = 0, hi = n_kept;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (key3[mid] < target) lo = mid + 1;
    else hi = mid;
  }
  wptr[i] = (int32_t)lo;
}

// Entry codes: -2 - (position among its window's staged columns), else the
// column; staged[p] = 1 for an entry that reads a staged column.
__global__ __launch_bounds__(256) void k_win_codes(const uint64_t *__restrict__ entry_key,
                                                   const int32_t *__restrict__ wptr, const int32_t *__restrict__ wcols,
                                                   int64_t E, int32_t *__restrict__ code, int32_t *__restrict__ staged) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= E) return;
  const int64_t w = (int64_t)(entry_key[p] >> 32);
  const int32_t col = (int32_t)(entry_key[p] & 0xffffffffull);
  int64_t lo = wptr[w], hi = wptr[w + 1];
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (wcols[mid] < col) lo = mid + 1;
    else hi = mid;
  }
  const bool hit = lo < wptr[w + 1] && wcols[lo] == col;
  code[p] = hit ? (int32_t)(-2 - (lo - wptr[w])) : col;
  staged[p] = hit ? 1 : 0;
}

}  // namespace

hipError_t dev_split_windows(const int32_t *lptr, int64_t n_light, int32_t *colidx, int32_t R, int32_t cap,
                             const std::function<void *(size_t)> &alloc, hipStream_t s, int32_t **wptr,
                             int32_t **wcols, int32_t *wmax, int64_t *n_staged, int64_t *staged_uses) {
  *wmax = 0;
  *n_staged = 0;
  *staged_uses = 0;
  const int64_t nw = (n_light + R - 1) / R;
  hipError_t e;
  int32_t E32 = 0;
  if (n_light > 0) {
    if ((e = hipMemcpyAsync(&E32, lptr + n_light, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
      return e;
  }
  const int64_t E = E32;
  *wptr = static_cast<int32_t *>(alloc(sizeof(int32_t) * (size_t)(nw + 1)));
  if (!*wptr) return hipErrorOutOfMemory;
  if (E == 0 || cap < 1 || R < 2) {  // nothing can be staged: every code is its column
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(nw + 1)), dim3(256), 0, s, *wptr, nw + 1, 0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    *wcols = static_cast<int32_t *>(alloc(sizeof(int32_t)));
    if (!*wcols) return hipErrorOutOfMemory;
    return hipStreamSynchronize(s);
  }
  if (E > INT32_MAX / 2) return hipErrorInvalidValue;
  const int n = (int)E;
  Scratch sc(s);
  // entry keys, sorted keys, run keys, run lengths + run count, candidate keys (x2), kept keys (x2), flags, temp
  if ((e = pool_alloc(&sc.p[0], sizeof(uint64_t) * (size_t)n)) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[1], sizeof(uint64_t) * (size_t)n)) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[2], sizeof(uint64_t) * (size_t)n)) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[3], sizeof(int32_t) * ((size_t)n + 1))) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[4], 2 * sizeof(uint64_t) * (size_t)n)) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[5], sizeof(int32_t) * (size_t)n)) != hipSuccess) return e;
  if ((e = pool_alloc(&sc.p[6], sizeof(int64_t))) != hipSuccess) return e;
  uint64_t *ekey = static_cast<uint64_t *>(sc.p[0]), *skey = static_cast<uint64_t *>(sc.p[1]);
  uint64_t *rkey = static_cast<uint64_t *>(sc.p[2]);
  int32_t *rlen = static_cast<int32_t *>(sc.p[3]), *nruns = rlen + n;
  uint64_t *k2 = static_cast<uint64_t *>(sc.p[4]), *k2s = k2 + n;
  int32_t *flag = static_cast<int32_t *>(sc.p[5]);
  int64_t *uses_d = static_cast<int64_t *>(sc.p[6]);
  int wbits = 1;
  while (wbits < 31 && ((int64_t)1 << wbits) < nw) ++wbits;
  int cbits = 1;  // uses are at most R (each row uses a column once)
  while (cbits < 31 && ((int64_t)1 << cbits) <= (int64_t)R) ++cbits;
  if (wbits + cbits > 32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_win_entry_keys, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, lptr, n_light, colidx, E, R,
                     ekey);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  size_t t1 = 0, t2 = 0, t3 = 0, t4 = 0, t5 = 0;
  if ((e = hipcub::DeviceRadixSort::SortKeys(nullptr, t1, ekey, skey, n, 0, 32 + wbits, s)) != hipSuccess) return e;
  if ((e = hipcub::DeviceRunLengthEncode::Encode(nullptr, t2, skey, rkey, rlen, nruns, n, s)) != hipSuccess) return e;
  if ((e = hipcub::DeviceRadixSort::SortKeys(nullptr, t3, k2, k2s, n, 0, 64, s)) != hipSuccess) return e;
  if ((e = hipcub::DeviceReduce::Sum(nullptr, t4, flag, uses_d, n, s)) != hipSuccess) return e;
  t5 = std::max({t1, t2, t3, t4, (size_t)1});
  if ((e = pool_alloc(&sc.p[7], t5)) != hipSuccess) return e;
  if ((e = hipcub::DeviceRadixSort::SortKeys(sc.p[7], t1, ekey, skey, n, 0, 32 + wbits, s)) != hipSuccess) return e;
  if ((e = hipcub::DeviceRunLengthEncode::Encode(sc.p[7], t2, skey, rkey, rlen, nruns, n, s)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_win_candidates, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, rkey, rlen, nruns, cbits,
                     k2);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int32_t runs = 0;
  if ((e = hipMemcpyAsync(&runs, nruns, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  if ((e = hipcub::DeviceRadixSort::SortKeys(sc.p[7], t3, k2, k2s, runs, 0, 64, s)) != hipSuccess) return e;
  // kept candidates re-keyed (window, column) into k2, then sorted into skey
  hipLaunchKernelGGL(k_win_keep, dim3((uint32_t)((runs + 255) / 256)), dim3(256), 0, s, k2s, nruns, cbits, cap, k2,
                     flag);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipcub::DeviceRadixSort::SortKeys(sc.p[7], t3, k2, skey, runs, 0, 64, s)) != hipSuccess) return e;
  int64_t n_kept = 0;  // the kept keys sort first
  if ((e = hipcub::DeviceReduce::Sum(sc.p[7], t4, flag, uses_d, runs, s)) != hipSuccess ||
      (e = hipMemcpyAsync(&n_kept, uses_d, sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  *wcols = static_cast<int32_t *>(alloc(sizeof(int32_t) * (size_t)std::max<int64_t>(1, n_kept)));
  if (!*wcols) return hipErrorOutOfMemory;
  hipLaunchKernelGGL(k_win_ptr_cols, dim3(grid_for(std::max<int64_t>(n_kept, nw + 1))), dim3(256), 0, s, skey, n_kept,
                     nw, *wptr, *wcols);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_win_codes, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, ekey, *wptr, *wcols, E, colidx,
                     flag);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipcub::DeviceReduce::Sum(sc.p[7], t4, flag, uses_d, n, s)) != hipSuccess) return e;
  std::vector<int32_t> hw((size_t)nw + 1);
  if ((e = hipMemcpyAsync(hw.data(), *wptr, sizeof(int32_t) * hw.size(), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(staged_uses, uses_d, sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  for (int64_t w = 0; w < nw; ++w) *wmax = std::max(*wmax, hw[(size_t)w + 1] - hw[(size_t)w]);
  *n_staged = n_kept;
  return hipSuccess;  // synchronised above; the scratch arrays are freed on return
}

hipError_t dev_block16(const int32_t *rowptr, const int32_t *colidx, const float *vals, int32_t m, int32_t k,
                       int64_t nnz, int64_t nnzb, int32_t ell_width, int32_t *bptr, int32_t *bcol, float *bval,
                       hipStream_t s) {
  (void)k;
  (void)nnz;
  const int64_t mb = ((int64_t)m + 15) / 16;
  const int64_t slots = ell_width >= 0 ? mb * ell_width : nnzb;
  hipError_t e;
  Scratch sc(s);  // counts and the longest block-row, scan temporary, bptr
  int32_t *ptr = bptr;
  if (!ptr) {
    if ((e = pool_alloc(&sc.p[2], sizeof(int32_t) * (size_t)(mb + 1))) != hipSuccess) return e;
    ptr = static_cast<int32_t *>(sc.p[2]);
  }
  if ((e = pool_alloc(&sc.p[0], sizeof(int32_t) * (size_t)(mb + 2))) != hipSuccess) return e;
  int32_t *count = static_cast<int32_t *>(sc.p[0]), *width = count + mb + 1;
  size_t tmp = 0;
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, s, width, (int64_t)1, 0);
  hipLaunchKernelGGL(k_blk_count, dim3((uint32_t)std::max<int64_t>(1, std::min<int64_t>(mb, 1 << 20))), dim3(256), 0, s, rowptr,
                     colidx, m, mb, count);
  if ((e = hipGetLastError()) != hipSuccess ||
      (e = hipcub::DeviceScan::ExclusiveSum(nullptr, tmp, count, ptr, (size_t)mb + 1, s)) != hipSuccess ||
      (e = pool_alloc(&sc.p[1], std::max<size_t>(tmp, 1))) != hipSuccess ||
      (e = hipcub::DeviceScan::ExclusiveSum(sc.p[1], tmp, count, ptr, (size_t)mb + 1, s)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(k_blk_width, dim3((uint32_t)std::min<int64_t>(mb / 256 + 1, 256)), dim3(256), 0, s, ptr, mb,
                     width);
  // nothing is written by block number before the counts agree with the
  // storage sized from the analysis
  int32_t total = 0, longest = 0;
  if ((e = hipGetLastError()) != hipSuccess ||
      (e = hipMemcpyAsync(&total, ptr + mb, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(&longest, width, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  if ((int64_t)total != nnzb || (ell_width >= 0 && longest > ell_width)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_blk_fill, dim3((uint32_t)std::min<int64_t>(mb + 1, 1 << 20)), dim3(256), 0, s, rowptr, colidx,
                     vals, m, mb, ptr, ell_width, slots, bcol, bval);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return hipStreamSynchronize(s);  // the scratch arrays are given back on return
}

hipError_t dev_sell(const int32_t *rowptr, const int32_t *colidx, const float *vals, int32_t m, int32_t row_max,
                    int32_t C, int32_t sigma, int64_t max_slots, const std::function<void *(size_t)> &alloc,
                    hipStream_t s, int32_t **perm, int64_t **sptr, int32_t **scol, float **sval, int64_t *slots) {
  *perm = nullptr;
  *sptr = nullptr;
  *scol = nullptr;
  *sval = nullptr;
  *slots = 0;
  const int64_t ns = ((int64_t)m + C - 1) / C;
  hipError_t e;
  *perm = static_cast<int32_t *>(alloc(sizeof(int32_t) * (size_t)std::max(1, m)));
  *sptr = static_cast<int64_t *>(alloc(sizeof(int64_t) * (size_t)(ns + 1)));
  if (!*perm || !*sptr) return hipErrorOutOfMemory;
  if (m == 0) {
    if ((e = hipMemsetAsync(*sptr, 0, sizeof(int64_t), s)) != hipSuccess) return e;
    *scol = static_cast<int32_t *>(alloc(sizeof(int32_t)));
    *sval = static_cast<float *>(alloc(sizeof(float)));
    if (!*scol || !*sval) return hipErrorOutOfMemory;
    return hipStreamSynchronize(s);
  }
  Scratch sc(s);  // keys, sorted keys, rows, slice sizes, temporary
  const size_t mm = (size_t)m;
  if ((e = pool_alloc(&sc.p[0], 8 * mm)) != hipSuccess || (e = pool_alloc(&sc.p[1], 8 * mm)) != hipSuccess ||
      (e = pool_alloc(&sc.p[2], 4 * mm)) != hipSuccess || (e = pool_alloc(&sc.p[3], 8 * (size_t)ns)) != hipSuccess)
    return e;
  uint64_t *keys = static_cast<uint64_t *>(sc.p[0]), *skeys = static_cast<uint64_t *>(sc.p[1]);
  int32_t *rows = static_cast<int32_t *>(sc.p[2]);
  int64_t *size = static_cast<int64_t *>(sc.p[3]);
  hipLaunchKernelGGL(k_sell_keys, dim3(grid_for(m)), dim3(256), 0, s, rowptr, m, sigma, row_max, keys, rows);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const uint64_t n_keys = (uint64_t)((m + (int64_t)sigma - 1) / sigma) * (uint64_t)(row_max + 1);
  int end_bit = 1;
  while (end_bit < 64 && ((uint64_t)1 << end_bit) < n_keys) ++end_bit;
  size_t tmp_sort = 0, tmp_scan = 0;
  if ((e = hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_sort, keys, skeys, rows, *perm, m, 0, end_bit, s)) !=
          hipSuccess ||
      (e = hipcub::DeviceScan::ExclusiveSum(nullptr, tmp_scan, size, *sptr, (int)ns, s)) != hipSuccess)
    return e;
  if ((e = pool_alloc(&sc.p[4], std::max<size_t>({tmp_sort, tmp_scan, 1}))) != hipSuccess) return e;
  if ((e = hipcub::DeviceRadixSort::SortPairs(sc.p[4], tmp_sort, keys, skeys, rows, *perm, m, 0, end_bit, s)) !=
      hipSuccess)
    return e;
  hipLaunchKernelGGL(k_sell_sizes, dim3(grid_for(ns)), dim3(256), 0, s, rowptr, *perm, m, C, ns, size);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipcub::DeviceScan::ExclusiveSum(sc.p[4], tmp_scan, size, *sptr, (int)ns, s)) != hipSuccess) return e;
  int64_t last[2] = {0, 0};
  if ((e = hipMemcpyAsync(&last[0], *sptr + (ns - 1), sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(&last[1], size + (ns - 1), sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  *slots = last[0] + last[1];
  if (*slots > max_slots) return hipSuccess;  // the caller rejects the plan; nothing more is built
  if ((e = hipMemcpyAsync(*sptr + ns, slots, sizeof(int64_t), hipMemcpyHostToDevice, s)) != hipSuccess) return e;
  *scol = static_cast<int32_t *>(alloc(sizeof(int32_t) * (size_t)std::max<int64_t>(1, *slots)));
  *sval = static_cast<float *>(alloc(sizeof(float) * (size_t)std::max<int64_t>(1, *slots)));
  if (!*scol || !*sval) return hipErrorOutOfMemory;
  if (*slots > 0) {
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(*slots)), dim3(256), 0, s, *scol, *slots, -1);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemsetAsync(*sval, 0, sizeof(float) * (size_t)*slots, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_sell_fill, dim3(grid_for(m)), dim3(256), 0, s, rowptr, colidx, vals, *perm, *sptr, m, C,
                       *scol, *sval);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipStreamSynchronize(s);  // the scratch arrays are freed on return
}

hipError_t dev_tag_cold(const int32_t *colidx, int64_t nnz, int32_t k, int64_t budget_rows, int32_t *tagged,
                        int64_t *hot_cols, int64_t *hot_nnz, hipStream_t s) {
  *hot_cols = *hot_nnz = 0;
  hipError_t e;
  Scratch sc(s);
  const size_t kk = (size_t)std::max(1, k);
  if ((e = pool_alloc(&sc.p[0], 4 * kk)) != hipSuccess) return e;
  int32_t *deg = static_cast<int32_t *>(sc.p[0]);
  if ((e = hipMemsetAsync(deg, 0, 4 * kk, s)) != hipSuccess) return e;
  if (nnz > 0) {
    hipLaunchKernelGGL(k_col_degree, dim3(grid_for(nnz)), dim3(256), 0, s, colidx, nnz, deg);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  std::vector<int32_t> h(kk);
  if ((e = hipMemcpyAsync(h.data(), deg, 4 * kk, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  h.resize((size_t)k);
  // smallest D >= 2 with #{deg >= D} <= budget_rows (the host conversion's rule)
  int32_t dmax = 0;
  for (int32_t d : h) dmax = std::max(dmax, d);
  std::vector<int64_t> hist((size_t)dmax + 2, 0);
  for (int32_t d : h) hist[d]++;
  int64_t above = 0;
  int32_t D = dmax + 1;
  for (int32_t d = dmax; d >= 2; --d) {
    if (above + hist[d] > budget_rows) break;
    above += hist[d];
    D = d;
  }
  int64_t hn = 0;
  for (int32_t d : h)
    if (d >= D) hn += d;
  *hot_cols = above;
  *hot_nnz = hn;
  if (nnz > 0) {
    hipLaunchKernelGGL(k_tag_cold, dim3(grid_for(nnz)), dim3(256), 0, s, colidx, nnz, deg, D, tagged);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipStreamSynchronize(s);
}

uint64_t pattern_hash_host(const int32_t *rowptr, const int32_t *colidx, int32_t m, int64_t nnz) {
  uint64_t h = 0;
  for (int64_t i = 0; i <= m; ++i) h += mix64(kPatternSalt[0] ^ ((uint64_t)i << 32 | (uint32_t)rowptr[i]));
  for (int64_t p = 0; p < nnz; ++p) h += mix64(kPatternSalt[1] ^ ((uint64_t)p << 32 | (uint32_t)colidx[p]));
  return h;
}

hipError_t dev_pattern_hash(const int32_t *rowptr, const int32_t *colidx, int32_t m, int64_t nnz, hipStream_t s,
                            uint64_t *out) {
  Scratch sc(s);
  hipError_t e;
  if ((e = pool_alloc(&sc.p[0], sizeof(unsigned long long))) != hipSuccess) return e;
  unsigned long long *sum = static_cast<unsigned long long *>(sc.p[0]);
  if ((e = hipMemsetAsync(sum, 0, sizeof(unsigned long long), s)) != hipSuccess) return e;
  const int64_t lens[2] = {(int64_t)m + 1, nnz};
  const int32_t *arrs[2] = {rowptr, colidx};
  for (int t = 0; t < 2; ++t) {
    if (lens[t] == 0) continue;
    const uint32_t grid = (uint32_t)std::min<int64_t>(2048, (lens[t] + 255) / 256);
    hipLaunchKernelGGL(k_pattern_hash, dim3(grid), dim3(256), 0, s, arrs[t], lens[t], kPatternSalt[t], sum);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  unsigned long long h = 0;
  if ((e = hipMemcpyAsync(&h, sum, sizeof(h), hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  *out = (uint64_t)h;
  return hipSuccess;
}

hipError_t dev_transpose(const int32_t *rowptr, const int32_t *colidx, const float *vals, int32_t m, int32_t k,
                         int64_t nnz, int32_t *t_rowptr, int32_t *t_colidx, float *t_vals, hipStream_t s) {
  hipError_t e;
  if (nnz > 0) {
    Scratch sc(s);  // sorted keys, (row, value) pairs in and out, sort temporary
    for (int t = 0; t < 3; ++t)
      if ((e = pool_alloc(&sc.p[t], (t == 0 ? sizeof(uint32_t) : sizeof(uint64_t)) * (size_t)nnz)) != hipSuccess)
        return e;
    uint32_t *keys_out = static_cast<uint32_t *>(sc.p[0]);
    uint64_t *pairs = static_cast<uint64_t *>(sc.p[1]), *sorted = static_cast<uint64_t *>(sc.p[2]);
    // the sort carries rows and values: gathering them afterwards by sorted position
    // is two random reads and a binary search per nonzero (the backward plan of a 2.4 M
    // row graph with 61 M nonzeros: 10.3 ms that way, 8.7 this; the sort bounds it)
    hipLaunchKernelGGL(k_transpose_pack, dim3(grid_for(nnz)), dim3(256), 0, s, rowptr, m, vals, nnz, pairs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int end_bit = 1;  // columns are in [0, k): sort on the bits that can be set
    while (end_bit < 31 && ((int64_t)1 << end_bit) < (int64_t)k) ++end_bit;
    const uint32_t *keys_in = reinterpret_cast<const uint32_t *>(colidx);  // valid columns are non-negative
    size_t tmp = 0;
    if ((e = hipcub::DeviceRadixSort::SortPairs(nullptr, tmp, keys_in, keys_out, pairs, sorted, (int)nnz, 0, end_bit,
                                                 s)) != hipSuccess)
      return e;
    if ((e = pool_alloc(&sc.p[3], std::max<size_t>(tmp, 1))) != hipSuccess) return e;
    if ((e = hipcub::DeviceRadixSort::SortPairs(sc.p[3], tmp, keys_in, keys_out, pairs, sorted, (int)nnz, 0, end_bit,
                                                 s)) != hipSuccess)
      return e;
    hipLaunchKernelGGL(k_transpose_rowptr, dim3(grid_for((int64_t)k + 1)), dim3(256), 0, s, keys_out, nnz, k,
                       t_rowptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_transpose_unpack, dim3(grid_for(nnz)), dim3(256), 0, s, sorted, nnz, t_colidx, t_vals);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipStreamSynchronize(s);  // the scratch arrays are freed on return
  }
  if ((e = hipMemsetAsync(t_rowptr, 0, sizeof(int32_t) * ((size_t)k + 1), s)) != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

}  // namespace sd
