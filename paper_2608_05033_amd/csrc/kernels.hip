// SpMM kernels for gfx950 (CDNA4, wave64).
//
// C = A.B with A sparse (CSR or 16x16 blocks) and B, C dense row-major fp32.
// The paper's SpMM mechanisms (Appendix "Compilation-Plan Design Space", SpMM
// row: reuse of dense rows across sparse nonzeros, accumulation in registers,
// one output write per row; Appendix "Case Studies": sub-warp row groups with
// shuffled sparse entries, and heavy rows split into chunks) are re-mapped
// onto wave64:
//
//  * A lane group of G lanes owns one sparse row (or chunk, or merge-path
//    piece) and covers G*VW output columns, VW = 4 giving one 128-bit load of
//    a B row per lane per nonzero.  64/G rows share a wave.  Pointers off 16 bytes
//    use the same loads (they need 4-byte alignment only), and so do widths that
//    are no multiple of 4: the last lane takes the row's last 4 columns and stores
//    those its neighbour does not.  One column per lane (VW = 1) issues four times
//    the loads (7-point Laplacian 60^3, N = 33: 77 us against 25; R-MAT 200 k
//    vertices, 3 M edges, N = 101: 279 against 129) and is the faster one, at such
//    widths, where waves are few or rows long or far; the planner tells them apart.
//  * The group loads G (column, value) pairs of its nonzero stream with one
//    coalesced load per lane, then broadcasts them inside the group with
//    ds_bpermute; up to 8 B-row loads are issued back to back
//    before the FMAs, so each lane keeps several 128-bit gathers in flight.
//  * Workgroup ids are remapped so that each of the 8 XCDs (each with its
//    own L2) walks one contiguous range of rows: neighbouring rows share B
//    rows, and consecutive hardware workgroup ids land on different XCDs.
//  * C is written once per element with non-temporal stores.
//  * Split heavy rows and merge-path carries are combined by separate fix-up
//    kernels that add partials in a fixed order: no atomics, bitwise
//    reproducible results.
//  * Dense 16x16 blocks use v_mfma_f32_16x16x4_f32 (fp32 matrix cores): the
//    only place where the work is a dense contraction.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "kernels.h"

namespace sd {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

typedef float f2 __attribute__((ext_vector_type(2)));

// T: a lane's registers.  M: the same in global memory, where rows of B and C of
// any width and any float pointer give 4-byte alignment only; the hardware takes
// its 8- and 16-byte accesses at any 4 bytes.
typedef f4 f4_mem __attribute__((aligned(4)));
typedef f2 f2_mem __attribute__((aligned(4)));
template <int VW>
struct VecOf;
template <>
struct VecOf<4> {
  using T = f4;
  using M = f4_mem;
};
template <>
struct VecOf<1> {
  using T = float;
  using M = float;
};
template <>
struct VecOf<2> {
  using T = f2;
  using M = f2_mem;
};

// Element t of a 1-, 2- or 4-wide lane vector.
__device__ __forceinline__ float elem(float x, int) { return x; }
__device__ __forceinline__ float elem(f2 x, int t) { return x[t]; }
__device__ __forceinline__ float elem(f4 x, int t) { return x[t]; }

constexpr int kWaves = 4;  // wave64s per 256-thread workgroup

// Hardware dispatches workgroup b to XCD b % 8.  Map it to logical id
// x*q + min(x, r) + b/8 (q = nb/8, r = nb%8): XCD x then owns one contiguous
// range of logical ids, and the map is a bijection on [0, nb).
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb) {
  const uint32_t q = nb >> 3, r = nb & 7u;
  const uint32_t x = b & 7u, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// Chunked round-robin: XCD x takes chunks x, x + 8, x + 16, ... of S
// consecutive ids, so at any time the 8 XCDs work on 8 adjacent sub-bands (the
// i-th workgroup sent to XCD x is id (i / S) 8S + x S + i % S).  Ids past the
// last whole round of 8S keep the hardware order, so the map is a bijection.
__device__ __forceinline__ uint32_t chunk_remap(uint32_t b, uint32_t nb, uint32_t S) {
  const uint32_t full = nb / (8u * S) * (8u * S);
  if (b >= full) return b;
  const uint32_t x = b & 7u, i = b >> 3;
  return (i / S) * 8u * S + x * S + i % S;
}

// Logical workgroup id.  order 1: each XCD one contiguous range of ids (each
// L2 sees neighbouring rows); order 0: the hardware's round-robin (the 8 XCDs
// work on one band of ids; what one XCD brings from HBM the others find in
// the shared Infinity Cache); order S >= 2: chunked round-robin with chunks
// of S ids (each XCD a contiguous sub-band, neighbouring XCDs the adjacent
// ones).
__device__ __forceinline__ uint32_t wg_index(int order) {
  if (order == 0) return blockIdx.x;
  if (order == 1) return xcd_remap(blockIdx.x, gridDim.x);
  return chunk_remap(blockIdx.x, gridDim.x, (uint32_t)order);
}

// Logical block of the heavy-split kernels.  The first cb8 (chunk_blocks
// rounded up to a multiple of 8) hardware workgroups take the chunks, the rest
// the light rows.  order 1: the chunk workgroups are dealt to the XCDs in
// contiguous ranges of the processing order (each XCD, with its own L2, works
// through its own stretch of columns); otherwise both parts keep the
// hardware's round-robin.  Returns false for the padding workgroups.
__device__ __forceinline__ bool split_block(int order, uint32_t chunk_blocks, uint32_t &blk) {
  if (order != 1) {
    blk = blockIdx.x;
    return true;
  }
  const uint32_t cb8 = (chunk_blocks + 7u) & ~7u;
  if (blockIdx.x < cb8) {
    blk = xcd_remap(blockIdx.x, cb8);
    return blk < chunk_blocks;
  }
  blk = blockIdx.x - cb8 + chunk_blocks;
  return true;
}

template <int VW>
__device__ __forceinline__ typename VecOf<VW>::T load_v(const float *p) {
  return *reinterpret_cast<const typename VecOf<VW>::M *>(p);
}

// ODD: widths that are no whole number of lanes.  Whole widths run code without the
// last lane's case, which costs short calls 1 to 3 % (rows of 9 around a band, 9,000 of
// them, N = 16: 5.16 / 5.07 us; the 64^3 stencil, N = 64: 25.9 / 25.2).
//
// First column a lane loads (of B, or of partial sums): its own.  ODD: the last VW
// columns of the row for the lane whose columns run past the width (it then repeats
// some of its neighbour's work).  Lanes wholly past it: a column that exists.  VW <= n.
template <int VW, bool ODD>
__device__ __forceinline__ int32_t load_col(int32_t col, int32_t n) {
  if constexpr (ODD) return min(col, n - VW);
  return col < n ? col : 0;
}

// Stores the lane's columns of a row; col < n is the lane's own first column and
// v starts at load_col(col, n).  Every column has one writer.
template <int VW, bool ODD, bool NT>
__device__ __forceinline__ void store_cols(float *row, int32_t col, int32_t n, typename VecOf<VW>::T v) {
  if (!ODD || col + VW <= n) {
    auto *p = reinterpret_cast<typename VecOf<VW>::M *>(row + col);
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
  } else {
    // the part of [n - VW, n) from col on
#pragma unroll
    for (int t = 1; t < VW; ++t)
      if (n - VW + t >= col) {
        if constexpr (NT) __builtin_nontemporal_store(elem(v, t), row + n - VW + t);
        else row[n - VW + t] = elem(v, t);
      }
  }
}

// Gathers the lane's slice of B row (raw & 0x7fffffff).  policy 0: normal
// loads; 1: tiered, a column tagged cold (bit 31 set by the plan) is loaded
// non-temporally so it is inserted for early eviction and the hot columns'
// rows stay in L2; 2: every gather non-temporal.
// The choice of load is an instruction bit, so a run-time policy costs a second
// load per slot; only the merge path has one.
template <int VW>
__device__ __forceinline__ typename VecOf<VW>::T gather_b(const float *__restrict__ Bl, int32_t raw, int32_t n,
                                                          int policy) {
  const float *p = Bl + (int64_t)(raw & 0x7fffffff) * n;
  if (policy == 2 || (policy == 1 && raw < 0))
    return __builtin_nontemporal_load(reinterpret_cast<const typename VecOf<VW>::M *>(p));
  return load_v<VW>(p);
}

// Loads the (column, value) tile of nonzeros [p, p + min(G, p1 - p)): lane
// glane of the group takes entry p + glane.  Plain loads: with the
// non-temporal hint the sparse stream is not kept in the Infinity Cache, and a
// line shared by two workgroups on different XCDs is read from HBM twice
// (measured on MI355X on the 7-point Laplacian: non-temporal entry loads made
// the ELL kernel up to 1.5x slower).
template <int G>
__device__ __forceinline__ void load_tile(const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                          int32_t p, int32_t p1, int glane, int32_t &c, float &v) {
  c = 0;
  v = 0.0f;
  if (glane < p1 - p && glane < G) {
    c = colidx[p + glane];
    v = vals[p + glane];
  }
}

// acc += sum over p in [p0, p1) of vals[p] * B[colidx[p], lane columns].
// (c, v) already holds the tile at p0 (from load_tile).  All G lanes of a
// group call this with the same p0, p1 (group-uniform control flow), so every
// ds_bpermute source lane is active.  One batch of up to 8 gathers in flight
// and no prefetch of the next tile: a second batch or tile raises the register
// count past 6 waves per SIMD, which costs more than it hides.
template <int G, int VW>
__device__ __forceinline__ void gather_rows(const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                            int32_t p0, int32_t p1, int32_t c, float v,
                                            const float *__restrict__ Bl, int32_t n, bool col_ok,
                                            typename VecOf<VW>::T &acc, int glane, int gbase) {
  using V = typename VecOf<VW>::T;
  if constexpr (G > 1) {
    constexpr int UNR = G < 8 ? G : 8;
    for (int32_t p = p0; p < p1; p += G) {
      const int32_t cnt = min(G, p1 - p);
      if (p != p0) load_tile<G>(colidx, vals, p, p1, glane, c, v);
      const int32_t cfirst = __shfl(c, gbase, 64);
#pragma unroll
      for (int t0 = 0; t0 < G; t0 += UNR) {
        if (t0 >= cnt) break;
        V bv[UNR];
        float av[UNR];
        int32_t ct[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          ct[u] = __shfl(c, gbase + t0 + u, 64);
          av[u] = __shfl(v, gbase + t0 + u, 64);
          ct[u] = (t0 + u < cnt) ? ct[u] : cfirst;  // an in-range address for the idle slots
        }
        __builtin_amdgcn_sched_barrier(0);  // broadcasts first, then the gathers back to back
#pragma unroll
        for (int u = 0; u < UNR; ++u) bv[u] = col_ok ? load_v<VW>(Bl + (int64_t)ct[u] * n) : (V)(0.0f);
#pragma unroll
        for (int u = 0; u < UNR; ++u)
          if (t0 + u < cnt) acc += av[u] * bv[u];
      }
      if (cnt < G) break;  // the next p could pass 2^31
    }
  } else {
    for (int32_t p = p0; p < p1; ++p) {
      if (p != p0) {
        c = colidx[p];
        v = vals[p];
      }
      if (col_ok) acc += v * load_v<VW>(Bl + (int64_t)c * n);
    }
  }
}

// A wave owns WR = (64/G) * J rows starting at wave-row w0 of the row space
// (rows w0.. of A, or entries w0.. of `rowlist`).  Lane l first fetches the
// bounds of wave-row l, so the whole wave's row pointers arrive with one
// load per lane; lane group g then takes wave-rows j*(64/G) + g, j < J
// (adjacent groups take adjacent rows, so their C stores are contiguous).
// The J rows of a group are processed together: their first (column, value)
// tiles are loaded back to back, then the B rows of the first UNR nonzeros of
// every one of the J rows are requested before any FMA, so J*UNR 128-bit
// gathers per lane are in flight.  Slots past a row's end issue no load.
// Nonzeros past the first UNR of a row (rare for the short rows this path
// is planned for) continue through gather_rows.
template <int G, int VW, bool ODD, int J, int UNR, bool LIST>
__device__ __forceinline__ void rows_wave(int64_t w0, const int32_t *__restrict__ rowptr,
                                          const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                          const int32_t *__restrict__ rowlist, int64_t nrows,
                                          const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                          int32_t col) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  constexpr int WR = RPW * J;
  static_assert(WR <= 64, "a wave holds at most 64 row descriptors");
  static_assert(UNR <= G, "a tile holds G nonzeros");
  const int lane = threadIdx.x & 63;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1), gidx = lane / G;
  const bool col_ok = col < n;
  const float *__restrict__ Bl = B + load_col<VW, ODD>(col, n);
  int32_t my_row = -1, my_p0 = 0, my_p1 = 0;
  if (lane < WR && w0 + lane < nrows) {
    // LIST: rowptr is indexed by list position (the heavy-split layout keeps
    // the listed rows' entries contiguous in list order); rowlist gives C's row
    my_row = LIST ? rowlist[w0 + lane] : (int32_t)(w0 + lane);
    const int64_t at = LIST ? w0 + lane : my_row;
    my_p0 = rowptr[at];
    my_p1 = rowptr[at + 1];
  }
  int32_t row[J], p0[J], p1[J], cnt[J], c[J];
  float v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int idx = j * RPW + gidx;
    row[j] = __shfl(my_row, idx, 64);
    p0[j] = __shfl(my_p0, idx, 64);
    p1[j] = __shfl(my_p1, idx, 64);
    cnt[j] = min(UNR, p1[j] - p0[j]);
  }
#pragma unroll
  for (int j = 0; j < J; ++j) load_tile<G>(colidx, vals, p0[j], p1[j], glane, c[j], v[j]);
  V acc[J];
  V bv[J][UNR];
  float av[J][UNR];
  int32_t ct[J][UNR];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    acc[j] = (V)(0.0f);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      ct[j][u] = __shfl(c[j], gbase + u, 64);
      av[j][u] = __shfl(v[j], gbase + u, 64);
    }
  }
  // all broadcasts first, then the gathers back to back
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      bv[j][u] = (V)(0.0f);
      if (u < cnt[j] && col_ok) bv[j][u] = load_v<VW>(Bl + (int64_t)ct[j][u] * n);
    }
#pragma unroll
  for (int j = 0; j < J; ++j) {
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (u < cnt[j]) acc[j] += av[j][u] * bv[j][u];
    if (p1[j] - p0[j] > UNR) {
      // rest of a long row: the tile at p0 + UNR is reloaded by gather_rows
      int32_t cc;
      float vv;
      load_tile<G>(colidx, vals, p0[j] + UNR, p1[j], glane, cc, vv);
      gather_rows<G, VW>(colidx, vals, p0[j] + UNR, p1[j], cc, vv, Bl, n, col_ok, acc[j], glane, gbase);
    }
    if (row[j] >= 0 && col_ok) store_cols<VW, ODD, true>(C + (int64_t)row[j] * n, col, n, acc[j]);
  }
}

// A workgroup's rows [first, first + rows) of the row space (or of the list
// positions), rows <= kStreamRows, taken in order by its lane groups as they
// become free (a counter in LDS).  A group takes one batch of up to 8 gathers per
// turn of whatever row it is at, and the next tile of entries - of the same row or
// of the row it takes next - is loaded before the current tile's gathers: a row
// start costs no memory round trip, no group waits for the longest row of its
// wave, and the rows in flight stay adjacent (which is what L2 lives on).
constexpr int kStreamRows = 256;
struct StreamLds {
  int32_t bounds[kStreamRows + 1], ids[kStreamRows];
  int32_t next;
};

template <int G, int VW, bool ODD, bool LIST>
__device__ __forceinline__ void rows_stream(StreamLds &lds, int64_t first, int rows,
                                            const int32_t *__restrict__ rowptr,
                                            const int32_t *__restrict__ colidx, const float *__restrict__ vals,
                                            const int32_t *__restrict__ rowlist, const float *__restrict__ B,
                                            float *__restrict__ C, int32_t n, int32_t col) {
  using V = typename VecOf<VW>::T;
  constexpr int UNR = G < 8 ? G : 8;
  constexpr int GROUPS = 256 / G;
  const int lane = threadIdx.x & 63;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const bool col_ok = col < n;
  const float *__restrict__ Bl = B + load_col<VW, ODD>(col, n);
  for (int t = threadIdx.x; t <= rows; t += 256) {
    lds.bounds[t] = rowptr[first + t];
    if (LIST && t < rows) lds.ids[t] = rowlist[first + t];
  }
  if (threadIdx.x == 0) lds.next = GROUPS;
  __syncthreads();
  int r = threadIdx.x / G, nr = rows;  // this row and the next one taken
  if (r >= rows) return;
  int32_t p = lds.bounds[r], e = lds.bounds[r + 1];
  int32_t c, nc = 0, np = 0, ne = 0, off = 0, cnt = min(G, e - p);
  float v, nv = 0.0f;
  load_tile<G>(colidx, vals, p, e, glane, c, v);
  V acc = (V)(0.0f);
  while (r < rows) {
    if (off == 0) {  // a new tile: request the one after it
      if (e - p > G) {
        np = p + G;
        ne = e;
      } else {
        if (glane == 0) nr = atomicAdd(&lds.next, 1);
        nr = __shfl(nr, gbase, 64);
        np = ne = 0;
        if (nr < rows) {
          np = lds.bounds[nr];
          ne = lds.bounds[nr + 1];
        }
      }
      load_tile<G>(colidx, vals, np, ne, glane, nc, nv);
    }
    V bv[UNR];
    float av[UNR];
    int32_t ct[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      ct[u] = __shfl(c, gbase + off + u, 64);
      av[u] = __shfl(v, gbase + off + u, 64);
    }
    __builtin_amdgcn_sched_barrier(0);  // broadcasts first, then the gathers back to back
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      bv[u] = (V)(0.0f);
      if (off + u < cnt && col_ok) bv[u] = load_v<VW>(Bl + (int64_t)ct[u] * n);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (off + u < cnt) acc += av[u] * bv[u];
    off += UNR;
    if (off >= cnt) {
      if (e - p <= G) {  // the row's last tile
        const int64_t row = LIST ? (int64_t)lds.ids[r] : first + r;
        if (col_ok) store_cols<VW, ODD, true>(C + row * n, col, n, acc);
        acc = (V)(0.0f);
        r = nr;
      }
      c = nc;
      v = nv;
      p = np;
      e = ne;
      cnt = min(G, e - p);
      off = 0;
    }
  }
}

// --------------------------------------------------------------- CSR rows ---
// J >= 1: J rows per lane group, batched (rows_wave).  J = 0: R rows per
// workgroup, streamed (rows_stream).
template <int G, int VW, bool ODD, int J, int UNR, bool LIST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(J <= 1 ? 6 : 1))) void k_csr_rows(const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ colidx,
                                                  const float *__restrict__ vals,
                                                  const int32_t *__restrict__ rowlist, int32_t nrows,
                                                  const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                                  int order, int R) {
  const int wave = threadIdx.x >> 6;
  const uint32_t blk = wg_index(order);
  const int32_t col = blockIdx.y * (G * VW) + (threadIdx.x & (G - 1)) * VW;
  if constexpr (J == 0) {
    __shared__ StreamLds lds;
    const int64_t first = (int64_t)blk * R;
    rows_stream<G, VW, ODD, LIST>(lds, first, (int)min((int64_t)R, nrows - first), rowptr, colidx, vals, rowlist, B, C, n,
                             col);
  } else {
    const int64_t w0 = ((int64_t)blk * kWaves + wave) * ((64 / G) * J);
    rows_wave<G, VW, ODD, J, UNR, LIST>(w0, rowptr, colidx, vals, rowlist, nrows, B, C, n, col);
  }
}

// ------------------------------------------------------- heavy-row split ---
// Workgroups [0, chunk_blocks) take chunks (row, begin, end), in the order
// corder gives, and write their partial sums to ws[chunk][*]; the rest take
// the light rows.
template <int G, int VW, bool ODD, int J, int UNR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(J <= 1 ? 6 : 1))) void k_csr_split(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx,
                                                   const float *__restrict__ vals,
                                                   const int32_t *__restrict__ light, int32_t nlight,
                                                   const int32_t *__restrict__ chunks, int32_t nchunks,
                                                   const int32_t *__restrict__ corder,
                                                   uint32_t chunk_blocks, float *__restrict__ ws,
                                                   const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                                   int order, int R) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  // Chunk workgroups come first; split_block deals them to the XCDs (a
  // remap over the whole grid would hand all heavy rows to a few XCDs).
  uint32_t blk;
  if (!split_block(order, chunk_blocks, blk)) return;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  V acc = (V)(0.0f);
  if (blk < chunk_blocks) {
    // processing slot t takes chunk corder[t]: chunks that cover the same
    // columns run side by side; the partial still lands at the chunk's own
    // workspace row, which the fix-up sums in one fixed order
    const int64_t t = ((int64_t)blk * kWaves + wave) * RPW + lane / G;
    int64_t q = nchunks;
    int32_t p0 = 0, p1 = 0;
    if (t < nchunks) {
      q = corder[t];
      p0 = chunks[3 * q + 1];
      p1 = chunks[3 * q + 2];
    }
    int32_t c0;
    float v0;
    load_tile<G>(colidx, vals, p0, p1, glane, c0, v0);
    gather_rows<G, VW>(colidx, vals, p0, p1, c0, v0, B + load_col<VW, ODD>(col, n), n, col_ok, acc, glane, gbase);
    if (q < nchunks && col_ok) store_cols<VW, ODD, false>(ws + q * n, col, n, acc);
  } else {
    const int64_t lb = (int64_t)(blk - chunk_blocks);
    if constexpr (J == 0) {
      __shared__ StreamLds lds;
      rows_stream<G, VW, ODD, true>(lds, lb * R, (int)min((int64_t)R, nlight - lb * R), rowptr, colidx, vals, light, B, C, n,
                               col);
    } else {
      rows_wave<G, VW, ODD, J, UNR, true>((lb * kWaves + wave) * (RPW * J), rowptr, colidx, vals, light, nlight, B, C, n,
                                     col);
    }
  }
}

// ------------------------------------------------------ sliced rows (small N) ---
// A narrow dense width needs few lanes per row (G <= 8 for N <= 32 with
// 128-bit accesses, G = 1 for N = 1), and one lane group per row then walks
// the row's nonzeros alone: long rows serialise and a wave holds many rows'
// dependent load chains.  Here S lane groups share a row: group s takes the
// nonzeros p0 + s, p0 + s + S, ..., UNR of them per round, and the S partial
// sums are added across lanes in a fixed butterfly (every lane of the row
// ends with the same, order-independent bits).  Lane l covers the columns of
// glane = l % G in slice s = (l / G) % S of row slot l / (G S).
//
// acc of slice s over [p0, p1).  The next round's (column, value) pairs are
// loaded behind the current round's gathers; every load uses an index clamped
// into [p0, p1), so no branch guards a load and the wait before the FMAs
// covers only the gathers.
template <int G, int VW, int S, int UNR>
__device__ __forceinline__ typename VecOf<VW>::T slice_sum(const int32_t *__restrict__ colidx,
                                                           const float *__restrict__ vals, int32_t p0, int32_t p1,
                                                           int s, const float *__restrict__ Bl, int32_t n) {
  using V = typename VecOf<VW>::T;
  V acc = (V)(0.0f);
  int32_t left = p1 - p0 - s;  // from p on; p itself may pass 2^31 behind the last round
  uint32_t p = (uint32_t)p0 + s;
  if (left <= 0) return acc;
  int32_t c[UNR];
  float v[UNR];
  auto fetch = [&]() {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int32_t q = (int32_t)(p + min(u * S, left - 1));
      c[u] = colidx[q];
      v[u] = vals[q];
    }
  };
  fetch();
  while (left > 0) {
    V b[UNR];
    float a[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      b[u] = load_v<VW>(Bl + (int64_t)c[u] * n);
      a[u] = v[u];
    }
    const int32_t here = left;
    p += S * UNR;
    left -= S * UNR;
    fetch();
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (u * S < here) acc += a[u] * b[u];
  }
  return acc;
}

__device__ __forceinline__ float xor_lanes(float x, int d) { return __shfl_xor(x, d, 64); }
__device__ __forceinline__ f4 xor_lanes(f4 x, int d) {
  return f4{__shfl_xor(x.x, d, 64), __shfl_xor(x.y, d, 64), __shfl_xor(x.z, d, 64), __shfl_xor(x.w, d, 64)};
}

// Sum over the S slices of a row; called by every lane of the wave.
template <int G, int S, typename V>
__device__ __forceinline__ V slice_reduce(V acc) {
#pragma unroll
  for (int d = G; d < G * S; d *= 2) acc += xor_lanes(acc, d);
  return acc;
}

// C[row] = the sum of its chunk partials.  One wave per heavy row: its S =
// 64/G lane groups take every S-th chunk, four partials in flight each, and
// meet in a fixed xor butterfly, so the sum is the same bits on every run
// (whatever order the chunks were computed in).  A heavy row of the power-law
// workloads has up to several hundred chunks; walked by one lane group in
// turn, they made the fix-up a tenth of the split's time.
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) void k_split_fixup(const int32_t *__restrict__ heavy_rows,
                                                     const int32_t *__restrict__ heavy_ptr, int32_t nheavy,
                                                     const float *__restrict__ ws, float *__restrict__ C,
                                                     int32_t n) {
  using V = typename VecOf<VW>::T;
  constexpr int S = 64 / G;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), s = lane / G;
  const int64_t h = (int64_t)blockIdx.x * kWaves + wave;
  if (h >= nheavy) return;  // wave-uniform
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ wl = ws + load_col<VW, ODD>(col, n);
  const int32_t q1 = heavy_ptr[h + 1];
  V a0 = (V)(0.0f), a1 = (V)(0.0f), a2 = (V)(0.0f), a3 = (V)(0.0f);
  int32_t q = heavy_ptr[h] + s;
  for (; q + 3 * S < q1; q += 4 * S) {
    a0 += load_v<VW>(wl + (int64_t)q * n);
    a1 += load_v<VW>(wl + (int64_t)(q + S) * n);
    a2 += load_v<VW>(wl + (int64_t)(q + 2 * S) * n);
    a3 += load_v<VW>(wl + (int64_t)(q + 3 * S) * n);
  }
  for (; q < q1; q += S) a0 += load_v<VW>(wl + (int64_t)q * n);
  const V acc = slice_reduce<G, S>((a0 + a1) + (a2 + a3));
  if (s == 0 && col_ok) store_cols<VW, ODD, true>(C + (int64_t)heavy_rows[h] * n, col, n, acc);
}

template <int G, int VW, bool ODD, int S, int UNR>
__global__ __launch_bounds__(256) void k_csr_slices(const int32_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ colidx,
                                                    const float *__restrict__ vals, int32_t nrows,
                                                    const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                                    int order) {
  using V = typename VecOf<VW>::T;
  constexpr int L = G * S, RPW = 64 / L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), s = (lane / G) & (S - 1);
  const uint32_t blk = wg_index(order);
  const int64_t r = ((int64_t)blk * kWaves + wave) * RPW + lane / L;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  int32_t p0 = 0, p1 = 0;
  if (r < nrows) {
    p0 = rowptr[r];
    p1 = rowptr[r + 1];
  }
  V acc = slice_sum<G, VW, S, UNR>(colidx, vals, p0, p1, s, B + load_col<VW, ODD>(col, n), n);
  acc = slice_reduce<G, S>(acc);
  if (r < nrows && s == 0 && col_ok) store_cols<VW, ODD, true>(C + r * n, col, n, acc);
}

// k_csr_split at narrow widths: a chunk takes a whole wave (64 / G slices;
// chunks are the long, few work items) and a light row S slices (the short,
// many ones).  Chunk partials go to ws, light rows to C: with non-temporal stores
// (nt) where C is large.  Its rows are written in no order, a few columns at a time,
// so a small C is better left to L2 to put together (us, plain / non-temporal: R-MAT
// 30 k vertices, 0.3 M edges, N = 1 and 4: 7.5 / 8.5, 8.0 / 8.5; 4,500 vertices, N = 20:
// 9.0 / 9.4), while a large one pushes out the rows of B (0.9 M vertices, 14 M edges,
// N = 8, 20, 32: 120 / 118, 227 / 206, 236 / 209; 100 k vertices, 0.6 M edges, N = 8: 12.5 /
// 11.8).
template <int G, int VW, bool ODD, int S, int UNR>
__global__ __launch_bounds__(256) void k_split_slices(const int32_t *__restrict__ rowptr,
                                                      const int32_t *__restrict__ colidx,
                                                      const float *__restrict__ vals,
                                                      const int32_t *__restrict__ light, int32_t nlight,
                                                      const int32_t *__restrict__ chunks, int32_t nchunks,
                                                      const int32_t *__restrict__ corder,
                                                      uint32_t chunk_blocks, float *__restrict__ ws,
                                                      const float *__restrict__ B, float *__restrict__ C,
                                                      int32_t n, int order, int nt) {
  using V = typename VecOf<VW>::T;
  constexpr int L = G * S, RPW = 64 / L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), s = (lane / G) & (S - 1);
  uint32_t blk;
  if (!split_block(order, chunk_blocks, blk)) return;  // as k_csr_split
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ Bl = B + load_col<VW, ODD>(col, n);
  if (blk < chunk_blocks) {
    constexpr int SC = 64 / G;
    const int sc = lane / G;
    const int64_t t = (int64_t)blk * kWaves + wave;  // processing slot; its chunk is corder[t]
    int64_t q = nchunks;
    int32_t p0 = 0, p1 = 0;
    if (t < nchunks) {
      q = corder[t];
      p0 = chunks[3 * q + 1];
      p1 = chunks[3 * q + 2];
    }
    V acc = slice_reduce<G, SC>(slice_sum<G, VW, SC, UNR>(colidx, vals, p0, p1, sc, Bl, n));
    if (q < nchunks && sc == 0 && col_ok) store_cols<VW, ODD, false>(ws + q * n, col, n, acc);
  } else {
    const int64_t i = ((int64_t)(blk - chunk_blocks) * kWaves + wave) * RPW + lane / L;
    int32_t row = -1, p0 = 0, p1 = 0;
    if (i < nlight) {  // rowptr by list position, as in rows_wave's LIST mode
      row = light[i];
      p0 = rowptr[i];
      p1 = rowptr[i + 1];
    }
    V acc = slice_reduce<G, S>(slice_sum<G, VW, S, UNR>(colidx, vals, p0, p1, s, Bl, n));
    if (row >= 0 && s == 0 && col_ok) {
      float *c = C + (int64_t)row * n;
      if (nt) {
        asm volatile("");  // before and after: merged with a plain store of another branch,
        store_cols<VW, ODD, true>(c, col, n, acc);
        asm volatile("");  // which the compiler does, the store loses its hint
      } else {
        store_cols<VW, ODD, false>(c, col, n, acc);
      }
    }
  }
}

// -------------------------------------------------------------- merge path ---
// Piece u covers path positions [start(u), start(u+1)).  A row that both
// starts and ends inside the piece is stored to C.  The piece's last,
// unfinished row leaves a carry (row, partial); the share of a row that began
// in an earlier piece and ends in this one is left as the piece's head
// (row, partial) instead of being stored.  The fix-up then stores each such
// row once: its carries in piece order, then the head of the piece that ends
// it.  So every element of C is written by exactly one store.
// rows[0, units): carry rows; rows[units, 2 units): head rows (-1: none).
// part[0, units n): carry partials; part[units n, 2 units n): head partials.
//
// The piece's nonzeros are one contiguous stream, so they are taken in tiles
// and in batches of 8 gathers whatever rows they belong to (the next tile is
// loaded behind the current gathers), and a row is closed when the running
// position reaches its end.  Walking row by row instead left each short row its
// own bounds -> entries -> gathers chain.
//
// The lane groups of a wave close their rows at different places of a batch, so a
// close may run up to 8 times a batch, each time for a few lanes: it waits on
// nothing.  The next row's end is at hand, the one after it requested from a tile
// held across the group's lanes, the next tile loaded ahead.  A close that fetched
// the end it needs made rows of equal length slower than walking them row by row
// (us, row by row / fetched / at hand, 60,000 rows of 12, N = 8, 16, 32: 27.1 / 35.6 /
// 30.1, 27.9 / 36.2 / 31.2, 27.2 / 35.5 / 28.1; R-MAT 100 k vertices, 2 M edges, N = 64:
// 139 / 70 / 57).  Two batches in flight on top cost 0 to 8 %.
//
// LONG (G = 64: one piece per wave): batches in which no row ends go without the
// test for a row's end behind every entry.
template <int G, int VW, bool ODD, bool LONG>
__global__ __launch_bounds__(256) void k_csr_merge(const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colidx,
                                                   const float *__restrict__ vals,
                                                   const int32_t *__restrict__ coords, int32_t units, int32_t m,
                                                   int32_t *__restrict__ rows, float *__restrict__ part,
                                                   const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                                   int policy, int order) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  constexpr int EPL = G >= 8 ? 1 : 8 / G;  // entries (and row ends) per lane and tile
  constexpr int T = G * EPL;               // tile: at least one batch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const uint32_t blk = wg_index(order);
  const int64_t u = ((int64_t)blk * kWaves + wave) * RPW + lane / G;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ Bl = B + load_col<VW, ODD>(col, n);
  int32_t i0 = 0, i1 = 0, j0 = 0, j1 = 0;
  if (u < units) {
    i0 = coords[2 * u];
    j0 = coords[2 * u + 1];
    i1 = coords[2 * u + 2];
    j1 = coords[2 * u + 3];
  }
  // the piece ends row i0, which began in an earlier piece
  const bool head = i0 < i1 && j0 > rowptr[i0];
  // Ends of the rows from i0 on, a tile of T held across the group's lanes and the next
  // one loaded ahead; rows from i1 on do not end in this piece.  Positions and rows are
  // unsigned: the last tile of almost 2^31 of either ends past INT32_MAX.
  constexpr uint32_t kNoEnd = UINT32_MAX;
  uint32_t ends[EPL], ends2[EPL], ahead = (uint32_t)i0 + T;
  auto load_ends = [&](uint32_t first, uint32_t(&x)[EPL]) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const uint32_t r = first + e * G + glane;
      x[e] = r < (uint32_t)i1 ? (uint32_t)rowptr[r + 1] : kNoEnd;
    }
  };
  auto end_at = [&](int k) {  // group-uniform k in [0, T)
    uint32_t v = ends[0];
#pragma unroll
    for (int e = 1; e < EPL; ++e) v = k / G == e ? ends[e] : v;
    return G == 1 ? v : __shfl(v, gbase + (k & (G - 1)), 64);
  };
  V acc = (V)(0.0f);
  load_ends((uint32_t)i0, ends);
  load_ends(ahead, ends2);
  // the row at hand ends at end, the one after it (place k of the tile) at next: closing a
  // row waits on neither memory nor a lane permute
  int k = 1;
  uint32_t end = end_at(0), next = end_at(1);
  float *dst = head ? part + ((int64_t)units + u) * n : C + (int64_t)i0 * n, *crow = C + ((int64_t)i0 + 1) * n;
  auto close_row = [&]() {
    if (col_ok) store_cols<VW, ODD, true>(dst, col, n, acc);
    dst = crow;
    crow += n;
    acc = (V)(0.0f);
    end = next;
    if (++k == T) {
      k = 0;
      ahead += T;
#pragma unroll
      for (int e = 0; e < EPL; ++e) ends[e] = ends2[e];
      load_ends(ahead, ends2);
    }
    next = end_at(k);
  };
  const uint32_t pe = (uint32_t)j1;
  while (end == (uint32_t)j0) close_row();
  int32_t c[EPL];
  float v[EPL];
  auto load_entries = [&](uint32_t p, int32_t(&cc)[EPL], float(&vv)[EPL]) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      cc[e] = 0;
      vv[e] = 0.0f;
      const uint32_t q = p + e * G + glane;
      if (q < pe) {
        cc[e] = colidx[q];
        vv[e] = vals[q];
      }
    }
  };
  load_entries((uint32_t)j0, c, v);
  for (uint32_t p = (uint32_t)j0; p < pe; p += T) {
    int32_t nc[EPL];
    float nv[EPL];
    load_entries(p + T, nc, nv);
#pragma unroll 1
    for (int t0 = 0; t0 < T; t0 += 8) {
      if (p + t0 >= pe) break;
      V bv[8];
      float av[8];
      int32_t ct[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {  // EPL > 1: one batch per tile, so t0 = 0
        if constexpr (EPL > 1) {
          ct[q] = G == 1 ? c[q / G] : __shfl(c[q / G], gbase + q % G, 64);
          av[q] = G == 1 ? v[q / G] : __shfl(v[q / G], gbase + q % G, 64);
        } else {
          ct[q] = __shfl(c[0], gbase + t0 + q, 64);
          av[q] = __shfl(v[0], gbase + t0 + q, 64);
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // broadcasts first, then the gathers back to back
      if (LONG && __all(p + t0 + 8 <= pe && end >= p + t0 + 8)) {  // 8 entries of the row at hand
        if (col_ok) {
#pragma unroll
          for (int q = 0; q < 8; ++q) bv[q] = gather_b<VW>(Bl, ct[q], n, policy);
#pragma unroll
          for (int q = 0; q < 8; ++q) acc += av[q] * bv[q];
        }
        while (end == p + t0 + 8) close_row();
        continue;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        bv[q] = (V)(0.0f);
        if (p + t0 + q < pe && col_ok) bv[q] = gather_b<VW>(Bl, ct[q], n, policy);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (p + t0 + q < pe) {
          acc += av[q] * bv[q];
          while (end == p + t0 + q + 1) close_row();  // this row, and empty rows after it
        }
    }
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      c[e] = nc[e];
      v[e] = nv[e];
    }
  }
  if (u < units) {
    // entries of row i1 in this piece: those after the last row it ends
    const bool has = i1 < m && j1 > max(j0, rowptr[i1]);
    if (glane == 0 && blockIdx.y == 0) {
      rows[u] = has ? i1 : -1;
      rows[units + u] = head ? i0 : -1;
    }
    if (has && col_ok) store_cols<VW, ODD, false>(part + u * n, col, n, acc);
  }
}

// The first piece of each run of pieces carrying into the same row r stores
// C[r]: the run's partials, then the head of the piece after the run, which
// ends r.  Row r's end is step rowptr[r + 1] + r of the path, so the run's end
// is known without reading the pieces between.  A run of up to 4 carries is
// added by its own lane group; a longer one (a heavy row: hundreds of pieces)
// by the whole wave, its 64/G lane groups taking every (64/G)-th carry, four
// in flight each, and meeting in a fixed xor butterfly.  Walked in turn by one
// lane group, the longest run set the kernel's time (R-MAT 200 k vertices,
// 3 M edges, n = 32: 71 us).
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) void k_merge_fixup(const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ coords,
                                                     const int32_t *__restrict__ rows,
                                                     const float *__restrict__ part, int32_t units,
                                                     float *__restrict__ C, int32_t n) {
  using V = typename VecOf<VW>::T;
  constexpr int S = 64 / G;
  constexpr int kAlone = 4;  // carries added by one lane group
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), s = lane / G;
  const int64_t u = ((int64_t)blockIdx.x * kWaves + wave) * S + s;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ pl = part + load_col<VW, ODD>(col, n);
  int32_t r = -1, end = 0;  // carries [u, end) go to row r
  if (u < units) {
    r = rows[u];
    if (r >= 0 && u > 0 && rows[u - 1] == r) r = -1;
    if (r >= 0) {
      const int64_t L = (int64_t)coords[2] + coords[3];  // path steps per piece
      end = (int32_t)min((int64_t)units, ((int64_t)rowptr[r + 1] + r) / L);
    }
  }
  auto add_head = [&](V sum, int32_t row, int32_t e) {
    if (e < units && rows[units + e] == row) sum += load_v<VW>(pl + ((int64_t)units + e) * n);
    return sum;
  };
  const bool alone = r >= 0 && end - u <= kAlone;
  if (alone) {
    V sum = load_v<VW>(pl + u * n);
#pragma unroll
    for (int t = 1; t < kAlone; ++t)
      if (u + t < end) sum += load_v<VW>(pl + (u + t) * n);
    sum = add_head(sum, r, end);
    if (col_ok) store_cols<VW, ODD, true>(C + (int64_t)r * n, col, n, sum);
  }
  uint64_t pending = __ballot(r >= 0 && !alone && glane == 0);
  while (pending) {  // wave-uniform
    const int src = __ffsll((long long)pending) - 1;
    pending &= pending - 1;
    const int32_t row = __shfl(r, src, 64), e = __shfl(end, src, 64);
    const int32_t u0 = (int32_t)__shfl((int32_t)u, src, 64);
    V a0 = (V)(0.0f), a1 = (V)(0.0f), a2 = (V)(0.0f), a3 = (V)(0.0f);
    int64_t q = (int64_t)u0 + s;
    for (; q + 3 * S < e; q += 4 * S) {
      a0 += load_v<VW>(pl + q * n);
      a1 += load_v<VW>(pl + (q + S) * n);
      a2 += load_v<VW>(pl + (q + 2 * S) * n);
      a3 += load_v<VW>(pl + (q + 3 * S) * n);
    }
    for (; q < e; q += S) a0 += load_v<VW>(pl + q * n);
    const V sum = add_head(slice_reduce<G, S>((a0 + a1) + (a2 + a3)), row, e);
    if (s == 0 && col_ok) store_cols<VW, ODD, true>(C + (int64_t)row * n, col, n, sum);
  }
}

// -------------------------------------------------------------------- ELL ---
// Lane group per row as in k_csr_rows, but the row's W slots sit at row * W:
// the (column, value) tile is requested as soon as the wave starts, with no
// row-pointer read before it.  The 64/G rows of a wave are consecutive, so
// their tiles form one contiguous segment.  Padding slots (column -1) issue
// no gather.
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_ell_rows(
    const int32_t *__restrict__ ecol, const float *__restrict__ eval, int32_t W, int32_t m,
    const float *__restrict__ B, float *__restrict__ C, int32_t n, int order) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  constexpr int UNR = G < 8 ? G : 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const uint32_t blk = wg_index(order);
  const int64_t r = ((int64_t)blk * kWaves + wave) * RPW + lane / G;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const bool row_ok = r < m;
  const float *__restrict__ Bl0 = B + load_col<VW, ODD>(col, n);  // lanes past n never store
  V acc = (V)(0.0f);
  for (int32_t t = 0; t < W; t += G) {
    const int32_t cnt = min(G, W - t);  // the same for every lane
    int32_t c = -1;
    float v = 0.0f;
    if (row_ok && glane < cnt) {
      c = ecol[r * W + t + glane];
      v = eval[r * W + t + glane];
    }
#pragma unroll
    for (int t0 = 0; t0 < G; t0 += UNR) {
      if (t0 >= cnt) break;
      V bv[UNR];
      float av[UNR];
      int32_t ct[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        ct[u] = __shfl(c, gbase + t0 + u, 64);
        av[u] = __shfl(v, gbase + t0 + u, 64);
      }
      // all broadcasts first, then the loads back to back (without the barrier the
      // compiler pairs each load with its own broadcast and waits on each)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {  // padding and slots past the row width issue no load
        bv[u] = (V)(0.0f);
        if (t0 + u < cnt && ct[u] >= 0) bv[u] = load_v<VW>(Bl0 + (int64_t)ct[u] * n);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
        if (t0 + u < cnt) acc += av[u] * bv[u];
    }
  }
  if (row_ok && col_ok) store_cols<VW, ODD, true>(C + r * n, col, n, acc);
}

// ELL with rows pipelined per lane group (W <= G: one entry load per lane
// covers a row).  Each workgroup makes `passes` passes of 4*64/G rows, pass p
// of workgroup b taking row block p * grid + b, so the resident workgroups
// sweep one contiguous band of rows together (neighbouring rows share B rows
// in L2).  While one pass's B-row gathers are in flight, the next pass's
// (column, value) entries are loaded.
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_ell_pipe(
    const int32_t *__restrict__ ecol, const float *__restrict__ eval, int32_t W, int32_t m, int32_t passes,
    const float *__restrict__ B, float *__restrict__ C, int32_t n, int order) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  constexpr int UNR = G < 8 ? G : 8;
  constexpr int PASS_ROWS = kWaves * RPW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const uint32_t blk = wg_index(order);
  const int64_t stride = (int64_t)gridDim.x * PASS_ROWS;
  int64_t r = (int64_t)blk * PASS_ROWS + wave * RPW + lane / G;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ Bl0 = B + load_col<VW, ODD>(col, n);  // lanes past n never store
  int32_t c = -1;
  float v = 0.0f;
  if (r < m && glane < W) {
    c = ecol[r * W + glane];
    v = eval[r * W + glane];
  }
  for (int32_t p = 0; p < passes; ++p) {  // the same trip count for the whole workgroup
    const int64_t rn = r + stride;
    int32_t cn = -1;
    float vn = 0.0f;
    V acc = (V)(0.0f);
#pragma unroll
    for (int t0 = 0; t0 < G; t0 += UNR) {
      if (t0 >= W) break;
      V bv[UNR];
      float av[UNR];
      int32_t ct[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        ct[u] = __shfl(c, gbase + t0 + u, 64);
        av[u] = __shfl(v, gbase + t0 + u, 64);
      }
      __builtin_amdgcn_sched_barrier(0);  // all broadcasts first, then the loads back to back
#pragma unroll
      for (int u = 0; u < UNR; ++u) {  // padding and slots past the row width issue no load
        bv[u] = (V)(0.0f);
        if (t0 + u < W && ct[u] >= 0) bv[u] = load_v<VW>(Bl0 + (int64_t)ct[u] * n);
      }
      if (t0 == 0 && p + 1 < passes && rn < m && glane < W) {  // next pass's entries, behind the gathers
        cn = ecol[rn * W + glane];
        vn = eval[rn * W + glane];
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
        if (t0 + u < W) acc += av[u] * bv[u];
    }
    if (r < m && col_ok) store_cols<VW, ODD, true>(C + r * n, col, n, acc);
    c = cn;
    v = vn;
    r = rn;
  }
}

// ------------------------------------------------------------ SELL-C-sigma ---
// Sorted row i = (wave id) * 64/G + lane group; its slice s = i / C holds
// min(C, m - sC) rows of width (slice_ptr[s+1] - slice_ptr[s]) / rows, stored
// row-major, so the group's entries are contiguous.  With C = 64/G (the plan's
// choice) each wave is one slice and every loop bound is wave-uniform; any
// other C (a launch with a different lane geometry) is still exact, with
// loop bounds that are uniform per lane group.  The result goes to C row
// perm[i].
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_sell_rows(
    const int32_t *__restrict__ perm, const int64_t *__restrict__ sptr, const int32_t *__restrict__ scol,
    const float *__restrict__ sval, int32_t C, int32_t m, const float *__restrict__ B, float *__restrict__ Cout,
    int32_t n, int order) {
  using V = typename VecOf<VW>::T;
  constexpr int RPW = 64 / G;
  constexpr int UNR = G < 8 ? G : 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const uint32_t blk = wg_index(order);
  const int64_t i = ((int64_t)blk * kWaves + wave) * RPW + lane / G;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  const float *__restrict__ Bl0 = B + load_col<VW, ODD>(col, n);  // lanes past n never store
  const bool row_ok = i < m;
  int64_t base = 0;
  int32_t W = 0, orow = 0;
  if (row_ok) {
    const int64_t sl = i / C, r0 = sl * C;
    const int64_t rows = min((int64_t)C, (int64_t)m - r0);
    base = sptr[sl];
    W = (int32_t)((sptr[sl + 1] - base) / rows);
    base += (i - r0) * W;
    orow = perm[i];
  }
  V acc = (V)(0.0f);
  for (int32_t t = 0; t < W; t += G) {  // uniform over the lane group
    const int32_t cnt = min(G, W - t);
    int32_t c = -1;
    float v = 0.0f;
    if (glane < cnt) {
      c = scol[base + t + glane];
      v = sval[base + t + glane];
    }
#pragma unroll
    for (int t0 = 0; t0 < G; t0 += UNR) {
      if (t0 >= cnt) break;
      V bv[UNR];
      float av[UNR];
      int32_t ct[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        ct[u] = __shfl(c, gbase + t0 + u, 64);
        av[u] = __shfl(v, gbase + t0 + u, 64);
      }
      __builtin_amdgcn_sched_barrier(0);  // broadcasts first, then the loads back to back
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        bv[u] = (V)(0.0f);
        if (t0 + u < cnt && ct[u] >= 0) bv[u] = load_v<VW>(Bl0 + (int64_t)ct[u] * n);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
        if (t0 + u < cnt) acc += av[u] * bv[u];
    }
  }
  if (row_ok && col_ok) store_cols<VW, ODD, true>(Cout + (int64_t)orow * n, col, n, acc);
}

// ---------------------------------------------------------- column windows ---
// The heavy-split layout with packed column windows over its light rows.  The
// chunk workgroups (the first ones, dealt as split_block says) run as in
// k_csr_split: heavy rows' entries carry plain columns.  Window workgroup w
// owns light-list positions [wR, wR + R).  Phase 1 copies the B rows of the
// window's staged columns (those two or more of its rows use) into LDS,
// [staged][G*VW] floats, with STAGE loads per lane group in flight.  After a
// barrier, phase 2 runs the window's rows, one per lane group in turn: an
// entry coded -2 - p reads staged row p from LDS, any other gathers B row
// `code` from memory.
template <int G, int VW, bool ODD>
__global__ __launch_bounds__(256) void k_win_split(
    const int32_t *__restrict__ rowptr, const int32_t *__restrict__ code, const float *__restrict__ vals,
    const int32_t *__restrict__ light, int32_t nlight, const int32_t *__restrict__ chunks,
    const int32_t *__restrict__ corder, int32_t nchunks, uint32_t chunk_blocks, float *__restrict__ ws,
    const int32_t *__restrict__ wptr, const int32_t *__restrict__ wcols, int32_t R, const float *__restrict__ B,
    float *__restrict__ C, int32_t n, int order) {
  using V = typename VecOf<VW>::T;
  extern __shared__ __align__(16) unsigned char win_lds[];
  V *__restrict__ tile = reinterpret_cast<V *>(win_lds);
  constexpr int RPW = 64 / G;
  constexpr int GROUPS = 256 / G;  // lane groups per workgroup
  constexpr int UNR = G < 8 ? G : 8;
  constexpr int STAGE = 8;         // staged rows per lane group per batch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int glane = lane & (G - 1), gbase = lane & ~(G - 1);
  const int grp = threadIdx.x / G;
  uint32_t blk;
  if (!split_block(order, chunk_blocks, blk)) return;  // workgroup-uniform
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool col_ok = col < n;
  if (blk < chunk_blocks) {
    const int64_t t = ((int64_t)blk * kWaves + wave) * RPW + lane / G;
    int64_t q = nchunks;
    int32_t p0 = 0, p1 = 0;
    if (t < nchunks) {
      q = corder[t];
      p0 = chunks[3 * q + 1];
      p1 = chunks[3 * q + 2];
    }
    int32_t c0;
    float v0;
    load_tile<G>(code, vals, p0, p1, glane, c0, v0);
    V acc = (V)(0.0f);
    gather_rows<G, VW>(code, vals, p0, p1, c0, v0, B + load_col<VW, ODD>(col, n), n, col_ok, acc, glane, gbase);
    if (t < nchunks && col_ok) store_cols<VW, ODD, false>(ws + q * n, col, n, acc);
    return;
  }
  const int64_t w = (int64_t)(blk - chunk_blocks);
  const float *__restrict__ Bl0 = B + load_col<VW, ODD>(col, n);  // lanes past n never store

  const int32_t s0 = wptr[w], D = wptr[w + 1] - s0;
  for (int32_t d0 = 0; d0 < D; d0 += GROUPS * STAGE) {
    V bv[STAGE];
#pragma unroll
    for (int u = 0; u < STAGE; ++u) {
      const int32_t d = d0 + u * GROUPS + grp;
      bv[u] = (V)(0.0f);
      if (d < D) bv[u] = load_v<VW>(Bl0 + (int64_t)wcols[s0 + d] * n);
    }
#pragma unroll
    for (int u = 0; u < STAGE; ++u) {
      const int32_t d = d0 + u * GROUPS + grp;
      if (d < D) tile[d * G + glane] = bv[u];
    }
  }
  __syncthreads();

  const int64_t t0 = w * R;
  const int32_t rows = (int32_t)min((int64_t)R, (int64_t)nlight - t0);
  for (int32_t r = 0; r < rows; r += GROUPS) {  // the same trip count for the whole workgroup
    const bool row_ok = r + grp < rows;
    int32_t p0 = 0, p1 = 0, crow = -1;
    if (row_ok) {
      const int64_t t = t0 + r + grp;
      p0 = rowptr[t];
      p1 = rowptr[t + 1];
      crow = light[t];
    }
    V acc = (V)(0.0f);
    for (int32_t p = p0; p < p1; p += G) {  // group-uniform bounds
      const int32_t cnt = min(G, p1 - p);
      int32_t c = -1;
      float v = 0.0f;
      if (glane < cnt) {
        c = code[p + glane];
        v = vals[p + glane];
      }
#pragma unroll
      for (int u0 = 0; u0 < G; u0 += UNR) {
        if (u0 >= cnt) break;
        V bv[UNR];
        float av[UNR];
        int32_t ct[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          ct[u] = __shfl(c, gbase + u0 + u, 64);
          av[u] = __shfl(v, gbase + u0 + u, 64);
        }
        __builtin_amdgcn_sched_barrier(0);  // broadcasts first, then the loads back to back
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          bv[u] = (V)(0.0f);
          if (u0 + u < cnt) {
            if (ct[u] >= 0)
              bv[u] = load_v<VW>(Bl0 + (int64_t)ct[u] * n);
            else
              bv[u] = tile[(-2 - ct[u]) * G + glane];
          }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
          if (u0 + u < cnt) acc += av[u] * bv[u];
      }
      if (cnt < G) break;  // as in gather_rows
    }
    if (row_ok && col_ok) store_cols<VW, ODD, true>(C + (int64_t)crow * n, col, n, acc);
  }
}

// ------------------------------------------------------------- BSR / MFMA ---
// One wave per (block-row, 16 NT NQ output columns), NT n-tiles of 16 columns;
// the width's last tile may be partial (RAG), mfma_shape chooses NT and NQ.
// For v_mfma_f32_16x16x4_f32 lane l supplies A[l%16][kk] and B[kk][l%16] for
// kk = l/16 and receives D[4(l/16)+v][l%16], v = 0..3.  The sum over the
// block's 16 columns is split into 4 MFMA k-steps s, lane group g = l/16
// taking block column 4g + s, so each lane's A operands are one float4 of its
// block row.  The 16 MFMA output columns c = l%16 of n-tile t map to dense
// columns NT c + t, so each lane's B operands for the NT n-tiles are NT
// consecutive floats of a B row, and the outputs of the NT n-tiles at one
// output row are NT consecutive floats of a C row.
// Accumulates the blocks q = first .. first + cnt - 1 of one block-row into
// acc (a 16 x 16 NT NQ tile of C at columns col0 ..).  RAG: the tile may run past
// the width n; lanes whose columns do read the last NT columns of B instead (so
// every address is in range).
// zrow: n zero floats owned by the plan, read in place of a B row by every
// slot that has no B row (a row past K, a Blocked-ELL padding block, the zero
// block past a block-row's end), so a non-finite B row never meets the zero
// fill of a block that does not use it.
template <int NQ, int NT, bool RAG = false>
__device__ __forceinline__ void bsr_mfma_blocks(int64_t first, int64_t cnt, int64_t zero_block,
                                                const int32_t *__restrict__ bcol, const float *__restrict__ bval,
                                                const float *__restrict__ B, const float *__restrict__ zrow,
                                                int32_t k, int32_t n, int32_t col0, int c, int g,
                                                f4 (&acc)[NQ][NT]) {
  using BV = typename VecOf<NT>::T;
  // Operand rings: NA value buffers and NB B-tile buffers, used in rotation by
  // a loop unrolled U = max(NA, NB) times (static buffer roles: no register
  // copies), so block q's values are in flight NA - 1 blocks ahead and its B
  // tile NB - 1 blocks ahead.  The values come from HBM and the B tiles mostly
  // from L2, so the values get the longer lead: the vector-memory counter
  // completes in issue order, and each step issues the B tile before the
  // values, so waiting for a B tile never waits for values issued later.
  // With one 64-column tile (NQ = 1) rings of 4 and 2 measured 7-8 % faster on
  // 32-block block-rows than rings of 3 and 3, at 6 instead of 5 waves per
  // SIMD.  A block's column index is a scalar load (its wait counter is not
  // the vector-memory one, so it never waits on blocks in flight).
  constexpr int NA = NQ == 1 ? 4 : 2, NB = 2;
  constexpr int U = NA > NB ? NA : NB;  // a multiple of both
  f4 abuf[NA];
  BV bbuf[NB][4][NQ];
  auto fetch_a = [&](int64_t q, f4 &a) {
    // block values are streamed once: non-temporal, so they do not push the
    // (reused) B tiles out of L2
    a = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(bval + q * 256 + c * 16 + 4 * g));
  };
  auto fetch_b = [&](int64_t q, BV (&b)[4][NQ]) {
    const int32_t bc = bcol[q];
    const bool valid = bc >= 0;  // Blocked-ELL padding has column -1 and zero values
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int32_t krow = bc * 16 + 4 * g + s;
#pragma unroll
      for (int qq = 0; qq < NQ; ++qq) {
        // No branch and no select on the loaded value (either makes the
        // compiler wait for the load at the join): the select is on the
        // address.  A row past K (last block-column) or a Blocked-ELL padding
        // block reads the zero row instead; its A values are the zero fill,
        // so it adds exactly zero.  The column is always in range: without RAG
        // n % (16 NT NQ) == 0, with it the last NT columns are the last read.
        const bool ok = valid && krow < k;
        const float *__restrict__ src = ok ? B + (int64_t)krow * n : zrow;
        const int32_t col = col0 + qq * 16 * NT + NT * c;
        b[s][qq] = load_v<NT>(src + (RAG ? load_col<NT, true>(col, n) : col));
      }
    }
  };
  auto mma = [&](const f4 &a, const BV (&b)[4][NQ]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int qq = 0; qq < NQ; ++qq)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[qq][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], elem(b[s][qq], t), acc[qq][t], 0, 0, 0);
  };
  // The loop runs whole rounds of U blocks and every fetch is unconditional:
  // slots past the range fetch the plan's zero block (column -1, zero
  // values), whose products add exactly zero.  Without branches around the
  // loads the compiler's wait before each block's MFMAs covers only that
  // block's loads, not the ones issued after it.
  const int64_t rounds = (cnt + U - 1) / U * U;
  auto slot = [&](int64_t i) { return i < cnt ? first + i : zero_block; };
#pragma unroll
  for (int i = 0; i < NB - 1; ++i) fetch_b(slot(i), bbuf[i]);
#pragma unroll
  for (int i = 0; i < NA - 1; ++i) fetch_a(slot(i), abuf[i]);
  for (int64_t q = 0; q < rounds; q += U) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      // the buffers refilled here were freed by the previous block
      fetch_b(slot(q + i + NB - 1), bbuf[(i + NB - 1) % NB]);
      fetch_a(slot(q + i + NA - 1), abuf[(i + NA - 1) % NA]);
      mma(abuf[i % NA], bbuf[i % NB]);
    }
  }
}

// One wave per (block-row, 16 NT NQ columns).  tx column tiles of a block-row are
// consecutive waves (blockIdx.y takes the next tx), so a workgroup's waves share
// a block-row's values in L1.
template <int NQ, int NT, bool ELL, bool RAG = false>
__global__ __launch_bounds__(256) void k_bsr_mfma(int32_t mb, int32_t m, int32_t k,
                                                  const int32_t *__restrict__ bptr, int32_t width,
                                                  const int32_t *__restrict__ bcol,
                                                  const float *__restrict__ bval,
                                                  const float *__restrict__ B, const float *__restrict__ zrow,
                                                  float *__restrict__ C, int32_t n, int32_t tx,
                                                  int64_t zero_block, int order) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const uint32_t blk = wg_index(order);
  const uint32_t unit = blk * kWaves + wave;
  const int32_t br = (int32_t)(unit / (uint32_t)tx);
  const int32_t col0 = (int32_t)(blockIdx.y * (uint32_t)tx + unit % (uint32_t)tx) * (16 * NT * NQ);
  if (br >= mb || col0 >= n) return;  // wave-uniform
  int64_t q0, q1;
  if (ELL) {
    q0 = (int64_t)br * width;
    q1 = q0 + width;
  } else {
    q0 = bptr[br];
    q1 = bptr[br + 1];
  }
  f4 acc[NQ][NT];
#pragma unroll
  for (int qq = 0; qq < NQ; ++qq)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[qq][t] = (f4)(0.0f);
  bsr_mfma_blocks<NQ, NT, RAG>(q0, q1 - q0, zero_block, bcol, bval, B, zrow, k, n, col0, c, g, acc);
#pragma unroll
  for (int qq = 0; qq < NQ; ++qq) {
    const int32_t col = col0 + qq * 16 * NT + NT * c;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t row = br * 16 + 4 * g + v;
      if (row < m && (!RAG || col < n)) {
        typename VecOf<NT>::T o;
        if constexpr (NT == 1) {
          o = acc[qq][0][v];
        } else {
#pragma unroll
          for (int t = 0; t < NT; ++t) o[t] = acc[qq][t][v];
        }
        if constexpr (RAG)
          store_cols<NT, true, true>(C + (int64_t)row * n, col, n, o);
        else
          __builtin_nontemporal_store(o, reinterpret_cast<typename VecOf<NT>::M *>(C + (int64_t)row * n + col));
      }
    }
  }
}

// ------------------------------------------------------------- BSR / VALU ---
// One wave per (block-row, G*VW output columns): lane group G covers the
// columns, 64/G row groups split the block's 16 rows.
template <int G, int VW, bool ODD, bool ELL>
__global__ __launch_bounds__(256) void k_bsr_valu(int32_t mb, int32_t m, int32_t k,
                                                  const int32_t *__restrict__ bptr, int32_t width,
                                                  const int32_t *__restrict__ bcol,
                                                  const float *__restrict__ bval,
                                                  const float *__restrict__ B, float *__restrict__ C, int32_t n,
                                                  int order) {
  using V = typename VecOf<VW>::T;
  constexpr int RG = 64 / G;                  // row groups per wave
  constexpr int RPL = RG >= 16 ? 1 : 16 / RG; // block rows per lane
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int glane = lane & (G - 1), rg = lane / G;
  const uint32_t blk = wg_index(order);
  const int32_t br = (int32_t)blk * kWaves + wave;
  if (br >= mb) return;
  const int32_t col = blockIdx.y * (G * VW) + glane * VW;
  const bool lane_ok = col < n && rg * RPL < 16;
  int64_t q0, q1;
  if (ELL) {
    q0 = (int64_t)br * width;
    q1 = q0 + width;
  } else {
    q0 = bptr[br];
    q1 = bptr[br + 1];
  }
  V acc[RPL];
#pragma unroll
  for (int t = 0; t < RPL; ++t) acc[t] = (V)(0.0f);
  if (lane_ok) {
    for (int64_t q = q0; q < q1; ++q) {
      const int32_t bc = bcol[q];
      if (bc < 0) continue;
#pragma unroll
      for (int kq = 0; kq < 4; ++kq) {
        V b[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int32_t krow = bc * 16 + 4 * kq + kk;
          b[kk] = krow < k ? load_v<VW>(B + (int64_t)krow * n + load_col<VW, ODD>(col, n)) : (V)(0.0f);
        }
#pragma unroll
        for (int t = 0; t < RPL; ++t) {
          const f4 a = *reinterpret_cast<const f4 *>(bval + q * 256 + (rg * RPL + t) * 16 + 4 * kq);
          acc[t] += a.x * b[0] + a.y * b[1] + a.z * b[2] + a.w * b[3];
        }
      }
    }
#pragma unroll
    for (int t = 0; t < RPL; ++t) {
      const int32_t row = br * 16 + rg * RPL + t;
      if (row < m) store_cols<VW, ODD, true>(C + (int64_t)row * n, col, n, acc[t]);
    }
  }
}

// ------------------------------------------------------------ dispatching ---
template <int G_, int VW_, bool ODD_>
struct Geo {
  static constexpr int G = G_, VW = VW_;
  static constexpr bool ODD = ODD_;  // the width is no whole number of lanes
};

template <int VW, bool ODD, typename F>
hipError_t with_lanes(int32_t G, F &&f) {
  switch (G) {
    case 1: return f(Geo<1, VW, ODD>{});
    case 2: return f(Geo<2, VW, ODD>{});
    case 4: return f(Geo<4, VW, ODD>{});
    case 8: return f(Geo<8, VW, ODD>{});
    case 16: return f(Geo<16, VW, ODD>{});
    case 32: return f(Geo<32, VW, ODD>{});
    case 64: return f(Geo<64, VW, ODD>{});
  }
  return hipErrorInvalidValue;
}

template <typename F>
hipError_t with_geometry(const Geometry &geo, F &&f) {
  if (geo.VW == 1) return with_lanes<1, false>(geo.G, f);
  return geo.odd ? with_lanes<4, true>(geo.G, f) : with_lanes<4, false>(geo.G, f);
}

inline uint32_t blocks_for(int64_t units, int G, int J = 1) {
  const int64_t per_block = (int64_t)kWaves * (64 / G) * J;
  return (uint32_t)((units + per_block - 1) / per_block);
}

// Rows per lane group J in {1, 2, 4} and B-row gathers per row per round
// UNR in {4, 8} (at most G); J * UNR <= 16 keeps the in-flight B data within
// 64 VGPRs at VW = 4.  J = 0: the streaming kernels (G >= 8).
template <int G, typename F>
hipError_t with_row_batch(int J, int UNR, F &&f) {
  if constexpr (G >= 8) {
    if (J == 0) return f(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
  }
  constexpr int U8 = G < 8 ? G : 8;
  constexpr int U4 = G < 4 ? G : 4;
  if constexpr (G >= 4) {
    if (J >= 4) return f(std::integral_constant<int, 4>{}, std::integral_constant<int, U4>{});
  }
  if constexpr (G >= 2) {
    if (J >= 2) {
      if (UNR >= 8) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, U8>{});
      return f(std::integral_constant<int, 2>{}, std::integral_constant<int, U4>{});
    }
  }
  if (UNR >= 8) return f(std::integral_constant<int, 1>{}, std::integral_constant<int, U8>{});
  return f(std::integral_constant<int, 1>{}, std::integral_constant<int, U4>{});
}

// Slices per row S for lane groups of G <= 8 lanes: a power of two with
// G * S <= 64.  UNR = 4 nonzeros per slice per round.
constexpr int kSliceUnroll = kSliceRound;
template <int G, typename F>
hipError_t with_slices(int S, F &&f) {
  if constexpr (G <= 8) {
    switch (S) {
      case 1: return f(std::integral_constant<int, 1>{});
      case 2: return f(std::integral_constant<int, 2>{});
      case 4: return f(std::integral_constant<int, 4>{});
      case 8: return f(std::integral_constant<int, 8>{});
      case 16:
        if constexpr (G <= 4) return f(std::integral_constant<int, 16>{});
        break;
      case 32:
        if constexpr (G <= 2) return f(std::integral_constant<int, 32>{});
        break;
      case 64:
        if constexpr (G == 1) return f(std::integral_constant<int, 64>{});
        break;
    }
  }
  return hipErrorInvalidValue;
}

// Reads `n4` float4s in a grid-stride loop, so the lines they occupy replace
// whatever L2 and the Infinity Cache held.  The store happens only if the sum
// is exactly -1.5 (never, for the zero-filled buffer the search uses), which
// keeps the reads from being optimised away.
__global__ __launch_bounds__(256) void k_cache_flush(const f4 *__restrict__ buf, int64_t n4,
                                                     float *__restrict__ sink) {
  f4 acc = (f4)(0.0f);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256) acc += buf[i];
  const float t = acc.x + acc.y + acc.z + acc.w;
  if (t == -1.5f) sink[0] = t;
}

}  // namespace

hipError_t launch_cache_flush(const void *buf, size_t bytes, float *sink, hipStream_t s) {
  const int64_t n4 = (int64_t)(bytes / 16);
  if (n4 == 0) return hipSuccess;
  hipLaunchKernelGGL(k_cache_flush, dim3(2048), dim3(256), 0, s, reinterpret_cast<const f4 *>(buf), n4, sink);
  return hipGetLastError();
}

Geometry geometry_for(int32_t n, int32_t vec4, int32_t col_tile) {
  Geometry g;
  g.VW = vec4 ? 4 : 1;
  g.odd = n % g.VW != 0;
  const int32_t width = (col_tile > 0 && col_tile < n) ? col_tile : n;
  const int32_t lanes = vec4 ? (width + 3) / 4 : width;
  int32_t G = 1;
  while (G < lanes && G < 64) G *= 2;
  g.G = G;
  g.coltiles = (n + G * g.VW - 1) / (G * g.VW);
  return g;
}

hipError_t launch_csr_rows(const CsrOperand &A, const DenseIO &io, int32_t rows_per_group, int32_t unroll,
                           int32_t slices, int32_t stream, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    if (slices > 1) {
      return with_slices<G>(slices, [&](auto ss) -> hipError_t {
        constexpr int S = decltype(ss)::value;
        const uint32_t nb = blocks_for(A.m, G * S);
        if (nb == 0) return hipSuccess;
        hipLaunchKernelGGL((k_csr_slices<G, VW, ODD, S, kSliceUnroll>), dim3(nb, geo.coltiles), dim3(256), 0, s,
                           A.rowptr, A.colidx, A.vals, A.m, io.B, io.C, io.n, io.order);
        return hipGetLastError();
      });
    }
    return with_row_batch<G>(stream > 0 ? 0 : rows_per_group, unroll, [&](auto jj, auto uu) -> hipError_t {
      constexpr int J = decltype(jj)::value, UNR = decltype(uu)::value;
      const int R = stream * (256 / G);
      const uint32_t nb = J == 0 ? (uint32_t)(((int64_t)A.m + R - 1) / R) : blocks_for(A.m, G, J);
      if (nb == 0) return hipSuccess;
      hipLaunchKernelGGL((k_csr_rows<G, VW, ODD, J, UNR, false>), dim3(nb, geo.coltiles), dim3(256), 0, s, A.rowptr,
                         A.colidx, A.vals, nullptr, A.m, io.B, io.C, io.n, io.order, R);
      return hipGetLastError();
    });
  });
}

hipError_t launch_csr_split(const CsrOperand &A, const int32_t *light, int32_t nlight, const int32_t *chunks,
                            const int32_t *corder, int32_t nchunks, const int32_t *heavy_rows,
                            const int32_t *heavy_ptr, int32_t nheavy, float *ws, const DenseIO &io,
                            int32_t rows_per_group, int32_t unroll, int32_t slices, int32_t stream, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    // narrow widths (G <= 8) take the sliced kernel, whose chunks get a whole wave
    hipError_t e = G <= 8 ? with_slices<G>(std::max(1, slices), [&](auto ss) -> hipError_t {
      constexpr int S = decltype(ss)::value;
      const uint32_t cb = blocks_for(nchunks, 64), lb = blocks_for(nlight, G * S);
      if (cb + lb == 0) return hipSuccess;
      const uint32_t grid = (io.order == 1 ? (cb + 7u) & ~7u : cb) + lb;
      hipLaunchKernelGGL((k_split_slices<G, VW, ODD, S, kSliceUnroll>), dim3(grid, geo.coltiles), dim3(256), 0, s,
                         A.rowptr, A.colidx, A.vals, light, nlight, chunks, nchunks, corder, cb, ws, io.B, io.C,
                         io.n, io.order == 1 ? 1 : 0, 4 * (int64_t)nlight * io.n >= (2 << 20) ? 1 : 0);
      return hipGetLastError();
    }) : with_row_batch<G>(stream > 0 ? 0 : rows_per_group, unroll, [&](auto jj, auto uu) -> hipError_t {
      constexpr int J = decltype(jj)::value, UNR = decltype(uu)::value;
      const int R = stream * (256 / G);
      const uint32_t cb = blocks_for(nchunks, G);
      const uint32_t lb = J == 0 ? (uint32_t)(((int64_t)nlight + R - 1) / R) : blocks_for(nlight, G, J);
      if (cb + lb == 0) return hipSuccess;
      const uint32_t grid = (io.order == 1 ? (cb + 7u) & ~7u : cb) + lb;
      hipLaunchKernelGGL((k_csr_split<G, VW, ODD, J, UNR>), dim3(grid, geo.coltiles), dim3(256), 0, s, A.rowptr,
                         A.colidx, A.vals, light, nlight, chunks, nchunks, corder, cb, ws, io.B, io.C, io.n,
                         io.order == 1 ? 1 : 0, R);
      return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    const uint32_t fb = (uint32_t)(((int64_t)nheavy + kWaves - 1) / kWaves);  // a wave per heavy row
    if (fb > 0) {
      hipLaunchKernelGGL((k_split_fixup<G, VW, ODD>), dim3(fb, geo.coltiles), dim3(256), 0, s, heavy_rows, heavy_ptr,
                         nheavy, ws, io.C, io.n);
      return hipGetLastError();
    }
    return hipSuccess;
  });
}

// Long rows, where a merge-path piece takes a whole wave (n > 128).  Batches without
// a row's end are told apart from 32 nonzeros a row on (us, not / so, rows around a
// band: 2,500 rows of 54, N = 180: 20.0 / 17.9; 9,000 of 130, N = 180: 72.2 / 63.0).
bool merge_long_rows(const Geometry &geo, int32_t m, int64_t nnz) { return geo.G == 64 && nnz >= 32 * (int64_t)m; }

// From 0.9 GB of gathered B rows on, LDS keeps such rows to two workgroups per CU: the
// pieces at work then lie in a quarter of the matrix, whose B rows L2 holds better (with
// the above, us: 18,000 rows of 54, N = 256: 120 / 97; 30,000 of 54, N = 180: 137 / 119;
// 60,000 of 130, N = 180: 712 / 575; 18,000 of 54, N = 180, 0.7 GB, loses: all that fit
// 1.21, two 1.03 times the speed of walking row by row).  So do odd widths that use
// every lane, whose rows of B straddle more lines than their neighbours' (n = 31, 63: 60,000
// rows of 130 1.00 / 1.45 and 0.72 / 0.89, 300,000 of 24 0.86 / 1.00 and 0.90 / 0.99 times
// that speed; n = 47 1.30 / 0.96; n = 125, 18,000 rows of 130: 89 / 120 us).  R-MAT
// graphs lose (100 k vertices, 21 a row, N = 180: 1.85 / 1.49); they have fewer nonzeros
// a row, and only m and nnz are known here.
size_t merge_lds_bytes(const Geometry &geo, int32_t m, int64_t nnz, int32_t n) {
  const double gathered = 4.0 * (double)nnz * n;
  if (merge_long_rows(geo, m, nnz)) return gathered >= 0.9e9 ? 65536 : 0;
  const bool last_lane_odd = geo.odd && geo.G <= 16 && geo.coltiles == 1 && n > (geo.G - 1) * geo.VW;
  return last_lane_odd && nnz >= 24 * (int64_t)m && gathered >= 0.7e9 ? 65536 : 0;
}

hipError_t launch_csr_merge(const CsrOperand &A, const int32_t *coords, int32_t units, int32_t *rows,
                            float *part, const DenseIO &io, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool odd = decltype(gg)::ODD;
    const uint32_t nb = blocks_for(units, G);
    if (nb == 0) return hipSuccess;
    // From 8 lanes a row on, whole widths run the odd ones' code: 1 to 5 % faster
    // (R-MAT 0.4 M vertices, 3.2 M edges, N = 32 and 96: 85 / 90, 200 / 232 us).
    constexpr bool ODD = odd || (VW == 4 && G >= 8);
    const size_t lds = merge_lds_bytes(geo, A.m, A.nnz, io.n);
    auto launch = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(nb, geo.coltiles), dim3(256), lds, s, A.rowptr, A.colidx, A.vals, coords, units,
                         A.m, rows, part, io.B, io.C, io.n, io.policy, io.order);
      return hipGetLastError();
    };
    hipError_t e;
    if (G == 64 && merge_long_rows(geo, A.m, A.nnz))
      e = launch(&k_csr_merge<G, VW, ODD, G == 64>);
    else
      e = launch(&k_csr_merge<G, VW, ODD, false>);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_merge_fixup<G, VW, ODD>), dim3(nb, geo.coltiles), dim3(256), 0, s, A.rowptr, coords, rows, part,
                       units, io.C, io.n);
    return hipGetLastError();
  });
}

hipError_t launch_ell(const int32_t *ecol, const float *eval, int32_t width, int32_t m, int32_t passes,
                      const DenseIO &io, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    if (passes >= 1 && width <= G) {
      const int64_t pass_rows = (int64_t)kWaves * (64 / G);
      const int64_t nb = ((int64_t)m + pass_rows * passes - 1) / (pass_rows * passes);
      if (nb == 0) return hipSuccess;
      hipLaunchKernelGGL((k_ell_pipe<G, VW, ODD>), dim3((uint32_t)nb, geo.coltiles), dim3(256), 0, s, ecol, eval,
                         width, m, passes, io.B, io.C, io.n, io.order);
      return hipGetLastError();
    }
    const uint32_t nb = blocks_for(m, G);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL((k_ell_rows<G, VW, ODD>), dim3(nb, geo.coltiles), dim3(256), 0, s, ecol, eval, width, m, io.B,
                       io.C, io.n, io.order);
    return hipGetLastError();
  });
}

hipError_t launch_sell(const int32_t *perm, const int64_t *sptr, const int32_t *scol, const float *sval,
                       int32_t C, int32_t m, const DenseIO &io, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  if (C < 1) return hipErrorInvalidValue;
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    const uint32_t nb = blocks_for(m, G);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL((k_sell_rows<G, VW, ODD>), dim3(nb, geo.coltiles), dim3(256), 0, s, perm, sptr, scol, sval, C, m,
                       io.B, io.C, io.n, io.order);
    return hipGetLastError();
  });
}

size_t window_lds_bytes(int32_t n, int32_t vec4, int32_t col_tile, int32_t staged) {
  const Geometry geo = geometry_for(n, vec4, col_tile);
  return (size_t)staged * (size_t)geo.G * (size_t)geo.VW * sizeof(float);
}

hipError_t launch_win_split(const CsrOperand &A, const int32_t *light, int32_t nlight, const int32_t *chunks,
                            const int32_t *corder, int32_t nchunks, const int32_t *heavy_rows,
                            const int32_t *heavy_ptr, int32_t nheavy, float *ws, const int32_t *wptr,
                            const int32_t *wcols, int32_t R, int32_t wmax, const DenseIO &io, hipStream_t s) {
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  if (R < 1) return hipErrorInvalidValue;
  const size_t lds = window_lds_bytes(io.n, io.vec4, io.col_tile, wmax);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    const uint32_t cb = blocks_for(nchunks, G);
    const uint32_t nw = (uint32_t)(((int64_t)nlight + R - 1) / R);
    if (cb + nw > 0) {
      const uint32_t grid = (io.order == 1 ? (cb + 7u) & ~7u : cb) + nw;
      hipLaunchKernelGGL((k_win_split<G, VW, ODD>), dim3(grid, geo.coltiles), dim3(256), lds, s, A.rowptr, A.colidx,
                         A.vals, light, nlight, chunks, corder, nchunks, cb, ws, wptr, wcols, R, io.B, io.C, io.n,
                         io.order == 1 ? 1 : 0);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    const uint32_t fb = (uint32_t)(((int64_t)nheavy + kWaves - 1) / kWaves);  // a wave per heavy row
    if (fb > 0) {
      hipLaunchKernelGGL((k_split_fixup<G, VW, ODD>), dim3(fb, geo.coltiles), dim3(256), 0, s, heavy_rows, heavy_ptr,
                         nheavy, ws, io.C, io.n);
      return hipGetLastError();
    }
    return hipSuccess;
  });
}

// Column tiles of one MFMA SpMM: every wave takes NQ NT n-tiles of 16 columns,
// the last tile partial (rag) where the width is no multiple of them.  One launch
// for the whole width: cut into 64-, 32- and 16-column launches, each streamed
// the block values again and left the chip idle at its end (24,011 rows, 21
// blocks of 16 per block-row, N = 100: 58 us in three launches, 31 in one;
// 131,072 rows, 32 blocks, N = 24, 48, 100: 144, 162, 307 us against 81, 109,
// 210).  The lines of the rule, in us at (64-column tiles / the other shape):
//   16 and 32 columns: as narrow as the width (131,072 rows, N = 16: 65 with 16,
//     77 with 32; N = 32: 78 with 32, 107 with 64);
//   32-column tiles while 64-column ones leave SIMDs without a wave (1,024 SIMDs;
//     500 block-rows, N = 64: 11.2 / 9.6; N = 96, 1,000 waves: 11.9 / 12.8);
//   128 columns per wave, which halves the value loads, where no half of it is
//     wasted and two waves per SIMD remain (8,192 block-rows, N = 256: 498 / 469,
//     N = 100: 234 / 210, N = 160 (three 64-column tiles): 323 / 398; 1,501
//     block-rows, N = 256: 61.4 / 58.5, N = 128 (1,501 waves): 31.6 / 36.0).
struct MfmaShape {
  int32_t NQ, NT, tiles;
  bool rag;
};
MfmaShape mfma_shape(int32_t mb, int32_t n, int32_t vec4) {
  MfmaShape s{1, 1, 0, false};
  if (vec4) {
    const int64_t t64 = (n + 63) / 64, waves64 = mb * t64, waves128 = mb * ((t64 + 1) / 2);
    s.NT = n <= 16 ? 1 : n <= 32 || waves64 < 768 ? 2 : 4;
    if (s.NT == 4 && t64 % 2 == 0 && waves128 >= 2048) s.NQ = 2;
  }
  const int32_t w = 16 * s.NT * s.NQ;
  s.tiles = (n + w - 1) / w;
  s.rag = n % w != 0;
  return s;
}

template <typename F>
hipError_t with_mfma_shape(const MfmaShape &sh, bool ell, F &&f) {
  auto pick = [&](auto nq, auto nt) -> hipError_t {
    constexpr int NQ = decltype(nq)::value, NT = decltype(nt)::value;
    if (sh.rag) return ell ? f(&k_bsr_mfma<NQ, NT, true, true>) : f(&k_bsr_mfma<NQ, NT, false, true>);
    return ell ? f(&k_bsr_mfma<NQ, NT, true, false>) : f(&k_bsr_mfma<NQ, NT, false, false>);
  };
  using std::integral_constant;
  if (sh.NQ == 2) return pick(integral_constant<int, 2>{}, integral_constant<int, 4>{});
  switch (sh.NT) {
    case 4: return pick(integral_constant<int, 1>{}, integral_constant<int, 4>{});
    case 2: return pick(integral_constant<int, 1>{}, integral_constant<int, 2>{});
    case 1: return pick(integral_constant<int, 1>{}, integral_constant<int, 1>{});
  }
  return hipErrorInvalidValue;
}

hipError_t launch_bsr(int32_t mb, int32_t m, int32_t k, const int32_t *bptr, int32_t width, const int32_t *bcol,
                      const float *bval, int64_t zero_block, const float *zrow, int32_t engine, const DenseIO &io,
                      hipStream_t s) {
  const uint32_t nb = (uint32_t)((mb + kWaves - 1) / kWaves);
  if (nb == 0) return hipSuccess;
  const bool ell = bptr == nullptr;
  if (engine == 1) {
    const MfmaShape sh = mfma_shape(mb, io.n, io.vec4);
    int32_t ny = (sh.tiles + kWaves - 1) / kWaves, tx = (sh.tiles + ny - 1) / ny;
    if ((int64_t)mb * tx * 64 > UINT32_MAX - 255) tx = 1, ny = sh.tiles;  // threads of a grid dimension
    const uint32_t grid = (uint32_t)(((int64_t)mb * tx + kWaves - 1) / kWaves);
    return with_mfma_shape(sh, ell, [&](auto kern) -> hipError_t {
      hipLaunchKernelGGL(kern, dim3(grid, (uint32_t)ny), dim3(256), 0, s, mb, m, k, bptr, width, bcol, bval, io.B,
                         zrow, io.C, io.n, tx, zero_block, io.order);
      return hipGetLastError();
    });
  }
  const Geometry geo = geometry_for(io.n, io.vec4, io.col_tile);
  return with_geometry(geo, [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    if (ell)
      hipLaunchKernelGGL((k_bsr_valu<G, VW, ODD, true>), dim3(nb, geo.coltiles), dim3(256), 0, s, mb, m, k, bptr, width,
                         bcol, bval, io.B, io.C, io.n, io.order);
    else
      hipLaunchKernelGGL((k_bsr_valu<G, VW, ODD, false>), dim3(nb, geo.coltiles), dim3(256), 0, s, mb, m, k, bptr, width,
                         bcol, bval, io.B, io.C, io.n, io.order);
    return hipGetLastError();
  });
}

hipError_t kernel_attributes(int32_t family, int32_t engine, int32_t n, int32_t vec4, int32_t rows_per_group,
                             int32_t unroll, int32_t slices, int32_t stream, int32_t col_tile, int32_t width,
                             int32_t block_rows, hipFuncAttributes *attr) {
  const int32_t G0 = geometry_for(n, vec4, col_tile).G;
  if ((family == 1 && slices > 1) || (family == 2 && G0 <= 8)) {
    return with_geometry(geometry_for(n, vec4, col_tile), [&](auto gg) -> hipError_t {
      constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
      constexpr bool ODD = decltype(gg)::ODD;
      return with_slices<G>(std::max(1, slices), [&](auto ss) -> hipError_t {
        constexpr int S = decltype(ss)::value;
        const void *fn = family == 2 ? (const void *)&k_split_slices<G, VW, ODD, S, kSliceUnroll>
                                     : (const void *)&k_csr_slices<G, VW, ODD, S, kSliceUnroll>;
        return hipFuncGetAttributes(attr, fn);
      });
    });
  }
  if (family == 6 || family == 7 || family == 8) {
    return with_geometry(geometry_for(n, vec4, col_tile), [&](auto gg) -> hipError_t {
      constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
      constexpr bool ODD = decltype(gg)::ODD;
      const void *fn = family == 8                          ? (const void *)&k_sell_rows<G, VW, ODD>
                       : family == 7                        ? (const void *)&k_win_split<G, VW, ODD>
                       : (rows_per_group >= 1 && width <= G) ? (const void *)&k_ell_pipe<G, VW, ODD>
                                                             : (const void *)&k_ell_rows<G, VW, ODD>;
      return hipFuncGetAttributes(attr, fn);
    });
  }
  if (family == 4 || family == 5) {
    const bool ell = family == 5;
    if (engine == 1)
      return with_mfma_shape(mfma_shape(block_rows, n, vec4), ell,
                             [&](auto kern) -> hipError_t { return hipFuncGetAttributes(attr, (const void *)kern); });
    return with_geometry(geometry_for(n, vec4, col_tile), [&](auto gg) -> hipError_t {
      constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
      constexpr bool ODD = decltype(gg)::ODD;
      const void *fn = ell ? (const void *)&k_bsr_valu<G, VW, ODD, true> : (const void *)&k_bsr_valu<G, VW, ODD, false>;
      return hipFuncGetAttributes(attr, fn);
    });
  }
  return with_geometry(geometry_for(n, vec4, col_tile), [&](auto gg) -> hipError_t {
    constexpr int G = decltype(gg)::G, VW = decltype(gg)::VW;
    constexpr bool ODD = decltype(gg)::ODD;
    return with_row_batch<G>(stream > 0 ? 0 : rows_per_group, unroll, [&](auto jj, auto uu) -> hipError_t {
      constexpr int J = decltype(jj)::value, UNR = decltype(uu)::value;
      const void *fn = family == 2   ? (const void *)&k_csr_split<G, VW, ODD, J, UNR>
                       : family == 3 ? (const void *)&k_csr_merge<G, VW, ODD || (VW == 4 && G >= 8), false>
                                     : (const void *)&k_csr_rows<G, VW, ODD, J, UNR, false>;
      return hipFuncGetAttributes(attr, fn);
    });
  });
}

}  // namespace sd
