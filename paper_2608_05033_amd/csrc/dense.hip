// Weight gradients: C = X^T Y for tall X (R x P) and Y (R x Q), fp32, on the
// fp32 matrix cores.  The dense transform of a graph layer has this shape in its
// backward pass: R is the number of vertices, P and Q are layer widths, so the
// whole output is a few 64 x 64 tiles and all the parallelism is in the rows.
//
// A wave owns one 64 x 64 output tile over a range of rows: with
// v_mfma_f32_16x16x4_f32, lane (c, g) = (l % 16, l / 16) supplies X[r + g][p] and
// Y[r + g][q] for the columns 4 c .. 4 c + 3 of the tile, one 16-byte load each
// per 4 rows, which feed 16 MFMAs (4 x 4 sub-tiles; sub-tile t of the tile is the
// columns 4 c + t).  So 2 KB of loads stand against 512 MFMA cycles and no LDS
// is needed; the loads of the next rows are in flight meanwhile.  Row ranges
// leave partial tiles, which a second kernel adds in a fixed order.
//
// Bound by fp32 MFMA at P = Q = 128 (2 R P Q flops against 4 R (P + Q) bytes: 32
// F/B, the ridge is near 30).  R = 262,144: the library's product for
// X^T Y runs on 13 workgroups and took 570 us at 128 x 128 and 547 at 128 x 64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;       // output tile edge of a wave
constexpr int kStepRows = 4;    // rows of one MFMA step
constexpr int kUnroll = 4;      // steps loaded ahead

// Tiles of one workgroup: GP x GQ (1 or 2 each); its 4 waves are GP GQ tiles
// times 4 / (GP GQ) row ranges.  blockIdx.y: the tile group.
struct Shape {
  int32_t gp, gq, groups_q, subs;
  int64_t parts, rows;  // row ranges (partial tiles per output tile), rows of one (a multiple of 16)
};

Shape shape_for(int64_t R, int32_t P, int32_t Q) {
  Shape s;
  const int32_t tp = (P + kTile - 1) / kTile, tq = (Q + kTile - 1) / kTile;
  s.gp = tp > 1 ? 2 : 1;
  s.gq = tq > 1 ? 2 : 1;
  s.groups_q = (tq + s.gq - 1) / s.gq;
  s.subs = 4 / (s.gp * s.gq);
  const int64_t groups = (int64_t)((tp + s.gp - 1) / s.gp) * s.groups_q;
  // two waves per SIMD over all tile groups, at least 128 rows each
  const int64_t waves = std::max<int64_t>(1, 512 * s.subs / groups);
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>(waves, (R + 127) / 128));
  s.rows = std::max<int64_t>(1, ((R + want - 1) / want + 15) / 16) * 16;
  s.parts = std::max<int64_t>(1, (R + s.rows - 1) / s.rows);
  return s;
}

// V4: 16-byte loads (both row strides and both bases are multiples of 16 bytes,
// P and Q multiples of 4); else four 4-byte loads with their own bounds.
template <bool V4>
__device__ __forceinline__ f4 load_row(const float *__restrict__ M, int64_t ld, int64_t r, int64_t r1, int32_t col,
                                       int32_t cols) {
  f4 v = (f4)(0.0f);
  if (r >= r1) return v;  // rows past the range add exactly zero
  if constexpr (V4) {
    if (col < cols) v = *reinterpret_cast<const f4 *>(M + r * ld + col);
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (col + t < cols) v[t] = M[r * ld + col + t];
  }
  return v;
}

template <bool V4>
__global__ __launch_bounds__(256) void k_gemm_tn(const float *__restrict__ X, int64_t ldx,
                                                 const float *__restrict__ Y, int64_t ldy, int64_t R, int32_t P,
                                                 int32_t Q, Shape sh, float *__restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int tiles = sh.gp * sh.gq, tile = wave % tiles;
  const int64_t range = (int64_t)blockIdx.x * sh.subs + wave / tiles;
  const int32_t p0 = ((int32_t)(blockIdx.y / sh.groups_q) * sh.gp + tile / sh.gq) * kTile;
  const int32_t q0 = ((int32_t)(blockIdx.y % sh.groups_q) * sh.gq + tile % sh.gq) * kTile;
  if (range >= sh.parts || p0 >= P || q0 >= Q) return;  // wave-uniform
  const int64_t r0 = range * sh.rows, r1 = min(R, r0 + sh.rows);
  f4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = (f4)(0.0f);
  f4 x[2][kUnroll], y[2][kUnroll];
  auto fetch = [&](int64_t r, f4(&xs)[kUnroll], f4(&ys)[kUnroll]) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      xs[u] = load_row<V4>(X, ldx, r + u * kStepRows + g, r1, p0 + 4 * c, P);
      ys[u] = load_row<V4>(Y, ldy, r + u * kStepRows + g, r1, q0 + 4 * c, Q);
    }
  };
  auto mma = [&](const f4(&xs)[kUnroll], const f4(&ys)[kUnroll]) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[u][a], ys[u][b], acc[a][b], 0, 0, 0);
  };
  constexpr int kRound = kUnroll * kStepRows;
  fetch(r0, x[0], y[0]);
  for (int64_t r = r0; r < r1; r += 2 * kRound) {  // two rounds: static buffer roles
    fetch(r + kRound, x[1], y[1]);
    mma(x[0], y[0]);
    fetch(r + 2 * kRound, x[0], y[0]);
    mma(x[1], y[1]);
  }
  // D[4 g + v][c] of sub-tile (a, b) is output row p0 + 4 (4 g + v) + a, column q0 + 4 c + b
  float *__restrict__ out = part + range * (int64_t)P * Q;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t p = p0 + 4 * (4 * g + v) + a;
      if (p >= P) continue;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (q0 + 4 * c + b < Q) out[(int64_t)p * Q + q0 + 4 * c + b] = acc[a][b][v];
    }
}

// C[e] = sum of the partial tiles' element e: 32 elements per workgroup, 8
// threads each taking every 8th partial, their sums added in order.
__global__ __launch_bounds__(256) void k_gemm_tn_sum(const float *__restrict__ part, int64_t parts, int64_t elems,
                                                     float *__restrict__ C) {
  __shared__ float sums[8][32];
  const int t = threadIdx.x & 31, s = threadIdx.x >> 5;
  const int64_t e = (int64_t)blockIdx.x * 32 + t;
  float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
  if (e < elems) {
    int64_t q = s;
    for (; q + 24 < parts; q += 32) {
      a0 += part[q * elems + e];
      a1 += part[(q + 8) * elems + e];
      a2 += part[(q + 16) * elems + e];
      a3 += part[(q + 24) * elems + e];
    }
    for (; q < parts; q += 8) a0 += part[q * elems + e];
  }
  sums[s][t] = (a0 + a1) + (a2 + a3);
  __syncthreads();
  if (s == 0 && e < elems) {
    float v = sums[0][t];
    for (int i = 1; i < 8; ++i) v += sums[i][t];
    C[e] = v;
  }
}

}  // namespace

extern "C" int sd_gemm_tn_workspace(int64_t rows, int32_t p, int32_t q, size_t *bytes) {
  if (!bytes || rows < 0 || p < 1 || q < 1) return SD_ERR_INVALID_VALUE;
  *bytes = (size_t)shape_for(rows, p, q).parts * (size_t)p * (size_t)q * sizeof(float);
  return SD_OK;
}

extern "C" int sd_gemm_tn(const float *X, int64_t ldx, const float *Y, int64_t ldy, int64_t rows, int32_t p, int32_t q,
                          float *C, void *workspace, size_t workspace_bytes, void *stream) {
  if (rows < 0 || p < 1 || q < 1 || ldx < p || ldy < q || !C || !workspace || (rows > 0 && (!X || !Y)))
    return SD_ERR_INVALID_VALUE;
  const Shape sh = shape_for(rows, p, q);
  if (workspace_bytes < (size_t)sh.parts * (size_t)p * (size_t)q * sizeof(float)) return SD_ERR_INVALID_VALUE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  float *part = static_cast<float *>(workspace);
  const int32_t tp = (p + kTile - 1) / kTile;
  const int64_t gy = (int64_t)((tp + sh.gp - 1) / sh.gp) * sh.groups_q, gx = (sh.parts + sh.subs - 1) / sh.subs;
  const int64_t elems = (int64_t)p * q;
  if (gy > 65535 || gx > INT32_MAX || (elems + 31) / 32 > INT32_MAX) return SD_ERR_OVERFLOW;
  const bool v4 = p % 4 == 0 && q % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 &&
                  (reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y)) % 16 == 0;
  if (v4)
    hipLaunchKernelGGL(k_gemm_tn<true>, dim3((uint32_t)gx, (uint32_t)gy), dim3(256), 0, s, X, ldx, Y, ldy, rows, p, q,
                       sh, part);
  else
    hipLaunchKernelGGL(k_gemm_tn<false>, dim3((uint32_t)gx, (uint32_t)gy), dim3(256), 0, s, X, ldx, Y, ldy, rows, p, q,
                       sh, part);
  hipLaunchKernelGGL(k_gemm_tn_sum, dim3((uint32_t)((elems + 31) / 32)), dim3(256), 0, s, part, sh.parts, elems, C);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? SD_OK : sd::report_hip_error((int)e);
}
