// Calibration-aware MWQ (Sec. 3.3.1: Eq. 3 and Eq. 5 minimise the output
// error ||WX - W^X||^2 over calibration activations X; Algorithm 1 quantizes
// the weights block by block and moves each block's quantization error onto
// the columns not yet quantized through H^c, the Cholesky factor of the
// inverse of H = 2 X X^T + lambda I).  Setup work, once per model.
//
// Factor (binary64): U = upper-triangular factor with H^-1 = U^T U.  With J
// the order-reversing permutation, J H J = L L^T (lower Cholesky factor L)
// gives H = V V^T with V = J L J upper triangular, so H^-1 = V^-T V^-1 and
// U = V^-1 = J L^-1 J: one Cholesky factorization and one triangular
// inverse.  Both are blocked in 64 x 64 tiles; every tile product sums in a
// fixed order, so the factor is deterministic.
//
// Calibrated pack (binary32): the integer codes are decided exactly as the
// plain pack decides them (same per-group rules, same arithmetic, no FMA
// contraction), on targets that the compensation has moved; the
// compensation E = D U_BB^-1, T_F -= E U_BF is written as fmaf chains in
// ascending index order, one chain per element, so the GPU reproduces the
// CPU definition of the algorithm bit for bit.  Rows are independent: the
// update of a row's later columns uses only that row's block error.
#pragma clang fp contract(off)

#include <type_traits>

#include "internal.h"

namespace d2moe {
namespace {

constexpr int FT = 64;  // factor tile

// ---- factor ----------------------------------------------------------------

__global__ void info_init_kernel(int32_t* info) { *info = 0; }

// Lower tiles of Hr = J H J, H[a][b] = 2 sum_t X[t][a] X[t][b] + lambda [a == b].
__global__ __launch_bounds__(256) void hessian_kernel(const float* __restrict__ X, int tokens,
                                                      int n, double lambda, double* __restrict__ A) {
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  __shared__ double xa[16][FT], xb[16][FT];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  double acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = 0.0;
  for (int t0 = 0; t0 < tokens; t0 += 16) {
    for (int idx = threadIdx.x; idx < 16 * FT; idx += 256) {
      const int tt = idx / FT, c = idx % FT, t = t0 + tt;
      const int fa = n - 1 - (ti * FT + c), fb = n - 1 - (tj * FT + c);
      xa[tt][c] = t < tokens ? (double)X[(size_t)t * n + fa] : 0.0;
      xb[tt][c] = t < tokens ? (double)X[(size_t)t * n + fb] : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int tt = 0; tt < 16; ++tt) {
      double a[4], b[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = xa[tt][ty * 4 + r];
#pragma unroll
      for (int c = 0; c < 4; ++c) b[c] = xb[tt][tx * 4 + c];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = fma(a[r], b[c], acc[r][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti * FT + ty * 4 + r, j = tj * FT + tx * 4 + c;
      A[(size_t)i * n + j] = 2.0 * acc[r][c] + (i == j ? lambda : 0.0);
    }
}

__device__ inline double lane_value(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Between one wave's LDS writes and other lanes' reads of them.  The hardware
// serves a wave's LDS accesses in order; this keeps the compiler to that order and
// costs no instruction.
__device__ inline void wave_handoff() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(integral_constant<int, w>) for w = FT, FT - kPhase, .., kPhase.
constexpr int kPhase = 16;
template <int W = FT, typename F>
__device__ __attribute__((always_inline)) inline void phases(F&& f) {
  f(std::integral_constant<int, W>{});
  if constexpr (W > kPhase) phases<W - kPhase>(f);
}

// Cholesky factorization of diagonal tile k (its trailing updates from the
// tiles left of it are already applied) by one wave: lane r holds row r in
// registers, column j's multipliers come from LDS, and no step waits on a
// barrier.  The columns are a loop: v[i] is column j + i of step j, and the
// update of a step moves every column down one register.  Written out column by
// column the code is run once only, and fetching it (about 60 KB) takes longer
// than the arithmetic; the loops of kPhase columns shorten with the columns
// left: 57 -> 31 us a tile.
// A non-positive pivot records its 1-based column in *info (first failure wins)
// and continues with pivot 1.
__global__ __launch_bounds__(64) void potrf_diag_kernel(double* __restrict__ A, int n, int k,
                                                        int32_t* __restrict__ info) {
  __shared__ double a[FT][FT + 1];
  // l[i] = L[j + i][j]; what lies past the last row is read and not used
  __shared__ __attribute__((aligned(16))) double l[FT];
  const size_t base = (size_t)k * FT;
  const int r = threadIdx.x;
#pragma unroll 16
  for (int i = 0; i < FT; ++i) a[i][r] = A[(base + i) * n + base + r];
  l[r] = 0.0;
  __syncthreads();
  double v[FT];
#pragma unroll
  for (int c = 0; c < FT; ++c) v[c] = a[r][c];
  phases([&](auto wc) {
    constexpr int W = decltype(wc)::value;  // columns left at the first step
#pragma clang loop unroll(disable)
    for (int j = FT - W; j < FT - W + kPhase; ++j) {
      double d = lane_value(v[0], j);
      if (!(d > 0.0)) {
        if (r == 0) atomicCAS(info, 0, (int32_t)(base + j + 1));
        d = 1.0;
      }
      d = sqrt(d);
      const double x = r == j ? d : v[0] / d;
      a[r][j] = r >= j ? x : 0.0;
      if (r >= j) l[r - j] = x;
      wave_handoff();
#pragma unroll
      for (int i = 1; i < W; ++i) v[i - 1] = fma(-x, l[i], v[i]);
      wave_handoff();
    }
  });
  __syncthreads();
#pragma unroll 8
  for (int i = 0; i < FT; ++i) A[(base + i) * n + base + r] = a[i][r];
}

// Panel tiles below diagonal tile k: A[i][k] <- A[i][k] L_kk^-T.  One lane
// per tile row, held in registers; each solved column is taken off the later
// ones at once (every element still sees its terms in ascending column order).  Written out,
// unlike the diagonal tile: 23 us a launch, 32 as loops of kPhase columns, as its
// workgroups share the instructions and a loop waits for its LDS reads.
__global__ __launch_bounds__(64) void trsm_kernel(double* __restrict__ A, int n, int k) {
  __shared__ __attribute__((aligned(16))) double lt[FT][FT + 2];  // lt[j][m] = L[m][j]
  __shared__ double b[FT][FT + 1];
  const size_t bk = (size_t)k * FT, bi = (size_t)(k + 1 + blockIdx.x) * FT;
  const int r = threadIdx.x;
#pragma unroll 8
  for (int i = 0; i < FT; ++i) {
    lt[r][i] = A[(bk + i) * n + bk + r];
    b[i][r] = A[(bi + i) * n + bk + r];
  }
  __syncthreads();
  double v[FT];
#pragma unroll
  for (int c = 0; c < FT; ++c) v[c] = b[r][c];
#pragma unroll
  for (int j = 0; j < FT; ++j) {
    v[j] = v[j] / lt[j][j];
#pragma unroll
    for (int m = j + 1; m < FT; ++m) v[m] = fma(-v[j], lt[j][m], v[m]);
  }
#pragma unroll
  for (int c = 0; c < FT; ++c) b[r][c] = v[c];
  __syncthreads();
#pragma unroll 8
  for (int i = 0; i < FT; ++i) A[(bi + i) * n + bk + r] = b[i][r];
}

// Trailing update of the lower tiles (i, j), k < j <= i:
// A[i][j] -= A[i][k] A[j][k]^T.
__global__ __launch_bounds__(256) void chol_update_kernel(double* __restrict__ A, int n, int k) {
  const int i = k + 1 + blockIdx.y, j = k + 1 + blockIdx.x;
  if (j > i) return;
  __shared__ double pa[FT][FT + 1], pb[FT][FT + 1];
  const size_t bk = (size_t)k * FT, bi = (size_t)i * FT, bj = (size_t)j * FT;
  for (int idx = threadIdx.x; idx < FT * FT; idx += 256) {
    const int r = idx / FT, c = idx % FT;
    pa[r][c] = A[(bi + r) * n + bk + c];
    pb[r][c] = A[(bj + r) * n + bk + c];
  }
  __syncthreads();
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  double acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = 0.0;
  for (int m = 0; m < FT; ++m) {
    double a[4], b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = pa[ty * 4 + r][m];
#pragma unroll
    for (int c = 0; c < 4; ++c) b[c] = pb[tx * 4 + c][m];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[r][c] = fma(a[r], b[c], acc[r][c]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const size_t o = (bi + ty * 4 + r) * n + bj + tx * 4 + c;
      A[o] = A[o] - acc[r][c];
    }
}

// Inverse of every lower-triangular diagonal tile: M_kk = L_kk^-1 (one lane
// per column, forward substitution).
__global__ __launch_bounds__(64) void trinv_diag_kernel(const double* __restrict__ L,
                                                        double* __restrict__ M, int n) {
  __shared__ double l[FT][FT + 1], y[FT][FT + 1];
  const size_t bk = (size_t)blockIdx.x * FT;
  for (int idx = threadIdx.x; idx < FT * FT; idx += 64) {
    const int r = idx / FT, c = idx % FT;
    l[r][c] = L[(bk + r) * n + bk + c];
  }
  __syncthreads();
  const int c = threadIdx.x;
  for (int r = 0; r < FT; ++r) {
    double v = r == c ? 1.0 : 0.0;
    for (int m = c; m < r; ++m) v = fma(-l[r][m], y[m][c], v);
    y[r][c] = r < c ? 0.0 : v / l[r][r];
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < FT * FT; idx += 64) {
    const int r = idx / FT, cc = idx % FT;
    M[(bk + r) * n + bk + cc] = y[r][cc];
  }
}

// M = L^-1 below the diagonal, M[i][k] = -M_ii (sum_{m=k}^{i-1} L[i][m] M[m][k]).
// Step m adds term m to the sums of every tile (i, k), k <= m < i, kept in M's
// own tiles, and finishes block row m + 1, whose sums are then complete: the
// terms of an element are added in ascending m as before, but one step is
// m + 1 columns of n/64 - m - 1 tiles in parallel instead of one serial row
// (n = 2048: 31 launches of
// 19 us, 163 us as rows).
__global__ __launch_bounds__(256) void trinv_step_kernel(const double* __restrict__ L,
                                                         double* __restrict__ M, int n, int m) {
  const int k = blockIdx.x, i = m + 1 + blockIdx.y;
  __shared__ double pa[FT][FT + 1], pb[FT][FT + 1];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const size_t bi = (size_t)i * FT, bk = (size_t)k * FT, bm = (size_t)m * FT;
  double acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = k < m ? M[(bi + ty * 4 + r) * n + bk + tx * 4 + c] : 0.0;
  auto load = [&](const double* A, size_t row, size_t col, double (&t)[FT][FT + 1]) {
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = A[(row + threadIdx.x / FT + 4 * q) * n + col + threadIdx.x % FT];
#pragma unroll
    for (int q = 0; q < 16; ++q) t[threadIdx.x / FT + 4 * q][threadIdx.x % FT] = v[q];
  };
  auto product = [&] {  // acc += pa pb
#pragma unroll 4
    for (int q = 0; q < FT; ++q) {
      double a[4], b[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = pa[ty * 4 + r][q];
#pragma unroll
      for (int c = 0; c < 4; ++c) b[c] = pb[q][tx * 4 + c];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = fma(a[r], b[c], acc[r][c]);
    }
  };
  load(L, bi, bm, pa);
  load(M, bm, bk, pb);
  __syncthreads();
  product();
  if (i == m + 1) {  // workgroup-uniform: the sums of this block row are complete
    __syncthreads();
    load(M, bi, bi, pa);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        pb[ty * 4 + r][tx * 4 + c] = acc[r][c];
        acc[r][c] = 0.0;
      }
    __syncthreads();
    product();
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[r][c] = -acc[r][c];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) M[(bi + ty * 4 + r) * n + bk + tx * 4 + c] = acc[r][c];
}

// U[a][b] = M[n-1-a][n-1-b] rounded to binary32 on and above the diagonal.
__global__ __launch_bounds__(256) void reverse_round_kernel(const double* __restrict__ M,
                                                            float* __restrict__ U, int n) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)n * n) return;
  const int a = (int)(idx / n), b = (int)(idx % n);
  U[idx] = b >= a ? (float)M[(size_t)(n - 1 - a) * n + (n - 1 - b)] : 0.0f;
}

// ---- calibrated pack ---------------------------------------------------------

__global__ __launch_bounds__(256) void copy_rows_kernel(const float* __restrict__ src,
                                                        float* __restrict__ dst, size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) dst[i] = src[i];
}

// Quantize block [b0, b0 + GAMMA) of level `lev` from the rows' current
// targets T, write the codes into the packed layout, update the rows' residual
// chains R, and solve E = D U_BB^-1 for their block errors D.
//   W: the expert's original rows [N][h]; T, R: [N][h]; E: [N][GAMMA].
// A wave takes kQuantRows rows with lane l holding columns l, l + 64 of each: a
// ballot is two plane words, and the solve takes column j's error (a lane
// broadcast, one division for all rows) off the later columns of every lane,
// U's row from LDS, so a column costs one step instead of j dependent ones.
// Every element still sees its terms in ascending column order.  Only the sum
// of magnitudes is one chain per (row, group), run by a lane each from LDS.
// 2816 x 2048, blocks of 128: 24 us a launch (26 with U in rounds of 4-byte
// loads, 228 with one lane per row).
constexpr int kQuantRows = 4, kQuantWaves = 4;
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // U: 4-byte aligned
template <int G, int GAMMA>
__global__ __launch_bounds__(64 * kQuantWaves) void calib_quant_kernel(
    const float* __restrict__ W, const float* __restrict__ T, float* __restrict__ R,
    const float* __restrict__ U, float* __restrict__ E, MwqView m, uint32_t* __restrict__ planes,
    uint16_t* __restrict__ scales, uint8_t* __restrict__ zeros, int e, int lev, int b0) {
  constexpr int C = GAMMA / 64, NG = GAMMA / G;  // columns per lane, groups per block
  constexpr int CG = G / 64;                     // lane columns per group
  constexpr int BR = 2048 / G;
  __shared__ __attribute__((aligned(16))) float us[GAMMA][GAMMA];
  __shared__ __attribute__((aligned(16))) float mag[kQuantWaves][kQuantRows][GAMMA + 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = (blockIdx.x * kQuantWaves + wave) * kQuantRows;
  const int h = m.cols;
  const int qmax = (1 << m.b_min) - 1;

  float t[kQuantRows][C], w[kQuantRows][C];  // targets; W (level 0) or the residual chain
#pragma unroll
  for (int r = 0; r < kQuantRows; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const size_t at = (size_t)(n0 + r) * h + b0 + 64 * c + lane;
      const bool ok = n0 + r < m.rows;
      t[r][c] = ok ? T[at] : 0.0f;
      w[r][c] = ok ? (lev == 0 ? W[at] : R[at]) : 0.0f;
    }
  // the block of U: all loads of a thread in flight at once, under the
  // quantization below
  constexpr int kUVec = GAMMA * GAMMA / 4 / (64 * kQuantWaves);
  f4u uv[kUVec];
#pragma unroll
  for (int q = 0; q < kUVec; ++q) {
    const int at = 4 * ((int)threadIdx.x + 64 * kQuantWaves * q);
    uv[q] = *(const f4u*)(U + (size_t)(b0 + at / GAMMA) * h + b0 + at % GAMMA);
  }

  float v[kQuantRows][C];  // block errors, then E
  if (lev == 0) {
#pragma unroll
    for (int r = 0; r < kQuantRows; ++r) {
      const int n = n0 + r;
      const bool ok = n < m.rows;  // wave-uniform
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float mn = 0.0f, mx = 0.0f;
#pragma unroll
        for (int c = g * CG; c < (g + 1) * CG; ++c) {
          mn = t[r][c] < mn ? t[r][c] : mn;
          mx = t[r][c] > mx ? t[r][c] : mx;
        }
        for (int off = 32; off > 0; off >>= 1) {
          const float a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
          mn = a < mn ? a : mn;
          mx = b > mx ? b : mx;
        }
        const float range = mx - mn;
        uint16_t s_h = f2h(range / (float)qmax);
        float s1 = h2f(s_h);
        if (!(s1 > 0.0f) || __builtin_isinf(s1)) {
          s_h = 0x3c00u;
          s1 = 1.0f;
        }
        float zf = rintf(-mn / s1);
        zf = zf < 0.0f ? 0.0f : zf;
        zf = zf > (float)qmax ? (float)qmax : zf;
        const int z = (int)zf;
        const size_t blk = m.block(e, ok ? n / BR : 0, b0 / G + g);
        const int i = n % BR;
        if (ok && lane == 0) {
          zeros[m.zero_idx(blk, i)] = (uint8_t)z;
          scales[m.scale_idx(blk, 0, i)] = s_h;
        }
#pragma unroll
        for (int c = g * CG; c < (g + 1) * CG; ++c) {
          const float x = t[r][c];
          float qf = rintf(x / s1 + (float)z);
          qf = qf < 0.0f ? 0.0f : qf;
          qf = qf > (float)qmax ? (float)qmax : qf;
          const int q = (int)qf;
          const float what = (float)(q - z) * s1;
          v[r][c] = x - what;
          w[r][c] = w[r][c] - what;
          for (int p = 0; p < m.b_min; ++p) {
            const uint64_t bits = __ballot((q >> p) & 1);
            if (ok && lane < 2)
              planes[m.plane_word(blk, p, (2 * (c - g * CG) + lane) * BR + i)] =
                  (uint32_t)(lane ? bits >> 32 : bits);
          }
        }
      }
    }
  } else {
#pragma unroll
    for (int r = 0; r < kQuantRows; ++r)
#pragma unroll
      for (int c = 0; c < C; ++c) mag[wave][r][64 * c + lane] = fabsf(t[r][c]);
    wave_handoff();
    // lane r NG + g sums group g of row r in ascending column order
    float acc = 0.0f;
    if (lane < kQuantRows * NG) {
      const float4* src = (const float4*)&mag[wave][lane / NG][(lane % NG) * G];
#pragma unroll 4
      for (int k = 0; k < G / 4; ++k) {
        const float4 x = src[k];
        acc = acc + x.x;
        acc = acc + x.y;
        acc = acc + x.z;
        acc = acc + x.w;
      }
    }
    const uint32_t sb_l = f2h(acc / (float)G);
#pragma unroll
    for (int r = 0; r < kQuantRows; ++r) {
      const int n = n0 + r;
      const bool ok = n < m.rows;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const uint16_t sb_h = (uint16_t)__builtin_amdgcn_readlane(sb_l, r * NG + g);
        const float sb = h2f(sb_h);
        const size_t blk = m.block(e, ok ? n / BR : 0, b0 / G + g);
        const int i = n % BR, p = m.b_min + lev - 1;
        if (ok && lane == 0) scales[m.scale_idx(blk, lev, i)] = sb_h;
#pragma unroll
        for (int c = g * CG; c < (g + 1) * CG; ++c) {
          const float x = t[r][c];
          const bool pos = x >= 0.0f;  // -0.0 >= 0: sign +1
          const uint64_t bits = __ballot(pos);
          if (ok && lane < 2)
            planes[m.plane_word(blk, p, (2 * (c - g * CG) + lane) * BR + i)] =
                (uint32_t)(lane ? bits >> 32 : bits);
          v[r][c] = pos ? (x - sb) : (x + sb);
          w[r][c] = pos ? (w[r][c] - sb) : (w[r][c] + sb);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kQuantRows; ++r)
    if (n0 + r < m.rows)
#pragma unroll
      for (int c = 0; c < C; ++c) R[(size_t)(n0 + r) * h + b0 + 64 * c + lane] = w[r][c];
#pragma unroll
  for (int q = 0; q < kUVec; ++q) {
    const int at = 4 * ((int)threadIdx.x + 64 * kQuantWaves * q);
    *(float4*)&us[at / GAMMA][at % GAMMA] = float4{uv[q].x, uv[q].y, uv[q].z, uv[q].w};
  }
  __syncthreads();  // the block of U is in LDS

  // E = D U_BB^-1, forward substitution in ascending order
#pragma unroll
  for (int cj = 0; cj < C; ++cj) {
    float un[C], dn = us[64 * cj][64 * cj];
#pragma unroll
    for (int c = cj; c < C; ++c) un[c] = us[64 * cj][64 * c + lane];
    for (int lj = 0; lj < 64; ++lj) {
      float u[C];
      const float diag = dn;
#pragma unroll
      for (int c = cj; c < C; ++c) u[c] = un[c];
      const int jn = 64 * cj + min(lj + 1, 63);  // the next row of U is read ahead
      dn = us[jn][jn];
#pragma unroll
      for (int c = cj; c < C; ++c) un[c] = us[jn][64 * c + lane];
      // the rows' column-j values side by side in lanes 0 .. kQuantRows - 1
      float x = 0.0f;
#pragma unroll
      for (int r = 0; r < kQuantRows; ++r) {
        const float vj =
            __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v[r][cj]), lj));
        x = lane == r ? vj : x;
      }
      x = x / diag;
#pragma unroll
      for (int r = 0; r < kQuantRows; ++r) {
        const float ej = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), r));
        const float upd = fmaf(-ej, u[cj], v[r][cj]);
        v[r][cj] = lane > lj ? upd : lane == lj ? ej : v[r][cj];
#pragma unroll
        for (int c = cj + 1; c < C; ++c) v[r][c] = fmaf(-ej, u[c], v[r][c]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kQuantRows; ++r)
    if (n0 + r < m.rows)
#pragma unroll
      for (int c = 0; c < C; ++c) E[(size_t)(n0 + r) * GAMMA + 64 * c + lane] = v[r][c];
}

// T[n][f] -= sum_j E[n][j] U[b0 + j][f] for the columns f >= b0 + gamma, as
// one fmaf chain per element in ascending j.  Tile: 64 rows x 64 columns,
// 4 x 4 per thread, E transposed in LDS so that a step reads two 16-byte
// vectors for 16 products; 32 columns of E at a time keep the tile at 16 KB,
// so that several workgroups share a compute unit.  2816 x 2048: 19 us a
// launch on average, 82 us with 64 x 32 tiles of 128 threads.
constexpr int kUpdTile = 64, kUpdDepth = 32;
__global__ __launch_bounds__(256) void calib_update_kernel(float* __restrict__ T,
                                                           const float* __restrict__ U,
                                                           const float* __restrict__ E, int N,
                                                           int h, int b0, int gamma) {
  __shared__ __attribute__((aligned(16))) float es[kUpdDepth][kUpdTile + 4];
  __shared__ __attribute__((aligned(16))) float us[kUpdDepth][kUpdTile];
  const int n0 = blockIdx.y * kUpdTile;
  const int f0 = b0 + gamma + blockIdx.x * kUpdTile;
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  float acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = n0 + ty * 4 + r;
    const float4 v = n < N ? *(const float4*)(T + (size_t)n * h + f0 + tx * 4)
                           : float4{0.f, 0.f, 0.f, 0.f};
    acc[r][0] = v.x; acc[r][1] = v.y; acc[r][2] = v.z; acc[r][3] = v.w;
  }
  // this thread's part of a depth step: E row er, columns 4 ej .. and + 16;
  // U rows uj, uj + 16, columns 4 uc ..
  const int er = threadIdx.x % 64, ej = threadIdx.x / 64;
  const int uj = threadIdx.x / 16, uc = threadIdx.x % 16;
  for (int j0 = 0; j0 < gamma; j0 += kUpdDepth) {
    float4 ev[2];
    f4u uv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ev[q] = n0 + er < N ? *(const float4*)(E + (size_t)(n0 + er) * gamma + j0 + 4 * ej + 16 * q)
                          : float4{0.f, 0.f, 0.f, 0.f};
      uv[q] = *(const f4u*)(U + (size_t)(b0 + j0 + uj + 16 * q) * h + f0 + 4 * uc);
    }
    __syncthreads();  // the previous depth step has been read
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int j = 4 * ej + 16 * q;
      es[j][er] = ev[q].x; es[j + 1][er] = ev[q].y; es[j + 2][er] = ev[q].z; es[j + 3][er] = ev[q].w;
      *(float4*)&us[uj + 16 * q][4 * uc] = float4{uv[q].x, uv[q].y, uv[q].z, uv[q].w};
    }
    __syncthreads();
#pragma unroll 8
    for (int j = 0; j < kUpdDepth; ++j) {
      const float4 a = *(const float4*)&es[j][4 * ty], b = *(const float4*)&us[j][4 * tx];
      const float ea[4] = {a.x, a.y, a.z, a.w}, ub[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(-ea[r], ub[c], acc[r][c]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = n0 + ty * 4 + r;
    if (n < N)
      *(float4*)(T + (size_t)n * h + f0 + tx * 4) =
          float4{acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
  }
}

}  // namespace

size_t calib_factor_workspace(int n) { return (size_t)2 * n * n * sizeof(double); }

hipError_t launch_calib_factor(const float* X, int tokens, int n, double lambda, float* U,
                               void* ws, int32_t* info, hipStream_t s) {
  double* A = (double*)ws;
  double* M = A + (size_t)n * n;
  const int nb = n / FT;
  info_init_kernel<<<1, 1, 0, s>>>(info);
  hessian_kernel<<<dim3(nb, nb), 256, 0, s>>>(X, tokens, n, lambda, A);
  for (int k = 0; k < nb; ++k) {
    potrf_diag_kernel<<<1, 64, 0, s>>>(A, n, k, info);
    if (k + 1 < nb) {
      trsm_kernel<<<nb - k - 1, 64, 0, s>>>(A, n, k);
      chol_update_kernel<<<dim3(nb - k - 1, nb - k - 1), 256, 0, s>>>(A, n, k);
    }
  }
  trinv_diag_kernel<<<nb, 64, 0, s>>>(A, M, n);
  for (int m = 0; m + 1 < nb; ++m)
    trinv_step_kernel<<<dim3(m + 1, nb - m - 1), 256, 0, s>>>(A, M, n, m);
  const size_t total = (size_t)n * n;
  reverse_round_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(M, U, n);
  return hipGetLastError();
}

size_t calib_pack_workspace(int rows, int cols, int gamma) {
  return ((size_t)2 * rows * cols + (size_t)rows * gamma) * sizeof(float);
}

hipError_t launch_pack_calibrated(const float* W, const float* U, int gamma,
                                  const d2moe_mwq* out, void* ws, hipStream_t s) {
  const MwqView m = view_of(out);
  const int N = m.rows, h = m.cols;
  float* T = (float*)ws;
  float* R = T + (size_t)N * h;
  float* E = R + (size_t)N * h;
  const size_t count = (size_t)N * h;
  const unsigned cgrid = (unsigned)((count + 255) / 256);
  const int rgrid = (N + kQuantRows * kQuantWaves - 1) / (kQuantRows * kQuantWaves);
  for (int e = 0; e < m.E; ++e) {
    const float* We = W + (size_t)e * count;
    for (int lev = 0; lev < m.levels(); ++lev) {
      copy_rows_kernel<<<cgrid, 256, 0, s>>>(lev == 0 ? We : R, T, count);
      for (int b0 = 0; b0 < h; b0 += gamma) {
        auto quant = m.group == 128 ? calib_quant_kernel<128, 128>
                     : gamma == 128 ? calib_quant_kernel<64, 128>
                                    : calib_quant_kernel<64, 64>;
        quant<<<rgrid, 64 * kQuantWaves, 0, s>>>(We, T, R, U, E, m, out->planes, out->scales,
                                                 out->zeros, e, lev, b0);
        if (b0 + gamma < h)
          calib_update_kernel<<<dim3((h - b0 - gamma) / kUpdTile, (N + kUpdTile - 1) / kUpdTile),
                                256, 0, s>>>(T, U, E, N, h, b0, gamma);
      }
    }
  }
  return hipGetLastError();
}

}  // namespace d2moe
