// MWQ quantize + bit-plane pack (Sec. 3.3.1: Eq. 2 asymmetric base level,
// Eq. 4-5 binary residual levels, Algorithm 1 with X = I) and the debug
// unpack hook.
//
// The packed codes are integers decided by binary32 arithmetic, so this file
// is compiled without FMA contraction and every step runs in the same order
// as the specification in d2moe.h: one lane owns one (row, group) and walks its
// group sequentially.
#pragma clang fp contract(off)

#include "internal.h"

namespace d2moe {
namespace {

constexpr int kPackWaves = 4;  // groups (one per wave) of the same 64 rows per workgroup

typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));  // W needs no more than 4 bytes

// One lane = one (row, group): the group's weights are held in registers from
// the load to the last level, so the only memory traffic is W in and the codes
// out.  A wave takes 64 consecutive rows, the workgroup's waves neighbouring
// groups of them (whose rows share DRAM pages).  The sums of Eq. 5 stay one
// sequential chain per lane.
//
// A residual's sign is read off its sign bit: the residuals are never -0.0
// (the base residual has +0.0 added, which turns a -0.0 weight's into +0.0, and
// v - s and v + s round an exact zero to +0.0), so the bit is clear exactly
// where v >= 0.  Only NaN weights differ; a wave that meets one (its sum of
// magnitudes is NaN) compares instead.
//
// Bound by the vector ALU (about 50 operations per weight at six residual
// levels).  One 28672 x 4096 matrix, 2-bit base to 8 bits, group 128: 200 us,
// 3.0 TB/s of weights and codes; 1297 us when a 64-thread workgroup staged one
// group in LDS and walked it once per level.
template <int G>
__global__ __launch_bounds__(64 * kPackWaves)
__attribute__((amdgpu_waves_per_eu(G == 64 ? 4 : 3))) void pack_kernel(const float* __restrict__ W,
                                                              MwqView m,
                                                              uint32_t* __restrict__ planes,
                                                              uint16_t* __restrict__ scales,
                                                              uint8_t* __restrict__ zeros) {
  constexpr int BR = 2048 / G;
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 64 + lane;
  const int kb = blockIdx.y * kPackWaves + (threadIdx.x >> 6), e = blockIdx.z;
  if (kb >= m.KB() || n >= m.rows) return;
  const int i = n % BR;
  const size_t blk = m.block(e, n / BR, kb);
  const int qmax = (1 << m.b_min) - 1;

  float r[G];
  {
    const f4* src = (const f4*)(W + ((size_t)e * m.rows + n) * m.cols + (size_t)kb * G);
#pragma unroll
    for (int c = 0; c < G / 4; ++c) {
      const f4 v = src[c];
#pragma unroll
      for (int j = 0; j < 4; ++j) r[4 * c + j] = v[j];
    }
  }

  // base level: min-max range including 0
  float mn = 0.0f, mx = 0.0f;
#pragma unroll
  for (int k = 0; k < G; ++k) {
    mn = r[k] < mn ? r[k] : mn;
    mx = r[k] > mx ? r[k] : mx;
  }
  const float range = mx - mn;
  const float s_raw = range / (float)qmax;
  uint16_t s_h = f2h(s_raw);
  float s1 = h2f(s_h);
  if (!(s1 > 0.0f) || __builtin_isinf(s1)) {
    s_h = 0x3c00u;
    s1 = 1.0f;
  }
  float zf = rintf(-mn / s1);
  zf = zf < 0.0f ? 0.0f : zf;
  zf = zf > (float)qmax ? (float)qmax : zf;
  const int z = (int)zf;
  zeros[m.zero_idx(blk, i)] = (uint8_t)z;
  uint16_t* sc = scales + m.scale_idx(blk, 0, i);  // of the current level
  *sc = s_h;
  uint32_t* pl = planes + m.plane_word(blk, 0, i);

  // base codes -> planes 0 .. b_min-1; residual kept.  Code j of a run of 32
  // goes to byte j / 8 of word j % 8; an 8 x 8 bit transpose in every byte
  // then leaves bit j of plane p's word in word p.
#pragma unroll
  for (int sub = 0; sub < G / 32; ++sub) {
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const int k = sub * 32 + j;
      const float v = r[k];
      // clamped to [0, qmax]; NaN gives 0
      const float qf = __builtin_amdgcn_fmed3f(rintf(v / s1 + (float)z), 0.0f, (float)qmax);
      const int q = (int)qf;
      const float what = (qf - (float)z) * s1;  // both small integers: exact
      r[k] = (v - what) + 0.0f;
      w[j & 7] |= (uint32_t)q << (8 * (j >> 3));
      // here, not sunk to their later uses (registers)
      asm volatile("" : "+v"(w[j & 7]), "+v"(r[k]));
      if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // bounds the live temporaries
    }
    auto swap = [&](int lo, int hi, uint32_t mask, int sh) {
      const uint32_t a = w[lo], b = w[hi];
      w[lo] = (a & mask) | ((b << sh) & ~mask);
      w[hi] = ((a >> sh) & mask) | (b & ~mask);
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) swap(t, t + 4, 0x0F0F0F0Fu, 4);
#pragma unroll
    for (int t = 0; t < 8; t += (t & 1) ? 3 : 1) swap(t, t + 2, 0x33333333u, 2);
#pragma unroll
    for (int t = 0; t < 8; t += 2) swap(t, t + 1, 0x55555555u, 1);
#pragma unroll
    for (int p = 0; p < 8; ++p)
      if (p < m.b_min) pl[64 * p + sub * BR] = w[p];
  }

  // residual levels: one sign plane + one scale per added bit
  pl += 64 * m.b_min;
  for (int lev = m.levels() - 1; lev > 0; --lev, pl += 64) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < G; ++k) acc = acc + fabsf(r[k]);
    const float s_mean = acc / (float)G;
    const uint16_t sb_h = f2h(s_mean);
    const float sb = h2f(sb_h);
    sc += BR;
    *sc = sb_h;
    const bool any_nan = __ballot(acc != acc) != 0;  // wave-uniform
#pragma unroll
    for (int sub = 0; sub < G / 32; ++sub) {
      uint32_t word = 0;
      if (any_nan) {
#pragma unroll
        for (int j = 31; j >= 0; --j) {
          const int k = sub * 32 + j;
          const bool pos = r[k] >= 0.0f;
          word = (word << 1) | (uint32_t)!pos;
          r[k] = pos ? (r[k] - sb) : (r[k] + sb);
          asm volatile("" : "+v"(r[k]));
        }
      } else {
#pragma unroll
        for (int j = 31; j >= 0; --j) {
          const int k = sub * 32 + j;
          word = __builtin_amdgcn_alignbit(word, __float_as_uint(r[k]), 31);  // word << 1 | sign
          r[k] = r[k] - copysignf(sb, r[k]);
          asm volatile("" : "+v"(r[k]));
        }
      }
      pl[sub * BR] = ~word;
    }
  }
}

// Element-wise unpack through the canonical addressing.
__global__ void debug_unpack_kernel(MwqView m, int e, int bits, uint8_t* __restrict__ q1,
                                    int8_t* __restrict__ signs) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t total = (size_t)m.rows * m.cols;
  if (idx >= total) return;
  const int n = (int)(idx / m.cols), k = (int)(idx % m.cols);
  const int BR = m.BR();
  const size_t blk = m.block(e, n / BR, k / m.group);
  const int w = ((k % m.group) / 32) * BR + n % BR;
  const int bit = k % 32;
  int q = 0;
  for (int p = 0; p < m.b_min; ++p) q |= (int)((m.planes[m.plane_word(blk, p, w)] >> bit) & 1u) << p;
  q1[idx] = (uint8_t)q;
  for (int p = m.b_min; p < bits; ++p) {
    const int s = (int)((m.planes[m.plane_word(blk, p, w)] >> bit) & 1u);
    signs[(size_t)(p - m.b_min) * total + idx] = s ? (int8_t)1 : (int8_t)-1;
  }
}

}  // namespace

hipError_t launch_pack(const float* W, const d2moe_mwq* out, hipStream_t s) {
  MwqView m = view_of(out);
  dim3 grid((m.rows + 63) / 64, (m.KB() + kPackWaves - 1) / kPackWaves, m.E);
  if (m.group == 64)
    pack_kernel<64><<<grid, 64 * kPackWaves, 0, s>>>(W, m, out->planes, out->scales, out->zeros);
  else
    pack_kernel<128><<<grid, 64 * kPackWaves, 0, s>>>(W, m, out->planes, out->scales, out->zeros);
  return hipGetLastError();
}

hipError_t launch_debug_unpack(const d2moe_mwq* w, int expert, int bits, uint8_t* q1,
                               int8_t* signs, hipStream_t s) {
  MwqView m = view_of(w);
  const size_t total = (size_t)m.rows * m.cols;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  debug_unpack_kernel<<<blocks, 256, 0, s>>>(m, expert, bits, q1, signs);
  return hipGetLastError();
}

}  // namespace d2moe
