// Lookup dequantization: two or three bit planes of many weights at once.
//
// The 2^n sums of n planes' signed scales are a table of binary16 values, held
// as one or two registers of low bytes and as many of high bytes, so that one
// byte permute looks up four weights' low (or high) bytes.  The indices of
// weights j, j + 8, j + 16, j + 24 are gathered in the four bytes of one word:
// the plane words are rotated so that a weight's bits follow one another,
// merged under masks that place several j in one word, and shifted down.
//
// Vector instructions for the 32 weights of a plane word, against the sign form
// (a shift, an and-or and a packed addition per plane and pair): three planes
// 70 / 144, two 55 / 96, and 16 more where the sum is added to an earlier one.
#pragma once
#include "internal.h"

namespace d2moe {
namespace lookup {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ inline h2 as_h2(uint32_t v) { return __builtin_bit_cast(h2, v); }
__device__ inline uint32_t as_u(h2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ inline uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }
__device__ inline uint32_t rotr(uint32_t v, int n) { return __builtin_amdgcn_alignbit(v, v, n); }

// Pairs (j, j + 16) and (j + 8, j + 24) of the table entries that the bytes of
// `idx` name; lo / hi hold the low / high bytes of entries 0..3 and 4..7.
__device__ inline void pairs(uint32_t idx, const uint32_t (&lo)[2], const uint32_t (&hi)[2], h2& a,
                             h2& b) {
  const uint32_t l = __builtin_amdgcn_perm(lo[1], lo[0], idx);
  const uint32_t h = __builtin_amdgcn_perm(hi[1], hi[0], idx);
  a = as_h2(__builtin_amdgcn_perm(h, l, 0x06020400u));
  b = as_h2(__builtin_amdgcn_perm(h, l, 0x07030501u));
}
// Splits entries (e0, e1), (e2, e3) into low and high bytes.
__device__ inline void split(h2 e01, h2 e23, uint32_t& lo, uint32_t& hi) {
  lo = __builtin_amdgcn_perm(as_u(e23), as_u(e01), 0x06040200u);
  hi = __builtin_amdgcn_perm(as_u(e23), as_u(e01), 0x07050301u);
}

// a[j] = pair (j, j + 16), a[NJ + j] = pair (j + 8, j + 24), j < NJ, of the planes
// w0, w1 (, w2) with scale pairs c0, c1 (, c2): a set bit adds its scale, a clear
// one subtracts it.  w1 comes rotated right by 31 and w2 by 30 (and all of them
// by 4 more to start at j = 4).  FIRST: the sum from `base`, plane after plane,
// the roundings of the sign form; otherwise the planes' own sum is added to
// a at once.
template <bool FIRST, int NJ>
__device__ __attribute__((always_inline)) inline void planes2(h2 (&a)[2 * NJ], uint32_t w0,
                                                              uint32_t w1, uint32_t c0,
                                                              uint32_t c1, h2 base) {
  const h2 s0 = as_h2(c0 ^ 0x00008000u), k1 = as_h2(c1);  // (-c0, +c0)
  const h2 e = FIRST ? base + s0 : s0;
  uint32_t lo[2], hi[2];
  split(e - k1, e + k1, lo[0], hi[0]);
  lo[1] = lo[0];
  hi[1] = hi[0];
  const uint32_t even = bfi(0x55555555u, w0, w1), odd = bfi(0xAAAAAAAAu, w0, w1);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const uint32_t d = j & 1 ? odd : even;
    h2 x, y;
    pairs((j ? rotr(d, j) : d) & 0x03030303u, lo, hi, x, y);
    a[j] = FIRST ? x : a[j] + x;
    a[NJ + j] = FIRST ? y : a[NJ + j] + y;
  }
}
template <bool FIRST, int NJ>
__device__ __attribute__((always_inline)) inline void planes3(h2 (&a)[2 * NJ], uint32_t w0,
                                                              uint32_t w1, uint32_t w2,
                                                              uint32_t c0, uint32_t c1,
                                                              uint32_t c2, h2 base) {
  const h2 s0 = as_h2(c0 ^ 0x00008000u), k1 = as_h2(c1), k2 = as_h2(c2);
  const h2 e = FIRST ? base + s0 : s0;
  const h2 e0 = e - k1, e1 = e + k1;
  uint32_t lo[2], hi[2];
  split(e0 - k2, e1 - k2, lo[0], hi[0]);
  split(e0 + k2, e1 + k2, lo[1], hi[1]);
  // word d holds the indices of weights d and d + 3 (d < 3), 6 and 7 of every
  // byte: bits j, j + 1, j + 2 of the rotated planes
  const uint32_t d0 = bfi(0x09090909u, w0, bfi(0x12121212u, w1, w2));
  const uint32_t d1 = bfi(0x12121212u, w0, bfi(0x24242424u, w1, w2));
  const uint32_t d2 = bfi(0x24242424u, w0, bfi(0x48484848u, w1, w2));
  const uint32_t d6 = bfi(0x40404040u, w0, bfi(0x80808080u, w1, w2));
  const uint32_t d7 = bfi(0x80808080u, w0, bfi(0x01010101u, w1, w2));
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const uint32_t d = j == 6 ? d6 : j == 7 ? d7 : j % 3 == 0 ? d0 : j % 3 == 1 ? d1 : d2;
    h2 x, y;
    pairs((j ? rotr(d, j) : d) & 0x07070707u, lo, hi, x, y);
    a[j] = FIRST ? x : a[j] + x;
    a[NJ + j] = FIRST ? y : a[NJ + j] + y;
  }
}

}  // namespace lookup
}  // namespace d2moe
