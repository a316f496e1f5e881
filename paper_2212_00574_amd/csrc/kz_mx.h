// Common-neighbour tests as 4-bit matrix products (gfx950), shared by the
// single-graph edge pass and the batched path.
//
// Whether rows u and v share a neighbour in a word is whether the product of
// their bits, sum_j u_j v_j, is non-zero: a contraction, 64 x 64 pairs of
// two blocks at a time.  The bits become FP4 (E2M1) codes with one AND per
// eight of them: a 32-bit half word splits into four registers by bit
// position modulo 4, and the positions 0, 1 and 2 of a nibble are themselves
// the codes of 0.5, 1 and 2 (position 3, the sign, shifts down to 2).  The
// order of the 64 elements is the same on both sides, so it does not matter.
// Products are 0.25, 1 or 4 and sums stay below 64 * 4 times the words of a
// class, whole multiples of 0.25 far below 2^22: exact in FP32, and zero
// exactly when there is no common neighbour.
#pragma once

#include "kz_internal.h"

namespace kzi {

typedef unsigned mx_u4 __attribute__((ext_vector_type(4)));  // two 64-bit words
typedef unsigned mx_u2 __attribute__((ext_vector_type(2)));
typedef unsigned short mx_us2 __attribute__((ext_vector_type(2)));
typedef int mx_v8i __attribute__((ext_vector_type(8)));
typedef float mx_v16f __attribute__((ext_vector_type(16)));

// FP4 codes of 32 bits of a row (see above).
__device__ __forceinline__ mx_v8i mx_codes(unsigned w) {
  mx_v8i v = {};
  v[0] = (int)(w & 0x11111111u);
  v[1] = (int)(w & 0x22222222u);
  v[2] = (int)(w & 0x44444444u);
  v[3] = (int)((w >> 1) & 0x44444444u);
  return v;
}

// A 64-bit word per lane (lane = row) to the matrix operand's layout, which
// wants the two halves of a row's 64 elements in lanes r and r + 32: after
// the swap x holds rows 0..31 (low halves in lanes 0..31, high halves in
// lanes 32..63) and y the rows 32..63.
__device__ __forceinline__ mx_u2 mx_split(unsigned lo, unsigned hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
  return mx_u2{r[0], r[1]};
}

// 32 x 32 pairs, one word: c + the products of a's and b's bits.
__device__ __forceinline__ mx_v16f mx_mma(const mx_v8i &a, const mx_v8i &b, const mx_v16f &c) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 4, 4, 0, 0, 0, 0);
}

__device__ __forceinline__ unsigned mx_bits(float x) { return __builtin_bit_cast(unsigned, x); }

// 16 zeros and ones, element e to bit e.
__device__ __forceinline__ unsigned mx_pack(const unsigned (&m)[16]) {
  unsigned x = m[15];
#pragma unroll
  for (int e = 14; e >= 0; --e) x = (x << 1) | m[e];
  return x;
}

// Two sums as half floats, rounded towards zero (their smallest value above
// zero, 0.25, stays above it), as whole numbers of the same order.
__device__ __forceinline__ mx_us2 mx_halves(float x, float y) {
  return __builtin_bit_cast(mx_us2, __builtin_amdgcn_cvt_pkrtz(x, y));
}

// 16 whole numbers, element e's "not zero" to bit e.
__device__ __forceinline__ unsigned mx_pack_halves(const mx_us2 (&m)[8]) {
  unsigned x = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    x |= __builtin_bit_cast(unsigned, __builtin_elementwise_min(m[e], mx_us2{1, 1})) << (2 * e);
  return (x & 0xffffu) | (x >> 15);  // the even elements' bits, the odd elements' one place up
}

// Which of 64 x 64 pairs are set, from four 32 x 32 quarters (quarter (i, j):
// rows 32i.., columns 32j..; bit e of lane l is row 8 (e / 4) + 4 (l / 32) +
// e % 4, column l % 32): lane c gets column c's bits, bit r for row r.
__device__ __forceinline__ unsigned long long mx_columns(const unsigned (&m)[2][2], int lane) {
  unsigned out[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    unsigned s[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      // bit 4a + b to bit 8a + b, then the half of the wave that holds it
      unsigned x = m[i][j] & 0xffffu;
      x = (x | (x << 8)) & 0x00ff00ffu;
      x = (x | (x << 4)) & 0x0f0f0f0fu;
      s[j] = x << ((lane >> 5) * 4);
    }
    const mx_u2 both = mx_split(s[0], s[1]);  // the halves of column `lane`
    out[i] = both.x | both.y;
  }
  return ((unsigned long long)out[1] << 32) | out[0];
}

}  // namespace kzi
