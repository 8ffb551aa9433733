// fp32 contractions on the bf16 matrix instructions, shared by the fp32 kernels (attention, calibration).
//
// A float is the exact sum of three bf16 numbers: x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2 (8 significant bits each;
// the differences are exact).  Of the nine products of two such sums six are taken; the others are together at most 2^-24 of
// x * y, half a unit in the last place of a float (6e-9 of a dot product of 128 ordinary numbers, whose fp32 sum is off by 2e-7).
// Six bf16 instructions do the work of sixteen fp32 ones of the same duration, and unlike those they overlap with vector
// instructions.  The sum of the five small products has an accumulator of its own where there is room for one.
//
// Valid for operands up to LARGEST in magnitude (products and their sums stay finite, no part rounds to infinity, infinities
// and the difference of two of them do not occur) and, where tiny ones count, from SMALLEST on; the caller checks and takes the
// fp32 instructions on the same operand layout (32x32x2) otherwise.  NaN stays NaN.
#pragma once

#include "device_util.h"

namespace heatkv {
namespace f32s {

// Whether a launch of fp32 scales takes a kernel on these parts (32 queries per workgroup, one workgroup per compute unit) or
// one on the fp32 instructions (16, up to four): the former where it needs fewer turns of 256 workgroups (blocks16, blocks32:
// workgroups of either; t: queries).  Attention, fp32 instructions -> parts:
//   d = 128: 1 turn, 16 pairs 400 x 1939 keys 66 -> 57 us; 2 turns, 529 x 2160 111 -> 106, 784 x 2194 129 -> 105; as many turns
//   of either, 264 against 504 workgroups 47 -> 64; full chip, 196 x 855 keys 261 -> 226, 625 x 2525 1221 -> 1039.
//   d = 64, where the parts cost as much for half the products: 1 turn, 16 pairs 400 x 1939 38 -> 35; more turns only where they
//   are at most 0.6 times as many (3 against 2: 529 x 2160 59 -> 61, 40 pairs 4 against 3: 400 x 2060 67 -> 72; 4 against 2: 784 x
//   2194 72 -> 61) and from 400 queries on, 500 on a full chip (64 pairs, 4 turns, 400 x 1996 109 -> 107; 128 pairs, 7 turns 200 ->
//   203; 256 pairs, 324 x 1660 317 -> 319, 529 x 2525 526 -> 504).
//   Below 196 queries start and merge, which are longer, show, and the update's workgroups, which take a unit each: 40 pairs,
//   169 x 659 (240 + 240 workgroups) 32.7 -> 27.8 without it, 35.4 -> 36.4 with it; 36 pairs, 144 x 490 (200 + 144) 26.1 -> 22.1.
// Calibration alike, and from a number of workgroups on (calibrate.hip).
// Not for a softmax scale above 2^20 (or NaN), which makes scores of keys or queries whose parts are inexact (SMALLEST): below
// it they are off by less than 128 x 2^60 x 2^-134 x 2^20, nothing in an exponent.
inline bool pays(int d, int t, unsigned long long blocks16, unsigned long long blocks32, float sm_scale) {
  if (!(fabsf(sm_scale) <= 0x1p20f)) return false;
  const unsigned long long turns16 = (blocks16 + 255) / 256, turns32 = (blocks32 + 255) / 256;
  if (turns32 >= turns16) return false;
  if (t < 196) return t >= 128 && blocks32 <= 224;
  return d == 128 || turns32 == 1 || (t >= (turns32 <= 4 ? 400 : 500) && 5 * turns32 <= 3 * turns16);
}

constexpr float LARGEST = 0x1p60f;
// Below 2^-110 the third part of a number is no longer exact: bf16 has no bits below 2^-133.  Where such a number can decide
// an output on its own (a column of tiny values next to ordinary ones, a value that only a tiny probability meets) the
// caller takes the fp32 instructions from this magnitude down; zero has parts.
constexpr float SMALLEST = 0x1p-100f;
// Orders like the magnitude, but for zero, which comes last.
__device__ __forceinline__ unsigned above_zero(float x) { return 2 * __float_as_uint(x) - 1; }

// Eight numbers in three parts: elements 2 i, 2 i + 1 of part k are the halves of w[k][i].
struct Parts {
  unsigned w[3][4];
  __device__ __forceinline__ bf16x8 part(int k) const {
    return __builtin_bit_cast(bf16x8, make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]));
  }
  __device__ __forceinline__ void set(int k, bf16x8 x) {
    const uint4 u = __builtin_bit_cast(uint4, x);
    w[k][0] = u.x;
    w[k][1] = u.y;
    w[k][2] = u.z;
    w[k][3] = u.w;
  }
};

// Two numbers rounded to a packed pair.  Opaque: the compiler otherwise rounds the low one once more by itself where only it
// is needed.
__device__ __forceinline__ unsigned round_pair(float lo, float hi) {
  unsigned u = __builtin_bit_cast(unsigned, bf16x2{static_cast<bf16_t>(lo), static_cast<bf16_t>(hi)});
  asm("" : "+v"(u));
  return u;
}
// x - (the low or high half of a pair), exact.  Not as a two-element dot product with (-1, 0) or (0, -1), which would spare
// the shift: that instruction does not overlap with matrix instructions (next to a 32x32x16 of 36 cycles one of them takes
// it to 62, four additions to 42).
__device__ __forceinline__ float minus_low(float x, unsigned h) { return x - __uint_as_float(h << 16); }
__device__ __forceinline__ float minus_high(float x, unsigned h) { return x - __uint_as_float(h & 0xffff0000u); }

// The split in six pieces, to go between the six products of another step.  x is used up.
__device__ __forceinline__ void split_piece(Parts& p, float (&x)[8], int piece) {
  auto round = [&](int k, int i) { p.w[k][i] = round_pair(x[2 * i], x[2 * i + 1]); };
  auto rest = [&](int k, int i) {
    x[2 * i] = minus_low(x[2 * i], p.w[k][i]);
    x[2 * i + 1] = minus_high(x[2 * i + 1], p.w[k][i]);
  };
  if (piece == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) round(0, i);
  } else if (piece == 1) {
#pragma unroll
    for (int i = 0; i < 3; ++i) rest(0, i);
  } else if (piece == 2) {
    rest(0, 3);
#pragma unroll
    for (int i = 0; i < 4; ++i) round(1, i);
  } else if (piece == 3) {
#pragma unroll
    for (int i = 0; i < 3; ++i) rest(1, i);
  } else if (piece == 4) {
    rest(1, 3);
    round(2, 0);
    round(2, 1);
  } else {
    round(2, 2);
    round(2, 3);
  }
}
__device__ __forceinline__ void split(Parts& p, float (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) split_piece(p, x, i);
}

// Product m = 0..5 of a 32 x 16 by 16 x 32 product, the large one last, which is added to `large`, the others to `small`
// (which may be the same).  b's part 2 is free after product 0, part 1 after 2, part 0 after 5.
constexpr int PRODUCTS = 6;
__device__ __forceinline__ void add_product(int m, f32x16& small, f32x16& large, const Parts& a, const Parts& b) {
  constexpr int A[PRODUCTS] = {0, 1, 0, 2, 1, 0}, B[PRODUCTS] = {2, 1, 1, 0, 0, 0};
  f32x16& acc = m == PRODUCTS - 1 ? large : small;
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.part(A[m]), b.part(B[m]), acc, 0, 0, 0);
}
// The same product on the fp32 instructions: step j takes element j of both operands.
__device__ __forceinline__ void add_f32(f32x16& acc, const float (&a)[8], const float (&b)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc, 0, 0, 0);
}

__device__ __forceinline__ float magnitude(float m, const float (&x)[8]) {
#pragma unroll
  for (int j = 0; j < 8; j += 2) m = fmaxf(m, fmaxf(fabsf(x[j]), fabsf(x[j + 1])));
  return m;
}

}  // namespace f32s
}  // namespace heatkv
