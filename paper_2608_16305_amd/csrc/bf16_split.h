// Float32 operands of the bfloat16 matrix instructions, as the sum of three bfloat16 parts.
//
// x = hi + mid + lo, each the nearest bfloat16 of what is left: 24 significant bits, so a product with
// bfloat16 weights is three exact products, and one of two float32 operands is six (the three smallest,
// below 2^-26 of the whole, are left out).  Below 2^-109 the low part loses bits (the smallest bfloat16 is 2^-133).
// A 16x16x32 instruction takes a sixteenth of the time that
// 16x16x4 float32 ones take for as many products, and rounds its float32 sum once per 32 of them instead
// of once per product.
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

namespace mtgnn {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Two floats to the nearest bfloat16s (one instruction).
__device__ __forceinline__ uint32_t cvt2_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}
__device__ __forceinline__ float lo_bf16(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }
constexpr float BF16_MAX = 3.3895313892515355e38f;

// The parts of eight floats (operands of one 16x16x32 instruction).  No arrays of vectors, which the compiler
// keeps in scratch memory.
struct Bf16Parts {
  bf16x8_t hi, mid, lo;
};
__device__ __forceinline__ bf16x8_t as_bf16x8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_bit_cast(bf16x8_t, u32x4_t{a, b, c, d});
}
__device__ __forceinline__ bf16x8_t round8_bf16(const float (&x)[8]) {   // values that are bfloat16 already: exact
  return as_bf16x8(cvt2_bf16(x[0], x[1]), cvt2_bf16(x[2], x[3]), cvt2_bf16(x[4], x[5]), cvt2_bf16(x[6], x[7]));
}
// ENDS: also for the ends of the range.  A finite x past the largest bfloat16 has that one as its high part; an
// infinite x has it too and an infinite middle part, and a finite low one, so that products with finite
// bfloat16 weights are what x's own would be.  Without: such an x gives infinite or NaN parts.
template <bool ENDS>
__device__ __forceinline__ void split_words(const float (&x)[8], uint32_t (&h)[4], uint32_t (&m)[4], uint32_t (&l)[4]) {
  auto high = [](float v) { return ENDS ? __builtin_amdgcn_fmed3f(v, -BF16_MAX, BF16_MAX) : v; };
  auto low = [](float v) { return ENDS ? __builtin_amdgcn_fmed3f(v, -1e34f, 1e34f) : v; };   // (at most 6e33; NaN: -1e34)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = cvt2_bf16(high(x[2 * i]), high(x[2 * i + 1]));
    const float a = x[2 * i] - lo_bf16(h[i]), b = x[2 * i + 1] - hi_bf16(h[i]);
    m[i] = cvt2_bf16(a, b);
    l[i] = cvt2_bf16(low(a - lo_bf16(m[i])), low(b - hi_bf16(m[i])));
  }
}
__device__ __forceinline__ Bf16Parts split_bf16(const float (&x)[8]) {
  uint32_t h[4], m[4], l[4];
  split_words<true>(x, h, m, l);
  return Bf16Parts{as_bf16x8(h[0], h[1], h[2], h[3]), as_bf16x8(m[0], m[1], m[2], m[3]),
                   as_bf16x8(l[0], l[1], l[2], l[3])};
}

// Both operands of a product of float32 values, as six instructions that each take one term for the first four
// and another for the last four of the eight: (hi hi | lo hi), (lo hi | hi hi), (hi mid | mid mid), (mid mid | hi mid),
// (mid hi | hi lo), (hi lo | mid hi).  Every instruction adds a sum of at least 2^-9 of the whole to its
// accumulator.  With an instruction a term the three smallest were a few units of a long sum's last place, and of
// nearly the same size in each step where a column hardly varies: rounded the same way every time, they
// left the attention's value gradient over 60,000 rows 2.6e-7 off (in pairs 1.4e-7, in one chain a block).
struct Bf16Left {
  bf16x8_t hl, lh, hm, mh;
};
struct Bf16Right {
  bf16x8_t hh, mm, hl, lh;
};
__device__ __forceinline__ Bf16Left split_left(const float (&x)[8]) {
  uint32_t h[4], m[4], l[4];
  split_words<false>(x, h, m, l);
  return Bf16Left{as_bf16x8(h[0], h[1], l[2], l[3]), as_bf16x8(l[0], l[1], h[2], h[3]),
                  as_bf16x8(h[0], h[1], m[2], m[3]), as_bf16x8(m[0], m[1], h[2], h[3])};
}
__device__ __forceinline__ Bf16Right split_right(const float (&x)[8]) {
  uint32_t h[4], m[4], l[4];
  split_words<false>(x, h, m, l);
  return Bf16Right{as_bf16x8(h[0], h[1], h[2], h[3]), as_bf16x8(m[0], m[1], m[2], m[3]),
                   as_bf16x8(h[0], h[1], l[2], l[3]), as_bf16x8(l[0], l[1], h[2], h[3])};
}

}  // namespace mtgnn
