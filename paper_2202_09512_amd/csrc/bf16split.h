// fp32 operands of the matrix products as sums of three bf16 terms.  v_mfma_f32_16x16x32_bf16 does eight times the
// work of v_mfma_f32_16x16x4_f32 in about half its cycles, so a product x y kept as six term products, accumulated in
// fp32, costs a third of the fp32 instructions' cycles, and vector instructions of the other wave run beside it, which
// they do not beside fp32 MFMA (measured on this GPU).
//   x = x1 + d1 + d2 and y = y1 + y2 + y3, both exactly: 24 bits in three terms of 8.  Terms below 2^-133 are lost, so
//   values below 2^-110 have fewer bits than in fp32.
//   Of x y, d1 y3 and d2 y2 are left out (and d2 y3): below 2^-23 of it each.  One product is off by at most 2^-22.2, 2^-24.8
//   in the root mean square (measured; an fp32 product, which is only rounded once: 2^-24, 2^-25.2), random in sign; sums
//   of thousands of products are as good as those of the fp32 instructions (see kernels_dense.hip).
// bf16 has fp32's exponent range, so that nothing is scaled; a head that would round up to infinity is cut instead.  An
// infinite operand gives NaN (its rest is infinity minus infinity).
#pragma once
#include "common.h"

namespace nnr {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float cut_to_bf16(float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }

// the upper half-words of two floats: bf16(a) in the low half, bf16(b) in the high half (both cut)
__device__ __forceinline__ uint32_t pack_cut(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}

// two floats rounded to bf16 (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_round(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

// v = hi + lo + rest of 2^-16 |v|, hi and lo rounded to bf16, for four values of a lane (two packed words each)
__device__ __forceinline__ void split2(const float (&v)[4], uintx2& hi, uintx2& lo) {
  hi = uintx2{pack_round(v[0], v[1]), pack_round(v[2], v[3])};
  lo = uintx2{pack_round(v[0] - __uint_as_float(hi.x << 16), v[1] - __uint_as_float(hi.x & 0xFFFF0000u)),
              pack_round(v[2] - __uint_as_float(hi.y << 16), v[3] - __uint_as_float(hi.y & 0xFFFF0000u))};
}

// v = x1 + d1 + d2, exactly: the head x1 is v cut to 8 bits, d1 the rest of 16 bits rounded to 8, and what is left then has 8
__device__ __forceinline__ void split3(const float (&v)[4], uintx2& x1, uintx2& d1, uintx2& d2) {
  x1 = uintx2{pack_cut(v[0], v[1]), pack_cut(v[2], v[3])};
  float r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = v[i] - cut_to_bf16(v[i]);
  d1 = uintx2{pack_round(r[0], r[1]), pack_round(r[2], r[3])};
  d2 = uintx2{pack_cut(r[0] - __uint_as_float(d1.x << 16), r[1] - __uint_as_float(d1.x & 0xFFFF0000u)),
              pack_cut(r[2] - __uint_as_float(d1.y << 16), r[3] - __uint_as_float(d1.y & 0xFFFF0000u))};
}

// The four values that a lane supplies to one 16-deep product, as right operands of depth-32 instructions, which take
// two terms at once (four of their eight slots each): (y1 | y2) and (y1 | y3), 16 bytes each.  With a left operand
// x1 + d1 + d2 the six term products are three instructions:
//   (d2 | x1) (y1 | y3),   (d1 | d1) (y1 | y2),   (x1 | x1) (y1 | y2).
// (Pairs that need only three different half operands on the right were measured as well: their overlapping register
// windows cost more copies than the loads they save.)
__device__ __forceinline__ uintx8 operand_terms(const float (&y)[4]) {
  float head[4], r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // rounded to bf16 in a float (values within 2^-9 of the largest finite one are cut: they would become infinite)
    const float h = __uint_as_float(pack_round(y[i], 0.0f) << 16);
    head[i] = __builtin_isinf(h) ? cut_to_bf16(y[i]) : h;
    r[i] = y[i] - head[i];
  }
  const uint32_t h0 = pack_cut(head[0], head[1]), h1 = pack_cut(head[2], head[3]);
  uintx2 m, l;
  split2(r, m, l);
  return uintx8{h0, h1, m.x, m.y, h0, h1, l.x, l.y};
}

// the two operands of one lane in memory: 64 lanes apart, so that a wave's loads are two contiguous KB
__device__ __forceinline__ void store_terms(uintx4* at, uintx8 c) {
  at[0] = __builtin_shufflevector(c, c, 0, 1, 2, 3);
  at[64] = __builtin_shufflevector(c, c, 4, 5, 6, 7);
}
__device__ __forceinline__ uintx8 load_terms(const uintx4* at) {
  const uintx4 a = at[0], b = at[64];
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// acc += instruction i = 0, 1, 2 of x y, with x1 (cut head), d1 and d2 (terms of the rest) of the left operand
__device__ __forceinline__ floatx4 mfma_terms(int i, uintx2 x1, uintx2 d1, uintx2 d2, uintx8 y, floatx4 acc) {
  const uintx4 a = i == 0 ? __builtin_shufflevector(d2, x1, 0, 1, 2, 3)
                          : (i == 1 ? __builtin_shufflevector(d1, d1, 0, 1, 2, 3) : __builtin_shufflevector(x1, x1, 0, 1, 2, 3));
  const uintx4 b = i == 0 ? __builtin_shufflevector(y, y, 4, 5, 6, 7) : __builtin_shufflevector(y, y, 0, 1, 2, 3);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

}  // namespace nnr
