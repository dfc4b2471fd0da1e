// An fp32 value as three bf16 values, for products on the bf16 matrix cores
// (the splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations",
// arXiv:1904.06376).
//
// 2^23 x = h + m + l to its last bit, h = bf16(2^23 x), m = bf16(2^23 x - h), l =
// bf16(2^23 x - h - m), each rounded to nearest, so |m| <= 2^-9 |h| and |l| <=
// 2^-18 |h|.  A product a b is formed as the six products hh, hm, mh, mm, hl,
// lh, each exact (8 x 8 significand bits), accumulated in fp32, and the sum is
// multiplied by 2^-46; what is left out (ml, lm, ll) is below 2^-25 |a b|.
//
// Why 2^23: the matrix cores read subnormal bf16 values as zeros.  Every fp32
// value is a multiple of 2^-149, so are its unscaled parts, and those below
// 2^-126 would be lost: 1e-36 times 1e13 came out 8e-4 off, 1e-39 times 1e30 as
// zero.  Scaled, a part that is not zero is at least 2^-126.  It costs a
// multiplication per value split (13 vector instructions for two, not 11).
#pragma once

#include <hip/hip_runtime.h>

namespace nf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const floatx2 f = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

// The three bf16 parts of two values times PARTS_SCALE, packed (a in the low half).
constexpr float PARTS_SCALE = 8388608.f;                       // 2^23
constexpr float PARTS_UNSCALE = 1.f / PARTS_SCALE / PARTS_SCALE;
__device__ __forceinline__ void split3(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  a *= PARTS_SCALE;
  b *= PARTS_SCALE;
  h = pack_bf16(a, b);
  const float a1 = a - __builtin_bit_cast(float, h << 16);
  const float b1 = b - __builtin_bit_cast(float, h & 0xffff0000u);
  m = pack_bf16(a1, b1);
  l = pack_bf16(a1 - __builtin_bit_cast(float, m << 16),
                b1 - __builtin_bit_cast(float, m & 0xffff0000u));
}

// The six products by part (0 h, 1 m, 2 l) of A and of B, the small ones first.
constexpr int PART_A[6] = {2, 0, 1, 1, 0, 0}, PART_B[6] = {0, 2, 1, 0, 1, 0};

// Whether a sum of six products cannot be trusted.  An operand that is not
// finite, or that rounds to infinity in bf16 once scaled (from 2^105 on),
// leaves a NaN or an infinity in every sum it enters, as does a sum past 2^82.
// Such sums are formed again on the fp32 matrix cores.
__device__ __forceinline__ bool parts_doubtful(float sum) {
  return !(fabsf(sum) < __builtin_inff());
}

}  // namespace nf
