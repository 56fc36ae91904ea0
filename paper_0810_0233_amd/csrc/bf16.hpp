// bf16.hpp -- FP32 numbers as sums of three bf16 ones, and the bf16 matrix
// instruction.
//
// x = x0 + x1 + x2 exactly, each the remainder rounded to bf16 (8 bits apiece,
// to nearest, so either sign): the remainders are exact FP32 numbers, and the
// last one has at most 8 bits left (the splitting of Henry, Tang and Heinecke, "Leveraging
// the bfloat16 artificial intelligence datatype for higher-precision
// computations", 2019).  Of the nine products of two such sums the six down to
// 2^-16 of the largest are formed; the other three are below 2^-25 of it and of
// either sign, under FP32's own rounding.  The range is FP32's, but below 2^-110
// the last piece is subnormal and loses bits: moments from 1e-35 up give the FP32
// form's error (order 6, 20,000 in a fluid and 73,728 of a film: 2.2e-7 and
// 1.3e-7), 1e-36 3.5e-7, 1e-37 3e-6.
#pragma once
#include "mfma.hpp"

namespace ccfmm {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// two FP32 numbers rounded to bf16 (to nearest even)
__device__ __forceinline__ bf16x2 to_bf16(float a, float b) {
  return __builtin_convertvector(f32x2{a, b}, bf16x2);
}
// -1 in the low or the high half, held in a register the compiler does not
// look into (its inline constant for such operands is a different number)
struct MinusOne {
  uint32_t lo = 0x0000bf80u, hi = 0xbf800000u;
  __device__ __forceinline__ MinusOne() { asm volatile("" : "+s"(lo), "+s"(hi)); }
};
// a and b minus the halves of h, exactly (h holds their roundings)
__device__ __forceinline__ void remainders(bf16x2 h, const MinusOne& one, float& a, float& b) {
  a = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, one.lo), a, false);
  b = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, one.hi), b, false);
}
__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace ccfmm
