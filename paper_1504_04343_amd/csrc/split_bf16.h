// fp32 operands on the bf16 matrix cores, without giving up fp32 precision.
//
// An fp32 value has 24 significant bits; x = h + m + l with h = bf16(x), m = bf16(x - h),
// l = bf16(x - h - m) is exact (each term takes 8 bits of what is left, rounding to nearest keeps
// the remainders short).  A product of two such sums needs six of the nine partial products,
//   h*h, h*m, m*h, h*l, l*h, m*m,
// the other three are below 2^-25 of the product.  bf16 products are exact in the matrix core's
// fp32 accumulation.  The partial products are kept in two accumulators: h*h alone in one, the five
// corrections (2^-8 and smaller) in the other, added once at the end.  The long chain then takes
// one rounding per 16 reduction indices instead of one per 2, so that the sums come out closer to
// 64 bits than those of v_mfma_f32_32x32x2_f32 (relative error in the 2-norm, 2304 products: 2.3e-7
// against 6.1e-7 on ReLU data, 43264 products: 1.25e-6 against 2.6e-6; with all six in one
// accumulator 7.1e-7 and 3.3e-6).
//
// Why: six v_mfma_f32_32x32x16_bf16 take 192 cycles where eight v_mfma_f32_32x32x2_f32 take 512.
//
// Not finite: inf - inf makes m and l NaN, and 0 * inf appears between the terms, so a result that
// an infinity (or a value above bf16's largest, 3.39e38) touches comes out NaN.  The kernels
// recompute every NaN result in plain fp32 before they end (a NaN that is real is met again).
#pragma once
#include "cct_internal.h"

namespace cct {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned cvt_pk_bf16(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }

// two values -> their h, m and l terms, each a pair of bf16 in one register
__device__ __forceinline__ void split_pair(float a, float b, unsigned* h, unsigned* m, unsigned* l) {
  *h = cvt_pk_bf16(a, b);
  const float ra = a - bf16_lo(*h), rb = b - bf16_hi(*h);
  *m = cvt_pk_bf16(ra, rb);
  *l = cvt_pk_bf16(ra - bf16_lo(*m), rb - bf16_hi(*m));
}

// one value -> h, m, l for a pack that the NaN recomputation reads back: h + m + l is the value
// itself also where it is not finite or rounds beyond bf16's range
__device__ __forceinline__ void split_value(float v, unsigned short* h, unsigned short* m,
                                            unsigned short* l) {
  unsigned hh = cvt_pk_bf16(v, 0.f) & 0xffffu;
  if ((hh & 0x7f80u) == 0x7f80u) {
    if ((__float_as_uint(v) & 0x7f800000u) == 0x7f800000u) {
      *h = (unsigned short)hh;
      *m = *l = 0;
      return;
    }
    hh = __float_as_uint(v) >> 16;  // finite: cut instead of rounding up to infinity
  }
  const float r = v - __uint_as_float(hh << 16);
  const unsigned mm = cvt_pk_bf16(r, 0.f) & 0xffffu;
  *h = (unsigned short)hh;
  *m = (unsigned short)mm;
  *l = (unsigned short)(cvt_pk_bf16(r - __uint_as_float(mm << 16), 0.f) & 0xffffu);
}

}  // namespace
}  // namespace cct
