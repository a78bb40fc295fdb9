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
// Range: bf16 has fp32's exponents, so the last bits of a value below 2^-110 would be lost in m and l.  Every
// value is therefore multiplied by 2^24 before it is split, which keeps the terms of the smallest fp32
// number normal, and every result by 2^-48 at the end.  (Without: values of about 2^-118 times 2^88
// came out with a relative error of 1.5e-5.)  It costs one multiplication per split value, at most 1 % of a pass.
//
// Not finite: inf - inf makes m and l NaN, and 0 * inf appears between the terms, so a result that an infinity
// touches comes out NaN; a value of 2^104 or a result of 2^80 overflows.  The kernels recompute every result
// that is not finite in plain fp32 before they end (redo_not_finite; one that is real is met again).
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

constexpr float kSplitScale = 0x1p24f;     // of a split value
constexpr float kSplitUnscale = 0x1p-48f;  // of a result

// two values -> their h, m and l terms, each a pair of bf16 in one register
__device__ __forceinline__ void split_pair(float a, float b, unsigned* h, unsigned* m, unsigned* l) {
  a *= kSplitScale;
  b *= kSplitScale;
  *h = cvt_pk_bf16(a, b);
  const float ra = a - bf16_lo(*h), rb = b - bf16_hi(*h);
  *m = cvt_pk_bf16(ra, rb);
  *l = cvt_pk_bf16(ra - bf16_lo(*m), rb - bf16_hi(*m));
}

// One value -> h, m, l for a pack that the recomputation reads back.  A value that does not split (not finite,
// or 2^104 and more) leaves NaN in h, which every result of its row meets, and its bits in m and l.
__device__ __forceinline__ void split_value(float v, unsigned short* h, unsigned short* m,
                                            unsigned short* l) {
  const float s = v * kSplitScale;
  const unsigned hh = cvt_pk_bf16(s, 0.f) & 0xffffu;
  if ((hh & 0x7f80u) == 0x7f80u) {
    *h = 0x7fc0u;
    *m = (unsigned short)(__float_as_uint(v) >> 16);
    *l = (unsigned short)(__float_as_uint(v) & 0xffffu);
    return;
  }
  const float r = s - __uint_as_float(hh << 16);
  const unsigned mm = cvt_pk_bf16(r, 0.f) & 0xffffu;
  *h = (unsigned short)hh;
  *m = (unsigned short)mm;
  *l = (unsigned short)(cvt_pk_bf16(r - __uint_as_float(mm << 16), 0.f) & 0xffffu);
}
__device__ __forceinline__ float join_value(unsigned short h, unsigned short m, unsigned short l) {
  if ((h & 0x7f80u) == 0x7f80u) return __uint_as_float(((unsigned)m << 16) | l);
  return ((__uint_as_float((unsigned)h << 16) + __uint_as_float((unsigned)m << 16)) + __uint_as_float((unsigned)l << 16)) *
         (1.0f / kSplitScale);
}

__device__ __forceinline__ bool finite(float v) { return __builtin_fabsf(v) < __builtin_inff(); }

}  // namespace
}  // namespace cct
