// fp32 operands on the bf16 matrix cores, without giving up fp32 precision.
//
// An fp32 value has 24 significant bits; x = h + m + l with h = bf16(x), m = bf16(x - h),
// l = bf16(x - h - m) is exact (each term takes 8 bits of what is left, rounding to nearest keeps
// the remainders short).  A product of two such sums needs six of the nine partial products,
//   h*h, h*m, m*h, h*l, l*h, m*m,
// the other three are below 2^-25 of the product.  bf16 products are exact in the matrix core's
// fp32 accumulation.  The partial products are kept in two accumulators: h*h alone in one, the five
// corrections (2^-8 and smaller) in the other, added once at the end.  The long chain then takes
// one rounding per 16 reduction indices instead of one per 2 (v_mfma_f32_16x16x32_bf16 takes 32, with the same
// errors), so that the sums come out closer to
// 64 bits than those of v_mfma_f32_32x32x2_f32 (relative error in the 2-norm, 2304 products: 2.3e-7
// against 6.1e-7 on ReLU data, 43264 products: 1.25e-6 against 2.6e-6; with all six in one
// accumulator 7.1e-7 and 3.3e-6).
//
// Why: six v_mfma_f32_32x32x16_bf16 (as twelve 16x16x32) take 192 cycles where eight v_mfma_f32_32x32x2_f32 take 512.
//
// Range: bf16 has fp32's exponents, so the last bits of a value below 2^-110 would be lost in m and l.  Every
// value is therefore multiplied by 2^24 before it is split, which keeps the terms of the smallest fp32
// number normal, and every result by 2^-48 at the end.  (Without: values of about 2^-118 times 2^88
// came out with a relative error of 1.5e-5.)  It costs one multiplication per split value, at most 1 % of a pass.
//
// Not finite: inf - inf makes m and l NaN, and 0 * inf appears between the terms, so a result that an infinity
// touches comes out NaN; a value of 2^104 or a result of 2^80 overflows.  The kernels recompute the blocks with
// results that are not finite in plain fp32 before they end (a value that is real is met again).
#pragma once
#include "cct_internal.h"
#include "gemm_common.h"

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

// A quarter of splitting a pair of 8 values, 3 or 4 instructions, for kernels that write it between their MFMAs: step
// n = 4 e + 0 .. 3 of pair e.  ra and rb hold what is left of the pair in between.
__device__ __forceinline__ void split_quarter(float (&v)[8], u32x4 (&q)[3], int n, float& ra, float& rb) {
  const int e = n >> 2;
  // keeps a step where it is written: it would be moved in front of all MFMAs
  if (n & 3)
    asm volatile("" : "+v"(ra), "+v"(rb));
  else
    asm volatile("" : "+v"(v[2 * e]), "+v"(v[2 * e + 1]));
  switch (n & 3) {
    case 0:
      ra = v[2 * e] * kSplitScale;
      rb = v[2 * e + 1] * kSplitScale;
      q[0][e] = cvt_pk_bf16(ra, rb);
      break;
    case 1:
      ra -= bf16_lo(q[0][e]);
      rb -= bf16_hi(q[0][e]);
      break;
    case 2:
      q[1][e] = cvt_pk_bf16(ra, rb);
      ra -= bf16_lo(q[1][e]);
      break;
    default:
      rb -= bf16_hi(q[1][e]);
      q[2][e] = cvt_pk_bf16(ra, rb);
  }
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

// The kernel's first argument, read again: what only the code behind it needs is not kept in scalar registers
// through the kernel.
template <class T>
__device__ __forceinline__ const T& first_argument() {
  auto at = __builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(at));
  return *(const T*)at;
}

// A 32 x 32 block of results in plain fp32: every step is two products, a(s) and b(s) those of a lane's row and
// column (lane & 31) and half (lane >> 5); 8 steps' loads are in flight.  open(acc): which of its results a lane
// still waits for (a NaN stays one).
template <class A, class B, class Open>
__device__ __forceinline__ floatx16 fp32_block(int steps, A a, B b, Open open) {
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll 1
  for (int s = 0; s < steps; s += 8) {
    float x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      x[u] = s + u < steps ? a(s + u) : 0.f;
      y[u] = s + u < steps ? b(s + u) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u], y[u], acc, 0, 0, 0);
    if (!__any(open(acc))) break;
  }
  return acc;
}
// the results among `todo` that are no NaN
__device__ __forceinline__ unsigned numbers(const floatx16& acc, unsigned todo) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (acc[r] != acc[r]) todo &= ~(1u << r);
  return todo;
}

// One result per lane with `todo` in plain fp32: what(lane) describes a lane's result (all lanes call it),
// term(that, k, &x, &y) gives its k-th product, false if there is none.  A NaN among the first 64 decides; the
// other results take the whole wave one by one.  Returns the lane's own sum.
template <class What, class Term>
__device__ __forceinline__ float fp32_sum(bool todo, int terms, What what, Term term) {
  const int lane = threadIdx.x & 63;
  float mine = 0.f;
  const auto own = what(lane);
  for (int k = 0; k < min(terms, 64) && todo; ++k) {
    float x, y;
    if (term(own, k, &x, &y)) mine = fmaf(x, y, mine);
    todo = mine == mine;
  }
  unsigned long long left = __ballot(todo);
  while (left) {
    const int who = __ffsll(left) - 1;
    left &= left - 1;
    const auto result = what(who);
    float sum = 0.f;
#pragma unroll 1
    for (int k0 = lane; k0 - lane < terms && !__any(sum != sum); k0 += 256) {
      float x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + u * 64 >= terms || !term(result, k0 + u * 64, &x[u], &y[u])) x[u] = y[u] = 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) sum = fmaf(x[u], y[u], sum);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == who) mine = sum;
  }
  return mine;
}

}  // namespace
}  // namespace cct
