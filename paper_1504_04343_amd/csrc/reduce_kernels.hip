// Lifting phase (Sec. 2.1, fused with the bias add) and the adjoint of the lowering phase:
// the two kernels that READ a lowered matrix once and write the (k or k^2 times smaller)
// tensor.  HBM-bound on the read stream.
#include <type_traits>

#include "cct_internal.h"
#include "index_common.h"

namespace cct {
namespace {

// Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each with an L2 of its own.
// Neighbouring runs of output elements read neighbouring (often line-sharing) stretches of the
// matrix rows, so the kernels below renumber their workgroups: every XCD gets one contiguous
// range of runs and walks it in order, and a cache line that two neighbouring runs share is
// fetched from HBM once instead of once per XCD.
__device__ __forceinline__ int xcd_contiguous_block() {
  const int total = gridDim.x;
  const int per = total >> 3, rem = total & 7;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  return xcd * per + min(xcd, rem) + slot;
}

// acc[e] += the taps of a TI x TJ window in row-major order, the taps of a row loaded together: all of a
// thread's loads of a row are in flight at once (TJ = 0: any width, one tap at a time).
template <int V, int TJ, class Tap>
__device__ __forceinline__ void add_taps(int ti_end, int tj_end, Tap tap, float (&acc)[V]) {
  constexpr int W = TJ > 0 ? TJ : 1;
  for (int ti = 0; ti < ti_end; ++ti)
    for (int tj = 0; tj < (TJ > 0 ? TJ : tj_end); tj += W) {
      float v[W][V];
#pragma unroll
      for (int u = 0; u < W; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) v[u][e] = tap(ti, tj + u, e);
#pragma unroll
      for (int u = 0; u < W; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += v[u][e];
    }
}

// ---------------------------------------------------------------------------------------
// Lifting phase fused with the bias add.  Each thread produces VEC consecutive output
// elements (one 16-byte store); for a fixed tap the lanes of a wave read consecutive
// (stride sw) columns of one R^ row, every R^ entry is read exactly once, and the VEC loads of
// a tap are independent, which keeps enough reads in flight to stream from HBM.
// ---------------------------------------------------------------------------------------
template <bool VSTORE, int V, int TJ>
__global__ __launch_bounds__(TPB) void lift_kernel(const float* __restrict__ rt, long long ld,
                                                   float* __restrict__ y,
                                                   const float* __restrict__ bias, int total, int O,
                                                   WinMap m, FastDiv divWt, FastDiv divPl,
                                                   FastDiv divO) {
  const int t0 = (xcd_contiguous_block() * TPB + threadIdx.x) * V;   // total < 2^31 checked by the launcher
  if (t0 >= total) return;
  const long long kk = (long long)m.Ki * m.Kj;
  const int PcG = m.Ha * m.Wb;
  long long base[V];
  int ra[V], cb[V];
  float acc[V];
  {
    int plane = fdiv(t0, divPl);               // n*O + o
    const int pix = t0 - plane * (m.Ht * m.Wt);
    int r = fdiv(pix, divWt);
    int c = pix - r * m.Wt;
    int n = fdiv(plane, divO);
    int o = plane - n * O;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const bool live = t0 + e < total;
      base[e] = (long long)o * kk * ld + (long long)n * PcG;
      ra[e] = live ? r * m.sh - m.ph : -(1 << 30);
      cb[e] = c * m.sw - m.pw;
      acc[e] = (bias && live) ? bias[o] : 0.0f;
      if (++c == m.Wt) {
        c = 0;
        if (++r == m.Ht) {
          r = 0;
          if (++o == O) {
            o = 0;
            ++n;
          }
        }
      }
    }
  }
  auto tap = [&](int i, int j, int e) {
    const int a = ra[e] + i, b = cb[e] + j;
    const bool ok = (unsigned)a < (unsigned)m.Ha && (unsigned)b < (unsigned)m.Wb;
    const float t = rt[ok ? base[e] + (long long)(i * m.Kj + j) * ld + a * m.Wb + b : 0];
    return ok ? t : 0.0f;
  };
  add_taps<V, TJ>(m.Ki, m.Kj, tap, acc);
  if (VSTORE && V == 4 && t0 + V <= total) {
    *reinterpret_cast<float4*>(y + t0) = make_float4(acc[0], acc[1 % V], acc[2 % V], acc[3 % V]);
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (t0 + e < total) y[t0 + e] = acc[e];
  }
}

// Adjoint of the lowering phase as a gather (no atomics): every dx pixel sums the entries of
// the lowered gradient that were copied from it.  Only taps i = (h+ph) mod sh, +sh, +2sh, ...
// (and likewise j) can have come from pixel (h, w), so the tap loops step by the stride.
template <bool VSTORE, int V, int TJ>
__global__ __launch_bounds__(TPB) void inv_lower_kernel(const float* __restrict__ ddt, long long ld,
                                                        float* __restrict__ dx, int total, int C,
                                                        WinMap m, FastDiv divWt, FastDiv divPl,
                                                        FastDiv divC, FastDiv divSh, FastDiv divSw) {
  const int t0 = (xcd_contiguous_block() * TPB + threadIdx.x) * V;
  if (t0 >= total) return;
  const long long kk = (long long)m.Ki * m.Kj;
  const int PcG = m.Ha * m.Wb;
  long long base[V];
  int i0[V], a0[V], j0[V], b0[V];
  float acc[V];
  {
    int plane = fdiv(t0, divPl);               // n*C + ch
    const int pix = t0 - plane * (m.Ht * m.Wt);
    int h = fdiv(pix, divWt);
    int w = pix - h * m.Wt;
    int n = fdiv(plane, divC);
    int ch = plane - n * C;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const bool live = t0 + e < total;
      base[e] = (long long)ch * kk * ld + (long long)n * PcG;
      // first admissible taps and the grid coordinates they map to
      a0[e] = fdiv(h + m.ph, divSh);
      i0[e] = live ? h + m.ph - a0[e] * m.sh : (1 << 30);
      b0[e] = fdiv(w + m.pw, divSw);
      j0[e] = w + m.pw - b0[e] * m.sw;
      acc[e] = 0.0f;
      if (++w == m.Wt) {
        w = 0;
        if (++h == m.Ht) {
          h = 0;
          if (++ch == C) {
            ch = 0;
            ++n;
          }
        }
      }
    }
  }
  const int nti = (m.Ki + m.sh - 1) / m.sh, ntj = (m.Kj + m.sw - 1) / m.sw;
  auto tap = [&](int ti, int tj, int e) {
    const int i = i0[e] + ti * m.sh, a = a0[e] - ti;
    const int j = j0[e] + tj * m.sw, b = b0[e] - tj;
    const bool ok = i < m.Ki && j < m.Kj && (unsigned)a < (unsigned)m.Ha && (unsigned)b < (unsigned)m.Wb;
    const float t = ddt[ok ? base[e] + (long long)(i * m.Kj + j) * ld + a * m.Wb + b : 0];
    return ok ? t : 0.0f;
  };
  add_taps<V, TJ>(nti, ntj, tap, acc);
  if (VSTORE && V == 4 && t0 + V <= total) {
    *reinterpret_cast<float4*>(dx + t0) = make_float4(acc[0], acc[1 % V], acc[2 % V], acc[3 % V]);
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (t0 + e < total) dx[t0 + e] = acc[e];
  }
}

// Elements per thread and unrolled taps of a launch.  Small tensors take one element per thread: four would
// leave most of the chip idle (one image of 13 x 13, 384 channels, 3 x 3 taps: 64 workgroups and 9.5 us).
constexpr long long kSmallTensor = 1 << 19;
template <class F>
void choose(long long total, bool aligned, int tj, F f) {
  auto taps = [&](auto vs, auto v) {
    if (tj == 2) return f(vs, v, std::integral_constant<int, 2>());
    if (tj == 3) return f(vs, v, std::integral_constant<int, 3>());
    if (tj == 5) return f(vs, v, std::integral_constant<int, 5>());
    return f(vs, v, std::integral_constant<int, 0>());
  };
  if (total < kSmallTensor) return taps(std::false_type(), std::integral_constant<int, 1>());
  if (aligned) return taps(std::true_type(), std::integral_constant<int, VEC>());
  return taps(std::false_type(), std::integral_constant<int, VEC>());
}

}  // namespace

int launch_lift(const float* rt, long long ld, float* y, const float* bias, int nimg, int O,
                const WinMap& m, hipStream_t st) {
  const long long total = (long long)nimg * O * m.Ht * m.Wt;
  const long long blocks = (total + TPB * VEC - 1) / (TPB * VEC);
  if (!grid_ok(blocks) || total >= 2147483647LL - TPB * VEC) return CCT_EUNSUPPORTED;
  ProfScope ps("lift_kernel", 0.0,
               4.0 * total + 4.0 * O * m.Ki * m.Kj * (double)nimg * m.Ha * m.Wb, st);
  choose(total, reinterpret_cast<uintptr_t>(y) % 16 == 0, m.Kj, [&](auto vs, auto v, auto tj) {
    constexpr auto kern = lift_kernel<decltype(vs)::value, decltype(v)::value, decltype(tj)::value>;
    const long long blocks = (total + TPB * v.value - 1) / (TPB * v.value);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(TPB), 0, st, rt, ld, y, bias, (int)total, O, m,
                       make_fastdiv(m.Wt), make_fastdiv(m.Ht * m.Wt), make_fastdiv(O));
  });
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int launch_inv_lower(const float* ddt, long long ld, float* dx, int nimg, int C, const WinMap& m,
                     hipStream_t st) {
  const long long total = (long long)nimg * C * m.Ht * m.Wt;
  const long long blocks = (total + TPB * VEC - 1) / (TPB * VEC);
  if (!grid_ok(blocks) || total >= 2147483647LL - TPB * VEC) return CCT_EUNSUPPORTED;
  ProfScope ps("inv_lower_kernel", 0.0,
               4.0 * total + 4.0 * C * m.Ki * m.Kj * (double)nimg * m.Ha * m.Wb, st);
  choose(total, reinterpret_cast<uintptr_t>(dx) % 16 == 0, (m.Kj + m.sw - 1) / m.sw, [&](auto vs, auto v, auto tj) {
    constexpr auto kern = inv_lower_kernel<decltype(vs)::value, decltype(v)::value, decltype(tj)::value>;
    const long long blocks = (total + TPB * v.value - 1) / (TPB * v.value);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(TPB), 0, st, ddt, ld, dx, (int)total, C, m,
                       make_fastdiv(m.Wt), make_fastdiv(m.Ht * m.Wt), make_fastdiv(C), make_fastdiv(m.sh),
                       make_fastdiv(m.sw));
  });
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace cct
