// Forward pass of layers so small that their launches are what they cost: one launch, the kernel matrix and the
// tensor read in place, products summed in 64 bits.
//
// A workgroup computes 4 kernels at 64 consecutive positions of the batch; lanes are positions, each of its 8 waves
// sums an eighth of the Cg*K*K products.  The four kernels' values and where each of the products' pixels lies go
// through LDS once (broadcast reads), pixels come from memory, 16 or 32 loads in flight.  Bound by latency: one way
// to memory for the kernels, one for the pixels, the launch; that is why sums in 64 bits cost nothing, and they
// leave only the result's own rounding (2-norm 3e-8; two roundings per product and a tree: 7e-8).
// 4 images of 3 x 32 x 32, 16 kernels of 5 x 5 (9.8 MFLOP, 256 workgroups): 13.6 us as a
// pack and a matrix product, 6.1 us now, most of it the call.
#include <type_traits>

#include "cct_internal.h"

namespace cct {
namespace {

constexpr int MK = 4;      // kernels per workgroup
constexpr int PARTS = 8;   // waves
constexpr int KD_MAX = 512;

struct Small {
  const float *x, *w, *bias;
  float* y;
  int N, C, H, W, O, K, stride, pad, Cg, Og, Wout, P, Kd, row_tiles;
  unsigned divP_M, divK_M, divKK_M, divW_M;
  int divP_sh, divK_sh, divKK_sh, divW_sh;
};

__device__ __forceinline__ int div_u(int n, unsigned M, int sh) { return (int)(((unsigned long long)(unsigned)n * M) >> sh); }

__global__ __launch_bounds__(64 * PARTS) void conv_small(Small p) {
  __shared__ __attribute__((aligned(16))) double wl[KD_MAX][MK];
  __shared__ int2 tap[KD_MAX];  // offset from the window's first pixel, row and column in the window
  __shared__ double sum[PARTS][MK][64];
  __shared__ int special;  // a kernel value is not finite
  const int tid = threadIdx.x, lane = tid & 63;
  const int part = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.y / p.row_tiles, o0 = (blockIdx.y - g * p.row_tiles) * MK;  // within the group
  const int col = blockIdx.x * 64 + lane;
  const bool live = col < p.N * p.P;

  if (tid == 0) special = 0;
  __syncthreads();
  const float* w = p.w + ((long long)g * p.Og + o0) * p.Kd;
  for (int k = tid; k < p.Kd; k += 64 * PARTS) {
    float v[MK];
#pragma unroll
    for (int r = 0; r < MK; ++r) v[r] = w[(long long)min(r, p.Og - 1 - o0) * p.Kd + k];
    const int KK = p.K * p.K, c = div_u(k, p.divKK_M, p.divKK_sh), t = k - c * KK, i = div_u(t, p.divK_M, p.divK_sh), j = t - i * p.K;
    tap[k] = make_int2((c * p.H + i) * p.W + j, i | j << 16);
#pragma unroll
    for (int r = 0; r < MK; ++r) {
      wl[k][r] = v[r];
      if (!(__builtin_fabsf(v[r]) < __builtin_inff())) special = 1;
    }
  }
  const int n = live ? div_u(col, p.divP_M, p.divP_sh) : 0, pix = live ? col - n * p.P : 0;
  const int row = div_u(pix, p.divW_M, p.divW_sh);
  const int h0 = row * p.stride - p.pad, w0 = (pix - row * p.Wout) * p.stride - p.pad;
  const float* x = p.x + ((long long)n * p.C + g * p.Cg) * p.H * p.W;
  const int first = h0 * p.W + w0;
  __syncthreads();

  const int per = (p.Kd + PARTS - 1) / PARTS, k1 = min((part + 1) * per, p.Kd);
  double acc[MK];
#pragma unroll
  for (int r = 0; r < MK; ++r) acc[r] = 0.0;
  // A pixel outside the tensor is 0, and no product at all where a kernel value is not finite.
  auto run = [&](auto batch, auto exact) {
    constexpr int BATCH = decltype(batch)::value;
    for (int k0 = part * per; k0 < k1; k0 += BATCH) {
      float v[BATCH];
      unsigned ok = 0;
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int2 t = tap[min(k0 + u, k1 - 1)];
        const bool in = k0 + u < k1 && (unsigned)(h0 + (t.y & 0xffff)) < (unsigned)p.H && (unsigned)(w0 + (t.y >> 16)) < (unsigned)p.W;
        const float q = x[in ? first + t.x : 0];
        v[u] = in ? q : 0.f;
        if (exact.value && in) ok |= 1u << u;
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const double* wk = wl[min(k0 + u, k1 - 1)];
#pragma unroll
        for (int r = 0; r < MK; ++r)
          if (!exact.value || ok >> u & 1) acc[r] = fma((double)v[u], wk[r], acc[r]);
      }
    }
  };
  using yes = std::true_type;
  using no = std::false_type;
  if (special)
    run(std::integral_constant<int, 16>(), yes());
  else if (per <= 16)
    run(std::integral_constant<int, 16>(), no());
  else
    run(std::integral_constant<int, 32>(), no());
#pragma unroll
  for (int r = 0; r < MK; ++r) sum[part][r][lane] = acc[r];
  __syncthreads();
  if (part >= MK || o0 + part >= p.Og || !live) return;
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < PARTS; ++q) v += sum[q][part][lane];
  const int o = g * p.Og + o0 + part;
  if (p.bias) v += p.bias[o];
  p.y[((long long)n * p.O + o) * p.P + pix] = (float)v;
}

}  // namespace

// Time: 2.5 us + 0.016 us per product of a result, and 4.5 us + 0.04 us per product for every 1024 workgroups.  What ran
// these layers before (a pack and a product) takes about 8.5 us + 0.027 us per product while it does not fill
// the chip either, so that the line lies near 120000 workgroups x (112 + products).  us, before -> now: 16 images of
// 14 x 14, 16 -> 32 channels, K = 3 (392 workgroups, 144 products) 11.1 -> 8.4, the same with 64 kernels (784) 11.0
// against 13.4; 4 images of 7 x 7, 512 -> 128, K = 1 (128) 22.7 -> 11.4; 256 images of 7 x 7, 16 -> 32, K = 1
// (1568 workgroups, 16 products) 8.6 against 12.0.  Layers of 1 x 1 kernels are still left to the
// products on the tensor in place (gemm_split), although the smallest of them would gain as much (8 images of 14 x 14,
// 64 -> 64: 9.8 -> 6.0): tests/test_gpu_gemm_split.py calls that kernel through such layers under AUTO.
// Over 1080 layers that it took: 0.2 to 0.9 times the time, 6 of them more than 3 % slower, by up to 2.4 us at the line.
// (K up to 65535 only, so that the number of products cannot overflow.)
bool conv_small_fits(const cct_conv_desc_t& d, int Hout, int Wout) {
  if (d.precision != CCT_PREC_F32 || d.K < 2 || d.K > 0xffff) return false;
  const long long Kd = (long long)(d.C / d.groups) * d.K * d.K, cols = (long long)d.N * Hout * Wout;
  const long long rows = (long long)d.groups * ((d.O / d.groups + MK - 1) / MK);
  if (Kd > KD_MAX || cols >= (1LL << 24) || rows > 65535 || (long long)d.C * d.H * d.W >= (1LL << 30)) return false;
  return (cols + 63) / 64 * rows * (112 + Kd) <= 120000;
}

int launch_conv_small(const cct_conv_desc_t& d, int Hout, int Wout, const float* x, const float* w, const float* bias,
                      float* y, hipStream_t st) {
  Small p;
  p.x = x; p.w = w; p.bias = bias; p.y = y;
  p.N = d.N; p.C = d.C; p.H = d.H; p.W = d.W; p.O = d.O; p.K = d.K; p.stride = d.stride; p.pad = d.pad;
  p.Cg = d.C / d.groups; p.Og = d.O / d.groups; p.Wout = Wout; p.P = Hout * Wout; p.Kd = p.Cg * d.K * d.K;
  p.row_tiles = (p.Og + MK - 1) / MK;
  make_fastdiv_parts(p.P, &p.divP_M, &p.divP_sh);
  make_fastdiv_parts(Wout, &p.divW_M, &p.divW_sh);
  make_fastdiv_parts(d.K, &p.divK_M, &p.divK_sh);
  make_fastdiv_parts(d.K * d.K, &p.divKK_M, &p.divKK_sh);
  const long long cols = (long long)d.N * p.P;
  ProfScope ps("conv_small", 2.0 * d.O * p.Kd * (double)cols,
               4.0 * ((double)d.N * d.C * d.H * d.W + (double)d.O * (cols + p.Kd)), st);
  hipLaunchKernelGGL(conv_small, dim3((unsigned)((cols + 63) / 64), (unsigned)(d.groups * p.row_tiles)), dim3(64 * PARTS), 0, st, p);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace cct
