// The layers between CaffeNet's convolutional layers, as library entry points: the rectified
// linear unit, max pooling and local response normalisation, forward and backward (Sec. 1: the other layers are built with the
// same techniques as the convolution and match Caffe layer by layer; Sec. 2.2: processing the
// whole batch at once applies to every layer).  All are pure streaming kernels: every element of
// the input is read once and every element of the output written once, the whole batch in one
// launch.  Semantics are Caffe's:
//   ReLU      y = max(x, 0);  dx = dy where x > 0, else 0.
//   LRN       across channels: scale = k + (alpha/size) * sum of x^2 over the `size` channels
//             centred on the channel (zero padded), y = x * scale^(-beta); backward is the exact
//             derivative.  A thread owns a segment of the channels of one pixel in registers:
//             x (and dy) are read once, apart from the few channels around a segment's ends,
//             and y (dx) is written once.
//   dropout   y = x * scale where the caller's mask is set, else 0 (both directions).
//   softmax loss  softmax over the classes of each image, mean negative log-likelihood of the
//             labels; backward (prob - onehot) / N.  One workgroup per image, fixed-order sums.
//   max pool  K x K windows with stride s and padding p, clipped to the image, output size
//             ceil((H + 2p - K)/s) + 1 (minus one if the last window would start beyond the
//             image); the FIRST maximum in row-major order of the window is the one that
//             receives the gradient.  The backward pass is a gather (no atomics): a pixel sums
//             dy over the at most ceil(K/s)^2 windows that contain it and chose it.
#include "cct_internal.h"
#include "index_common.h"

namespace cct {
namespace {


__global__ __launch_bounds__(TPB) void relu_forward_kernel(const float* __restrict__ x,
                                                           float* __restrict__ y, long long n4,
                                                           long long n) {
  const long long stride = (long long)gridDim.x * TPB;
  for (long long i = (long long)blockIdx.x * TPB + threadIdx.x; i < n4; i += stride) {
    float4 v = reinterpret_cast<const float4*>(x)[i];
    v.x = v.x > 0.f ? v.x : 0.f;
    v.y = v.y > 0.f ? v.y : 0.f;
    v.z = v.z > 0.f ? v.z : 0.f;
    v.w = v.w > 0.f ? v.w : 0.f;
    reinterpret_cast<float4*>(y)[i] = v;
  }
  // tail (and everything, when the pointers are not 16-byte aligned: then n4 == 0)
  for (long long i = n4 * 4 + (long long)blockIdx.x * TPB + threadIdx.x; i < n; i += stride) {
    const float v = x[i];
    y[i] = v > 0.f ? v : 0.f;
  }
}

__global__ __launch_bounds__(TPB) void relu_backward_kernel(const float* __restrict__ x,
                                                            const float* __restrict__ dy,
                                                            float* __restrict__ dx, long long n4,
                                                            long long n) {
  const long long stride = (long long)gridDim.x * TPB;
  for (long long i = (long long)blockIdx.x * TPB + threadIdx.x; i < n4; i += stride) {
    const float4 v = reinterpret_cast<const float4*>(x)[i];
    float4 g = reinterpret_cast<const float4*>(dy)[i];
    g.x = v.x > 0.f ? g.x : 0.f;
    g.y = v.y > 0.f ? g.y : 0.f;
    g.z = v.z > 0.f ? g.z : 0.f;
    g.w = v.w > 0.f ? g.w : 0.f;
    reinterpret_cast<float4*>(dx)[i] = g;
  }
  for (long long i = n4 * 4 + (long long)blockIdx.x * TPB + threadIdx.x; i < n; i += stride)
    dx[i] = x[i] > 0.f ? dy[i] : 0.f;
}

struct PoolGeom {
  int H, W, K, s, p, Ho, Wo;
};

// one thread per output element, consecutive threads along the output row
__global__ __launch_bounds__(TPB) void maxpool_forward_kernel(const float* __restrict__ x,
                                                              float* __restrict__ y,
                                                              int* __restrict__ argmax,
                                                              long long total, PoolGeom g) {
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= total) return;
  const int q = (int)(t % g.Wo);
  const long long u = t / g.Wo;
  const int r = (int)(u % g.Ho);
  const long long plane = u / g.Ho;
  const float* __restrict__ xp = x + plane * g.H * g.W;
  const int h0 = max(r * g.s - g.p, 0), w0 = max(q * g.s - g.p, 0);
  const int h1 = min(r * g.s - g.p + g.K, g.H), w1 = min(q * g.s - g.p + g.K, g.W);
  int best = -1;
  float bv = 0.f;
  for (int h = h0; h < h1; ++h)
    for (int w = w0; w < w1; ++w) {
      const float v = xp[h * g.W + w];
      if (best < 0 || v > bv) {
        bv = v;
        best = h * g.W + w;
      }
    }
  y[t] = bv;
  if (argmax) argmax[t] = best;
}

// one thread per input pixel: windows (r, q) with r*s - p <= h < r*s - p + K (same for w)
__global__ __launch_bounds__(TPB) void maxpool_backward_kernel(const float* __restrict__ dy,
                                                               const int* __restrict__ argmax,
                                                               float* __restrict__ dx,
                                                               long long total, PoolGeom g) {
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= total) return;
  const int w = (int)(t % g.W);
  const long long u = t / g.W;
  const int h = (int)(u % g.H);
  const long long plane = u / g.H;
  const int me = h * g.W + w;
  const int rlo = h + g.p - g.K + 1 <= 0 ? 0 : (h + g.p - g.K + g.s) / g.s;   // ceil((h+p-K+1)/s)
  const int qlo = w + g.p - g.K + 1 <= 0 ? 0 : (w + g.p - g.K + g.s) / g.s;
  const int rhi = min((h + g.p) / g.s, g.Ho - 1), qhi = min((w + g.p) / g.s, g.Wo - 1);
  const long long base = plane * g.Ho * g.Wo;
  float acc = 0.f;
  for (int r = rlo; r <= rhi; ++r)
    for (int q = qlo; q <= qhi; ++q) {
      const long long o = base + (long long)r * g.Wo + q;
      if (argmax[o] == me) acc += dy[o];
    }
  dx[t] = acc;
}

// A workgroup takes kWalk consecutive elements of the flat (plane, row, column) range of a kernel, kPer per
// thread: the plane of its first one by a 64-bit division of uniform values, everything per thread in 32
// bits with multiplicative division.  A tensor is then a uniform pointer and a 32-bit offset.  `load` runs
// for all elements of a thread before `use` does, so that their loads are in flight together: the bytes
// in flight on a CU are what bounds these kernels.  load(u, plane0, dp, r, c), use(u, ...) with the
// plane relative to the workgroup's first one.
constexpr int kPer = 4, kWalk = kPer * TPB;
template <class Load, class Use>
__device__ __forceinline__ void walk_planes(long long total, int per_plane, const FastDiv& divP, const FastDiv& divC,
                                            Load load, Use use) {
  const long long t0 = (long long)blockIdx.x * kWalk, plane0 = t0 / per_plane;
  const int rem0 = (int)(t0 - plane0 * per_plane), left = (int)min((long long)kWalk, total - t0);
  int dp[kPer], r[kPer], c[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int rem = rem0 + min(u * TPB + (int)threadIdx.x, left - 1);  // past the end: the last one, unused
    dp[u] = fdiv(rem, divP);
    const int o = rem - dp[u] * per_plane;
    r[u] = fdiv(o, divC);
    c[u] = o - r[u] * divC.d;
    load(u, plane0, dp[u], r[u], c[u]);
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (u * TPB + (int)threadIdx.x < left) use(u, plane0, dp[u], r[u], c[u]);
}
// the planes of one workgroup within 32-bit offsets
inline bool walk_fits(long long per_plane, long long in_plane, long long out_plane) {
  return per_plane < (1LL << 30) && (kWalk / per_plane + 2) * std::max(in_plane, out_plane) < (1LL << 29);
}

// Windows of K x K pixels, K >= stride.  CLIP: some windows reach past the image; none is empty, and rows
// and columns past a clipped window's end repeat its last one (a repeated value is never greater).  Pool1
// at batch 256 (297 MB in, 143 MB out): 183 us with one dependent load at a time and 64-bit divisions per
// thread, 144 with all loads of four windows in flight but nine of 4 bytes each, 114 with pairs.
// PAIRS (K = 3, stride 2, no clipping): a lane loads the first two columns of its window, 8 bytes next to
// its neighbour's, and takes the third from the neighbour; lanes at the end of a row or wave load it (the others ask
// for an offset that the buffer's range check answers: behind a branch every row's load was a trip to memory of its own,
// 116 -> 99 us).  The last element's window ends its row, so that no lane in use takes a column from one past the end.
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));  // 8 bytes, dword aligned
template <int K, bool CLIP, bool PAIRS = false>
__global__ __launch_bounds__(TPB) void maxpool_forward_window(const float* __restrict__ x, float* __restrict__ y,
                                                              int* __restrict__ argmax, long long total, PoolGeom g,
                                                              FastDiv divP, FastDiv divC) {
  const int Po = g.Ho * g.Wo, P = g.H * g.W;
  float v[kPer][K * K];
  auto corner = [&](int r, int q, int* h0, int* w0, int* h1, int* w1) {
    *h0 = CLIP ? max(r * g.s - g.p, 0) : r * g.s;
    *w0 = CLIP ? max(q * g.s - g.p, 0) : q * g.s;
    *h1 = min(r * g.s - g.p + K, g.H) - 1;
    *w1 = min(q * g.s - g.p + K, g.W) - 1;
  };
  auto edge = [&](int q) { return (threadIdx.x & 63) == 63 || q == g.Wo - 1; };
  // offset of a pixel from the window's first one
  auto off = [&](int e, int h0, int w0, int h1, int w1) {
    const int i = e / K, j = e % K;
    return CLIP ? (min(h0 + i, h1) - h0) * g.W + min(w0 + j, w1) - w0 : i * g.W + j;
  };
  walk_planes(
      total, Po, divP, divC,
      [&](int u, long long plane0, int dp, int r, int q) {
        int h0, w0, h1, w1;
        corner(r, q, &h0, &w0, &h1, &w1);
        const float* __restrict__ xp = x + plane0 * P;
        const unsigned base = (unsigned)(dp * P + h0 * g.W + w0);
        if constexpr (PAIRS) {
          const __amdgpu_buffer_rsrc_t rs =
              __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xp), 0, 0x7fffffff, 0x00020000);
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const unsigned at = (base + (unsigned)(i * g.W)) * 4u;
            const f32x2u two = __builtin_bit_cast(f32x2u, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, 0, 0));
            v[u][3 * i] = two[0];
            v[u][3 * i + 1] = two[1];
            v[u][3 * i + 2] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(edge(q) ? at + 8u : 0x80000000u), 0, 0));
          }
          return;
        }
#pragma unroll
        for (int e = 0; e < K * K; ++e) v[u][e] = xp[base + (unsigned)off(e, h0, w0, h1, w1)];
      },
      [&](int u, long long plane0, int dp, int r, int q) {
        int h0, w0, h1, w1;
        corner(r, q, &h0, &w0, &h1, &w1);
        if constexpr (PAIRS) {
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const float next = __shfl_down(v[u][3 * i], 1, 64);
            v[u][3 * i + 2] = edge(q) ? v[u][3 * i + 2] : next;
          }
        }
        float bv = v[u][0];
        int best = 0;
#pragma unroll
        for (int e = 1; e < K * K; ++e) {
          const bool more = v[u][e] > bv;
          bv = more ? v[u][e] : bv;
          best = more ? off(e, h0, w0, h1, w1) : best;
        }
        const unsigned t = (unsigned)(dp * Po + r * g.Wo + q);
        (y + plane0 * Po)[t] = bv;
        if (argmax) (argmax + plane0 * Po)[t] = h0 * g.W + w0 + best;
      });
}

// Stride 2, windows of 2 or 3 pixels: a thread owns the 2 x 2 pixels (2a - p + 0..1, 2b - p + 0..1), which
// only the windows a - 1 (K = 3) and a, b - 1 and b contain: at most four, read once for four pixels.
// The windows of a pixel are added in row-major order, as the general kernels do.  Pool1 at batch 256
// (143 MB in, 297 MB out): 155 us with the planes staged in LDS and a loop per pixel, 109 now.
template <int K>
__global__ __launch_bounds__(TPB) void maxpool_backward_cells(const float* __restrict__ dy,
                                                              const int* __restrict__ argmax, float* __restrict__ dx,
                                                              long long total, int cells, PoolGeom g, FastDiv divP,
                                                              FastDiv divC) {
  constexpr int NW = K - 1;  // windows per axis
  const int Po = g.Ho * g.Wo, P = g.H * g.W;
  float v[kPer][NW][NW];
  int m[kPer][NW][NW];
  walk_planes(
      total, cells, divP, divC,
      [&](int u, long long plane0, int dp, int a, int b) {
        const float* __restrict__ dyp = dy + plane0 * Po;
        const int* __restrict__ ap = argmax + plane0 * Po;
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
          for (int j = 0; j < NW; ++j) {
            // a window outside the grid: load the nearest one, it is ignored below
            const int rc = min(max(a - NW + 1 + i, 0), g.Ho - 1), qc = min(max(b - NW + 1 + j, 0), g.Wo - 1);
            const unsigned o = (unsigned)(dp * Po + rc * g.Wo + qc);
            m[u][i][j] = ap[o];
            v[u][i][j] = dyp[o];
          }
      },
      [&](int u, long long plane0, int dp, int a, int b) {
        float* __restrict__ out = dx + plane0 * P;
        const int h0 = 2 * a - g.p, w0 = 2 * b - g.p;
        bool rok[NW], qok[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          rok[i] = a - NW + 1 + i >= 0 && a - NW + 1 + i < g.Ho;
          qok[i] = b - NW + 1 + i >= 0 && b - NW + 1 + i < g.Wo;
        }
#pragma unroll
        for (int eh = 0; eh < 2; ++eh) {
          const int h = h0 + eh;
          float acc[2];
#pragma unroll
          for (int ew = 0; ew < 2; ++ew) {
            const int me = h * g.W + w0 + ew;
            float sum = 0.f;
#pragma unroll
            for (int i = eh ? NW - 1 : 0; i < NW; ++i)
#pragma unroll
              for (int j = ew ? NW - 1 : 0; j < NW; ++j)
                sum += rok[i] && qok[j] && m[u][i][j] == me ? v[u][i][j] : 0.f;
            acc[ew] = sum;
          }
          if (h < 0 || h >= g.H) continue;
          const unsigned o = (unsigned)(dp * P + h * g.W + w0);
          if (w0 >= 0 && w0 + 1 < g.W) {
            const f32x2u two = {acc[0], acc[1]};
            *reinterpret_cast<f32x2u*>(out + o) = two;
          } else if (w0 >= 0) {
            if (w0 < g.W) out[o] = acc[0];
          } else if (w0 + 1 >= 0 && w0 + 1 < g.W) {
            out[o + 1] = acc[1];
          }
        }
      });
}

// The same gather with the output planes staged in LDS: a workgroup owns `np` consecutive
// (image, channel) planes, copies their dy and argmax (np*Ho*Wo values each, contiguous in memory)
// into LDS with coalesced loads and then walks the np*H*W input pixels, which gather from LDS in
// the same window order.  dy and argmax are read from memory once, and all index arithmetic is
// 32-bit with multiplicative division.
__global__ __launch_bounds__(TPB) void maxpool_backward_lds_kernel(
    const float* __restrict__ dy, const int* __restrict__ argmax, float* __restrict__ dx,
    long long planes, int np, PoolGeom g, FastDiv divP, FastDiv divW, FastDiv divS) {
  extern __shared__ float pool_smem[];
  const int Po = g.Ho * g.Wo, P = g.H * g.W;
  const long long pl0 = (long long)blockIdx.x * np;
  const int n_here = (int)min((long long)np, planes - pl0);
  float* sdy = pool_smem;
  int* sarg = reinterpret_cast<int*>(pool_smem + np * Po);
  const float* __restrict__ dyp = dy + pl0 * Po;
  const int* __restrict__ ap = argmax + pl0 * Po;
  for (int i = threadIdx.x; i < n_here * Po; i += TPB) {
    sdy[i] = dyp[i];
    sarg[i] = ap[i];
  }
  __syncthreads();
  float* __restrict__ dxp = dx + pl0 * P;
  for (int i = threadIdx.x; i < n_here * P; i += TPB) {
    const int pl = fdiv(i, divP), me = i - pl * P;
    const int h = fdiv(me, divW), w = me - h * g.W;
    const int rlo = h + g.p - g.K + 1 <= 0 ? 0 : fdiv(h + g.p - g.K + g.s, divS);
    const int qlo = w + g.p - g.K + 1 <= 0 ? 0 : fdiv(w + g.p - g.K + g.s, divS);
    const int rhi = min(fdiv(h + g.p, divS), g.Ho - 1), qhi = min(fdiv(w + g.p, divS), g.Wo - 1);
    const int ob = pl * Po;
    float acc = 0.f;
    for (int r = rlo; r <= rhi; ++r)
      for (int q = qlo; q <= qhi; ++q) {
        const int o = ob + r * g.Wo + q;
        if (sarg[o] == me) acc += sdy[o];
      }
    dxp[i] = acc;
  }
}

bool pool_geom(const cct_pool_desc_t* d, PoolGeom* g) {
  if (!d || d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->K <= 0 || d->stride <= 0 ||
      d->pad < 0 || d->pad >= d->K)
    return false;
  auto out = [&](int in) {
    const long long t = std::max<long long>((long long)in + 2LL * d->pad - d->K, 0);
    long long o = (t + d->stride - 1) / d->stride + 1;
    if (d->pad > 0 && (o - 1) * d->stride >= (long long)in + d->pad) --o;
    return o;
  };
  const long long ho = out(d->H), wo = out(d->W);
  if ((long long)d->H * d->W >= 2147483647LL || ho >= 2147483647LL || wo >= 2147483647LL) return false;
  *g = PoolGeom{d->H, d->W, d->K, d->stride, d->pad, (int)ho, (int)wo};
  return true;
}

inline long long vec4_count(const void* a, const void* b, const void* c, long long n) {
  const uintptr_t bits = reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) |
                         reinterpret_cast<uintptr_t>(c);
  return bits % 16 == 0 ? n / 4 : 0;
}

inline unsigned stream_blocks(long long work_items) {
  // enough workgroups to fill the chip several times over; the kernels loop (ReLU) or are
  // launched with one thread per element (pooling)
  const long long want = (work_items + TPB - 1) / TPB;
  return (unsigned)std::max<long long>(1, std::min<long long>(want, 256LL * 64));
}


// ---- local response normalisation -------------------------------------------------------------
struct LrnGeom {
  int C;
  unsigned segments;     // of the channels, one per thread and grid row
  long long hw, pixels;  // H*W, N*H*W
  float a, beta, k, coef;  // alpha/size; 2*alpha*beta/size
};

constexpr long long kLrnThreads = 1 << 18;
constexpr unsigned kMaxGridRows = 65535;

// s^-beta.  P34: beta = 3/4 (Caffe's default), where Newton's step for z^4 s^3 = 1 makes a result good to
// half a unit in the last place out of the hardware's approximate exponential and logarithm: with the
// rounding errors of z*z, z*z*s and its square carried along, e = z^4 s^3 - 1 is known to 2^-40, and
// z - z*e/4 rounds once.  About 15 instructions against powf's hundred, which were the kernels' bound.
// Outside [2^-30, 2^30] the intermediate powers could leave the range of fp32: powf.
template <bool P34>
__device__ __forceinline__ float neg_power(float s, float beta) {
  if (!P34 || !(s >= 0x1p-30f && s <= 0x1p30f)) return powf(s, -beta);
  const float z = __builtin_amdgcn_exp2f(-0.75f * __builtin_amdgcn_logf(s));
  const float a = z * z, al = fmaf(z, z, -a);
  const float b = a * s, bl = fmaf(al, s, fmaf(a, s, -b));
  const float c = b * b, cl = fmaf(2.f * b, bl, fmaf(b, b, -c));
  const float e = fmaf(cl, s, fmaf(c, s, -1.f));
  return fmaf(-0.25f * e, z, z);
}

template <int SIZE, bool P34, int CS>
__global__ __launch_bounds__(TPB) void lrn_forward_kernel(const float* __restrict__ x,
                                                          float* __restrict__ y, LrnGeom g) {
  constexpr int HALF = (SIZE - 1) / 2;
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= g.pixels) return;
  const long long n = t / g.hw, pix = t - n * g.hw;
  const float* xp = x + n * g.C * g.hw + pix;  // channel c of this pixel is xp[c*hw]
  float* yp = y + n * g.C * g.hw + pix;
  // one turn unless there are more segments than a grid has rows
  for (unsigned seg = blockIdx.y; seg < g.segments; seg += gridDim.y) {
    const int c0 = (int)(seg * CS);
    float xs[CS + 2 * HALF];  // x of channels c0-HALF ..
#pragma unroll
    for (int i = 0; i < CS + 2 * HALF; ++i) {
      const int ch = c0 + i - HALF;
      xs[i] = (ch >= 0 && ch < g.C) ? xp[ch * g.hw] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < CS; ++i) {
      if (c0 + i >= g.C) break;
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < SIZE; ++k) sum += xs[i + k] * xs[i + k];
      yp[(c0 + i) * g.hw] = xs[i + HALF] * neg_power<P34>(g.k + g.a * sum, g.beta);
    }
  }
}

// dx[c] = dy[c]*scale[c]^-beta - coef * x[c] * sum_{|c'-c| <= HALF} dy[c'] x[c'] scale[c']^(-beta-1).
template <int SIZE, bool P34, int CS>
__global__ __launch_bounds__(TPB) void lrn_backward_kernel(const float* __restrict__ x,
                                                           const float* __restrict__ dy,
                                                           float* __restrict__ dx, LrnGeom g) {
  constexpr int HALF = (SIZE - 1) / 2;
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= g.pixels) return;
  const long long n = t / g.hw, pix = t - n * g.hw;
  const float* xp = x + n * g.C * g.hw + pix;
  const float* gp = dy + n * g.C * g.hw + pix;
  float* op = dx + n * g.C * g.hw + pix;
  for (unsigned seg = blockIdx.y; seg < g.segments; seg += gridDim.y) {
    const int c0 = (int)(seg * CS);
    float xs[CS + 4 * HALF];  // x of channels c0-2*HALF ..
    float gs[CS + 2 * HALF];  // dy of channels c0-HALF .., then the direct terms dy*scale^-beta
    float tr[CS + 2 * HALF];  // cross terms of the same channels
#pragma unroll
    for (int i = 0; i < CS + 4 * HALF; ++i) {
      const int ch = c0 + i - 2 * HALF;
      xs[i] = (ch >= 0 && ch < g.C) ? xp[ch * g.hw] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < CS + 2 * HALF; ++i) {
      const int ch = c0 + i - HALF;
      gs[i] = (ch >= 0 && ch < g.C) ? gp[ch * g.hw] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < CS + 2 * HALF; ++i) {
      const int ch = c0 + i - HALF;
      tr[i] = 0.f;
      if (ch >= 0 && ch < g.C) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < SIZE; ++k) sum += xs[i + k] * xs[i + k];
        const float scale = g.k + g.a * sum;
        const float pw = neg_power<P34>(scale, g.beta);
        tr[i] = gs[i] * xs[i + HALF] * pw / scale;
        gs[i] *= pw;
      }
    }
#pragma unroll
    for (int i = 0; i < CS; ++i) {
      if (c0 + i >= g.C) break;
      float cross = 0.f;
#pragma unroll
      for (int k = 0; k < SIZE; ++k) cross += tr[i + k];
      op[(c0 + i) * g.hw] = gs[i + HALF] - g.coef * xs[i + 2 * HALF] * cross;
    }
  }
}

bool lrn_geom(const cct_lrn_desc_t* d, LrnGeom* g) {
  if (!d || d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0) return false;
  if (d->size < 1 || !(d->size & 1) || !(d->k > 0.f) || !(d->alpha >= 0.f)) return false;
  g->C = d->C;
  g->hw = (long long)d->H * d->W;
  g->pixels = g->hw * d->N;
  g->a = d->alpha / (float)d->size;
  g->beta = d->beta;
  g->k = d->k;
  g->coef = 2.0f * d->alpha * d->beta / (float)d->size;
  return true;
}

template <int SIZE, bool P34, int CS>
void launch_lrn_kernel(bool backward, const float* x, const float* dy, float* out, const LrnGeom& g,
                       dim3 grid, hipStream_t st) {
  if (backward)
    hipLaunchKernelGGL((lrn_backward_kernel<SIZE, P34, CS>), grid, dim3(TPB), 0, st, x, dy, out, g);
  else
    hipLaunchKernelGGL((lrn_forward_kernel<SIZE, P34, CS>), grid, dim3(TPB), 0, st, x, out, g);
}
template <int SIZE>
void launch_lrn(bool backward, const float* x, const float* dy, float* out, const LrnGeom& g, int cs,
                dim3 grid, hipStream_t st) {
  const bool p34 = g.beta == 0.75f;
  if (cs == 16)
    p34 ? launch_lrn_kernel<SIZE, true, 16>(backward, x, dy, out, g, grid, st)
        : launch_lrn_kernel<SIZE, false, 16>(backward, x, dy, out, g, grid, st);
  else
    p34 ? launch_lrn_kernel<SIZE, true, 4>(backward, x, dy, out, g, grid, st)
        : launch_lrn_kernel<SIZE, false, 4>(backward, x, dy, out, g, grid, st);
}

int run_lrn(const cct_lrn_desc_t* desc, bool backward, const float* x, const float* dy, float* out,
            hipStream_t st) {
  LrnGeom g;
  if (!lrn_geom(desc, &g) || !x || !out || (backward && !dy)) return CCT_EINVAL;
  const long long blocks = (g.pixels + TPB - 1) / TPB;
  if (blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  const double elems = (double)g.pixels * g.C;
  ProfScope ps(backward ? "lrn_backward_kernel" : "lrn_forward_kernel", 0.0,
               (backward ? 12.0 : 8.0) * elems, st);
  // A thread takes 16 channels of its pixel, all loaded before the first result, so that a CU has enough
  // bytes in flight; the size-1 (backward: 2*(size-1)) channels around them come from L2 once more.  With
  // few pixels 4, for more threads.  norm1 at batch 256 (72 MB): forward 72 us walking the channels with one
  // load ahead and powf, 32 now; backward 97 -> 49.
  const int cs = (g.pixels * ((g.C + 15) / 16) >= kLrnThreads) ? 16 : 4;
  g.segments = (unsigned)(((long long)g.C + cs - 1) / cs);
  const dim3 grid((unsigned)blocks, std::min(g.segments, kMaxGridRows));
  switch (desc->size) {
    case 1: launch_lrn<1>(backward, x, dy, out, g, cs, grid, st); break;
    case 3: launch_lrn<3>(backward, x, dy, out, g, cs, grid, st); break;
    case 5: launch_lrn<5>(backward, x, dy, out, g, cs, grid, st); break;
    case 7: launch_lrn<7>(backward, x, dy, out, g, cs, grid, st); break;
    case 9: launch_lrn<9>(backward, x, dy, out, g, cs, grid, st); break;
    default: return CCT_EUNSUPPORTED;  // window sizes are compiled in: 1, 3, 5, 7, 9
  }
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// Dropout with the caller's mask: y = x * scale where mask != 0, else 0 (both directions).
__global__ __launch_bounds__(TPB) void dropout_kernel(const float* __restrict__ x,
                                                      const unsigned char* __restrict__ mask,
                                                      float scale, float* __restrict__ y,
                                                      long long n) {
  const long long stride = (long long)gridDim.x * TPB;
  for (long long i = (long long)blockIdx.x * TPB + threadIdx.x; i < n; i += stride)
    y[i] = mask[i] ? x[i] * scale : 0.f;
}

// Combines one value per thread over the workgroup, always in the same order: lanes by
// shuffles, the four waves through LDS.  Every thread gets the result.
template <bool MAX>
__device__ __forceinline__ float block_combine(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off, 64);
    v = MAX ? fmaxf(v, o) : v + o;
  }
  __syncthreads();   // red may still be read from an earlier call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const float a = red[0], b = red[1], c = red[2], d = red[3];
  return MAX ? fmaxf(fmaxf(a, b), fmaxf(c, d)) : (a + b) + (c + d);
}

// Softmax over the C scores of image blockIdx.x and its loss term
// -(x[label] - max - log(sum exp(x - max))); NaN for a label outside [0, C).
__global__ __launch_bounds__(TPB) void softmax_loss_forward_kernel(const float* __restrict__ x,
                                                                   const int* __restrict__ label,
                                                                   float* __restrict__ prob,
                                                                   float* __restrict__ image_loss,
                                                                   int C) {
  __shared__ float red[4];
  const float* xr = x + (long long)blockIdx.x * C;
  float* pr = prob + (long long)blockIdx.x * C;
  float mx = -__builtin_inff();
  for (int c = threadIdx.x; c < C; c += TPB) mx = fmaxf(mx, xr[c]);
  mx = block_combine<true>(mx, red);
  float sum = 0.f;
  for (int c = threadIdx.x; c < C; c += TPB) sum += expf(xr[c] - mx);
  sum = block_combine<false>(sum, red);
  const float inv = 1.0f / sum;
  for (int c = threadIdx.x; c < C; c += TPB) pr[c] = expf(xr[c] - mx) * inv;
  if (threadIdx.x == 0) {
    const int l = label[blockIdx.x];
    image_loss[blockIdx.x] =
        (l >= 0 && l < C) ? -(xr[l] - mx - logf(sum)) : __builtin_nanf("");
  }
}

// loss = (1/N) * sum of the per-image terms, added in a fixed order by one workgroup.
__global__ __launch_bounds__(TPB) void mean_kernel(const float* __restrict__ v,
                                                   float* __restrict__ out, int N) {
  __shared__ float red[4];
  float acc = 0.f;
  for (int i = threadIdx.x; i < N; i += TPB) acc += v[i];
  acc = block_combine<false>(acc, red);
  if (threadIdx.x == 0) out[0] = acc / (float)N;
}

__global__ __launch_bounds__(TPB) void softmax_loss_backward_kernel(const float* __restrict__ prob,
                                                                    const int* __restrict__ label,
                                                                    float* __restrict__ dx,
                                                                    long long total, FastDiv divC,
                                                                    float inv_n) {
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= total) return;
  const int n = fdiv((int)t, divC), c = (int)t - n * divC.d;
  dx[t] = (prob[t] - (c == label[n] ? 1.f : 0.f)) * inv_n;
}

int run_dropout(const float* x, const unsigned char* mask, float scale, float* y, long long n,
                hipStream_t st) {
  if (!x || !mask || !y || n < 0 || !(scale > 0.f)) return CCT_EINVAL;
  if (n == 0) return CCT_OK;
  const long long blocks = std::min<long long>((n + TPB - 1) / TPB, 1 << 16);
  ProfScope ps("dropout_kernel", 0.0, 9.0 * (double)n, st);
  hipLaunchKernelGGL(dropout_kernel, dim3((unsigned)blocks), dim3(TPB), 0, st, x, mask, scale, y, n);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace
}  // namespace cct

using namespace cct;

extern "C" {

int cct_relu_forward(const float* x, float* y, int64_t n, void* hip_stream) {
  if (!x || !y || n < 0) return CCT_EINVAL;
  if (n == 0) return CCT_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const long long n4 = vec4_count(x, y, nullptr, n);
  ProfScope ps("relu_forward_kernel", 0.0, 8.0 * (double)n, st);
  hipLaunchKernelGGL(relu_forward_kernel, dim3(stream_blocks(n4 ? n4 : n)), dim3(TPB), 0, st, x, y,
                     n4, (long long)n);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int cct_relu_backward(const float* x, const float* dy, float* dx, int64_t n, void* hip_stream) {
  if (!x || !dy || !dx || n < 0) return CCT_EINVAL;
  if (n == 0) return CCT_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const long long n4 = vec4_count(x, dy, dx, n);
  ProfScope ps("relu_backward_kernel", 0.0, 12.0 * (double)n, st);
  hipLaunchKernelGGL(relu_backward_kernel, dim3(stream_blocks(n4 ? n4 : n)), dim3(TPB), 0, st, x,
                     dy, dx, n4, (long long)n);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int cct_pool_output_dims(const cct_pool_desc_t* desc, int32_t* Hout, int32_t* Wout) {
  PoolGeom g;
  if (!Hout || !Wout || !pool_geom(desc, &g)) return CCT_EINVAL;
  *Hout = g.Ho;
  *Wout = g.Wo;
  return CCT_OK;
}

int cct_maxpool_forward(const cct_pool_desc_t* desc, const float* x, float* y, int32_t* argmax,
                        void* hip_stream) {
  PoolGeom g;
  if (!pool_geom(desc, &g) || !x || !y) return CCT_EINVAL;
  const long long total = (long long)desc->N * desc->C * g.Ho * g.Wo;
  const long long blocks = (total + TPB - 1) / TPB;
  if (blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)hip_stream;
  ProfScope ps("maxpool_forward_kernel", 0.0,
               4.0 * (double)desc->N * desc->C * g.H * g.W + (argmax ? 8.0 : 4.0) * (double)total, st);
  const long long Po = (long long)g.Ho * g.Wo;
  if ((g.K == 3 || g.K == 2) && g.s <= g.K && walk_fits(Po, (long long)g.H * g.W, Po)) {
    const dim3 grid((unsigned)((total + kWalk - 1) / kWalk));
    const FastDiv divP = make_fastdiv((int)Po), divC = make_fastdiv(g.Wo);
    const bool clip = g.p > 0 || (g.Ho - 1) * g.s + g.K > g.H || (g.Wo - 1) * g.s + g.K > g.W;
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(TPB), 0, st, x, y, argmax, total, g, divP, divC);
    };
    if (g.K == 3 && g.s == 2 && !clip)
      run(maxpool_forward_window<3, false, true>);
    else if (g.K == 3)
      clip ? run(maxpool_forward_window<3, true>) : run(maxpool_forward_window<3, false>);
    else
      clip ? run(maxpool_forward_window<2, true>) : run(maxpool_forward_window<2, false>);
  } else {
    hipLaunchKernelGGL(maxpool_forward_kernel, dim3((unsigned)blocks), dim3(TPB), 0, st, x, y, argmax,
                       total, g);
  }
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int cct_maxpool_backward(const cct_pool_desc_t* desc, const float* dy, const int32_t* argmax,
                         float* dx, void* hip_stream) {
  PoolGeom g;
  if (!pool_geom(desc, &g) || !dy || !argmax || !dx) return CCT_EINVAL;
  const long long total = (long long)desc->N * desc->C * g.H * g.W;
  const long long blocks = (total + TPB - 1) / TPB;
  if (blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)hip_stream;
  ProfScope ps("maxpool_backward_kernel", 0.0,
               4.0 * (double)total + 8.0 * (double)desc->N * desc->C * g.Ho * g.Wo, st);
  const long long ca = ((long long)g.H - 1 + g.p) / 2 + 1, cb = ((long long)g.W - 1 + g.p) / 2 + 1;
  if (g.s == 2 && (g.K == 3 || g.K == 2) &&
      walk_fits(ca * cb, (long long)g.H * g.W, (long long)g.Ho * g.Wo)) {
    const long long cells = (long long)desc->N * desc->C * ca * cb;
    const dim3 grid((unsigned)((cells + kWalk - 1) / kWalk));
    const FastDiv divP = make_fastdiv((int)(ca * cb)), divC = make_fastdiv((int)cb);
    if (g.K == 3)
      hipLaunchKernelGGL(maxpool_backward_cells<3>, grid, dim3(TPB), 0, st, dy, argmax, dx, cells, (int)(ca * cb), g,
                         divP, divC);
    else
      hipLaunchKernelGGL(maxpool_backward_cells<2>, grid, dim3(TPB), 0, st, dy, argmax, dx, cells, (int)(ca * cb), g,
                         divP, divC);
    CCT_CHECK_LAUNCH();
    return CCT_OK;
  }
  // planes whose dy and argmax fit 64 KiB of LDS: about 4096 input pixels per workgroup
  const long long P = (long long)g.H * g.W, Po = (long long)g.Ho * g.Wo;
  const long long planes = (long long)desc->N * desc->C;
  if (Po * 8 <= 65536 && P <= 65536) {
    long long np = std::max<long long>(1, 4096 / P);
    np = std::min({np, 65536 / (Po * 8), planes});
    const long long wgs = (planes + np - 1) / np;
    if (wgs >= 2147483647LL) return CCT_EUNSUPPORTED;
    hipLaunchKernelGGL(maxpool_backward_lds_kernel, dim3((unsigned)wgs), dim3(TPB),
                       (size_t)(np * Po * 8), st, dy, argmax, dx, planes, (int)np, g,
                       make_fastdiv((int)P), make_fastdiv(g.W), make_fastdiv(g.s));
    CCT_CHECK_LAUNCH();
    return CCT_OK;
  }
  hipLaunchKernelGGL(maxpool_backward_kernel, dim3((unsigned)blocks), dim3(TPB), 0, st, dy, argmax,
                     dx, total, g);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int cct_lrn_forward(const cct_lrn_desc_t* desc, const float* x, float* y, void* hip_stream) {
  return run_lrn(desc, false, x, nullptr, y, (hipStream_t)hip_stream);
}

int cct_lrn_backward(const cct_lrn_desc_t* desc, const float* x, const float* dy, float* dx,
                     void* hip_stream) {
  return run_lrn(desc, true, x, dy, dx, (hipStream_t)hip_stream);
}

int cct_dropout_forward(const float* x, const uint8_t* mask, float scale, float* y, int64_t n,
                        void* hip_stream) {
  return run_dropout(x, mask, scale, y, n, (hipStream_t)hip_stream);
}

int cct_dropout_backward(const float* dy, const uint8_t* mask, float scale, float* dx, int64_t n,
                         void* hip_stream) {
  return run_dropout(dy, mask, scale, dx, n, (hipStream_t)hip_stream);
}

int cct_softmax_loss_forward(int32_t N, int32_t C, const float* x, const int32_t* label, float* prob,
                             float* image_loss, float* loss, void* hip_stream) {
  if (N <= 0 || C <= 0 || !x || !label || !prob || !image_loss || !loss) return CCT_EINVAL;
  hipStream_t st = (hipStream_t)hip_stream;
  ProfScope ps("softmax_loss_forward_kernel", 0.0, 8.0 * (double)N * C, st);
  hipLaunchKernelGGL(softmax_loss_forward_kernel, dim3((unsigned)N), dim3(TPB), 0, st, x, label, prob,
                     image_loss, C);
  CCT_CHECK_LAUNCH();
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(TPB), 0, st, image_loss, loss, N);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int cct_softmax_loss_backward(int32_t N, int32_t C, const float* prob, const int32_t* label,
                              float* dx, void* hip_stream) {
  if (N <= 0 || C <= 0 || !prob || !label || !dx) return CCT_EINVAL;
  const long long total = (long long)N * C;
  if (total >= 2147483647LL) return CCT_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)hip_stream;
  ProfScope ps("softmax_loss_backward_kernel", 0.0, 8.0 * (double)total, st);
  hipLaunchKernelGGL(softmax_loss_backward_kernel, dim3((unsigned)((total + TPB - 1) / TPB)), dim3(TPB),
                     0, st, prob, label, dx, total, make_fastdiv(C), 1.0f / (float)N);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // extern "C"
