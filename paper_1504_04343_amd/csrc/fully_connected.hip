// Fully connected layers through the convolution entry points.
//
// A layer whose kernel covers its whole unpadded input (K = H = W, one output pixel per image)
// is the m = 1 case of the lowering of Sec. 2.1: the lowered matrix D^ is the batch itself viewed
// as [N][F], F = C*K*K, the kernel matrix K^ is w viewed as [O][F] and lifting is a reshape, so
// the three passes are the plain matrix products
//     y = D^ K^T + b          (contract over F: both operands are F-contiguous in place)
//     dD^ = dy K^             (contract over O: w is read in place, dy^T is packed: N*O values)
//     dK^ = dy^T D^           (contract over N: x is read in place, dy is packed)
// with no lowered copy, no kernel-matrix pack and no chunking.  The forward product has only
// N*O outputs (few tiles) and a long contraction, so it is split over F into partial products
// that a second kernel sums in split order together with the bias (bit-reproducible, no atomics).
// The backward-data product has N*F outputs, still too few tiles at CaffeNet's batch, and is split
// over O the same way (the splits run as the groups of one launch).  The products run on gemm_split, over few
// images as plain fp32 products that read or write the kernels once (fc_forward_few, fc_backward_data_few,
// fc_outer_kernel); the fp32 matrix kernels are for workspaces without room for gemm_split's packed operand and for
// backward-weights passes over 17 to 32 images of more than 2^22 weights.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "cct_internal.h"
#include "index_common.h"

namespace cct {
namespace {

constexpr long long kAlign = 256;
constexpr int kIntMax = 2147483647;
constexpr int kDbiasBlocks = 64;
// workgroups the split forward product aims for, and the shortest split worth a workgroup
constexpr int kFcTargetBlocks = 1024;
constexpr int kFcMinSplit = 256;
constexpr long long kFcMaxPartBytes = 256LL << 20;
// backward-data: workgroups that fill the chip, and the fewest kernels a split may hold
constexpr int kFcFillBlocks = 1024;
constexpr int kFcMinSplitRows = 128;

inline long long align_up(long long v, long long a) { return (v + a - 1) / a * a; }

// pack[r][m] (Kpad x Mpad, zero padded) = transposed ? src[m][k] : src[k][m], src compact, where
// row r = g*Kpad_s + kk stands for k = g*Ks + kk (kk < Ks; the other rows of a split are zero):
// the K indices are cut into splits of Ks, each padded to Kpad_s rows.  32 x 32 tiles through LDS
// so that reads and writes are both row-contiguous.
__global__ __launch_bounds__(TPB) void fc_pack_kernel(const float* __restrict__ src,
                                                      float* __restrict__ pack, int K, int M,
                                                      int Kpad, int Mpad, int transposed, int Ks,
                                                      int Kpad_s) {
  __shared__ float tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = blockIdx.y * 32, m0 = blockIdx.x * 32;
  if (transposed) {
    const int r = r0 + tx, g = r / Kpad_s, kk = r - g * Kpad_s, k = g * Ks + kk;
    const bool kok = r < Kpad && kk < Ks && k < K;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + ty + j * 8;
      tile[ty + j * 8][tx] = (m < M && kok) ? src[(long long)m * K + k] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rr = r0 + ty + j * 8, m = m0 + tx;
      if (rr < Kpad && m < Mpad) pack[(long long)rr * Mpad + m] = tile[tx][ty + j * 8];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + ty + j * 8, m = m0 + tx;
      const int g = r / Kpad_s, kk = r - g * Kpad_s, k = g * Ks + kk;
      if (r < Kpad && m < Mpad)
        pack[(long long)r * Mpad + m] = (kk < Ks && k < K && m < M) ? src[(long long)k * M + m] : 0.0f;
    }
  }
}

// y[n][o] = sum_s part[s][n][o] + bias[o], splits added in order.
__global__ __launch_bounds__(TPB) void fc_sum_splits_kernel(const float* __restrict__ part,
                                                            float* __restrict__ y, int S,
                                                            long long total, FastDiv divO,
                                                            const float* __restrict__ bias) {
  const long long t = (long long)blockIdx.x * TPB + threadIdx.x;
  if (t >= total) return;
  const float* src = part + t;
  // In 64 bits: 31 parts of 32 kernels each added in 32 are what such a sum's error came from.  Four loads in flight, past
  // the end the last one again.
  double acc = 0.0;
  const float shift = bias ? bias[(int)t - fdiv((int)t, divO) * divO.d] : 0.f;
  for (int s = 0; s < S; s += 4) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = src[(long long)min(s + u, S - 1) * total];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = s + u < S ? acc + v[u] : acc;
  }
  y[t] = (float)(acc + shift);
}

// (In profiles this kernel and fc_backward_data_few are gemm_split_k and gemm_split_k_columns, as readers of
// cct_profile_read know them; they split nothing and use no matrix core.)
typedef float fc_f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes, dword aligned

// The product of up to 8 rows with a k-contiguous B (a fully connected layer's forward pass on few images) in one launch
// and without splitting: C[m][col] = sum_k A[m][k] * B[col][k] + bias[col].  A workgroup owns 4 columns; the contraction is
// split over its lanes and 8 waves, 4 consecutive k each, whose sums meet in a tree.  Bound by reading B once: a matrix
// instruction would be 16 or 32 rows of which most are none, and splitting B costs more than 8 multiplications.
// One image: fc6's 151 MB 46.3 us on gemm_split with its partial sums and their launch, 26.9 now; 4096 -> 1000 12.9 -> 6.7.
// Up to 4 rows at any size (4 rows of fc6 41.8 -> 36.3), up to 8 where B has up to 2^22 values in rows of 256 and more: beyond that each
// column's share of A, which comes from the L1, weighs (8 rows, 4096 -> 4096 27.9 and 23.8, 9216 -> 4096 51.1 and 41.6).
constexpr int kCols = 4, kWaves = 8;
struct FewRows {
  const float *A, *B, *bias;
  float* C;
  int M, N, K;
};
template <int N, int OFF>
__device__ __forceinline__ void fold(double* v, int lane, int* mine) {
  if constexpr (N > 1) {
    const bool upper = lane & OFF;
#pragma unroll
    for (int q = 0; q < N / 2; ++q) {
      const double keep = upper ? v[q + N / 2] : v[q], give = upper ? v[q] : v[q + N / 2];
      v[q] = keep + __shfl_xor(give, OFF, 64);
    }
    *mine += upper ? N / 2 : 0;
  } else {
    v[0] += __shfl_xor(v[0], OFF, 64);
  }
  if constexpr (OFF > 1) fold<(N > 1 ? N / 2 : 1), OFF / 2>(v, lane, mine);
}
// ALONE: every wave has 4 columns and their whole contraction to itself, of less than one step of all waves.  Many columns
// of few features are workgroups that share out next to nothing and meet for it.
template <int ROWS, bool ALONE = false>
__global__ __launch_bounds__(64 * kWaves) void fc_forward_few(FewRows p) {
  __shared__ double red[ALONE ? 1 : kWaves][ROWS * kCols];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n0 = (ALONE ? (int)blockIdx.x * kWaves + wave : (int)blockIdx.x) * kCols;
  constexpr int STEP = (ALONE ? 1 : kWaves) * 64 * 4;
  const float *a[ROWS], *b[kCols];
#pragma unroll
  for (int m = 0; m < ROWS; ++m) a[m] = p.A + (long long)min(m, p.M - 1) * p.K;
#pragma unroll
  for (int c = 0; c < kCols; ++c) b[c] = p.B + (long long)min(n0 + c, p.N - 1) * p.K;
  double acc[ROWS][kCols];
#pragma unroll
  for (int m = 0; m < ROWS; ++m)
#pragma unroll
    for (int c = 0; c < kCols; ++c) acc[m][c] = 0.0;
  const int k_first = ((ALONE ? 0 : wave * 64) + lane) * 4;
  const int whole = p.K / STEP * STEP;  // up to here every lane has its 4
  fc_f32x4u bv[2][kCols], av[2][ROWS];
  auto load = [&](int set, int k) {
#pragma unroll
    for (int c = 0; c < kCols; ++c) bv[set][c] = *reinterpret_cast<const fc_f32x4u*>(b[c] + k);
#pragma unroll
    for (int m = 0; m < ROWS; ++m) av[set][m] = *reinterpret_cast<const fc_f32x4u*>(a[m] + k);
  };
  // Sums in 64 bits: lanes' chains and their tree in 32 rounded more than the matrix cores' chains do (2-norm, 2 rows of 136:
  // 7.0e-8, 5.7e-8 there, 2.4e-8 so; 3 of 1000 with 32 columns 1.3e-7, 8.3e-8, 2.6e-8).  In whole steps of all waves, which
  // are of rows of 2048 and more, four products are summed in 32 first (4.7e-8; 4 rows, 4096 -> 4096: 21 us without, 16).
  auto multiply = [&](int set, auto four) {
#pragma unroll
    for (int m = 0; m < ROWS; ++m)
#pragma unroll
      for (int c = 0; c < kCols; ++c) {
        if constexpr (decltype(four)::value) {
          float sum = av[set][m][0] * bv[set][c][0];
#pragma unroll
          for (int e = 1; e < 4; ++e) sum = fmaf(av[set][m][e], bv[set][c][e], sum);
          acc[m][c] += sum;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[m][c] = fma((double)av[set][m][e], (double)bv[set][c][e], acc[m][c]);
        }
      }
  };
  constexpr std::bool_constant<!ALONE> four;
  constexpr std::false_type single;
  if (whole) {
    const int last = whole - STEP;
    load(0, k_first);
    for (int k = 0; k < whole; k += 2 * STEP) {
      load(1, k_first + min(k + STEP, last));
      multiply(0, four);
      load(0, k_first + min(k + 2 * STEP, last));
      if (k + STEP < whole) multiply(1, four);
    }
  }
  const int k_rest = whole + k_first;
  if (k_rest + 4 <= p.K) {
    load(0, k_rest);
    multiply(0, single);
  } else {
    for (int k = k_rest; k < p.K; ++k) {
      double x[ROWS];
#pragma unroll
      for (int m = 0; m < ROWS; ++m) x[m] = a[m][k];
#pragma unroll
      for (int c = 0; c < kCols; ++c) {
        const double y = b[c][k];
#pragma unroll
        for (int m = 0; m < ROWS; ++m) acc[m][c] = fma(x[m], y, acc[m][c]);
      }
    }
  }
  // sums over the lanes: in every step a lane passes on half of its values and keeps the other half
  constexpr int VALUES = ROWS * kCols;
  double v[VALUES];
#pragma unroll
  for (int q = 0; q < VALUES; ++q) v[q] = acc[q / kCols][q % kCols];
  int mine = 0;
  fold<VALUES, 32>(v, lane, &mine);
  constexpr int REST = 64 / VALUES;  // lanes that hold the same value
  auto store = [&](int t, double sum) {
    const int m = t / kCols, col = n0 + t % kCols;
    if (m < p.M && col < p.N) p.C[(long long)m * p.N + col] = (float)(sum + (p.bias ? p.bias[col] : 0.f));
  };
  if constexpr (ALONE) {
    if (lane % REST == 0) store(mine, v[0]);
    return;
  }
  if (lane % REST == 0) red[wave][mine] = v[0];
  __syncthreads();
  const int t = threadIdx.x;
  if (t >= VALUES) return;
  double u[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) u[w] = red[w][t];
  store(t, ((u[0] + u[1]) + (u[2] + u[3])) + ((u[4] + u[5]) + (u[6] + u[7])));
}

// Columns from which the waves work alone: there it is 0.35 to 0.75 times the time with all waves, below as much or more.
// As times of gemm_split, which ran these layers before there was this kernel (20800 layers), with all waves and alone: 3 or
// 4 rows of up to 63 -> 4096 to 8191 1.32 and 1.00, of 256 to 511 -> 8192 and more 1.45 and 0.62; 5 to 8 rows of 256 to
// 511 -> 4096 to 8191 1.56 and 0.57, of 1024 to 2047 -> 2048 to 4095 0.99 and 0.79, of fewer columns 0.70 and 0.86.
bool few_alone(int M, int N, int K) { return K < 2048 && N >= (M <= 4 ? 4096 : 2048); }
bool forward_few_fits(int M, int N, int K) { return M <= 4 || (M <= 8 && K >= 256 && (long long)N * K <= (1LL << 22)); }

int launch_forward_few(const float* A, const float* B, const float* bias, float* C, int M, int N, int K, hipStream_t st) {
  if (M < 1 || M > 8 || N < 1 || K < 1) return CCT_EUNSUPPORTED;
  const FewRows p{A, B, bias, C, M, N, K};
  const bool alone = few_alone(M, N, K);
  const int cols = alone ? kCols * kWaves : kCols;
  const dim3 grid((unsigned)(((long long)N + cols - 1) / cols)), block(64 * kWaves);
  const int rows = M <= 2 ? M : M <= 4 ? 4 : 8;
  ProfScope ps(2.0 * M * N * K, 4.0 * ((double)M * K + (double)N * K + (double)M * N), st, alone ? "gemm_split_k<%d, alone>" : "gemm_split_k<%d>", rows);
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, st, p); };
  switch (rows) {
    case 1: launch(alone ? fc_forward_few<1, true> : fc_forward_few<1>); break;
    case 2: launch(alone ? fc_forward_few<2, true> : fc_forward_few<2>); break;
    case 4: launch(alone ? fc_forward_few<4, true> : fc_forward_few<4>); break;
    default: launch(alone ? fc_forward_few<8, true> : fc_forward_few<8>);
  }
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// dw[o][f] = sum_n dy[n][o] * x[n][f] and dbias[o] = sum_n dy[n][o] over up to IMAGES images, in fp32: a workgroup owns ROWS
// kernels x 1024 features, a thread 4 consecutive ones; dy's values are the same for all threads and come from LDS.
// Bound by writing dw, and in layers of some MB and less by one trip to memory: the loads of up to 16 images are on their
// way at once (four at a time, dy's values by scalar loads between them, was a trip for every four images or even every one,
// 32 images of 25 -> 3252 29.2 us).  In us, as a pack of dy, a matrix product whose stages are mostly padding and the bias
// gradient's launch, and so: 9216 -> 4096 on one image 39.0 and 24.4, on 16 39.7 and 27.7; 4096 -> 1000 on 16 13.6 and
// 7.9; 32 of 1024 -> 4096 15.7 and 10.8, of 25 -> 3252 12.0 and 11.8.  Of 6300 layers of 1 to 32 images none is slower.
constexpr int kOuterMost = 32;  // images
// From 17 images on 4 kernels: a thread's multiplications are what short launches take then (8: of 17 to 32 images an eighth
// of the layers up to 1.5 times as long as behind a pack)
constexpr int outer_rows(int N) { return N <= 16 ? 8 : 4; }
template <int IMAGES>
__global__ __launch_bounds__(TPB) void fc_outer_kernel(const float* __restrict__ x, const float* __restrict__ dy,
                                                       float* __restrict__ dw, float* __restrict__ dbias, int N, int O, int F) {
  constexpr int ROWS = outer_rows(IMAGES), AHEAD = IMAGES < 16 ? IMAGES : 16;  // images whose loads are in flight
  __shared__ __attribute__((aligned(16))) float g[kOuterMost][ROWS];
  const int o0 = blockIdx.y * ROWS;
  const int f0 = (int)(blockIdx.x * TPB + threadIdx.x) * 4;
  const bool whole = f0 + 4 <= F;
  float v[AHEAD][4];
  auto load = [&](int u) {  // images past the last one: that one again, times nothing
    const float* xn = x + (long long)min(u, N - 1) * F + min(f0, F - 1);
    if (whole) {
      const fc_f32x4u t = *reinterpret_cast<const fc_f32x4u*>(xn);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[u % AHEAD][e] = t[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[u % AHEAD][e] = f0 + e < F ? xn[e] : 0.f;
    }
  };
  {
    const int n = (int)threadIdx.x / ROWS, o = (int)threadIdx.x % ROWS;
    const float q = dy[(long long)min(n, N - 1) * O + min(o0 + o, O - 1)];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load(u);
    if (n < kOuterMost) g[n][o] = n < N ? q : 0.f;
  }
  __syncthreads();
  if (dbias && blockIdx.x == 0 && threadIdx.x < 8 * ROWS) {  // a lane sums 4 images of a kernel
    const int o = (int)threadIdx.x % ROWS, strip = (int)threadIdx.x / ROWS;
    float sum = (g[strip * 4][o] + g[strip * 4 + 1][o]) + (g[strip * 4 + 2][o] + g[strip * 4 + 3][o]);
#pragma unroll
    for (int off = ROWS; off < 8 * ROWS; off *= 2) sum += __shfl_xor(sum, off, 64);
    if (strip == 0 && o0 + o < O) dbias[o0 + o] = sum;
  }
  if (f0 >= F) return;
  float acc[ROWS][4];
#pragma unroll
  for (int o = 0; o < ROWS; ++o)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[o][e] = 0.f;
  // the products of 4 images are summed before they are added
#pragma unroll
  for (int n0 = 0; n0 < IMAGES; n0 += 4) {
    if (n0 >= N) break;
    float t[ROWS][4];
#pragma unroll
    for (int u = n0; u < n0 + 4; ++u) {
      float d[ROWS];
#pragma unroll
      for (int o = 0; o < ROWS; ++o) d[o] = g[u][o];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float xv = u < N ? v[u % AHEAD][e] : 0.f;
#pragma unroll
        for (int o = 0; o < ROWS; ++o) t[o][e] = fmaf(d[o], xv, u == n0 ? 0.f : t[o][e]);
      }
      if (u + AHEAD < IMAGES) load(u + AHEAD);
    }
#pragma unroll
    for (int o = 0; o < ROWS; ++o)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[o][e] += t[o][e];
  }
#pragma unroll
  for (int o = 0; o < ROWS; ++o) {
    if (o0 + o >= O) break;
    float* to = dw + (long long)(o0 + o) * F + f0;
    if (whole) {
      *reinterpret_cast<fc_f32x4u*>(to) = fc_f32x4u{acc[o][0], acc[o][1], acc[o][2], acc[o][3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f0 + e < F) to[e] = acc[o][e];
    }
  }
}

int launch_outer(const float* x, const float* dy, float* dw, float* dbias, int N, int O, int F, hipStream_t st) {
  const int rows = outer_rows(N);
  const dim3 grid((unsigned)((F + 4 * TPB - 1) / (4 * TPB)), (unsigned)((O + rows - 1) / rows)), block(TPB);
  ProfScope ps("fc_outer_kernel", 2.0 * N * (double)O * F, 4.0 * ((double)O * F + (double)N * (F + O)), st);
  if (N <= 4) hipLaunchKernelGGL(fc_outer_kernel<4>, grid, block, 0, st, x, dy, dw, dbias, N, O, F);
  else if (N <= 8) hipLaunchKernelGGL(fc_outer_kernel<8>, grid, block, 0, st, x, dy, dw, dbias, N, O, F);
  else if (N <= 16) hipLaunchKernelGGL(fc_outer_kernel<16>, grid, block, 0, st, x, dy, dw, dbias, N, O, F);
  else hipLaunchKernelGGL(fc_outer_kernel<kOuterMost>, grid, block, 0, st, x, dy, dw, dbias, N, O, F);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// dx[n][f] = sum_o dy[n][o] * w[o][f] over up to 8 images (S > 1: one of S shares of the kernels, to part): a
// workgroup owns 256 features, a lane 4 consecutive ones, its 8 waves share out the kernels; dy's values, the same for a whole
// wave, come from the lane that holds them (by scalar loads in front of every four kernels 5 to 8 images took 1.04 times
// as long).  Bound by reading w once; the kernels are split over workgroups where the features are too few to fill the
// chip.  One image of fc6 (151 MB) 38.2 us on 32-row tiles of the matrix cores behind a pack, 31.4 now; 4096 -> 1000
// 14.8 -> 11; with 16 images registers leave too few waves in flight (41 and 77).
constexpr int kRowsWaves = 8, kRowsFeatures = 256;
// Fewer kernels add every product in 64 bits, as a wave has at most 8 of them then: 2.5e-8 in the 2-norm at any number of
// kernels, where sums of four are 4.7e-8 (8 images, 32 to 256 kernels).
constexpr int kFourKernels = 64;
template <int ROWS, class Acc = double>
__global__ __launch_bounds__(64 * kRowsWaves) void fc_backward_data_few(const float* __restrict__ w, const float* __restrict__ dy,
                                                                  float* __restrict__ out, int N, int O, int F, int share) {
  __shared__ double red[kRowsWaves][kRowsFeatures];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int f0 = blockIdx.x * kRowsFeatures + lane * 4, fb = min(f0, F - 1);
  const bool whole = f0 + 4 <= F;
  const int per = (share + kRowsWaves - 1) / kRowsWaves;
  const int o_begin = blockIdx.y * share + wave * per, o_end = min(min(O, (int)(blockIdx.y + 1) * share), o_begin + per);
  Acc acc[ROWS][4];
#pragma unroll
  for (int n = 0; n < ROWS; ++n)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[n][e] = 0;
  // 4 kernels at a time: their loads in flight together, from kFourKernels on their products summed in 32 bits and all in
  // 64 (8 images of 512 -> 64: 2-norm 6.8e-8 in 32 bits, 4.8e-8 so and on the matrix cores)
  // dy's values of 64 kernels: a lane's of one each, for the whole wave by a lane's number
  float dv[ROWS], next[ROWS];
  auto load_dy = [&](float (&to)[ROWS], int o) {
#pragma unroll
    for (int n = 0; n < ROWS; ++n) to[n] = dy[(long long)min(n, N - 1) * O + min(o + lane, O - 1)];
  };
  load_dy(next, o_begin);
  for (int o = o_begin; o < o_end; o += 4) {
    const int at = (o - o_begin) & 63;
    if (at == 0) {
#pragma unroll
      for (int n = 0; n < ROWS; ++n) dv[n] = next[n];
      if (o + 64 < o_end) load_dy(next, o + 64);
    }
    auto d = [&](int n, int u) {
      return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dv[n]), at + u));
    };
    float v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* wo = w + (long long)min(o + u, o_end - 1) * F + fb;
      if (whole) {
        const fc_f32x4u q = *reinterpret_cast<const fc_f32x4u*>(wo);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = q[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = f0 + e < F ? wo[e] : 0.f;
      }
    }
    const int live = min(4, o_end - o);
    auto add = [&](auto full) {
      constexpr bool FULL = decltype(full)::value;
#pragma unroll
      for (int n = 0; n < ROWS; ++n) {
        if constexpr (FULL) {
          const float d0 = d(n, 0), d1 = d(n, 1), d2 = d(n, 2), d3 = d(n, 3);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[n][e] += fmaf(d3, v[3][e], fmaf(d2, v[2][e], fmaf(d1, v[1][e], d0 * v[0][e])));
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (u >= live) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[n][e] = fma((Acc)d(n, u), (Acc)v[u][e], acc[n][e]);
          }
        }
      }
    };
    if (live == 4 && O >= kFourKernels) add(std::integral_constant<bool, true>());
    else add(std::integral_constant<bool, false>());
  }
  // the waves' sums, a row of dx at a time
  const int t = threadIdx.x, f = blockIdx.x * kRowsFeatures + t;
  float* to = out + (long long)blockIdx.y * N * F;
#pragma unroll
  for (int n = 0; n < ROWS; ++n) {
    if (n < N) {  // the same for all
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][lane * 4 + e] = acc[n][e];
      __syncthreads();
      if (t < kRowsFeatures && f < F)
        to[(long long)n * F + f] = (float)(((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) + ((red[4][t] + red[5][t]) + (red[6][t] + red[7][t])));
      __syncthreads();
    }
  }
}

// How many workgroups share a feature's kernels: at most 1024 workgroups of at least 32 kernels, none shared where a wave's
// chain of 16 kernels is shorter than the second launch, which adds the shares.
// (5 to 8 images of 4096 and more -> 4096 and more features take 1.20 times as long as on gemm_split, 1.13 with 512 workgroups;
// their sums in 32 bits, twice as close to 64 bits as there, would be a tenth further off.)
int backward_data_few_shares(int O, int F) {
  const int blocks = (F + kRowsFeatures - 1) / kRowsFeatures;
  return O <= 128 ? 1 : std::max(1, std::min({1024 / blocks, O / 32, 64}));
}

int launch_backward_data_few(const float* w, const float* dy, float* out, int N, int O, int F, int S, hipStream_t st) {
  const int share = (O + S - 1) / S;
  const dim3 grid((unsigned)((F + kRowsFeatures - 1) / kRowsFeatures), (unsigned)((O + share - 1) / share)), block(64 * kRowsWaves);
  ProfScope ps("gemm_split_k_columns", 2.0 * N * (double)O * F, 4.0 * ((double)O * F + (double)N * (O + (double)S * F)), st);
  if (N <= 1) hipLaunchKernelGGL(fc_backward_data_few<1>, grid, block, 0, st, w, dy, out, N, O, F, share);
  else if (N <= 2) hipLaunchKernelGGL(fc_backward_data_few<2>, grid, block, 0, st, w, dy, out, N, O, F, share);
  else if (N <= 4) hipLaunchKernelGGL(fc_backward_data_few<4>, grid, block, 0, st, w, dy, out, N, O, F, share);
  // (8 rows of 64-bit sums leave too few waves in flight, fc6 38 -> 53 us; in 32 bits its error is 1.1e-7, 1.2e-7 on the matrix cores)
  else if (O < 512) hipLaunchKernelGGL(fc_backward_data_few<8>, grid, block, 0, st, w, dy, out, N, O, F, share);
  else hipLaunchKernelGGL((fc_backward_data_few<8, float>), grid, block, 0, st, w, dy, out, N, O, F, share);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// Kpad = total rows of the pack = splits * Kpad_s
int launch_fc_pack(const float* src, float* pack, int K, int M, int Kpad, int Mpad, int transposed,
                   int Ks, int Kpad_s, hipStream_t st) {
  dim3 grid((unsigned)((Mpad + 31) / 32), (unsigned)((Kpad + 31) / 32));
  if (grid.y > 65535) return CCT_EUNSUPPORTED;
  ProfScope ps("fc_pack_kernel", 0.0, 4.0 * ((double)K * M + (double)Kpad * Mpad), st);
  hipLaunchKernelGGL(fc_pack_kernel, grid, dim3(TPB), 0, st, src, pack, K, M, Kpad, Mpad, transposed,
                     Ks, Kpad_s);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

int launch_fc_sum_splits(const float* part, float* out, int S, long long total, int O,
                         const float* bias, hipStream_t st) {
  const long long blocks = (total + TPB - 1) / TPB;
  if (!grid_ok(blocks) || (bias && total >= kIntMax)) return CCT_EUNSUPPORTED;
  ProfScope ps("fc_sum_splits_kernel", 0.0, 4.0 * total * (S + 1), st);
  hipLaunchKernelGGL(fc_sum_splits_kernel, dim3((unsigned)blocks), dim3(TPB), 0, st, part, out, S,
                     total, make_fastdiv(O), bias);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace

namespace {

// The fewest splits by precision: a sum's rounding grows with the length of its chain (256 images of 9216 features, 2-norm:
// chains of 1152 products 1.6e-7, of 2304 2.3e-7).  Chains are as short as tiles of 128, 64 or 32 rows need to fill the
// chip: rounds of workgroups (512 of 128 rows, 1024 of fewer) times their stages of 32, 4 us to fill and drain a round.
double chain_seconds(int Mpad, long long tiles_n, int K, long long G) {
  int BM = Mpad % 128 == 0 && K > 128 ? 128 : Mpad % 64 == 0 ? 64 : 32;
  long long wgs = tiles_n * ((unsigned)Mpad / (unsigned)BM) * G;
  for (; BM > 32 && wgs < 256; BM /= 2) wgs *= 2;
  const int log_slots = BM == 128 ? 9 : 10, slots = 1 << log_slots;
  const double flops = BM == 128 ? 1.0 / 230.0e12 : BM == 64 ? 1.0 / 200.0e12 : 1.0 / 120.0e12;
  const double stage = 2.0 * BM * 128 * 32 * flops * slots;
  const double share = std::min(1.0, 0.3 + 0.7 * (double)((wgs + 255) >> 8) * (256.0 / slots));
  return (double)((wgs + slots - 1) >> log_slots) * ((K + 31) / 32 * stage * share + 4.0e-6);
}

// The plan on gemm_split.  The row operand (x of the forward pass, dy of the others) is packed as three bf16 terms or
// split in place, as gemm_split's estimates say; w and x are read in place.  The contraction is cut into the number of
// splits S that is estimated fastest, but for precision no fewer than chain_seconds asks for: rounds of workgroups
// times their stages, against the partial products that are written and read once more.  Measured, fc6 at batch 256
// (19.3 GFLOP per pass): forward 1 / 2 / 8 / 27 splits 320 / 175 / 113 / 148 us, backward-data 1 / 3 / 11 / 27 splits
// 163 / 116 / 137 / 181; a 4096 -> 1000 layer forward 1 / 4 / 8 splits 127 / 41 / 27.  false = sizes or a workspace that it
// cannot take, or a backward-weights pass over up to 32 images, whose product is one short stage, mostly padding.
// *estimate: its seconds; *limited: without the workspace's limit there is a faster one.
bool fc_plan_split(const cct_conv_desc_t& d, int pass, long long max_bytes, long long F, FcPlan* P, double* estimate,
                   bool* limited) {
  const long long NO = 4LL * d.N * d.O;
  const long long cap = max_bytes < 0 ? kFcMaxPartBytes : std::min(kFcMaxPartBytes, max_bytes);
  const bool fwd = pass == CCT_PASS_FORWARD, bwdw = pass == CCT_PASS_BACKWARD_WEIGHTS;
  if (bwdw && d.N <= 32) return false;
  const int M = bwdw ? d.O : d.N;                                  // rows
  const long long Kd = fwd ? F : bwdw ? d.N : d.O, cols = fwd ? d.O : F;
  const long long out = 4LL * M * cols;
  GemmTN p;
  std::memset(&p, 0, sizeof(p));
  p.M = M; p.Mpad = gemm_split_mpad(M);
  p.Ncols = (int)cols; p.b_ks = F;
  p.bmap = ColMap{kIntMax, 0};
  // A split of S, the number of them, and their workspace.  The sizes keep the form that they had when all splits
  // were equal, which callers may count on: forward a multiple of y, backward-data a number of dx that divides the
  // contraction.  The kernels need neither; up to one y, and up to twice the partial products, are spare.
  // (Kd < 2^31: 32-bit divisions, this runs for every number of splits of every call)
  auto len = [&](long long S) { return S == 1 ? Kd : align_up(((unsigned)Kd + (unsigned)S - 1) / (unsigned)S, 32); };
  auto count = [&](long long S) -> long long { return ((unsigned)Kd + (unsigned)len(S) - 1) / (unsigned)len(S); };
  auto room = [&](long long S) {
    const long long n = count(S);
    for (long long v = n; !fwd && v < 2 * n; ++v)
      if (Kd % v == 0) return v;
    return n;
  };
  auto pack = [&](long long S) {
    if (fwd && d.N <= 32) return 0LL;  // few rows: read in place by every workgroup
    const long long bytes = 6LL * count(S) * p.Mpad * gemm_split_kpad((int)len(S));
    // forward: whole multiples of y, like the partial products behind it
    return fwd ? (bytes + NO - 1) / NO * NO : align_up(bytes, kAlign);
  };
  auto need = [&](long long S) {
    return align_up(pack(S) + (count(S) > 1 ? room(S) * out : 0), kAlign) +
           (bwdw ? align_up(4LL * d.O * kDbiasBlocks, kAlign) : 0);
  };
  auto seconds = [&](long long S) {
    const long long n = count(S);
    return gemm_split_seconds(fwd, !fwd || d.N > 32, M, (int)len(S), cols, n) +
           (n > 1 ? 2.0 * n * out / 5.5e12 + 2.5e-6 : 0.0);
  };
  long long S = 1;
  double best = 1e30;
  *limited = false;
  auto each = [&](auto visit) {
    visit(1LL);
    for (int sp = 2; sp <= 64 && Kd >= (long long)sp * kFcMinSplitRows; sp += sp < 16 ? 1 : 4) visit((long long)sp);
  };
  auto choose = [&](long long most) {
    long long least = 1;
    double shortest = 1e30;
    each([&](long long sp) {
      const long long n = count(sp);
      const double t = chain_seconds(p.Mpad, (cols + 127) / 128, (int)len(sp), n) + (n > 1 ? 2.0 * n * out / 6.0e12 : 0.0);
      if (t >= shortest) return;
      if (need(sp) <= most) {
        shortest = t;
        least = sp;
      } else {
        *limited = true;
      }
    });
    S = least;
    best = 1e30;
    each([&](long long sp) {
      if (sp < least || need(sp) > most) return;
      const double t = seconds(sp);
      if (t >= best) return;
      best = t;
      S = sp;
    });
  };
  // The recommended plan wherever it fits: fewer splits may need more room than it does, and must not turn it down then.
  if (!bwdw) choose(kFcMaxPartBytes);
  *limited = false;
  if (!bwdw && max_bytes >= 0 && need(S) > max_bytes) choose(cap);
  *estimate = best;
  if (max_bytes >= 0 && need(S) > max_bytes) return false;
  p.Kdim = (int)len(S); p.Kpad = gemm_split_kpad(p.Kdim);
  if (!gemm_split_fits(p, fwd)) return false;
  P->split = 1;
  P->split_len = p.Kdim;
  P->S = (int)count(S);
  P->Mpad = p.Mpad;
  P->Kpad = p.Kpad;
  P->pack_off = 0;
  P->part_off = pack(S);
  P->scratch_off = pack(S);  // backward-weights: no partial products
  P->total = std::max<long long>(need(S), kAlign);
  return true;
}

GemmTN fc_split_problem(const FcPlan& P, int M, int Ncols, const float* B, float* C) {
  GemmTN p;
  std::memset(&p, 0, sizeof(p));
  p.Mpad = P.Mpad; p.Kpad = P.Kpad;
  p.B = B; p.b_ks = P.F;
  p.bmap = ColMap{kIntMax, 0};
  p.C = C; p.c_ms = Ncols; p.c_gs = (long long)M * Ncols;
  p.cmap = ColMap{kIntMax, 0};
  p.M = M; p.Ncols = Ncols; p.Kdim = P.split_len; p.G = P.S;
  return p;
}

}  // namespace

// The plan on the fp32 matrix instructions.
namespace {
bool fc_plan_f32(const cct_conv_desc_t& d, int pass, long long max_bytes, long long F, FcPlan* P, double* estimate) {
  long long off = 0;
  auto take = [&](long long bytes, long long* o) {
    *o = off;
    off += align_up(bytes, kAlign);
  };
  int BM, BN, BK;
  if (pass == CCT_PASS_FORWARD) {
    // the split product reads whole K tiles of both operands without column guards
    gemm_nt_tile(d.N, d.O, &BM, &BN, &BK);
    if (F % BK) return false;
    const long long tiles = (long long)((d.N + BM - 1) / BM) * ((d.O + BN - 1) / BN);
    long long S = std::max<long long>(1, std::min<long long>((kFcTargetBlocks + tiles - 1) / tiles,
                                                             F / kFcMinSplit));
    // fewer, longer splits when the partial products would not fit
    const long long cap = max_bytes < 0 ? kFcMaxPartBytes : std::min(kFcMaxPartBytes, max_bytes);
    long long smax = cap / (4LL * d.N * d.O);
    while (smax > 1 && align_up(4LL * smax * d.N * d.O, kAlign) > cap) --smax;
    S = std::min(S, std::max<long long>(1, smax));
    P->split_len = (int)align_up((F + S - 1) / S, BK);
    P->S = (int)((F + P->split_len - 1) / P->split_len);
    take(4LL * P->S * d.N * d.O, &P->part_off);
  } else if (pass == CCT_PASS_BACKWARD_DATA) {
    // rows = images.  Too few tiles to fill the chip: 64-row tiles, and the contraction split into
    // S equal parts (the smallest divisor S of O that gives kFcFillBlocks workgroups, else the
    // largest one with parts of at least kFcMinSplitRows kernels) whose partial products are summed
    // afterwards.  Measured on fc6 at batch 256 (19.3 GFLOP): unsplit 0.33 ms, 4 splits of 128-row
    // tiles 0.24 ms, 4 splits of 64-row tiles 0.22 ms.
    gemm_tn_tile(d.N, (int)F, &BM, &BN, &BK);
    if (BM == 128 && d.N % 64 == 0 && (long long)((d.N + 127) / 128) * ((F + BN - 1) / BN) < 512) BM = 64;
    const long long tiles = (long long)((d.N + BM - 1) / BM) * ((F + BN - 1) / BN);
    const long long cap = max_bytes < 0 ? kFcMaxPartBytes : std::min(kFcMaxPartBytes, max_bytes);
    // workspace of a plan with sp splits: the packed dy and, when split, the partial products
    auto need = [&](long long sp) {
      const long long pack = 4LL * sp * align_up(d.O / sp, BK) * align_up(d.N, BM);
      return align_up(pack, kAlign) + (sp > 1 ? align_up(4LL * sp * d.N * F, kAlign) : 0);
    };
    int S = 1;
    for (int sp = 2; sp <= 64 && tiles * S < kFcFillBlocks; ++sp)
      if (d.O % sp == 0 && d.O / sp >= kFcMinSplitRows && need(sp) <= cap) S = sp;
    P->BM = BM;
    P->S = S;
    P->split_len = d.O / S;
    P->Mpad = (int)align_up(d.N, BM);
    P->Kpad = (int)align_up(P->split_len, BK);   // rows of one split
    take(4LL * S * P->Kpad * P->Mpad, &P->pack_off);
    if (S > 1) take(4LL * S * d.N * F, &P->part_off);
  } else {
    gemm_tn_tile(d.O, (int)F, &BM, &BN, &BK);
    P->BM = BM;
    P->Mpad = (int)align_up(d.O, BM);
    P->Kpad = (int)align_up(d.N, BK);
    P->S = 1;
    take(4LL * P->Kpad * P->Mpad, &P->pack_off);
    take(4LL * d.O * kDbiasBlocks, &P->scratch_off);
  }
  P->total = std::max<long long>(off, kAlign);
  // Rounds of 512 workgroups at 110 TFLOP/s.  Forward: up to one per CU, a workgroup takes 0.6 of the time it takes
  // beside another (37 images, 4640 features, 3076 kernels, 4 splits: 50 us).  Backward-data: 1.2 in any number (12
  // images, 5184 features, 359 kernels: 37 us; 458, 1728 and 1556: 77).
  const long long rows = pass == CCT_PASS_BACKWARD_WEIGHTS ? d.O : d.N, cols = pass == CCT_PASS_FORWARD ? d.O : F;
  const long long len = pass == CCT_PASS_BACKWARD_WEIGHTS ? d.N : P->split_len;
  const long long wgs = ((rows + BM - 1) / BM) * ((cols + BN - 1) / BN) * P->S;
  *estimate = (double)((wgs + 511) / 512) * 2.0 * BM * BN * (double)len / (110.0e12 / 512) * (pass == CCT_PASS_BACKWARD_DATA ? 1.2 : wgs <= 256 ? 0.6 : 1.0) +
              (P->S > 1 ? 8.0 * P->S * rows * cols / 6.0e12 : 0.0);
  return max_bytes < 0 || P->total <= max_bytes;
}
}  // namespace

bool fc_plan(const cct_conv_desc_t& d, int pass, long long max_bytes, FcPlan* P) {
  if (d.K != d.H || d.K != d.W || d.pad != 0 || d.groups != 1) return false;
  if (d.precision != CCT_PREC_F32) return false;
  if (d.lowering != CCT_LOWER_AUTO && d.lowering != CCT_LOWER_TYPE1) return false;
  const long long F = (long long)d.C * d.K * d.K;
  if (F >= kIntMax - 256 || (long long)d.N * d.O >= kIntMax || (long long)d.N * F >= (1LL << 40) ||
      (long long)d.O * F >= (1LL << 40))
    return false;
  std::memset(P, 0, sizeof(*P));
  P->F = (int)F;
  // Fewer splits than are worth it, because their partial products and the packed operand (1.5 times the fp32
  // one) do not fit: the fp32 plan may split more (37 images, 4640 features, 3076 kernels in a quarter of the
  // workspace: 150 us unsplit, 52 with four fp32 splits).
  FcPlan f32 = *P;
  double split_seconds, f32_seconds;
  bool limited;
  if (!fc_plan_split(d, pass, max_bytes, F, P, &split_seconds, &limited))
    return fc_plan_f32(d, pass, max_bytes, F, P, &f32_seconds);
  if (limited && max_bytes >= 0 && fc_plan_f32(d, pass, max_bytes, F, &f32, &f32_seconds) && f32_seconds < split_seconds)
    *P = f32;
  return true;
}

int fc_forward(const cct_conv_desc_t& d, const FcPlan& P, const float* x, const float* w,
               const float* bias, float* y, char* ws, hipStream_t st) {
  if (P.F % 32 == 0 && reinterpret_cast<uintptr_t>(w) % 16) return CCT_EINVAL;
  if (P.split && forward_few_fits(d.N, d.O, P.F))
    return launch_forward_few(x, w, bias, y, d.N, d.O, P.F, st);
  if (P.split) {
    void* pack = ws + P.pack_off;
    float* part = reinterpret_cast<float*>(ws + P.part_off);
    GemmTN p = fc_split_problem(P, d.N, d.O, w, P.S > 1 ? part : y);
    int rc = gemm_split_operand(&p, true, x, d.N <= 32 ? nullptr : pack, P.F, P.F, 1, P.split_len, 1, st);
    if (rc) return rc;
    p.b_gs = P.split_len;
    if (P.S == 1) {
      p.bias = bias; p.bias_gs = -1;
    }
    rc = launch_gemm_split(p, P.F, true, st);
    if (rc || P.S == 1) return rc;
    return launch_fc_sum_splits(part, y, P.S, (long long)d.N * d.O, d.O, bias, st);
  }
  GemmNT q;
  std::memset(&q, 0, sizeof(q));
  q.A = x; q.a_ms = P.F;
  q.amap = ColMap{kIntMax, 0};
  q.B = w; q.b_ns = P.F;
  q.Cpart = reinterpret_cast<float*>(ws + P.part_off);
  q.M = d.N; q.N = d.O; q.Ncols = P.F;
  q.G = 1; q.S = P.S; q.split_len = P.split_len;
  int rc = launch_gemm_nt(q, st);
  if (rc) return rc;
  return launch_fc_sum_splits(q.Cpart, y, P.S, (long long)d.N * d.O, d.O, bias, st);
}

int fc_backward_data(const cct_conv_desc_t& d, const FcPlan& P, const float* w, const float* dy,
                     float* dx, char* ws, hipStream_t st) {
  if (P.split && d.N <= 8) {
    // the shares whose partial products the plan's workspace holds
    const long long out = 4LL * d.N * P.F;
    int S = backward_data_few_shares(d.O, P.F);
    if (S > 1) S = (int)std::max(1LL, std::min<long long>(S, P.total / out));
    const int share = (d.O + S - 1) / S;
    S = (d.O + share - 1) / share;
    float* part = reinterpret_cast<float*>(ws);
    const int rc = launch_backward_data_few(w, dy, S > 1 ? part : dx, d.N, d.O, P.F, S, st);
    if (rc || S == 1) return rc;
    return launch_fc_sum_splits(part, dx, S, (long long)d.N * P.F, 1, nullptr, st);
  }
  if (P.split) {
    void* pk = ws + P.pack_off;
    float* part = reinterpret_cast<float*>(ws + P.part_off);
    GemmTN p = fc_split_problem(P, d.N, P.F, w, P.S > 1 ? part : dx);
    int rc = gemm_split_operand(&p, false, dy, pk, d.O, d.O, 1, P.split_len, 1, st);
    if (rc) return rc;
    p.b_gs = (long long)P.split_len * P.F;
    rc = launch_gemm_split(p, d.O, false, st);
    if (rc || P.S == 1) return rc;
    return launch_fc_sum_splits(part, dx, P.S, (long long)d.N * P.F, 1, nullptr, st);
  }
  float* pack = reinterpret_cast<float*>(ws + P.pack_off);
  // pack[s][oo][n] = dy[n][s*split_len + oo]
  int rc = launch_fc_pack(dy, pack, d.O, d.N, P.S * P.Kpad, P.Mpad, 1, P.split_len, P.Kpad, st);
  if (rc) return rc;
  float* part = reinterpret_cast<float*>(ws + P.part_off);
  GemmTN p;
  std::memset(&p, 0, sizeof(p));
  p.A = pack;
  p.a_gs = (long long)P.Kpad * P.Mpad;
  p.Mpad = P.Mpad; p.Kpad = P.Kpad;
  p.B = w; p.b_ks = P.F;
  p.b_gs = (long long)P.split_len * P.F;     // a split = the next split_len kernels
  p.bmap = ColMap{kIntMax, 0};
  p.b_ld_guard = P.F % 128 == 0 ? P.F : 0;   // whole column tiles can be read as vectors
  p.C = P.S > 1 ? part : dx;
  p.c_ms = P.F;
  p.c_gs = (long long)d.N * P.F;
  p.cmap = ColMap{kIntMax, 0};
  p.M = d.N; p.Ncols = P.F; p.Kdim = P.split_len; p.G = P.S;
  p.force_bm = P.BM;
  rc = launch_gemm_tn(p, st);
  if (rc || P.S == 1) return rc;
  return launch_fc_sum_splits(part, dx, P.S, (long long)d.N * P.F, 1, nullptr, st);
}

namespace {
// The product on the fp32 matrix instructions, for workspaces that hold dy once.
int fc_weights_f32(const cct_conv_desc_t& d, const FcPlan& P, const float* x, const float* dy, float* dw,
                   float* pack, hipStream_t st) {
  int rc = launch_fc_pack(dy, pack, d.N, d.O, P.Kpad, P.Mpad, 0, d.N, P.Kpad, st);  // pack[n][o] = dy[n][o]
  if (rc) return rc;
  GemmTN p;
  std::memset(&p, 0, sizeof(p));
  p.A = pack;
  p.Mpad = P.Mpad; p.Kpad = P.Kpad;
  p.B = x; p.b_ks = P.F;
  p.bmap = ColMap{kIntMax, 0};
  p.b_ld_guard = P.F % 128 == 0 ? P.F : 0;
  p.C = dw; p.c_ms = P.F;
  p.cmap = ColMap{kIntMax, 0};
  p.M = d.O; p.Ncols = P.F; p.Kdim = d.N; p.G = 1;
  p.force_bm = P.BM;
  return launch_gemm_tn(p, st);
}

}  // namespace

int fc_backward_weights(const cct_conv_desc_t& d, const FcPlan& P, const float* x, const float* dy,
                        float* dw, float* dbias, char* ws, hipStream_t st) {
  float* pack = reinterpret_cast<float*>(ws + P.pack_off);
  int rc;
  const long long oy = ((long long)d.O + outer_rows(d.N) - 1) / outer_rows(d.N);
  if (!P.split && (d.N <= 16 || (d.N <= 32 && (long long)d.O * P.F <= (1LL << 22))) && oy <= 65535)
    return launch_outer(x, dy, dw, dbias, d.N, d.O, P.F, st);
  if (P.split) {
    GemmTN p = fc_split_problem(P, d.O, P.F, x, dw);
    rc = gemm_split_operand(&p, false, dy, pack, d.N, 1, d.O, 0, 1, st);
    if (rc) return rc;
    rc = launch_gemm_split(p, d.N, false, st);
  } else {
    rc = fc_weights_f32(d, P, x, dy, dw, pack, st);
  }
  if (rc) return rc;
  if (dbias) {
    const int nblk = std::max(1, std::min({d.N, kDbiasBlocks, (2048 + d.O - 1) / d.O}));
    rc = launch_dbias(dy, dbias, reinterpret_cast<float*>(ws + P.scratch_off), d.N, d.O, 1, nblk, st);
  }
  return rc;
}

}  // namespace cct
