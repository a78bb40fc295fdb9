// Backward-weights pass of layers with few channels (the first layer of a network) on the bf16 matrix cores, fp32
// operands as three bf16 terms (split_bf16.h): x and dy read in place, once, no granules in memory.
//
//     dw[o][(i,j,ci)] = sum_{n, r, c} dy[n, o, r, c] * xpad[n, ci, r*s + i, c*s + j]
//
// As in conv_bwdw_img 8 images at one pixel are the 8 consecutive reduction indices of a lane, so that every tap is
// aligned.  There the granules go through memory, 32 channels at a time; with 3 channels that is eleven times the
// products.  Here a workgroup owns ALL taps of all channels (up to 384 columns) and BM kernels, and builds the
// granules in LDS: it takes 8 images and a strip of 8 output columns and walks down the output rows.  Per output row it
// stages dy's 8 positions (two slots) and the stride's worth of new input rows (a ring of K + stride rows); the loads
// of the row after next are in flight meanwhile, and splitting is written between the MFMAs.  The neighbouring strips of the
// same images run next to it on the same XCD: they share the lines of dy and x through L2.
//   - a wave owns all rows of CB blocks of 16 columns; an MFMA (16x16x32) takes four positions;
//   - granules of x lie as [ring row][column][channel][term], 48 bytes from one to the next, those of dy as
//     [position][term][kernel]: reads of consecutive columns or rows do not conflict.
// The bias gradient is summed from the values that are staged anyway.  Partial sums go to bwdw_img_reduce.
//
// Bound by the matrix cores at the clock the card holds under it (MfmaUtil 55 % at 1.83 GHz, LDS a third busy) and
// by what stands still at the ends of a row's stage: 224 workgroups, 5.4 us per row and workgroup, of it 3.0 MFMAs.
// CaffeNet's first layer at batch 256 with its bias gradient: gather-fed fp32 matrix product 600 us, reduction 12,
// bias gradient 65 before; 278 and 10 now.  388 layers of 1 to 16 channels per group: 0.66 times the time in the mean.
// Tried: rows of all strips shared evenly over 256 workgroups instead of strips on 224 (conv1 1119 -> 1289 us: the strips
// of the same images no longer run side by side, and dy's lines are fetched for every strip).
#include <algorithm>
#include <climits>

#include "cct_internal.h"
#include "gemm_common.h"
#include "split_bf16.h"

namespace cct {
namespace {

constexpr int kImg = 8;   // images per granule
constexpr int kPos = 8;   // output columns of a strip
constexpr int NT = 512;
constexpr long long kPartialBytes = 256LL << 20;  // of the partial sums of a launch
constexpr int kCell = 48;  // bytes of a granule's three terms

struct Few {
  const float *x, *dy;
  float* part;  // [S][G][Og][N], n = (tap, channel), scaled as they are
  float* sums;  // [S][O], or null
  int N, Cg, Og, C, O, H, W, Hout, Wout, K, s, pad, G, nimg;
  int strips, segs, seg_rows, S, tiles_m;
  int WX, ring, row_b;  // staged columns, ring rows and their bytes
};

// (narrow tiles: two workgroups per CU where LDS allows it, as the plan counts on)
template <int RB, int CB>
__global__ __launch_bounds__(NT, RB * CB <= 6 && CB < 3 ? 4 : 2) void conv_bwdw_few(Few p) {
  constexpr int BM = 16 * RB;
  constexpr int UD = (BM * kPos + NT - 1) / NT;  // granules of dy per thread and stage
  constexpr int PH = UD + 1;                     // and one of x
  constexpr int DPOS = (3 * BM + 1) * 16;        // bytes between positions: writes of 8 positions do not conflict
  constexpr int DSLOT = kPos * DPOS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_f[];
  unsigned char* Ds = smem_f;
  double* Bs = reinterpret_cast<double*>(smem_f + 2 * DSLOT);  // the bias gradient by kernel and pair of positions
  unsigned char* Xs = smem_f + 2 * DSLOT + BM * kPos * 4;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = lane & 15, kg = lane >> 4;

  int idx = blockIdx.x;
  {
    const int total = p.tiles_m * p.S;
    const int per = total >> 3, rem = total & 7;
    const int xcd = idx & 7;
    idx = xcd * per + min(xcd, rem) + (idx >> 3);
  }
  const int s = idx / p.tiles_m, m0 = (idx - s * p.tiles_m) * BM;
  const int g = blockIdx.y;
  const int is = s / p.strips, strip = s - is * p.strips, ig = is / p.segs, seg = is - ig * p.segs;
  const int r0 = seg * p.seg_rows, r1 = min(p.Hout, r0 + p.seg_rows), c0 = strip * kPos;
  const int nv = min(kImg, p.nimg - ig * kImg);

  // images past the last one lie beyond the range and load as zeros
  const long long x_img = (long long)p.C * p.H * p.W, y_img = (long long)p.O * p.Hout * p.Wout;
  const int plane = p.H * p.W, P = p.Hout * p.Wout;
  const unsigned xi_b = (unsigned)x_img * 4u, yi_b = (unsigned)y_img * 4u;
  const __amdgpu_buffer_rsrc_t x_rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.x + ig * kImg * x_img + (long long)g * p.Cg * plane), 0,
      (int)((nv - 1) * xi_b + (unsigned)(p.Cg * plane) * 4u), 0x00020000);
  const __amdgpu_buffer_rsrc_t y_rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.dy + ig * kImg * y_img + (long long)g * p.Og * P), 0,
      (int)((nv - 1) * yi_b + (unsigned)(p.Og * P) * 4u), 0x00020000);
  constexpr unsigned kDead = 0x80000000u;

  // ---- dy: granule q = tid + 512 u is (kernel q / 8, position q % 8).  Kernels past the last one read what lies there
  // (their results are not stored), positions past the last one are zero.
  // (what follows from the thread alone is computed where it is needed: there is no register to keep it)
  auto mine = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  auto y_voff = [&]() {
    const int t = mine();
    return c0 + (t & 7) < p.Wout ? (unsigned)((m0 + (t >> 3)) * P + c0 + (t & 7)) * 4u : kDead;
  };
  auto y_lds = [&]() {
    const int t = mine();
    return (t & 7) * DPOS + (t >> 3) * 16;
  };
  const unsigned y_next = (unsigned)(NT / kPos * P) * 4u;
  auto y_mine = [&](int u) { return wave * 64 + u * NT < BM * kPos; };
  // ---- x: the new rows of a stage, granule tid is (channel, row, column), columns fastest
  const int cells = p.WX * p.Cg;                // granules of a ring row
  const int xcol = tid % p.WX, xt = tid / p.WX, xrow = xt % p.s, xc = xt / p.s;
  const bool x_live = xc < p.Cg;
  const int xw = c0 * p.s - p.pad + xcol;
  const unsigned x_voff = x_live && xw >= 0 && xw < p.W ? (unsigned)(xc * plane + xw) * 4u : kDead;

  float raw[PH][kImg];
  // (the range is checked against the vector offset alone; the sums are not kept in registers between the stages)
  auto load_y = [&](float (&v)[kImg], int u, int r) {
    unsigned yi = yi_b, row = u * y_next + (unsigned)(r * p.Wout) * 4u;
    asm volatile("" : "+s"(yi), "+s"(row));
    const unsigned vo = y_voff() + row;
#pragma unroll
    for (int e = 0; e < kImg; ++e)
      v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(y_rs, (int)(vo + e * yi), 0, 0));
  };
  // row h of the padded tensor
  auto load_x = [&](float (&v)[kImg], unsigned voff, int h) {
    const int hh = h - p.pad;
    const unsigned vo = voff != kDead && hh >= 0 && hh < p.H ? voff + (unsigned)(hh * p.W) * 4u : kDead;
    unsigned xi = xi_b;
    asm volatile("" : "+s"(xi));
#pragma unroll
    for (int e = 0; e < kImg; ++e)
      v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(x_rs, (int)(vo + e * xi), 0, 0));
  };
  auto split8 = [](const float (&v)[kImg], u32x4 (&q)[3]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned h, m, l;
      split_pair(v[2 * e], v[2 * e + 1], &h, &m, &l);
      q[0][e] = h;
      q[1][e] = m;
      q[2][e] = l;
    }
  };
  auto put = [](unsigned char* at, int term, const u32x4 (&q)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4*>(at + k * term) = q[k];
  };
  // The bias gradient's part of a granule: 8 images of two positions in a tree, added up over the rows in 64 bits.  In 32
  // bits, a position's chain of rows by itself, the sum's error was up to 1.8 times that of the bias gradient's own kernel, in
  // a quarter of 2900 layers more than 5 % above it (2-norm, geometric mean 1.28e-7 there, 1.17e-7 so, 9.5e-8 now).
  auto add_sum = [&](const float (&v)[kImg], int u, bool first) {
    float own = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    own += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, own), 0xb1, 0xf, 0xf, true));  // the neighbour's
    double* at = Bs + u * (NT / 2) + mine() / 2;  // of both, with the same sum: no branch between the MFMAs
    *at = first ? (double)own : *at + own;
  };
  // ---- the first stage: all K rows of x
  {
    const int all = p.K * cells;
    for (int q = tid; q < all; q += NT) {
      const int col = q % p.WX, t = q / p.WX, row = t % p.K, c = t / p.K;
      const int w = c0 * p.s - p.pad + col, h = r0 * p.s + row;
      float v[kImg];
      load_x(v, w >= 0 && w < p.W ? (unsigned)(c * plane + w) * 4u : kDead, h);
      u32x4 t3[3];
      split8(v, t3);
      put(Xs + (h % p.ring) * p.row_b + (col * p.Cg + c) * kCell, 16, t3);
    }
#pragma unroll
    for (int u = 0; u < UD; ++u) {
      load_y(raw[0], u, r0);
      if (y_mine(u)) add_sum(raw[0], u, true);
      u32x4 t3[3];
      split8(raw[0], t3);
      if (y_mine(u)) put(Ds + y_lds() + u * (NT / kPos * 16), BM * 16, t3);
    }
  }
  const int last = r1 - 1;
  const int x_ahead = p.K - p.s + xrow;  // the thread's new row of a stage, from the stage's first
  // A stage is staged in PH phases: dy's granules of a thread, then that of x
  auto load_phase = [&](float (&v)[kImg], int f, int r, int row) {
    if (f < UD) load_y(v, f, min(r, last));
    else load_x(v, x_voff, min(r, last) * p.s + row);
  };
#pragma unroll
  for (int f = 0; f < PH; ++f) load_phase(raw[f], f, r0 + 1, x_ahead);

  // ---- operands: where a lane's columns begin, in the stage's ring rows
  const int row_b = p.row_b, ring_b = p.ring * row_b;
  const int base = (r0 * p.s) % p.ring;  // ring row of the first stage's first row
  auto wrap = [&](int at) { return at >= ring_b ? at - ring_b : at; };
  int b_at[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int n = min((wave * CB + j) * 16 + lo, p.N - 1), tap = n / p.Cg, c = n - tap * p.Cg, i = tap / p.K;
    b_at[j] = wrap((base + i) * row_b + ((tap - i * p.K + kg * p.s) * p.Cg + c) * kCell);
  }
  // where this thread's next row of x goes, and which row of a stage it is, in one register
  int x_to = wrap(wrap((base + p.K + xrow) * row_b + (xcol * p.Cg + xc) * kCell)) << 8 | x_ahead;
  const int a_lds = kg * DPOS + lo * 16;
  const int step_b = 4 * p.s * p.Cg * kCell;

  f32x4 acc_h[RB][CB], acc_c[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc_h[i][j][r] = acc_c[i][j][r] = 0.f;
  u32x4 a[3], b[CB][3];
  u32x4 q[3];
  float ra = 0.f, rb = 0.f;

  for (int r = r0; r < r1; ++r) {
    const int slot = (r - r0) & 1;
    __syncthreads();  // this stage's granules are visible, nobody reads those before them any more
    auto read_a = [&](int ks, int i, int k) {
      a[k] = *reinterpret_cast<const u32x4*>(Ds + slot * DSLOT + a_lds + ks * 4 * DPOS + (k * BM + i * 16) * 16);
    };
    auto read_b = [&](int ks, int j, int k) {
      b[j][k] = *reinterpret_cast<const u32x4*>(Xs + b_at[j] + ks * step_b + k * 16);
    };
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      read_a(0, 0, k);
#pragma unroll
      for (int j = 0; j < CB; ++j) read_b(0, j, 2 - k);
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int TOTAL = 2 * RB * CB * 6, SPAN = TOTAL / PH;  // MFMAs, and of them for a phase of staging
    constexpr int PER = SPAN >= 18 ? 1 : SPAN >= 10 ? 2 : 4;  // steps behind an MFMA
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const bool end = i == RB - 1;
        auto mfma = [&](int k, int x, int y, f32x4 (&acc)[CB]) {
#pragma unroll
          for (int j = 0; j < CB; ++j) {
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[x]),
                                                             __builtin_bit_cast(bf16x8, b[j][y]), acc[j], 0, 0, 0);
            const int at = (ks * RB + i) * CB * 6 + k * CB + j, f = at / SPAN, n = at - f * SPAN;
            if (f < PH) {
              float (&v)[kImg] = raw[f < PH ? f : 0];
              if (n == 16 / PER) {
                unsigned char* to = f < UD ? Ds + (slot ^ 1) * DSLOT + y_lds() + f * (NT / kPos * 16) : Xs + (x_to >> 8);
                if (f < UD ? y_mine(f) : x_live) put(to, f < UD ? BM * 16 : 16, q);
              }
              if (n * PER < 16)
#pragma unroll
                for (int e = 0; e < PER; ++e) split_quarter(v, q, n * PER + e, ra, rb);
              if (n == 16 / PER) {  // the buffer is free
                if (f < UD && r + 1 < r1 && y_mine(f)) add_sum(v, f, false);
                load_phase(v, f, r + 2, x_to & 255);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        auto next_a = [&](int k) {
          if (!end) read_a(ks, i + 1, k);
          else if (ks == 0) read_a(1, 0, k);
        };
        // every operand is read three products or two before it is needed, into the registers that its predecessor leaves
        auto next_b = [&](int k) {
          if (!end || ks == 1) return;
#pragma unroll
          for (int j = 0; j < CB; ++j) read_b(1, j, k);
        };
        mfma(0, 0, 2, acc_c[i]);
        next_b(2);
        mfma(1, 0, 1, acc_c[i]);
        mfma(2, 0, 0, acc_h[i]);
        next_a(0);
        mfma(3, 1, 1, acc_c[i]);
        next_b(1);
        mfma(4, 1, 0, acc_c[i]);
        next_a(1);
        mfma(5, 2, 0, acc_c[i]);
        next_a(2);
        next_b(0);
      }
    const int down = p.s * row_b;
#pragma unroll
    for (int j = 0; j < CB; ++j) b_at[j] = wrap(b_at[j] + down);
    x_to += down << 8;
    x_to -= x_to >= ring_b << 8 ? ring_b << 8 : 0;
  }

  float* __restrict__ C = p.part + ((long long)s * p.G + g) * p.Og * p.N;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + i * 16 + kg * 4 + r, n = (wave * CB + j) * 16 + lo;
        if (m < p.Og && n < p.N) C[(long long)m * p.N + n] = acc_h[i][j][r] + acc_c[i][j][r];
      }
  if (!p.sums) return;
  __syncthreads();
  if (wave * 64 >= BM * kPos / 2) return;
  double v = Bs[tid];
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  const int o = tid >> 2;
  if ((tid & 3) == 0 && m0 + o < p.Og) p.sums[(long long)s * p.O + g * p.Og + m0 + o] = (float)v;
}

template <int RB, int CB>
int launch_few(const Few& p, size_t lds, hipStream_t st) {
  constexpr auto kern = conv_bwdw_few<RB, CB>;
  if (const int rc = ensure_dynamic_lds<kern>(160 * 1024)) return rc;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.S * p.tiles_m), (unsigned)p.G), dim3(NT), lds, st, p);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// us: what a round of workgroups takes per output row, and per row and block of 16 x 16 results for every workgroup on a
// CU; to fill and drain, and that per block; bytes per us of the partial sums, twice; the launches.  Fitted to 388 layers of
// 1 to 16 channels per group (1 to 700 images, K = 3 to 11): off by 7 % in the mean, 15 % in nine of ten.
constexpr double kRowUs = 1.17, kBlockUs = 0.216, kFillUs = 7.1, kFillBlockUs = 0.2, kPartialRate = 5.27e6, kLaunchUs = 0.8;

inline int column_blocks(long long N) { return (int)((N + 127) / 128); }

// Bytes of a ring row: the first tap of a kernel's next row continues the last one's walk over the banks
inline int row_bytes(int WX, int Cg, int K) { return WX * Cg * kCell + ((K - WX) * Cg * 3 & 7) * 16; }

// LDS of a workgroup with rows of 16 * rb kernels
inline long long lds_bytes(int rb, int ring, int row_b) {
  return 2LL * kPos * (3 * 16 * rb + 1) * 16 + 16LL * rb * kPos * 4 + (long long)ring * row_b;
}

}  // namespace

bool bwdw_few_plan(const cct_conv_desc_t& d, long long nimg, BwdwFewPlan* P) {
  const long long Hout = (d.H + 2LL * d.pad - d.K) / d.stride + 1, Wout = (d.W + 2LL * d.pad - d.K) / d.stride + 1;
  const int Cg = d.C / d.groups, Og = d.O / d.groups, s = d.stride;
  const long long N = (long long)Cg * d.K * d.K;
  if (d.precision != CCT_PREC_F32 || d.K > 64 || s > d.K || N > 384 || Cg > 32) return false;
  const int WX = (kPos - 1) * s + d.K, ring = d.K + s;
  if ((long long)s * WX * Cg > NT) return false;  // a granule of x per thread and stage
  // 32-bit byte offsets from the first of 8 images, rows of a tile past the last kernel among them
  const long long xi = (long long)d.C * d.H * d.W, yi = (long long)d.O * Hout * Wout;
  if (kImg * xi >= (1LL << 28) || kImg * yi + 96 * Hout * Wout >= (1LL << 28) || d.W + 2LL * d.pad >= (1LL << 20)) return false;
  P->cb = column_blocks(N);
  const long long strips = (Wout + kPos - 1) / kPos, out = 4LL * d.O * N;
  auto tiles_of = [&](int rb) { return (Og + 16 * rb - 1) / (16 * rb); };
  auto count = [&](long long images, long long segs) { return (images + kImg - 1) / kImg * strips * segs; };
  double best = 0.0;
  // Segments of the output rows, from the whole batch: what the rounds of workgroups (one per CU, or two where registers
  // and LDS allow it) are estimated to take, partial sums within 256 MiB.
  auto consider = [&](int rb) {
    const int blocks = rb * P->cb;
    const long long lds = lds_bytes(rb, ring, row_bytes(WX, Cg, d.K));
    if (lds > 160 * 1024) return;
    const int per_cu = blocks <= 6 && P->cb < 3 && lds <= 80 * 1024 ? 2 : 1;
    for (long long n = 1; n <= std::min(Hout, 64LL); ++n) {
      const long long rows = (Hout + n - 1) / n, segs = (Hout + rows - 1) / rows, S = count(d.N, segs);
      if (n > 1 && S * out > kPartialBytes) break;
      const long long wgs = S * tiles_of(rb) * d.groups, full = 256 * per_cu, rest = wgs % full;
      auto round = [&](int on) { return rows * (kRowUs + kBlockUs * blocks * on) + (kFillUs + kFillBlockUs * blocks) * on; };
      const double us = (double)(wgs / full) * round(per_cu) + (rest > 256 ? round(2) : rest ? round(1) : 0.0) +
                        2.0 * (double)(S * out) / kPartialRate;
      if (best == 0.0 || us < best) {
        best = us;
        P->rb = rb;
        P->lds = lds;
        P->segs = (int)segs;
        P->seg_rows = (int)rows;
      }
    }
  };
  consider(Og > 64 ? 6 : Og > 32 ? 4 : 2);
  // A few kernels past 96: two tiles of 64 instead of two of 96 (700 such layers 0.76 times the time, 0.93 at most; before,
  // they were the ones that took up to 1.15 times as long as without this kernel: 47 images of 97 x 96, two groups of 14 -> 100
  // channels, 3 x 3, 387 us for 335).  193 to 256 in four tiles instead of three still gain (464 layers, 0.83) and stay.
  if (Og > 96 && Og <= 128) consider(4);
  if (best == 0.0) return false;
  const long long tiles = tiles_of(P->rb);
  // The whole batch in one launch where its partial sums are no more than that, else as many images at a time as are (batch
  // 4096 of CaffeNet's first layer: 477 MiB)
  const long long eight = count(kImg, P->segs) * out;
  if (eight > kPartialBytes) return false;
  P->images = (int)std::min<long long>(kPartialBytes / eight * kImg, INT_MAX / kImg * kImg);
  const long long S = count(std::min<long long>(nimg, P->images), P->segs);
  if (S * tiles >= (1LL << 30) || S * d.O >= (1LL << 30) || d.groups > 65535) return false;
  P->S = (int)S;
  P->seconds = 1e-6 * (best + kLaunchUs);
  return true;
}

int launch_bwdw_few(const cct_conv_desc_t& d, const BwdwFewPlan& P, int nimg, const float* x, const float* dy, float* part,
                    float* sums, hipStream_t st) {
  Few q;
  memset(&q, 0, sizeof(q));
  q.x = x; q.dy = dy; q.part = part; q.sums = sums;
  q.Cg = d.C / d.groups; q.Og = d.O / d.groups; q.C = d.C; q.O = d.O; q.H = d.H; q.W = d.W;
  q.Hout = (d.H + 2 * d.pad - d.K) / d.stride + 1; q.Wout = (d.W + 2 * d.pad - d.K) / d.stride + 1;
  q.K = d.K; q.s = d.stride; q.pad = d.pad; q.G = d.groups; q.nimg = nimg;
  q.N = q.Cg * d.K * d.K;
  q.strips = (q.Wout + kPos - 1) / kPos; q.segs = P.segs; q.seg_rows = P.seg_rows; q.S = P.S;
  q.tiles_m = (q.Og + 16 * P.rb - 1) / (16 * P.rb);
  q.WX = (kPos - 1) * d.stride + d.K; q.ring = d.K + d.stride;
  q.row_b = row_bytes(q.WX, q.Cg, d.K);
  const double yn = (double)nimg * d.O * q.Hout * q.Wout;
  ProfScope ps(2.0 * yn * q.N, 4.0 * ((double)nimg * d.C * d.H * d.W + yn + (double)q.S * d.O * q.N), st, "conv_bwdw_few<%d, %d>",
               16 * P.rb, P.cb);
  switch (P.rb * 4 + P.cb) {
    case 25: return launch_few<6, 1>(q, P.lds, st);
    case 26: return launch_few<6, 2>(q, P.lds, st);
    case 27: return launch_few<6, 3>(q, P.lds, st);
    case 17: return launch_few<4, 1>(q, P.lds, st);
    case 18: return launch_few<4, 2>(q, P.lds, st);
    case 19: return launch_few<4, 3>(q, P.lds, st);
    case 9: return launch_few<2, 1>(q, P.lds, st);
    case 10: return launch_few<2, 2>(q, P.lds, st);
    case 11: return launch_few<2, 3>(q, P.lds, st);
    default: return CCT_EUNSUPPORTED;
  }
}

}  // namespace cct
