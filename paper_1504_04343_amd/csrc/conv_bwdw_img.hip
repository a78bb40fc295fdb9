// Backward-weights pass on the bf16 matrix cores with the images as the contiguous reduction index.
//
//     dw[o][(ci,i,j)] = sum_{n, r, c} dy[n, o, r, c] * xpad[n, ci, r*s + i, c*s + j]
//
// A lane of v_mfma_f32_16x16x32_bf16 takes 8 consecutive reduction indices of its row as one 16-byte
// operand.  Taken along a row of the image those 8 values would start at any column (the tap shifts
// them); taken over 8 IMAGES at one pixel they are one aligned granule whatever the tap.  So the pass is
//   1. bwdw_img_prep: x (zero padded) and dy are rewritten once as granules of 8 images,
//          xs[image group][padded row][padded column][term][channel],  ds[image group][pixel][term][kernel],
//      in bf16: one term (bf16 operands), or three whose sum is the fp32 value (split_bf16.h).  The same
//      kernel sums dy for the bias gradient, which reads all of dy anyway;
//   2. conv_bwdw_img: the matrix product, column = (image group, output pixel) = 8 reduction indices;
//      row n of the second operand is a tap of a channel, i.e. a constant offset from the column's cell;
//   3. bwdw_img_reduce: the splits' partial products are added in split order.
// Nothing of the size of the lowered matrix exists (no K*K blow-up).
//
// The product (granule_product.h): a workgroup owns BM kernels x 256 lowered rows, ordered (block of 32
// channels, tap, channel) so that neighbouring lanes read neighbouring granules.
//
// Measured (whole pass with the bias gradient; before: dy and x read in place by fp32 matrix
// instructions, or bf16 lowered matrices): conv3 at batch 1024 2880 -> 1550 us, of it 1255 the product
// (244 TFLOP/s of fp32 results, 1460 of bf16 MFMAs: the card's power limit) and 240 the rewriting
// (4.6 TB/s); conv2 at batch 256 1215 -> 690; conv4 at batch 256 with bf16 operands 355 -> 125.
#include <algorithm>

#include "cct_internal.h"
#include "granule_product.h"

namespace cct {
namespace {

constexpr int kImg = 8;       // images per granule
constexpr int kChanBlock = 32;
constexpr int kPrepPx = 32, kPrepCh = 32;  // pixels and channels a workgroup of the first step rewrites

// ---- 1. granules of 8 images ------------------------------------------------------------------

// One tensor of the first step: [nimg][C][H][W] -> [group][H + 2*pad][W + 2*pad][TERMS][C] granules.
struct PrepJob {
  const float* src;
  uint4* dst;
  float* sums;  // bias gradient: [group * pixel tiles][C] partial sums, or null
  int C, H, W, pad, Wp, pixels;  // pixels: (H + 2*pad) * (W + 2*pad)
  int tiles_px, tiles_c;
  unsigned mWp, mTpx, mTc;
  int sWp, sTpx, sTc;
};

// Bound by memory: every value is read once (rows of 32 pixels) and written as 2 * TERMS bytes (runs of
// 32 granules); the transposition goes through LDS.
template <int TERMS>
__global__ __launch_bounds__(256) void bwdw_img_prep(PrepJob j0, PrepJob j1, int blocks0, int nimg) {
  constexpr int ROW = kPrepCh + 1;  // granules between pixels in LDS: 16-byte accesses spread over the banks
  __shared__ uint4 buf[TERMS][kPrepPx * ROW];
  const bool second = (int)blockIdx.x >= blocks0;
  const PrepJob& j = second ? j1 : j0;
  const int b = second ? (int)blockIdx.x - blocks0 : (int)blockIdx.x;
  // channel tile fastest: the tiles of one pixel range write the same lines
  const int bp = fdiv_u(b, j.mTc, j.sTc), tc = b - bp * j.tiles_c;
  const int ig = fdiv_u(bp, j.mTpx, j.sTpx), tp = bp - ig * j.tiles_px;
  const int tid = threadIdx.x;
  const int px = tid & 31, cr = tid >> 5;
  const int q = tp * kPrepPx + px;
  const int hp = fdiv_u(q, j.mWp, j.sWp), wp = q - hp * j.Wp;
  const int h = hp - j.pad, w = wp - j.pad;
  const bool inside = q < j.pixels && h >= 0 && h < j.H && w >= 0 && w < j.W;
  const long long plane = (long long)j.H * j.W, img = (long long)j.C * plane;
  const float* src = j.src + (long long)ig * kImg * img + (long long)tc * kPrepCh * plane;
  const int nv = min(kImg, nimg - ig * kImg);
  // Buffer loads whose range check supplies the zeros, so that all are on their way before the first is waited for: with
  // a branch around each, whole groups of them were waited for in turn (conv2 at batch 256 145 -> 118 us).  A plane is
  // less than 2^24 pixels: 32-bit byte offsets inside a tile of channels.
  float v[kPrepCh / 8][kImg];
  const unsigned first = (unsigned)((cr * (int)plane + h * j.W + w) * 4);
#pragma unroll
  for (int it = 0; it < kPrepCh / 8; ++it) {
    const unsigned off = inside && tc * kPrepCh + it * 8 + cr < j.C ? first + (unsigned)it * 8u * (unsigned)plane * 4u : 0x80000000u;
#pragma unroll
    for (int e = 0; e < kImg; ++e) {
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(src + e * img), 0, e < nv ? 0x7fffffff : 0, 0x00020000);
      v[it][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
    }
  }
#pragma unroll
  for (int it = 0; it < kPrepCh / 8; ++it) {
    const int cl = it * 8 + cr;
    uint4 t[TERMS];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = v[it][2 * e], c = v[it][2 * e + 1];
      unsigned hh, mm, ll;
      if (TERMS == 3) {
        split_pair(a, c, &hh, &mm, &ll);
        reinterpret_cast<unsigned*>(&t[1])[e] = mm;
        reinterpret_cast<unsigned*>(&t[TERMS - 1])[e] = ll;
      } else {
        hh = cvt_pk_bf16(a, c);
      }
      reinterpret_cast<unsigned*>(&t[0])[e] = hh;
    }
#pragma unroll
    for (int k = 0; k < TERMS; ++k) buf[k][px * ROW + cl] = t[k];
    if (j.sums) {
      float s = ((v[it][0] + v[it][1]) + (v[it][2] + v[it][3])) + ((v[it][4] + v[it][5]) + (v[it][6] + v[it][7]));
#pragma unroll
      for (int off = 16; off > 0; off >>= 1) s += __shfl_down(s, off, 32);
      const int c = tc * kPrepCh + cl;
      if (px == 0 && c < j.C) j.sums[(long long)bp * j.C + c] = s;
    }
  }
  __syncthreads();
  const int c = tid & 31, r0 = tid >> 5;
  const int ch = tc * kPrepCh + c;
  if (ch >= j.C) return;
#pragma unroll
  for (int it = 0; it < kPrepPx * TERMS / 8; ++it) {
    const int u = it * 8 + r0, p = u / TERMS, k = u - p * TERMS;
    const int qq = tp * kPrepPx + p;
    if (qq < j.pixels) j.dst[(((long long)ig * j.pixels + qq) * TERMS + k) * j.C + ch] = buf[k][p * ROW + c];
  }
}

// ---- 2. the product -----------------------------------------------------------------------------

struct ImgGemm {
  const unsigned char *xs, *ds;
  float* part;  // [S][G][M][N], n = (channel block, tap, channel); three terms: scaled as they are
  int M, N, G;
  int Cg, Og, C, O, K, KK, s, Wp;
  long long img_cells;  // padded pixels per image
  int P, Wout;
  int ncols, split_cols, S, tiles_m, tiles_n;
  unsigned mP, mWout;
  int sP, sWout;
};

template <int BM, int TERMS, int SLOTS>
__global__ __launch_bounds__(granule_waves(BM, TERMS) * 64, 2) void conv_bwdw_img(ImgGemm p) {
  using GP = GranuleProduct<BM, TERMS, SLOTS, 16>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_i[];  // [2][A: SLOTS*BMP | B: SLOTS*BN]
  GP gp;

  const int lane = threadIdx.x & 63;
  // consecutive workgroup ids go round-robin over the 8 XCDs: give every XCD a contiguous run of
  // (split, tile) pairs, tile fastest, so that the tiles of one split share both operands through L2
  int bid = blockIdx.x;
  {
    const int total = p.tiles_m * p.tiles_n * p.S;
    const int per = total >> 3, rem = total & 7;
    const int xcd = bid & 7, slot = bid >> 3;
    bid = xcd * per + min(xcd, rem) + slot;
  }
  const int ntiles = p.tiles_m * p.tiles_n;
  const int s = bid / ntiles, tile = bid - s * ntiles;
  const int tile_m = tile / p.tiles_n, tile_n = tile - tile_m * p.tiles_n;
  const int g = blockIdx.y;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int c_begin = s * p.split_cols, c_end = min(p.ncols, c_begin + p.split_cols);

  // rows past the last one repeat it (their products are not stored)
#pragma unroll
  for (int u = 0; u < GP::A_PARTS; ++u) gp.a_voff[u] = (unsigned)min(m0 + u * 64 + lane, p.M - 1) * kGran;
#pragma unroll
  for (int u = 0; u < GP::B_PARTS; ++u) {
    const int n = min(n0 + gp.b_part(u) * 64 + lane, p.N - 1);
    const int cb = n / (p.KK * kChanBlock), width = min(kChanBlock, p.Cg - cb * kChanBlock);
    const int rem = n - cb * p.KK * kChanBlock, tap = rem / width, cl = rem - tap * width;
    const int i = tap / p.K, j = tap - i * p.K;
    gp.b_voff[u] = (unsigned)(((long long)(i * p.Wp + j) * TERMS * p.C + cb * kChanBlock + cl) * kGran);
  }
  const unsigned char* Bg = p.xs + (long long)g * p.Cg * kGran;
  const long long b_cell = (long long)TERMS * p.C * kGran;
  gp.run(smem_i, c_begin, c_end, p.ds + (long long)g * p.Og * kGran, (long long)TERMS * p.O * kGran, p.O * kGran,
         p.C * kGran, [&](int col) {
           const int ig = fdiv_u(col, p.mP, p.sP), pix = col - ig * p.P;
           const int r = fdiv_u(pix, p.mWout, p.sWout), c = pix - r * p.Wout;
           return Bg + (ig * p.img_cells + (long long)(r * p.s) * p.Wp + c * p.s) * b_cell;
         });

  float* __restrict__ C = p.part + ((long long)s * p.G + g) * p.M * p.N;
  gp.for_each([&](int row, int column, float v) {
    const int m = m0 + row, n = n0 + column;
    if (m < p.M && n < p.N) C[(long long)m * p.N + n] = v;
  });
}

// ---- 3. sum of the splits -----------------------------------------------------------------------

struct ImgReduce {
  const float* part;
  float* dw;
  const float* sums;  // bias partial sums [nsums][O], or null
  float* dbias;
  const float *x, *dy;  // the chunk's tensors, for results that are not finite
  int M, N, G, S, K, KK, Cg, Og, C, O, H, W, P, Wout, s, pad, nimg;
  unsigned mWout;
  int sWout;
  int nsums, accumulate, blocks_dw, split, strips;
};

constexpr int kSumCh = 4, kStrips = 256 / kSumCh;

// The last blocks sum the bias gradient.
// split: the operands were split and scaled; results that are not finite are summed again in plain fp32
// (split_bf16.h), the whole workgroup on one at a time.
__global__ __launch_bounds__(256) void bwdw_img_reduce(ImgReduce p) {
  __shared__ float red[256];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= p.blocks_dw) {
    // strips of partial sums per kernel, four loads of a strip in flight
    const int o = ((int)blockIdx.x - p.blocks_dw) * kSumCh + tid % kSumCh;
    float v = 0.f;
    if (o < p.O) {
      const float* src = p.sums + o;
      int k = tid / kSumCh;
      for (; k + 3 * kStrips < p.nsums; k += 4 * kStrips) {
        float u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = src[(long long)(k + e * kStrips) * p.O];
        v += (u[0] + u[1]) + (u[2] + u[3]);
      }
      for (; k < p.nsums; k += kStrips) v += src[(long long)k * p.O];
    }
    // the strips in a tree: one after the other they would add as much error as 32 levels of it
    red[tid] = v;
    __syncthreads();
#pragma unroll
    for (int off = 128; off >= kSumCh; off >>= 1) {
      if (tid < off) red[tid] += red[tid + off];
      __syncthreads();
    }
    if (tid < kSumCh && o < p.O) p.dbias[o] = p.accumulate ? p.dbias[o] + red[tid] : red[tid];
    return;
  }
  // a workgroup takes 256 weights, or 64 with a quarter of the splits per wave
  const int wid = p.strips == 4 ? tid & 63 : tid, strip = p.strips == 4 ? tid >> 6 : 0;
  const long long total = (long long)p.M * p.N * p.G;
  const long long t0 = (long long)blockIdx.x * (256 / p.strips), t = t0 + wid;
  float sum = 0.f;
  int o = 0, ci = 0, tap = 0;
  long long wi = 0;
  if (t < total) {
    const float* src = p.part + t;
    const int share = (p.S + p.strips - 1) / p.strips, end = min(p.S, (strip + 1) * share);
    int k = strip * share;
    for (; k + 8 <= end; k += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = src[(k + u) * total];
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += v[u];
    }
    for (; k < end; ++k) sum += src[k * total];
    // A group may hold more than 2^31 weights: the workgroup's first row (of all groups) in 64 bits, the
    // rest from there.
    const long long row0 = t0 / p.N;
    const int n0 = (int)(t0 - row0 * p.N) + wid, rows = n0 / p.N, n = n0 - rows * p.N;
    o = (int)row0 + rows;
    const int cb = n / (p.KK * kChanBlock), width = min(kChanBlock, p.Cg - cb * kChanBlock);
    const int rem = n - cb * p.KK * kChanBlock;
    tap = rem / width;
    ci = cb * kChanBlock + rem - tap * width;
    wi = ((long long)o * p.Cg + ci) * p.KK + tap;
  }
  if (p.strips == 4) {
    red[tid] = sum;
    __syncthreads();
    sum = ((red[wid] + red[64 + wid]) + red[128 + wid]) + red[192 + wid];
  }
  if (p.split) {
    __shared__ int redo[256];
    __shared__ int any;
    const int P = p.P;
    // the operands of weight (oo, channel cc, tap i, j) at pixel pix of image n, zeros outside the image: the loads
    // do not depend on a branch, so that a thread has several in flight
    auto operands = [&](int oo, int cc, int i, int j, int n, int pix, float* a, float* b) {
      const int r = fdiv_u(pix, p.mWout, p.sWout), c = pix - r * p.Wout;
      const int h = r * p.s + i - p.pad, w = c * p.s + j - p.pad;
      const bool ok = n < p.nimg && h >= 0 && h < p.H && w >= 0 && w < p.W;
      const float va = p.dy[ok ? ((long long)n * p.O + oo) * P + pix : 0];
      const float vb = p.x[ok ? (((long long)n * p.C + cc) * p.H + h) * p.W + w : 0];
      *a = ok ? va : 0.f;
      *b = ok ? vb : 0.f;
    };
    bool bad = strip == 0 && t < total && !finite(sum);
    sum *= kSplitUnscale;
    if (bad) {  // where a NaN went in, most weights are decided here, all at once
      float v = 0.f;
      for (int q = 0; q < 64 && q < P && v == v; ++q) {
        float a, b;
        operands(o, o / p.Og * p.Cg + ci, tap / p.K, tap % p.K, 0, q, &a, &b);
        v = fmaf(a, b, v);
      }
      if (v != v) {
        sum = v;
        bad = false;
      }
    }
    if (tid == 0) any = 0;
    __syncthreads();
    redo[tid] = bad;
    if (bad) any = 1;
    __syncthreads();
    if (any) {
      __shared__ int key[3];
      __shared__ int found;  // a NaN, which no other product changes: the threads stop as they see it
      volatile int* stop = &found;
#pragma unroll 1
      for (int who = 0; who < 256; ++who) {
        if (!redo[who]) continue;  // the same for all threads
        if (tid == who) {
          key[0] = o;
          key[1] = o / p.Og * p.Cg + ci;
          key[2] = tap;
          found = 0;
        }
        __syncthreads();
        const int i = key[2] / p.K, jj = key[2] - i * p.K;
        // a thread's pixels advance by 4 * 256: image and pixel by adding, no division by P
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        int n[4], pix[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          n[u] = (tid + u * 256) / p.P;
          pix[u] = tid + u * 256 - n[u] * p.P;
        }
        const int dn = 1024 / p.P, dpix = 1024 - dn * p.P;
        while (n[0] < p.nimg && !*stop) {
          float a[4], b[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            operands(key[0], key[1], i, jj, n[u], pix[u], &a[u], &b[u]);
            n[u] += dn;
            pix[u] += dpix;
            if (pix[u] >= p.P) {
              pix[u] -= p.P;
              ++n[u];
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = fmaf(a[u], b[u], v[u]);
          const float sum4 = (v[0] + v[1]) + (v[2] + v[3]);
          if (sum4 != sum4) *stop = 1;
        }
        red[tid] = (v[0] + v[1]) + (v[2] + v[3]);
        __syncthreads();
#pragma unroll 1
        for (int off = 128; off > 0; off >>= 1) {
          if (tid < off) red[tid] += red[tid + off];
          __syncthreads();
        }
        if (tid == who) sum = red[0];
        __syncthreads();
      }
    }
  }
  if (strip == 0 && t < total) p.dw[wi] = p.accumulate ? p.dw[wi] + sum : sum;
}

// ---- host -----------------------------------------------------------------------------------------

inline int out_size(int in, int K, int s, int pad) { return (in + 2 * pad - K) / s + 1; }

// What a tile of three terms costs, in rows of a 128-row one: with fewer rows the same columns are read for fewer
// products (256 images of 28 x 28, 64 channels, 3 x 3: 128 kernels 155 us, 96 in a tile of 96 rows 129 and of 128 rows
// 154, 64 96; 384 kernels in two groups as 4 tiles of 96 267, as 6 of 64 293).
constexpr int tile_weight(int bm) { return bm == 128 ? 128 : bm == 96 ? 104 : 76; }

inline int row_tile(int M, int terms) {
  if (terms == 1) return M % 128 == 0 || M % 128 > 64 ? 128 : 64;
  int best = 128;
  for (int bm : {96, 64})
    if ((M + bm - 1) / bm * tile_weight(bm) < (M + best - 1) / best * tile_weight(best)) best = bm;
  return best;
}

template <int BM, int TERMS, int SLOTS>
int launch_product(const ImgGemm& p, dim3 grid, hipStream_t st) {
  constexpr int lds = GranuleProduct<BM, TERMS, SLOTS, 16>::LDS;
  constexpr auto kern = conv_bwdw_img<BM, TERMS, SLOTS>;
  if (const int rc = ensure_dynamic_lds<kern>(lds)) return rc;
  hipLaunchKernelGGL(kern, grid, dim3(granule_waves(BM, TERMS) * 64), lds, st, p);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace

bool bwdw_img_plan(const cct_conv_desc_t& d, long long nimg, BwdwImgPlan* P) {
  const int Hout = out_size(d.H, d.K, d.stride, d.pad), Wout = out_size(d.W, d.K, d.stride, d.pad);
  const int Cg = d.C / d.groups, Og = d.O / d.groups;
  const long long terms = d.precision == CCT_PREC_F32 ? 3 : 1;
  const long long Hp = d.H + 2LL * d.pad, Wp = d.W + 2LL * d.pad;
  const long long pix = (long long)Hout * Wout, N = (long long)Cg * d.K * d.K;
  const long long groups_of_images = (nimg + kImg - 1) / kImg;
  const long long cols = groups_of_images * pix;
  if (d.groups > 65535 || N >= (1LL << 30) || Hp * Wp >= (1LL << 24) || cols >= (1LL << 30)) return false;
  // a tap's offset from its column's cell, a term's from its granule: 32-bit byte offsets
  if (((d.K - 1) * Wp + d.K) * terms * d.C * kGran >= (1LL << 31) || terms * d.O * kGran >= (1LL << 31) ||
      terms * d.C * kGran >= (1LL << 31))
    return false;
  const long long tx = (Hp * Wp + kPrepPx - 1) / kPrepPx, ty = (pix + kPrepPx - 1) / kPrepPx;
  const long long ctx = (d.C + kPrepCh - 1) / kPrepCh, cty = (d.O + kPrepCh - 1) / kPrepCh;
  if (groups_of_images * (tx * ctx + ty * cty) >= (1LL << 30)) return false;
  auto at_most = [&](long long ncols, long long ncol) { return (ncols + 2 * ncol - 1) / (2 * ncol); };
  const long long all = (d.N + kImg - 1) / kImg * pix, tiles_64 = ((Og + 63) / 64) * ((N + BN - 1) / BN) * d.groups;
  // Where even tiles of 64 rows and two stages are few, the chain of one counts (up to 512 of them larger tiles take
  // 1.1 times the time, 1.05 up to 1024, 0.99 up to 4096, 0.89 beyond)
  P->BM = terms == 3 && std::min(tiles_64, 768LL) * std::min(at_most(all, 4), 768LL) < 768 ? 64 : row_tile(Og, (int)terms);
  P->terms = (int)terms;
  const long long ncol = terms == 1 ? 8 : 4;  // columns per stage
  const long long tiles = ((Og + P->BM - 1) / P->BM) * ((N + BN - 1) / BN) * d.groups;
  const long long slots = terms == 3 || P->BM == 128 ? 256 : 512;  // workgroups the chip holds
  const long long out_bytes = 4LL * d.O * N;
  // Splits, from the whole batch: whole rounds of workgroups (a last round that is nearly empty costs as
  // much as a full one), the number of rounds that is estimated fastest, partial products within 256 MiB,
  // at least two stages each.  A smaller chunk takes at most as many, so that its plan is no larger.
  // (Rows as they are: 64 of three terms take 0.94 times what they took as two workgroups of four waves per CU; priced
  // at their weight, 76, layers went to other kernels that this one runs in 0.7 times the time, 2 % of 9156.)
  const double sec_col = 2.0 * P->BM * BN * kImg / ((terms == 3 ? 245.0e12 : 600.0e12) / slots);
  auto cut = [&](long long ncols, long long want, long long* S, long long* len) {
    *len = ((ncols + want - 1) / want + ncol - 1) / ncol * ncol;
    *S = (ncols + *len - 1) / *len;
  };
  long long want = 0, S, len;
  double best = 0.0;
  for (int rounds = 1; rounds <= 4; ++rounds) {
    long long w = std::max(1LL, rounds * slots / tiles);
    w = std::min(w, std::max(1LL, (256LL << 20) / out_bytes));
    w = std::min(w, at_most(all, ncol));
    cut(all, w, &S, &len);
    const double sec = (double)((tiles * S + slots - 1) / slots) * ((double)len * sec_col + 9.0e-6) +
                       (double)out_bytes * S * 2.0 / 8.0e12 + (double)S * 1.5e-8;
    if (want == 0 || sec < best) {
      best = sec;
      want = w;
    }
  }
  want = std::min(want, at_most(cols, ncol));
  cut(cols, want, &S, &len);
  if (all >= (1LL << 30) || tiles * S >= (1LL << 31)) return false;
  P->S = (int)S;
  P->split_cols = (int)len;
  // a pixel with few channels is a short run of granules: 3 channels measured 1.2 TB/s
  const double runs = std::max(1.0, 10.0 / d.C);
  const double moved = (double)groups_of_images * kImg *
                       ((double)d.C * (4.0 * d.H * d.W + 2.0 * terms * Hp * Wp) * runs + (double)d.O * pix * (4.0 + 2.0 * terms));
  P->seconds = best + moved / 4.0e12 + 2.0e-6;
  long long off = 0;
  auto take = [&](long long bytes, long long* o) {
    *o = off;
    off += (bytes + 255) / 256 * 256;
  };
  take(groups_of_images * Hp * Wp * terms * d.C * kGran, &P->xs_off);
  take(cols * terms * d.O * kGran, &P->ds_off);
  take(want * out_bytes, &P->part_off);
  take(groups_of_images * ty * d.O * 4, &P->sums_off);
  P->total = off;
  // Few channels (with kFewMargin 2 of 388 layers take more than 4 % longer than without this kernel; at 1.0 none do, but
  // those that stay off it lose 2 % in the mean).  Decided for the whole batch, so that a shorter last chunk runs the same way.
  P->few = bwdw_few_plan(d, nimg, &P->fp) && (nimg < d.N || P->fp.seconds < kFewMargin * P->seconds);
  if (nimg < d.N && P->few) {
    BwdwImgPlan whole;
    P->few = bwdw_img_plan(d, d.N, &whole) && whole.few;
  }
  if (P->few) {
    P->seconds = P->fp.seconds;
    P->S = P->fp.S;
    off = 0;
    take(P->S * out_bytes, &P->part_off);
    take((long long)P->S * d.O * 4, &P->sums_off);
    P->total = off;
  }
  return true;
}

int launch_bwdw_img(const cct_conv_desc_t& d, const BwdwImgPlan& P, int nimg, const float* x, const float* dy,
                    float* dw, float* dbias, int accumulate, char* ws, hipStream_t st) {
  const int Hout = out_size(d.H, d.K, d.stride, d.pad), Wout = out_size(d.W, d.K, d.stride, d.pad);
  const int Cg = d.C / d.groups, Og = d.O / d.groups, KK = d.K * d.K, pix = Hout * Wout;
  if (P.few && nimg > P.fp.images) {
    for (int n0 = 0; n0 < nimg; n0 += P.fp.images) {
      const int ni = std::min(P.fp.images, nimg - n0);
      BwdwImgPlan part;
      if (!bwdw_img_plan(d, ni, &part)) return CCT_EUNSUPPORTED;
      const int rc = launch_bwdw_img(d, part, ni, x + (long long)n0 * d.C * d.H * d.W, dy + (long long)n0 * d.O * pix, dw, dbias,
                                     accumulate || n0 > 0, ws, st);
      if (rc) return rc;
    }
    return CCT_OK;
  }
  const int Hp = d.H + 2 * d.pad, Wp = d.W + 2 * d.pad, igs = (nimg + kImg - 1) / kImg;
  auto job = [&](const float* src, long long dst_off, int C, int H, int W, int pad) {
    PrepJob j;
    memset(&j, 0, sizeof(j));
    j.src = src;
    j.dst = reinterpret_cast<uint4*>(ws + dst_off);
    j.C = C; j.H = H; j.W = W; j.pad = pad;
    j.Wp = W + 2 * pad;
    j.pixels = (H + 2 * pad) * j.Wp;
    j.tiles_px = (j.pixels + kPrepPx - 1) / kPrepPx;
    j.tiles_c = (C + kPrepCh - 1) / kPrepCh;
    make_fastdiv_parts(j.Wp, &j.mWp, &j.sWp);
    make_fastdiv_parts(j.tiles_px, &j.mTpx, &j.sTpx);
    make_fastdiv_parts(j.tiles_c, &j.mTc, &j.sTc);
    return j;
  };
  float* part = reinterpret_cast<float*>(ws + P.part_off);
  float* sums = dbias ? reinterpret_cast<float*>(ws + P.sums_off) : nullptr;
  int nsums = P.S;
  if (P.few) {
    if (const int rc = launch_bwdw_few(d, P.fp, nimg, x, dy, part, sums, st)) return rc;
  } else {
    const PrepJob jx = job(x, P.xs_off, d.C, d.H, d.W, d.pad);
    PrepJob jy = job(dy, P.ds_off, d.O, Hout, Wout, 0);
    jy.sums = sums;
    nsums = igs * jy.tiles_px;
    const int bx = igs * jx.tiles_px * jx.tiles_c, by = igs * jy.tiles_px * jy.tiles_c;
    const double xn = (double)nimg * d.C * d.H * d.W, yn = (double)nimg * d.O * pix;
    {
      ProfScope ps(P.terms == 3 ? "bwdw_img_prep<3>" : "bwdw_img_prep<1>", 0.0, (4.0 + 2.0 * P.terms) * (xn + yn), st);
      if (P.terms == 3)
        hipLaunchKernelGGL(bwdw_img_prep<3>, dim3((unsigned)(bx + by)), dim3(256), 0, st, jx, jy, bx, nimg);
      else
        hipLaunchKernelGGL(bwdw_img_prep<1>, dim3((unsigned)(bx + by)), dim3(256), 0, st, jx, jy, bx, nimg);
      CCT_CHECK_LAUNCH();
    }
    ImgGemm q;
    memset(&q, 0, sizeof(q));
    q.xs = reinterpret_cast<const unsigned char*>(ws + P.xs_off);
    q.ds = reinterpret_cast<const unsigned char*>(ws + P.ds_off);
    q.part = part;
    q.M = Og; q.N = Cg * KK; q.G = d.groups;
    q.Cg = Cg; q.Og = Og; q.C = d.C; q.O = d.O; q.K = d.K; q.KK = KK; q.s = d.stride; q.Wp = Wp;
    q.img_cells = (long long)Hp * Wp;
    q.P = pix; q.Wout = Wout;
    q.ncols = igs * pix;
    q.split_cols = P.split_cols;
    q.S = P.S;
    q.tiles_m = (Og + P.BM - 1) / P.BM;
    q.tiles_n = (q.N + BN - 1) / BN;
    make_fastdiv_parts(pix, &q.mP, &q.sP);
    make_fastdiv_parts(Wout, &q.mWout, &q.sWout);
    const long long blocks = (long long)q.tiles_m * q.tiles_n * q.S;
    if (blocks <= 0 || blocks >= 2147483647LL || d.groups > 65535) return CCT_EUNSUPPORTED;
    {
      ProfScope ps(2.0 * yn * Cg * KK, 2.0 * P.terms * (xn + yn) + 4.0 * q.S * (double)d.O * q.N, st,
                   "conv_bwdw_img<%d, %d, %d>", P.BM, P.terms, P.terms == 1 ? 8 : 12);
      const dim3 grid((unsigned)blocks, (unsigned)d.groups);
      int rc;
      if (P.BM == 128)
        rc = P.terms == 3 ? launch_product<128, 3, 12>(q, grid, st) : launch_product<128, 1, 8>(q, grid, st);
      else if (P.BM == 96)
        rc = launch_product<96, 3, 12>(q, grid, st);
      else
        rc = P.terms == 3 ? launch_product<64, 3, 12>(q, grid, st) : launch_product<64, 1, 8>(q, grid, st);
      if (rc) return rc;
    }
  }
  ImgReduce r;
  memset(&r, 0, sizeof(r));
  r.part = part; r.dw = dw; r.sums = sums; r.dbias = dbias; r.x = x; r.dy = dy;
  r.M = Og; r.N = Cg * KK; r.G = d.groups; r.S = P.S; r.K = d.K; r.KK = KK; r.Cg = Cg; r.Og = Og;
  r.C = d.C; r.O = d.O; r.H = d.H; r.W = d.W; r.P = pix; r.Wout = Wout; r.s = d.stride; r.pad = d.pad;
  make_fastdiv_parts(Wout, &r.mWout, &r.sWout);
  r.nimg = nimg;
  r.nsums = nsums;
  r.accumulate = accumulate;
  r.split = P.terms == 3;
  const long long total = (long long)d.O * r.N;
  // few weights: more loads in flight per weight
  r.strips = total < 256 * 1024 && P.S >= 8 ? 4 : 1;
  const long long rb = (total * r.strips + 255) / 256, db = dbias ? (d.O + kSumCh - 1) / kSumCh : 0;
  if (rb + db >= 2147483647LL) return CCT_EUNSUPPORTED;
  r.blocks_dw = (int)rb;
  ProfScope ps("bwdw_img_reduce", 0.0, 4.0 * total * (P.S + 1), st);
  hipLaunchKernelGGL(bwdw_img_reduce, dim3((unsigned)(rb + db)), dim3(256), 0, st, r);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace cct
