// Forward and stride-1 backward-data passes for bf16 operands as a product of granules (8 channels of a
// pixel, granule_product.h):
//     C[m][pos] = sum_{channels, taps} K^[m][channels, tap] * xpad[n, channels, r*s + i, c*s + j]
//   1. granule_prep: x (or dy) is rounded and rewritten once as xs[image][8 channels][padded row][padded
//      column], the kernels as ks[8 channels, tap][row]; both are plain streaming copies;
//   2. conv_granules: a column of the reduction is (8 channels, tap); a row of the second operand is an
//      output position, a constant offset from the tap's first pixel, and neighbouring positions are
//      neighbouring granules.  The epilogue writes NCHW and adds the bias.
// The fused kernel (conv_fused_kc_bf16) rounds x again in every workgroup and waits for it once per 16
// channels; here nothing but operand reads and MFMAs is left in the loop, for one extra pass over x.
// Measured at batch 256, the pass with its rewriting: conv4 (57.4 GFLOP) forward 170 -> 96 us (of it 72 the
// product, 800 TFLOP/s), backward-data 157 -> 95; conv2 (115 GFLOP) 244 -> 227 and 251 -> 221; a 1 x 1 layer,
// 69 images of 42 x 42, 452 -> 58 channels, 175 -> 95 and 174 -> 74.
#include <algorithm>

#include "cct_internal.h"
#include "granule_product.h"

namespace cct {
namespace {

constexpr int kCh = 8;      // channels per granule
constexpr int SLOTS = 8;    // columns per stage

// ---- 1. granules of 8 channels -------------------------------------------------------------------

struct GranPrep {
  const float* src;  // [nimg][Ctot][H][W], Cg channels per group
  const float* w;
  u32x4 *xs, *ks;
  int C, G, Cg, n8, H, W, pad, Wp, pixels;       // n8 = granules of a group's channels
  int M, K, KK, Og_w, Cg_w, flipped;             // kernels: rows per group, w is [G*Og_w][Cg_w][K][K]
  long long x_total, blocks_x;
  unsigned mWp, mPx, mPer, mN8;                  // by the row width, the pixels, the granules of an image and of a group
  int sWp, sPx, sPer, sN8;
  double per_px, per_img;                        // 1 / pixels, 1 / granules of an image
};

// floor(n / d) for n < 2^38, the same in a whole wave, with r = 1.0 / d: the product is off by less than one
__device__ __forceinline__ long long uniform_div(long long n, int d, double r) {
  long long q = (long long)((double)n * r);
  const long long rem = n - q * d;
  q += rem < 0 ? -1 : rem >= d ? 1 : 0;
  return (long long)__builtin_amdgcn_readfirstlane((int)(q >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)q);
}

__device__ __forceinline__ u32x4 granule_of(const float (&v)[kCh]) {
  return u32x4{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7])};
}

__global__ __launch_bounds__(256) void granule_prep(GranPrep p, int kernel_granules) {
  if ((long long)blockIdx.x >= p.blocks_x) {
    // kernels: ks[group][granule of channels, tap][row]
    const int t = (int)(blockIdx.x - p.blocks_x) * 256 + threadIdx.x;
    if (t >= kernel_granules) return;
    const int m = t % p.M, q = t / p.M;
    const int tap = q % p.KK, gc = q / p.KK, g = gc / p.n8, c0 = (gc - g * p.n8) * kCh;
    const int i = tap / p.K, j = tap - i * p.K;
    float v[kCh];
#pragma unroll
    for (int e = 0; e < kCh; ++e) {
      const int c = c0 + e;
      // forward: row = kernel, channel = input channel; backward-data: the roles change and the taps flip
      const int oo = p.flipped ? c : m, ci = p.flipped ? m : c;
      const int at = p.flipped ? p.KK - 1 - (i * p.K + j) : i * p.K + j;
      v[e] = c < p.Cg ? p.w[(((long long)g * p.Og_w + oo) * p.Cg_w + ci) * p.KK + at] : 0.f;
    }
    p.ks[t] = granule_of(v);
    return;
  }
  // Bound by memory.  64-bit divisions in every lane had been as long as the copy itself: those of a workgroup's first
  // granule are uniform, the lanes' own start from it.  All loads are on their way at once; zeros come from the buffer's
  // range check.
  const long long t0 = (long long)blockIdx.x * 256, plane0 = uniform_div(t0, p.pixels, p.per_px);  // (image, group, granule)
  const int rem = (int)(t0 - plane0 * p.pixels) + threadIdx.x;
  if (t0 + threadIdx.x >= p.x_total) return;
  const int dp = fdiv_u(rem, p.mPx, p.sPx), q = rem - dp * p.pixels;
  const int hp = fdiv_u(q, p.mWp, p.sWp), h = hp - p.pad, w = q - hp * p.Wp - p.pad;
  const int per = p.G * p.n8;
  const long long n0 = uniform_div(plane0, per, p.per_img);
  const int gc0 = (int)(plane0 - n0 * per), g0 = fdiv_u(gc0, p.mN8, p.sN8), ch0 = g0 * p.Cg + (gc0 - g0 * p.n8) * kCh;
  const int dn = fdiv_u(gc0 + dp, p.mPer, p.sPer), gc = gc0 + dp - dn * per, g = fdiv_u(gc, p.mN8, p.sN8);
  const int c0 = (gc - g * p.n8) * kCh, ch = g * p.Cg + c0;
  const bool inside = h >= 0 && h < p.H && w >= 0 && w < p.W;
  // 32-bit byte offsets from the first granule's channels: more than two granules only of planes of up to 256 pixels
  const long long HW = (long long)p.H * p.W;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.src + (n0 * p.C + ch0) * HW), 0, 0x7fffffff, 0x00020000);
  const unsigned first = (unsigned)(((dn * p.C + ch - ch0) * (int)HW + h * p.W + w) * 4);
  float v[kCh];
#pragma unroll
  for (int e = 0; e < kCh; ++e)
    v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
        rs, (int)(inside && c0 + e < p.Cg ? first + (unsigned)e * (unsigned)HW * 4u : 0x80000000u), 0, 0));
  p.xs[t0 + threadIdx.x] = granule_of(v);
}

// ---- 2. the product --------------------------------------------------------------------------------

struct GranGemm {
  const unsigned char *xs, *ks;
  float* out;
  const float* bias;  // [G*M] or null
  int M, G, n8, K, KK, s, Wp, P, Wout, ncols, npos;
  int tiles_m, tiles_n;
  long long pixels, out_img, out_group;  // elements
  unsigned mP, mWout, mKK, mK;
  int sP, sWout, sKK, sK;
};

template <int BM>
__global__ __launch_bounds__(BM * 4, 2) void conv_granules(GranGemm p) {
  using GP = GranuleProduct<BM, 1, SLOTS, 32>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_g[];
  GP gp;
  const int lane = threadIdx.x & 63;
  // every XCD gets a contiguous run of position tiles, the row tiles of one next to each other (they share x)
  int bid = blockIdx.x;
  {
    const int total = p.tiles_m * p.tiles_n;
    const int per = total >> 3, rem = total & 7;
    const int xcd = bid & 7, slot = bid >> 3;
    bid = xcd * per + min(xcd, rem) + slot;
  }
  const int tile_n = bid / p.tiles_m, tile_m = bid - tile_n * p.tiles_m;
  const int g = blockIdx.y;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const long long img_gran = (long long)p.G * p.n8 * p.pixels;  // granules of an image
  const int n_f = fdiv_u(n0, p.mP, p.sP);
  // rows past the last one repeat it (their products are not stored)
#pragma unroll
  for (int u = 0; u < GP::A_PARTS; ++u) gp.a_voff[u] = (unsigned)min(m0 + u * 64 + lane, p.M - 1) * kGran;
#pragma unroll
  for (int u = 0; u < GP::B_PARTS; ++u) {
    const int pos = min(n0 + gp.b_part(u) * 64 + lane, p.npos - 1);
    const int n = fdiv_u(pos, p.mP, p.sP), pix = pos - n * p.P;
    const int r = fdiv_u(pix, p.mWout, p.sWout), c = pix - r * p.Wout;
    gp.b_voff[u] = (unsigned)(((n - n_f) * img_gran + (long long)(r * p.s) * p.Wp + c * p.s) * kGran);
  }
  const unsigned char* Bg = p.xs + (n_f * img_gran + (long long)g * p.n8 * p.pixels) * kGran;
  gp.run(smem_g, 0, p.ncols, p.ks + (long long)g * p.ncols * p.M * kGran, (long long)p.M * kGran, 0, 0, [&](int col) {
    const int c8 = fdiv_u(col, p.mKK, p.sKK), tap = col - c8 * p.KK;
    const int i = fdiv_u(tap, p.mK, p.sK), j = tap - i * p.K;
    return Bg + (c8 * p.pixels + i * p.Wp + j) * kGran;
  });

  const float* bias = p.bias ? p.bias + (long long)g * p.M : nullptr;
  const int row0 = m0 + gp.row(0, 0);
  float bv[GP::RB * 16];
  load_bias(bv, bias, p.M - 1, [&](int r) { return m0 + gp.row(r / 16, r % 16); });
  float* __restrict__ out = p.out + g * p.out_group;
#pragma unroll
  for (int j = 0; j < GP::JB; ++j) {
    const int pos = n0 + gp.column(j);
    if (pos >= p.npos) continue;
    const int n = fdiv_u(pos, p.mP, p.sP);
    float* __restrict__ at = out + n * p.out_img + (pos - n * p.P) + (long long)row0 * p.P;
#pragma unroll
    for (int i = 0; i < GP::RB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (m0 + gp.row(i, r) < p.M) at[(long long)(gp.row(i, r) - gp.row(0, 0)) * p.P] = gp.acc[i][j][r] + bv[i * 16 + r];
  }
}

template <int BM>
int launch_product(const GranGemm& p, dim3 grid, hipStream_t st) {
  constexpr auto kern = conv_granules<BM>;
  constexpr int lds = GranuleProduct<BM, 1, SLOTS, 32>::LDS;
  if (const int rc = ensure_dynamic_lds<kern>(lds)) return rc;
  hipLaunchKernelGGL(kern, grid, dim3(BM * 4), lds, st, p);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

inline int row_tile(int M) { return M % 128 == 0 || M % 128 > 64 ? 128 : 64; }

// The pass as a convolution: input channels, output rows and planes.
struct Conv {
  int C, Cg, H, W, M, K, s, pad, Hout, Wout;
};
Conv conv_of(const cct_conv_desc_t& d, int pass) {
  const int Hout = (d.H + 2 * d.pad - d.K) / d.stride + 1, Wout = (d.W + 2 * d.pad - d.K) / d.stride + 1;
  if (pass == CCT_PASS_FORWARD) return {d.C, d.C / d.groups, d.H, d.W, d.O / d.groups, d.K, d.stride, d.pad, Hout, Wout};
  return {d.O, d.O / d.groups, Hout, Wout, d.C / d.groups, d.K, 1, d.K - 1 - d.pad, d.H, d.W};
}

}  // namespace

bool granules_plan(const cct_conv_desc_t& d, int pass, long long nimg, GranulesPlan* P) {
  if (d.precision != CCT_PREC_BF16_IN_F32_ACC || d.groups > 65535) return false;
  if (pass == CCT_PASS_BACKWARD_WEIGHTS) return false;
  if (pass == CCT_PASS_BACKWARD_DATA && (d.stride > 1 || d.pad > d.K - 1)) return false;
  const Conv c = conv_of(d, pass);
  const long long n8 = (c.Cg + kCh - 1) / kCh, KK = (long long)d.K * d.K, cols = n8 * KK;
  const long long Hp = c.H + 2LL * c.pad, Wp = c.W + 2LL * c.pad, pix = Hp * Wp, pos = (long long)c.Hout * c.Wout;
  const long long planes = nimg * d.groups * n8;
  if (pix >= (1LL << 24) || cols >= (1LL << 24) || nimg * pos >= (1LL << 30) || planes * pix >= (1LL << 38)) return false;
  // 32-bit byte offsets from a tile's first image; the kernels of a group
  const long long T = (BN - 1) / pos + 2;
  if (T * d.groups * n8 * pix * kGran >= (1LL << 31) || d.groups * cols * c.M >= (1LL << 30)) return false;
  P->BM = row_tile(c.M);
  const long long tiles_n = (nimg * pos + BN - 1) / BN, tiles = tiles_n * ((c.M + P->BM - 1) / P->BM) * d.groups;
  if (tiles >= (1LL << 30)) return false;
  const long long slots = P->BM == 128 ? 256 : 512;
  const double sec_col = 2.0 * P->BM * BN * kCh / (600.0e12 / slots);
  const double product = (double)((tiles + slots - 1) / slots) * ((double)((cols + SLOTS - 1) / SLOTS * SLOTS) * sec_col + 6.0e-6);
  const double out = 4.0 * nimg * c.M * d.groups * pos;
  const double moved = 4.0 * nimg * c.C * c.H * c.W + 16.0 * planes * pix;
  P->seconds = std::max(product, out / 4.0e12) + moved / 4.0e12 + 8.0e-6;
  long long off = 0;
  auto take = [&](long long bytes, long long* o) {
    *o = off;
    off += (bytes + 255) / 256 * 256;
  };
  take(planes * pix * kGran, &P->xs_off);
  take(d.groups * cols * c.M * kGran, &P->ks_off);
  P->total = off;
  return true;
}

int launch_granules(const cct_conv_desc_t& d, int pass, const GranulesPlan& P, int nimg, const float* in,
                    const float* w, const float* bias, float* out, char* ws, hipStream_t st) {
  const Conv c = conv_of(d, pass);
  const int n8 = (c.Cg + kCh - 1) / kCh, KK = d.K * d.K;
  GranPrep q;
  memset(&q, 0, sizeof(q));
  q.src = in; q.w = w;
  q.xs = reinterpret_cast<u32x4*>(ws + P.xs_off);
  q.ks = reinterpret_cast<u32x4*>(ws + P.ks_off);
  q.C = c.C; q.G = d.groups; q.Cg = c.Cg; q.n8 = n8; q.H = c.H; q.W = c.W; q.pad = c.pad;
  q.Wp = c.W + 2 * c.pad;
  q.pixels = (c.H + 2 * c.pad) * q.Wp;
  q.M = c.M; q.K = d.K; q.KK = KK; q.Og_w = d.O / d.groups; q.Cg_w = d.C / d.groups;
  q.flipped = pass == CCT_PASS_BACKWARD_DATA;
  q.x_total = (long long)nimg * d.groups * n8 * q.pixels;
  q.blocks_x = (q.x_total + 255) / 256;
  make_fastdiv_parts(q.Wp, &q.mWp, &q.sWp);
  make_fastdiv_parts(q.pixels, &q.mPx, &q.sPx);
  make_fastdiv_parts(d.groups * n8, &q.mPer, &q.sPer);
  make_fastdiv_parts(n8, &q.mN8, &q.sN8);
  q.per_px = 1.0 / q.pixels;
  q.per_img = 1.0 / (d.groups * n8);
  const int kg = d.groups * n8 * KK * c.M;
  const long long blocks = q.blocks_x + (kg + 255) / 256;
  if (blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  {
    ProfScope ps("granule_prep", 0.0, 4.0 * nimg * c.C * c.H * c.W + 16.0 * q.x_total, st);
    hipLaunchKernelGGL(granule_prep, dim3((unsigned)blocks), dim3(256), 0, st, q, kg);
    CCT_CHECK_LAUNCH();
  }
  GranGemm p;
  memset(&p, 0, sizeof(p));
  p.xs = reinterpret_cast<const unsigned char*>(q.xs);
  p.ks = reinterpret_cast<const unsigned char*>(q.ks);
  p.out = out; p.bias = bias;
  p.M = c.M; p.G = d.groups; p.n8 = n8; p.K = d.K; p.KK = KK; p.s = c.s; p.Wp = q.Wp;
  p.P = c.Hout * c.Wout; p.Wout = c.Wout; p.ncols = n8 * KK; p.npos = nimg * p.P;
  p.pixels = q.pixels;
  p.out_img = (long long)c.M * d.groups * p.P;
  p.out_group = (long long)c.M * p.P;
  p.tiles_m = (c.M + P.BM - 1) / P.BM;
  p.tiles_n = (p.npos + BN - 1) / BN;
  make_fastdiv_parts(p.P, &p.mP, &p.sP);
  make_fastdiv_parts(p.Wout, &p.mWout, &p.sWout);
  make_fastdiv_parts(KK, &p.mKK, &p.sKK);
  make_fastdiv_parts(d.K, &p.mK, &p.sK);
  const long long tiles = (long long)p.tiles_m * p.tiles_n;
  if (tiles <= 0 || tiles >= 2147483647LL || d.groups > 65535) return CCT_EUNSUPPORTED;
  ProfScope ps(2.0 * c.M * (double)p.npos * c.Cg * KK * d.groups,
               16.0 * q.x_total + 4.0 * p.out_img * nimg + 16.0 * kg, st, "conv_granules<%d>", P.BM);
  const dim3 grid((unsigned)tiles, (unsigned)d.groups);
  return P.BM == 128 ? launch_product<128>(p, grid, st) : launch_product<64>(p, grid, st);
}

}  // namespace cct
