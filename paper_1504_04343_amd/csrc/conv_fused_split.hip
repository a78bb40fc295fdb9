// Fused forward / backward-data pass (the "Fusion" of Sec. 2.1) for fp32 operands on the bf16 matrix
// cores: every operand is the exact sum of three bf16 terms and a product is six
// bf16 MFMAs (split_bf16.h).
//
// Product: C[m][pos] = sum_{grp, tap, c} K^[grp][tap][m][c] * xpad[n, grp*16 + c, r*s + i, c*s + j]
//   - a workgroup owns BM rows x 128 consecutive positions (48 rows: x 192, 64: also x 160); a wave owns 32 or 48 rows x (all |
//     half | a quarter of them) positions, two accumulators per block of results;
//   - per channel group of 16 it stages the zero-padded input rows its positions can touch as cells
//     (row, column) in a two-slot LDS ring, split while they are staged.  A cell is three terms of 16 bytes
//     for each half of its 16 channels; the halves lie apart, so that cells are 48 bytes = three 16-byte
//     slots from the next and reads of consecutive cells do not conflict;
//   - a tile is one tap of one channel group: 16 reduction indices.  The B operand of a lane is 16 bytes per
//     term of its position's cell at its tap, read ahead of the MFMAs;
//   - the kernel matrix comes packed and split as [group][tile][term][row][16] and never passes
//     through LDS: a lane loads the 16 bytes of its row, tile and term straight from the pack, some tiles
//     ahead, the tile and term in the scalar offset.  With all four waves stacked along the rows
//     no two waves read the same rows, which is why a wave is 32 x 128 and not 64 x 64: the pack is
//     read once per workgroup and tile (12 KiB per 768 MFMA cycles of a wave) and the cells four
//     times from LDS (48 of 128 bytes per cycle), where 64 x 64 waves would ask 24 KiB of the L1;
//   - the cells of the next group are fetched and written in up to four steps of 8 channels, spread over the
//     tiles; the workgroup meets when they are published.
// Two forms, by the edge MB of the blocks of results (which runs where: split_block):
//   - 16: v_mfma_f32_16x16x32_bf16 takes a pair of tiles, lanes 0-31 supply the first and lanes 32-63 the second;
//     where a tile's cells begin stands in a table in LDS.  Any K.  An odd number of taps (3 x 3, 5 x 5) makes pairs
//     that take the last tap of one group and the first of the next one; with an odd number of tiles the last one is
//     paired with zeros.  It does more per watt (granule_product.h), which large launches are bound by, and rows come
//     in blocks of 16: 96 kernels run as 2 x 48 rows.  Measured, us, 32 -> 16: conv1 forward (96 rows) 472 -> 403,
//     conv2 forward 490 -> 450, backward-data 613 -> 586, conv3 at batch 1024 1238 -> 1141 and 1273 -> 1182; 64 images
//     of 28 x 28, 64 channels: K = 7 to 64 kernels 149 -> 111.
//   - 32: v_mfma_f32_32x32x16_bf16 takes one tile; 3 x 3 and 5 x 5 kernels, all taps of a group unrolled, so that
//     nothing is looked up or decided between the MFMAs of a lone wave.  16 -> 32, in us: 50 images of conv5 forward
//     71.7 -> 67.9, 4 images of 28 x 28, 64 -> 128, K = 3, 18.9 -> 18.4, 48 workgroups of K = 5 24.4 -> 21.1, 20 images of
//     27 x 27, 192 -> 192, K = 3, 72.3 -> 67.4.
// 48 rows (conv2's and conv1's backward-data) are a tile of their own, with 192 positions, 48 of a wave: four waves then
// ask the L1 for the same 9 KiB each per 864 MFMA cycles.  With 128 positions (per 576 cycles) it was slower than the
// padding to 64 rows, 800 against 730 us.  Splitting and loading in pieces between the MFMAs gave
// nothing (conv5 75 -> 78), nor did kernel values four pairs ahead.
//   - KT: the kernel size where it is compiled in (3, 5); 0 = any K.
//   - S: 1 = the tensor itself; 2, 4 = space to depth: the padded input is read as a tensor of S*S
//     times as many channels on a grid S times as coarse (channel = (ci, dh, dw)), which turns a
//     layer of stride S into an unpadded one of stride 1 with ceil(K/S) taps.
#include <algorithm>
#include <cmath>

#include "cct_internal.h"
#include "conv_fused_kc_common.h"
#include "gemm_common.h"
#include "split_bf16.h"

namespace cct {
namespace {

using namespace kc;
constexpr int CB = 48;  // bytes between cells in LDS, of each half of their channels
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes, dword aligned

// K tiles per channel group: the taps; an even number (a zero tile) where K is not compiled in and pairs of tiles stay
// inside a group
__host__ __device__ constexpr int tiles_per_group(int K) {
  return K == 3 || K == 5 ? K * K : (K * K + 1) / 2 * 2;
}

// For results that are not finite: the operands of a product (channel, tap i, j) in plain fp32.
__device__ __forceinline__ float kernel_value(const GemmTN& p, int g, int m, int ch, int tap) {
  const int grp = ch / CG;
  const unsigned short* a = reinterpret_cast<const unsigned short*>(p.A) + (long long)g * p.a_gs * 3 +
                            (((long long)(grp * tiles_per_group(p.gK) + tap) * 3) * p.Mpad + m) * CG + (ch - grp * CG);
  const long long term = (long long)p.Mpad * CG;
  return join_value(a[0], a[term], a[2 * term]);
}
struct Output {
  int m, n, r, c;
};
// The pixel that tap (i, j) of channel ch reads for output (n, r, c); null outside the tensor and for taps that
// exist only in the regrouped kernel of a strided layer (index >= oK).
template <int S>
__device__ __forceinline__ const float* pixel_of(const GemmTN& p, int g, int n, int r, int c, int ch, int i, int j) {
  int h = r * p.gs + i - p.gp, w = c * p.gs + j - p.gp;
  if (S > 1) {
    const int dh = (ch % (S * S)) / S, dw = ch % S;
    if (i * S + dh >= p.oK || j * S + dw >= p.oK) return nullptr;
    h = h * S + dh - p.x_pad;
    w = w * S + dw - p.x_pad;
  }
  if (h < 0 || h >= p.x_h || w < 0 || w >= p.x_w) return nullptr;
  return reinterpret_cast<const float*>(p.B) + (long long)n * p.x_img +
         (long long)((g * p.gCg + ch) / (S * S)) * p.x_plane + (long long)h * p.x_w + w;
}

// positions of a workgroup on 48 rows, four waves with 48 each, and of the wide form on 64 rows, two with 80
constexpr int kWide48 = 192, kWide64 = 160;
// cells per thread: sizes that are not compiled in take a third one (7 x 7 windows on wide rows)
constexpr int kCells(int KT) { return KT ? 2 : 3; }

template <int WAVES_M, int RB, int KT, int S, int MB, int BN>
__global__ __launch_bounds__(NT, 2) void conv_fused_split(GemmTN p, KcGeom fg, int tiles_m, int tiles_n) {
  constexpr int QU = kCells(KT);  // cells per thread and slot
  constexpr int MW = 16 * RB;     // rows of a wave
  constexpr int BM = MW * WAVES_M;
  constexpr int WAVES_N = 4 / WAVES_M;
  constexpr int WN = BN / (MB * WAVES_N);  // blocks of MB positions of a wave
  constexpr int QB = MW * MB / 256;        // a lane's results in a block column: quads of consecutive rows
  static_assert(WAVES_M * WAVES_N == 4, "4 waves per workgroup");
  static_assert(MB == 16 || (MB == 32 && RB == 2 && KT != 0), "32 x 32 blocks: waves of 32 rows, unrolled taps");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem_b[];
  unsigned char* Xs = smem_b;  // [2 slots][2 halves][R][CB]
  const int half_b = fg.R * CB, slot_b = 2 * half_b;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int lane_lo = lane & (MB - 1);                             // row / column inside a block
  const int lane_hi = lane >> 5;                                   // which tile of a pair the lane supplies
  const int lane_ch = MB == 16 ? (lane >> 4) & 1 : lane_hi;        // which half of a tile's 16 channels
  const int row4 = MB == 16 ? (lane >> 4) * 4 : lane_hi * 4;       // the lane's rows of a block: row4 .. row4 + 3
  auto quad = [](int i) { return MB == 16 ? 16 * i : 8 * i; };     // + this, for quad i

  // consecutive workgroup ids go round-robin over the 8 XCDs: give every XCD a contiguous run of
  // column tiles with the M tiles of one column tile next to each other (they share x through L2)
  int bid = blockIdx.x;
  {
    const int total = tiles_m * tiles_n;
    const int per = total >> 3, rem = total & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    bid = xcd * per + min(xcd, rem) + idx;
  }
  const int tile_n = bid / tiles_m;
  const int tile_m = bid - tile_n * tiles_m;
  const int g = blockIdx.y;
  const int m0 = tile_m * BM;

  // ---- which positions, images and output rows does this workgroup cover ---------------------
  const int P = p.gHout * p.gWout;
  int n0, ce;  // positions [n0, ce) of the chunk
  if (fg.tpi > 0) {
    const int img = tile_n / fg.tpi;
    n0 = img * P + (tile_n - img * fg.tpi) * BN;
    ce = min(n0 + BN, (img + 1) * P);
  } else {
    n0 = tile_n * BN;
    ce = min(n0 + BN, p.Ncols);
  }
  const int n_f = n0 / P;
  const int a_f = (n0 - n_f * P) / p.gWout;
  const int n_l = (ce - 1) / P;
  const int a_l = ((ce - 1) - n_l * P) / p.gWout;
  const int rows_first = ((n_f == n_l ? a_l : p.gHout - 1) - a_f) * p.gs + p.gK;
  const int len_first = rows_first * fg.Wp;
  const int len_full = ((p.gHout - 1) * p.gs + p.gK) * fg.Wp;
  const int rows_last = n_l == n_f ? rows_first : a_l * p.gs + p.gK;
  const int r_actual = (n_l == n_f ? 0 : len_first + (n_l - n_f - 1) * len_full) + rows_last * fg.Wp;

  // ---- staging: a thread owns cells tid and tid + 256 of every group.  A cell's byte offset inside
  // the tensor never changes; dead cells (padding, rows this workgroup does not need) get an offset
  // that fails the buffer range check and load as zero; the channel enters through the scalar offset
  // of the buffer load.  With S > 1 the pixels of a cell are dead one by one: rows lo_h .. ok_h - 1 and
  // columns lo_w .. ok_w - 1 of the cell exist.
  // (`slack` elements before the first image, so that a cell that starts in the padding has an offset)
  const long long slack = S > 1 ? (long long)p.x_pad * (p.x_w + 1) : 0;
  const float* Xb = reinterpret_cast<const float*>(p.B) + (long long)n_f * p.x_img - slack;
  unsigned voff[QU];
  int lo_h[QU], ok_h[QU], lo_w[QU], ok_w[QU];
#pragma unroll
  for (int u = 0; u < QU; ++u) {
    const int q = tid + u * NT;
    voff[u] = 0x80000000u;
    lo_h[u] = ok_h[u] = lo_w[u] = ok_w[u] = 0;
    if (q < r_actual) {
      int seg = 0, rem = q, a_lo = a_f;
      if (q >= len_first) {
        const int qq = q - len_first;
        seg = 1 + qq / len_full;
        rem = qq - (seg - 1) * len_full;
        a_lo = 0;
      }
      const int row = rem / fg.Wp, wp = rem - row * fg.Wp;
      int h = a_lo * p.gs + row - p.gp, w = wp - p.gp;
      if (h >= 0 && h < p.gH && w >= 0 && w < p.gW) {
        if (S > 1) {
          h = h * S - p.x_pad;
          w = w * S - p.x_pad;
          lo_h[u] = -h;
          lo_w[u] = -w;
          ok_h[u] = p.x_h - h;
          ok_w[u] = p.x_w - w;
        }
        voff[u] = (unsigned)((seg * p.x_img + slack + (long long)h * p.x_w + w) * 4);
      }
    }
  }
  // byte offset of channel c of group grp: a channel past the last one repeats it (its kernel values
  // are zero); S > 1: 16 channels are 16 / (S*S) whole planes
  const unsigned plane_b = (unsigned)p.x_plane * 4u, row_b = (unsigned)p.x_w * 4u;
  const __amdgpu_buffer_rsrc_t x_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Xb), 0, 0x7fffffff, 0x00020000);
  auto chan_b = [&](int grp, int c) -> unsigned {
    if (S == 1) return (unsigned)(g * p.gCg + min(grp * CG + c, p.gCg - 1)) * plane_b;
    constexpr int SS = S * S;
    const int pl = min(grp * (CG / SS) + c / SS, p.gCg / SS - 1);
    return (unsigned)(g * (p.gCg / SS) + pl) * plane_b + (unsigned)((c / S) % S) * row_b + (c % S) * 4u;
  };
  // no cell of this workgroup lies in the tensor's last image (padded: nor in its first), so loads of S
  // pixels may run past the ends of a row
  const bool inner = S > 1 && n_l + 1 < p.Ncols / P && (p.x_pad == 0 || n_f > 0);
  // step = 2 * (cell u) + (channel half): 8 channels of a cell
  auto stage_load = [&](float (&stg)[8], int grp, int step) {
    const int u = step >> 1, v = step & 1;
    if ((tid & ~63) + u * NT < fg.R) {  // whole waves; lanes past R hold dead cells
      const unsigned vo = voff[u];
      if (S > 1 && inner) {
        // S consecutive pixels of a row of the cell are S channels: one load; pixels beyond the
        // row (its neighbours', inside the tensor) are cleared when they are stored
#pragma unroll
        for (int e = 0; e < 8; e += S) {
          const int c = v * 8 + e;
          const int dh = (c / S) % S, vv = (int)(dh >= lo_h[u] && dh < ok_h[u] ? vo : 0x80000000u), co = (int)chan_b(grp, c);
          if constexpr (S == 4) {
            const f32x4 t = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, vv, co, 0));
#pragma unroll
            for (int k = 0; k < 4; ++k) stg[e + k] = t[k];
          } else if constexpr (S == 2) {
            const f32x2 t = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(x_rs, vv, co, 0));
            stg[e] = t[0];
            stg[e + 1] = t[1];
          }
        }
        return;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = v * 8 + e;
        unsigned vv = vo;
        if (S > 1) {
          const int dh = (c / S) % S, dw = c % S;
          vv = dh >= lo_h[u] && dh < ok_h[u] && dw >= lo_w[u] && dw < ok_w[u] ? vo : 0x80000000u;
        }
        stg[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(x_rs, (int)vv, (int)chan_b(grp, c), 0));
      }
    }
  };
  auto stage_store = [&](const float (&stg)[8], int slot, int step) {
    const int u = step >> 1, v = step & 1;
    const int q = tid + u * NT;
    if (q < fg.R) {
      u32x4 h, m, l;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        unsigned a, b, c;
        float x0 = stg[2 * e], x1 = stg[2 * e + 1];
        if (S > 1) {
          const int d0 = (2 * e) % S, d1 = (2 * e + 1) % S;
          x0 = d0 >= lo_w[u] && d0 < ok_w[u] ? x0 : 0.f;
          x1 = d1 >= lo_w[u] && d1 < ok_w[u] ? x1 : 0.f;
        }
        split_pair(x0, x1, &a, &b, &c);
        h[e] = a;
        m[e] = b;
        l[e] = c;
      }
      u32x4* dst = reinterpret_cast<u32x4*>(Xs + slot * slot_b + v * half_b + q * CB);
      dst[0] = h;
      dst[1] = m;
      dst[2] = l;
    }
  };
  {
    float first[2 * QU][8];
#pragma unroll
    for (int s = 0; s < 2 * QU; ++s) stage_load(first[s], 0, s);
#pragma unroll
    for (int s = 0; s < 2 * QU; ++s) stage_store(first[s], 0, s);
  }
  // per-lane byte offset of each owned position's cell
  const int bn = wave_n * WN * MB + lane_lo;
  int bbase[WN];
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const int col = n0 + bn + j * MB;
    int cb = 0;
    if (col < ce) {
      const int n = col / P, pix = col - n * P;
      const int r = pix / p.gWout, c = pix - r * p.gWout;
      const int seg = n == n_f ? 0 : len_first + (n - n_f - 1) * len_full;
      const int a_lo = n == n_f ? a_f : 0;
      cb = seg + (r - a_lo) * p.gs * fg.Wp + c * p.gs;
    }
    bbase[j] = cb * CB + lane_ch * half_b;
  }

  // ---- kernel-matrix operands straight from the pack (L2)
  const int tpg = KT ? KT * KT : tiles_per_group(p.gK);
  const int ktiles = fg.ngroups * tpg;
  const unsigned short* Abase = reinterpret_cast<const unsigned short*>(p.A) +
                                ((long long)g * p.a_gs * 3 + (long long)(m0 + wave_m * MW) * CG);
  const __amdgpu_buffer_rsrc_t a_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(Abase), 0, 0x7fffffff, 0x00020000);
  const unsigned term_b = (unsigned)p.Mpad * CG * 2u;
  const unsigned a_row = (lane_lo * CG + lane_ch * 8) * 2;  // bytes inside a term

  f32x4 out[QB][WN];  // the results
  if constexpr (MB == 16) {
    // The next group's four steps, FL at a time: loaded before one pair of tiles, stored before a later one, so that
    // the MFMAs between cover the way to memory.  Register budget decides FL; where it is short, 5 x 5 kernels have
    // the tiles to go one by one.
    constexpr int FL = KT != 0 && WAVES_M * RB <= 4 && RB == 2 && S == 1 && WN < 5 ? 4 : KT == 5 && RB * WN > 10 ? 1 : 2;  // KT == 0: one cell
    float stg[FL][8];

    // operands two pairs of tiles ahead
    const int pairs = (ktiles + 1) / 2;
    const unsigned a_voff = a_row + lane_hi * (3u * term_b);
    const unsigned a_half = lane_hi ? 0x80000000u : a_voff;  // the last tile has no partner: zeros
    u32x4 a[2][RB][3];
    const unsigned a_last = (unsigned)(pairs - 1) * (6u * term_b);
    unsigned so = 0;
    auto load_a = [&](int set) {  // the next pair, at the end the last one again
      const unsigned vo = so == a_last && (ktiles & 1) ? a_half : a_voff;
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          a[set][i][q] = __builtin_bit_cast(
              u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rs, (int)(vo + i * 16 * CG * 2), (int)(so + q * term_b), 0));
      so = min(so + 6u * term_b, a_last);
    };

    f32x4 acc_h[RB][WN], acc_c[RB][WN];  // h*h, and the corrections
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc_h[i][j][r] = acc_c[i][j][r] = 0.f;
    // The h*h chain rounds as it goes.  Waves with few blocks have the registers to break it every 8 pairs, which keeps
    // the error of small layers below that of the lowered layouts (their sums come in K or K*K parts: 11 images of
    // 27 x 27, two groups of 128 -> 48 channels, K = 5: 2-norm 2.2e-7 there, 3.4e-7 with one chain, 1.2e-7 with parts;
    // the time is the same within 1 %).  Against one fp32 chain a single one is a third of the error already.
    constexpr bool PARTS = RB * WN <= 10;
    f32x4 total[PARTS ? RB : 1][PARTS ? WN : 1];
    int left = 8;
    if constexpr (PARTS) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) total[i][j][r] = 0.f;
    }
    auto end_pair = [&]() {
      if constexpr (PARTS) {
        if (--left > 0) return;
        left = 8;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              total[i][j][r] += acc_h[i][j][r];
              acc_h[i][j][r] = 0.f;
            }
      }
    };

    load_a(0);
    load_a(1);

    // operand sets of B: FAR blocks are multiplied together while the next FAR are read; two where the registers
    // allow it, so that an accumulator's MFMAs are further apart (conv2's backward-data 612 -> 600 us; 32 rows need
    // more than the 168 registers of three workgroups per CU for it: held to them the loop spilled, 64 images of
    // 28 x 28, 256 -> 21 channels, K = 3, 125 us instead of 67).  `off`: where the lane's tile of the pair lies from
    // the position's first cell
    constexpr int NB = RB * WN <= 8 && S < 4 ? 4 : 2, FAR = NB / 2;
    u32x4 b[NB][3];
    auto read_b = [&](int set, int j, int off) {
      const u32x4* src = reinterpret_cast<const u32x4*>(Xs + bbase[j] + off);
#pragma unroll
      for (int q = 0; q < 3; ++q) b[set][q] = src[q];
    };
    auto mfma6 = [&](int set, int j, int bs) {  // FAR blocks from j
      __builtin_amdgcn_sched_barrier(0);
#define CCT_M(X, Y, ACC)                                                                                  \
    _Pragma("unroll") for (int jj = 0; jj < FAR; ++jj) _Pragma("unroll") for (int i = 0; i < RB; ++i)       \
        ACC[i][j + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                                           \
            __builtin_bit_cast(bf16x8, a[set][i][X]), __builtin_bit_cast(bf16x8, b[bs + jj][Y]), ACC[i][j + jj], 0, 0, 0)
      CCT_M(2, 0, acc_c);
      CCT_M(0, 2, acc_c);
      CCT_M(1, 1, acc_c);
      CCT_M(1, 0, acc_c);
      CCT_M(0, 1, acc_c);
      CCT_M(0, 0, acc_h);
#undef CCT_M
      __builtin_amdgcn_sched_barrier(0);
    };
    // One pair of tiles: FAR blocks' operands are read while the FAR before them are multiplied, the next pair's first
    // ones (at byte offset `nxt`) behind the last but FAR.  Where the next pair reads cells that were staged meanwhile
    // (`turn`) the workgroup meets before that read: every one of them has been published by then.
    auto multiply = [&](int set, int cur, int nxt, bool turn) {
#pragma unroll
      for (int j = 0; j < WN; j += FAR) {
        const int ahead = j + FAR, bs = (set * WN + ahead) % NB;
        if (ahead == WN && turn) __syncthreads();
#pragma unroll
        for (int jj = 0; jj < FAR; ++jj) {
          if (ahead < WN)
            read_b(bs + jj, ahead + jj, cur);
          else
            read_b(bs + jj, jj, nxt);
        }
        mfma6(set, j, (set * WN + j) % NB);
      }
    };
    static_assert(2 * WN % NB == 0, "block 0 of every other pair uses operand set 0");

    // ---- the tiles in turn: channel group, tap; groups alternate between the two slots.  A period of pairs begins
    // with channel group `grp`.  An odd number of taps (KT) makes it two groups, KK pairs, of which pair H takes the
    // last tap of the one and the first of the other; otherwise it is one group.
    constexpr int KK = KT * KT, H = KK / 2, NP = 2 * QU / FL;
    const int period = KT ? KK : tpg / 2;
    int* offsets = reinterpret_cast<int*>(Xs + 2 * slot_b);  // of a period's tiles, from the position's first cell
    for (int e = tid; e < 2 * period; e += NT) {
      const int tap = KT ? e % KK : e < fg.KK ? e : 0;  // zero tile: any cell of the group
      int off = (tap / p.gK * fg.Wp + tap % p.gK) * CB;
      // the only group's last tile has no partner: any cells, its kernel values are zeros
      if (KT && e >= KK) off = fg.ngroups == 1 ? 0 : off + slot_b;
      offsets[e] = off;
    }
    __syncthreads();  // slot 0 and the offsets are visible

    // Staging, before pair `pp` of a period; true: the next pair reads cells that this staged.  In the odd form the
    // workgroup meets once more behind pair H, before it stages into the slot that is free then.
    auto stage = [&](int pp, int grp) -> bool {
      if constexpr (KT != 0) {
        // phase f is stored before the (f + 1)-th of NP pairs spread over the group's share of the period; the next
        // phase's loads go out at once
        constexpr int N1 = H - 1, N2 = KK - 1 - H;
        unsigned events = 0;
#pragma unroll
        for (int f = 0; f < NP; ++f) events |= 1u << (f + 1) * N1 / NP | 1u << (H + (f + 1) * N2 / NP);
        if (!(events >> pp & 1)) return false;
        const bool late = pp >= H;
        const int to = grp + (late ? 2 : 1);
        if (to >= fg.ngroups) return false;
#pragma unroll
        for (int f = 0; f < NP; ++f) {
          if (pp == (f + 1) * N1 / NP || pp == H + (f + 1) * N2 / NP) {
            if (f == 0 && late) __syncthreads();  // nobody reads slot 0 any more
#pragma unroll
            for (int s = 0; s < FL; ++s) stage_store(stg[s], late ? 0 : 1, f * FL + s);
            if (f + 1 < NP || to + 1 < fg.ngroups)
#pragma unroll
              for (int s = 0; s < FL; ++s) stage_load(stg[s], f + 1 < NP ? to : to + 1, (f + 1) % NP * FL + s);
          }
        }
        return pp == H - 1 || pp == KK - 1;
      } else {
        static_assert(FL == 2 || KT != 0, "a cell at a time");
        if (grp + 1 >= fg.ngroups) return false;
        // cell f is loaded in pair f * step and stored in pair (f + 1) * step, the last one (and what a short group
        // leaves no pair for) in the group's last pair
        const int step = max(1, period / QU), slot = (grp + 1) & 1;
#pragma unroll
        for (int f = 0; f < QU; ++f) {
          if (f > 0 && pp == f * step) {
#pragma unroll
            for (int s = 0; s < 2; ++s) stage_store(stg[s], slot, 2 * (f - 1) + s);
          }
          if (pp == f * step) {
#pragma unroll
            for (int s = 0; s < 2; ++s) stage_load(stg[s], grp + 1, 2 * f + s);
          }
        }
        if (pp != period - 1) return false;
#pragma unroll
        for (int f = 0; f < QU; ++f) {
          if (f * step >= period) {
#pragma unroll
            for (int s = 0; s < 2; ++s) stage_load(stg[s], grp + 1, 2 * f + s);
          }
          if ((f + 1) * step >= period || f == QU - 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) stage_store(stg[s], slot, 2 * f + s);
          }
        }
        return true;
      }
    };
    if (KT != 0 && fg.ngroups > 1)
#pragma unroll
      for (int s = 0; s < FL; ++s) stage_load(stg[s], 1, s);
    int pp = 0, grp = 0, slot = 0;  // slot: KT == 0
    // the lane's offset of the pair `ahead` of this one, read from LDS a pair before it is needed
    auto offset = [&](int ahead) {
      const bool wraps = pp + ahead >= period;
      return offsets[2 * (wraps ? pp + ahead - period : pp + ahead) + lane_hi] + (!KT && wraps ? slot_b - slot : slot);
    };
    int cur = offset(0), nxt = offset(1);
#pragma unroll
    for (int j = 0; j < FAR; ++j) read_b(j, j, cur);
    auto pair = [&](int set) {
      const bool wraps = pp + 1 == period;
      const int then = offset(2);
      const bool turn = stage(pp, grp);
      multiply(set, cur, nxt, turn);
      load_a(set);
      cur = nxt;
      nxt = then;
      if (!KT && wraps) slot = slot_b - slot;
      pp = wraps ? 0 : pp + 1;
      grp += wraps ? (KT ? 2 : 1) : 0;
      end_pair();
    };
    for (int t = pairs; t > 1; t -= 2) {
      pair(0);
      pair(1);
    }
    if (pairs & 1) pair(0);

#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (PARTS) acc_h[i][j][r] += total[i][j][r];
          out[i][j][r] = acc_h[i][j][r] + acc_c[i][j][r];
        }
  } else {
    // The next group's four steps, FL at a time: loaded in one tile, stored in a later one
    constexpr int FL = KT == 5 ? 1 : S == 1 ? 4 : 2;
    float stg[FL][8];

    // kernel values AD tiles ahead
    constexpr int AD = KT == 3 ? 3 : 5;
    u32x4 a[AD][3];
    auto load_a = [&](int set, int t) {
      const unsigned so = (unsigned)min(t, ktiles - 1) * (3u * term_b);
#pragma unroll
      for (int q = 0; q < 3; ++q)
        a[set][q] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rs, (int)a_row, (int)(so + q * term_b), 0));
    };

    floatx16 acc_h[WN], acc_c[WN];  // h*h, and the corrections
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc_h[j][r] = acc_c[j][r] = 0.f;
    // Parts as above: a group of 3 x 3 or two, half a group of 5 x 5 or a whole one, the longer ones where there are many,
    // whose sum rounds too (2-norm, parts of 16 tiles -> these: 4 images of 28 x 28, 64 channels, K = 3 9.2e-8 -> 8.0e-8;
    // 49 of 13 x 13, 192 channels, K = 3 1.00e-7 -> 1.02e-7, with one group 0.95e-7, but 463 -> 480 us in conv1's
    // backward-data; 11 of 27 x 27, 48 channels, K = 5 9.6e-8 -> 9.2e-8; 4 of 13 x 13, 256 channels, K = 5 1.26e-7
    // -> 1.27e-7).  A group's part is added in the first tile of the next one, behind that tile's corrections: its last
    // MFMA is long done by then.
    constexpr bool PARTS = WN <= 2;
    floatx16 total[PARTS ? WN : 1];
    if constexpr (PARTS) {
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) total[j][r] = 0.f;
    }
    const bool short_parts = fg.ngroups <= (KT == 3 ? 4 : 8);
    auto end_part = [&](int j) {
      if constexpr (PARTS) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          total[j][r] += acc_h[j][r];
          acc_h[j][r] = 0.f;
        }
      }
    };

#pragma unroll
    for (int e = 0; e < AD; ++e) load_a(e, e);
    __syncthreads();  // slot 0 is visible

    // operand sets of B: the two blocks that are read and multiplied in turn; with one block per tile
    // the set goes with the tile
    constexpr int NB = WN == 1 ? AD : 2;
    u32x4 b[NB][3];
    auto read_b = [&](int set, int j, int off) {
      const u32x4* src = reinterpret_cast<const u32x4*>(Xs + bbase[j] + off);
#pragma unroll
      for (int q = 0; q < 3; ++q) b[set][q] = src[q];
    };
    read_b(0, 0, 0);
    int slot = 0;

    // One tile: block j's operand is read while block j - 1 is multiplied, the next tile's first
    // block (at byte offset `nxt`) behind the last but one; the registers of this tile's A operand are
    // reloaded with tile t + AD behind its last MFMA.  In the last tile of a group (`turn`) the
    // workgroup meets before the next group's first read: every cell of it has been published by
    // then, and nobody reads the other slot's old cells any more.
    auto mfma6 = [&](int set, int bs, int j, bool next_part) {
      __builtin_amdgcn_sched_barrier(0);
#define CCT_M(X, Y, ACC)                                                                       \
    ACC = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[set][X]),          \
                                                  __builtin_bit_cast(bf16x8, b[bs][Y]), ACC, 0, 0, 0)
      CCT_M(2, 0, acc_c[j]);
      CCT_M(0, 2, acc_c[j]);
      CCT_M(1, 1, acc_c[j]);
      CCT_M(1, 0, acc_c[j]);
      CCT_M(0, 1, acc_c[j]);
      if (next_part) end_part(j);
      CCT_M(0, 0, acc_h[j]);
#undef CCT_M
      __builtin_amdgcn_sched_barrier(0);
    };
    auto tile = [&](int set, int t, int cur, int nxt, bool turn, bool next_part) {
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        if (j + 1 < WN) {
          read_b((j + 1) & 1, j + 1, cur);
        } else {
          if (turn) __syncthreads();
          read_b(WN == 1 ? (set + 1) % AD : 0, 0, nxt);
        }
        mfma6(set, WN == 1 ? set : j & 1, j, next_part);
      }
      load_a(set, t + AD);
    };
    static_assert(WN == 1 || WN % 2 == 0, "block 0 of every tile uses operand set 0");

    constexpr int KK = KT * KT;
    for (int grp = 0; grp < fg.ngroups; ++grp) {
      const bool more = grp + 1 < fg.ngroups;
      const int base = slot * slot_b, other = (slot ^ 1) * slot_b;
#pragma unroll
      for (int tt = 0; tt < KK; ++tt) {
        if (more) {
          constexpr int NP = 2 * QU / FL;  // phases; phase f is loaded at f * KK / NP, stored before the next
#pragma unroll
          for (int f = 0; f < NP; ++f) {
            if (tt == (f + 1) * (KK - 1) / NP)
#pragma unroll
              for (int s = 0; s < FL; ++s) stage_store(stg[s], slot ^ 1, f * FL + s);
            if (tt == f * (KK - 1) / NP)
#pragma unroll
              for (int s = 0; s < FL; ++s) stage_load(stg[s], grp + 1, f * FL + s);
          }
        }
        const int ti = tt / KT, tj = tt % KT, ni = (tt + 1) / KT, nj = (tt + 1) % KT;
        const bool last = tt == KK - 1;
        tile(tt % AD, grp * KK + tt, base + (ti * fg.Wp + tj) * CB,
             last ? (more ? other : base) : base + (ni * fg.Wp + nj) * CB, last && more,
             tt == 0 && (KT == 5 || short_parts || !(grp & 1)));
        if (KT == 5 && tt == KK / 2 && short_parts)
#pragma unroll
          for (int j = 0; j < WN; ++j) end_part(j);
      }
      if (more) slot ^= 1;
    }
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (PARTS) acc_h[j][r] += total[j][r];
        out[r / 4][j][r % 4] = acc_h[j][r] + acc_c[j][r];
      }
  }

  // ---- epilogue: Type-1 lifting + bias, or the depth-to-space store of a strided backward-data
  // pass
  const int mw = m0 + wave_m * MW;
  float check = 0.f;  // NaN once a result is not finite
#pragma unroll
  for (int i = 0; i < QB; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        check = fmaf(out[i][j][r], 0.f, check);
        out[i][j][r] *= kSplitUnscale;
      }
  if (p.d2s) {
    float* __restrict__ D = p.C;
    const int ss = p.dS * p.dS;
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int col = n0 + bn + j * MB;
      if (col >= ce) continue;
      const int n = col / P, pix = col - n * P;
      const int ga = pix / p.gWout, gb = pix - ga * p.gWout;
      const long long img = ((long long)n * p.dCtot + (long long)g * p.dCg) * p.dH;
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        // the lane's four consecutive rows m .. m+3 (m a multiple of 4)
        const int m = mw + quad(i) + row4;
        if (m >= p.M) continue;
        const int ci = fdiv_u(m, p.d_divSS_M, p.d_divSS_sh), rem = m - ci * ss;
        const int rh = fdiv_u(rem, p.d_divS_M, p.d_divS_sh), rw = rem - rh * p.dS;
        const int h = ga * p.dS + rh - p.dP, w = gb * p.dS + rw - p.dP;
        float* dst = D + ((img + (long long)ci * p.dH) + h) * p.dW + w;
        if ((p.dS & 3) == 0) {
          // stride a multiple of 4: the four rows are four consecutive pixels of one row of dx
          if ((unsigned)h >= (unsigned)p.dH) continue;
          if (w >= 0 && w + 3 < p.dW && m + 3 < p.M) {
            *reinterpret_cast<f32x4u*>(dst) = out[i][j];  // 4-byte aligned
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (m + e < p.M && (unsigned)(w + e) < (unsigned)p.dW) dst[e] = out[i][j][e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int me = m + e;
            if (me < p.M) {
              const int cie = fdiv_u(me, p.d_divSS_M, p.d_divSS_sh), reme = me - cie * ss;
              const int rhe = fdiv_u(reme, p.d_divS_M, p.d_divS_sh), rwe = reme - rhe * p.dS;
              const int he = ga * p.dS + rhe - p.dP, we = gb * p.dS + rwe - p.dP;
              if ((unsigned)he < (unsigned)p.dH && (unsigned)we < (unsigned)p.dW)
                D[((img + (long long)cie * p.dH) + he) * p.dW + we] = out[i][j][e];
            }
          }
        }
      }
    }
  } else {
    float* __restrict__ C = p.C + (long long)g * p.c_gs;
    const float* bias = p.bias ? p.bias + (long long)g * p.bias_gs : nullptr;
    const bool full_m = m0 + BM <= p.M;
    float bv[QB * 4];
    load_bias(bv, bias, p.M - 1, [&](int r) { return mw + row4 + quad(r / 4) + r % 4; });
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int col = n0 + bn + j * MB;
      if (col >= ce) continue;
      float* __restrict__ cl = C + col_offset(p.cmap, col) + (long long)(mw + row4) * p.c_ms;
#pragma unroll
      for (int i = 0; i < QB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = quad(i) + r;  // relative to mw + row4
          if (full_m || mw + row + row4 < p.M) cl[(long long)row * p.c_ms] = out[i][j][r] + bv[i * 4 + r];
        }
    }
  }
  if (!__any(check != check)) return;
  __threadfence_block();  // what the other lanes have stored is read below

  // ---- Blocks with results that are not finite: again in plain fp32 (split_bf16.h).  A block of fp32 products
  // costs a few times one of split ones whatever is in it (256 images of conv3 with one infinity each: 331 us
  // without, 4.3 ms with it).  It also multiplies zeros that stand for no pixel or no tap: where one may have met
  // a value that is not finite, a NaN is summed once more without them.
  constexpr int WB = (WN * MB + 31) / 32;
  const int wave_end = min(ce, n0 + (wave_n + 1) * WN * MB);
#pragma unroll 1
  for (int blk = 0; blk < WB * ((RB + 1) / 2); ++blk) {
    // 32 rows x 32 positions (the last ones may be another wave's: not looked at)
    const int r0 = mw + blk / WB * 32, rows_end = min(mw + MW, p.M), lo = lane & 31;
    const int col = n0 + wave_n * WN * MB + blk % WB * 32 + lo;
    const int n = min(col, ce - 1) / P, pix = min(col, ce - 1) - n * P, r_ = pix / p.gWout, c_ = pix - r_ * p.gWout;
    auto address = [&](int m) -> float* {  // null: no such result
      if (col >= wave_end || m >= rows_end) return nullptr;
      if (!p.d2s) return p.C + (long long)g * p.c_gs + col_offset(p.cmap, col) + (long long)m * p.c_ms;
      const int ss = p.dS * p.dS, ci = m / ss, rem = m - ci * ss;
      const int h = r_ * p.dS + rem / p.dS - p.dP, w = c_ * p.dS + rem % p.dS - p.dP;
      if ((unsigned)h >= (unsigned)p.dH || (unsigned)w >= (unsigned)p.dW) return nullptr;
      return p.C + (((long long)n * p.dCtot + (long long)g * p.dCg + ci) * p.dH + h) * p.dW + w;
    };
    int first = r0 + lane_hi * 4;
    asm volatile("" : "+v"(first));  // what depends on the rows is not kept for all blocks
    auto row = [&](int r) { return first + (r >> 2) * 8 + (r & 3); };
    auto store = [&](int r, float v) {
      if (!p.d2s && p.bias) v += p.bias[(long long)g * p.bias_gs + row(r)];
      *address(row(r)) = v;
    };
    unsigned todo = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* at = address(row(r));
      if (at && !finite(*at)) todo |= 1u << r;
    }
    if (!__any(todo)) continue;
    // step = (pair of channels, tap); which rows and columns hold values that are not finite, which columns
    // read outside the tensor
    bool a_bad = false, b_bad = false, b_out = false;
    auto doubts = [&]() {  // the results whose NaN may come from a zero that is no product
      const unsigned long long bad_rows = __ballot(a_bad), bad_cols = __ballot(b_bad), out_cols = __ballot(b_out);
      auto halves = [](unsigned long long v) { return (unsigned)(v | v >> 32); };
      if (p.d2s && halves(bad_cols) >> lo & 1) return 0xffffu;
      if (!(halves(out_cols) >> lo & 1)) return 0u;
      const unsigned rows = halves(bad_rows) >> (lane_hi * 4);
      return (rows & 0xfu) | (rows >> 4 & 0xf0u) | (rows >> 8 & 0xf00u) | (rows >> 12 & 0xf000u);
    };
    const floatx16 v = fp32_block(
        (p.gCg + 1) / 2 * fg.KK,
        [&](int s) {
          const int ch = s / fg.KK * 2 + lane_hi;
          const float a = ch < p.gCg ? kernel_value(p, g, min(r0 + lo, p.Mpad - 1), ch, s % fg.KK) : 0.f;
          a_bad |= !finite(a);
          return a;
        },
        [&](int s) {
          const int ch = s / fg.KK * 2 + lane_hi, tap = s % fg.KK;
          const float* at = ch < p.gCg ? pixel_of<S>(p, g, n, r_, c_, ch, tap / p.gK, tap % p.gK) : nullptr;
          b_out |= !at;
          const float b = at ? *at : 0.f;
          b_bad |= !finite(b);
          return b;
        },
        [&](const floatx16& acc) { return numbers(acc, todo) | (todo & doubts()); });
    const unsigned doubt = doubts();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (!(todo >> r & 1) || (v[r] != v[r] && (doubt >> r & 1))) continue;
      store(r, v[r]);
      todo &= ~(1u << r);
    }
    for (int r = 0; r < 16; ++r) {
      const bool mine = todo >> r & 1;
      if (!__any(mine)) continue;
      const float sum = fp32_sum(
          mine, p.gCg * fg.KK,
          [&](int who) {
            return Output{r0 + (r >> 2) * 8 + (who >> 5) * 4 + (r & 3), __shfl(n, who, 64), __shfl(r_, who, 64),
                          __shfl(c_, who, 64)};
          },
          [&](const Output& o, int k, float* x, float* y) {
            const int ch = k / fg.KK, tap = k - ch * fg.KK, i = tap / p.gK, jj = tap - i * p.gK;
            const float* at = pixel_of<S>(p, g, o.n, o.r, o.c, ch, i, jj);
            if (!at) return false;
            if (p.d2s) {
              const int rem = o.m % (p.dS * p.dS), rh = rem / p.dS, rw = rem % p.dS;
              if (rh + p.dS * (p.gK - 1 - i) >= p.oK || rw + p.dS * (p.gK - 1 - jj) >= p.oK) return false;
            }
            *x = kernel_value(p, g, o.m, ch, tap);
            *y = *at;
            return true;
          });
      if (mine) store(r, sum);
    }
  }
}

// The three terms of a kernel matrix in the layout above: pack[q][tile][term][m][16], zero padded in
// m, in the channels of the last group and in the tiles beyond a group's taps.
//   kind 0: m = kernel oo, channel = input channel ci, value w[oo, ci, i, j]
//   kind 1 (backward-data, stride 1): m = input channel, channel = kernel, w[oo, ci, K-1-i, K-1-j]
//   kind 2 (backward-data, stride s): m = (ci*s + rh)*s + rw, channel = kernel,
//           w[oo, ci, rh + s*(U-1-i), rw + s*(U-1-j)], 0 where that index reaches K
//   kind 3 (space to depth): m = kernel, channel = (ci*s + dh)*s + dw, w[oo, ci, i*s + dh, j*s + dw],
//           0 where that index reaches K
struct SplitPack {
  int kind, G, Og, Cg, K, s, U, Mpad, tpg, ngroups;
};
__global__ __launch_bounds__(256) void pack_split_kernel(const float* __restrict__ w,
                                                         unsigned short* __restrict__ pack, SplitPack d) {
  const long long per_group = (long long)d.ngroups * d.tpg * d.Mpad * CG;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= per_group * d.G) return;
  const int q = (int)(t / per_group);
  long long e = t - q * per_group;
  const int c = (int)(e % CG);
  e /= CG;
  const int m = (int)(e % d.Mpad);
  const int tile = (int)(e / d.Mpad);
  const int grp = tile / d.tpg, tap = tile - grp * d.tpg;
  const int i = tap / d.U, j = tap - i * d.U;
  const int ch = grp * CG + c;
  int oo = m, ci = ch, wi = i, wj = j;
  if (d.kind == 1) {
    oo = ch; ci = m; wi = d.K - 1 - i; wj = d.K - 1 - j;
  } else if (d.kind == 2) {
    const int ss = d.s * d.s, rem = m % ss;
    oo = ch; ci = m / ss;
    wi = rem / d.s + d.s * (d.U - 1 - i);
    wj = rem % d.s + d.s * (d.U - 1 - j);
  } else if (d.kind == 3) {
    const int ss = d.s * d.s, rem = ch % ss;
    ci = ch / ss;
    wi = i * d.s + rem / d.s;
    wj = j * d.s + rem % d.s;
  }
  float v = 0.0f;
  if (i < d.U && oo < d.Og && ci < d.Cg && wi >= 0 && wi < d.K && wj >= 0 && wj < d.K)
    v = w[((((long long)q * d.Og + oo) * d.Cg + ci) * d.K + wi) * d.K + wj];
  unsigned short h, mm, l;
  split_value(v, &h, &mm, &l);
  unsigned short* dst = pack + ((((long long)q * d.ngroups * d.tpg + tile) * 3) * d.Mpad + m) * CG + c;
  const long long term = (long long)d.Mpad * CG;
  dst[0] = h;
  dst[term] = mm;
  dst[2 * term] = l;
}

inline long long column_tiles(const GemmTN& p, const KcGeom& fg, long long nimg, int bn = BN) {
  const long long P = (long long)p.gHout * p.gWout;
  return fg.tpi > 0 ? fg.tpi * nimg : (P * nimg + bn - 1) / bn;
}

template <int WAVES_M, int RB, int KT, int S, int MB, int POS = BN>
int launch_variant(const GemmTN& p, const KcGeom& fg, size_t lds, hipStream_t st) {
  constexpr int BM = 16 * RB * WAVES_M;
  const int tiles_m = (p.M + BM - 1) / BM;
  if (tiles_m * BM > p.Mpad) return CCT_EINVAL;  // the pack's rows
  const long long tn = column_tiles(p, fg, p.Ncols / (p.gHout * p.gWout), POS);
  const long long blocks = (long long)tiles_m * tn;
  if (blocks <= 0 || blocks >= 2147483647LL || p.G > 65535) return CCT_EUNSUPPORTED;
  dim3 grid((unsigned)blocks, (unsigned)p.G);
  const double nimg = (double)p.Ncols / (p.gHout * p.gWout);
  const double x_bytes = 4.0 * nimg * p.x_img;
  const double y_bytes = p.d2s ? 4.0 * nimg * p.dCtot * p.dH * p.dW : 4.0 * (double)p.M * p.Ncols * p.G;
  ProfScope ps(p.prof_flops > 0 ? p.prof_flops : 2.0 * p.M * p.Ncols * p.Kdim * p.G,
               x_bytes + y_bytes + 4.0 * (double)p.M * p.Kdim * p.G, st,
               "conv_fused_split<%d, %d, %d, %d, %d%s>%s", WAVES_M, RB, KT, S, MB,
               POS == kWide64 ? ", wide" : "", p.d2s ? " strided" : "");
  constexpr auto kern = conv_fused_split<WAVES_M, RB, KT, S, MB, POS>;
  if (const int rc = ensure_dynamic_lds<kern>(2 * kLdsCap)) return rc;
  hipLaunchKernelGGL(kern, grid, dim3(NT), lds, st, p, fg, tiles_m, (int)tn);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

template <int WAVES_M, int RB, int MB>
int launch_rows(const GemmTN& p, const KcGeom& fg, size_t lds, hipStream_t st) {
  if (p.s2d == 4) {
    if (p.gK == 3) return launch_variant<WAVES_M, RB, 3, 4, MB>(p, fg, lds, st);
    return p.gK == 5 ? CCT_EUNSUPPORTED : launch_variant<WAVES_M, RB, 0, 4, 16>(p, fg, lds, st);
  }
  if (p.s2d == 2) {
    if (p.gK == 3) return launch_variant<WAVES_M, RB, 3, 2, MB>(p, fg, lds, st);
    return p.gK == 5 ? CCT_EUNSUPPORTED : launch_variant<WAVES_M, RB, 0, 2, 16>(p, fg, lds, st);
  }
  if (p.gK == 3) return launch_variant<WAVES_M, RB, 3, 1, MB>(p, fg, lds, st);
  if (p.gK == 5) return launch_variant<WAVES_M, RB, 5, 1, MB>(p, fg, lds, st);
  return launch_variant<WAVES_M, RB, 0, 1, 16>(p, fg, lds, st);
}

// the kernel size where it is compiled in
inline int compiled_k(const GemmTN& p) { return p.gK == 3 || (p.gK == 5 && !p.s2d) ? p.gK : 0; }

bool split_geom(const GemmTN& p, KcGeom* fg, size_t* lds, int bn = BN) {
  // one tap: a period of one pair, while the kernel reads offsets two pairs ahead (1 x 1 kernels have no windows to stage)
  if (p.gK < 2) return false;
  // the pack of one group is addressed with 32-bit byte offsets
  if (p.bf16 || (long long)p.Mpad * p.Kpad * 6 >= (1LL << 31)) return false;
  // Rows and channels are padded to whole tiles and groups: below two fifths of useful work the fp32 fused
  // kernels and the products on materialised matrices are the faster ones (160 images of 55 x 55, 8 channels
  // padded to 16 and 38 kernels to 64: 124 us against 184; half of it useful, 16 kernels on 352 channels,
  // 30 images of 52 x 52: 222 against 117).
  if (5LL * p.M * p.gCg < 2LL * p.Mpad * ((p.gCg + CG - 1) / CG * CG)) return false;
  // Regrouped, an image holds only the pixels that the kernels reach: the real one, which the staged cells are
  // addressed in (32-bit byte offsets from the workgroup's first image), may be larger.
  if (p.s2d) {
    const long long T = (bn - 1) / ((long long)p.gHout * p.gWout) + 2;  // images bn positions can touch
    if ((T + 1) * p.x_img + (long long)p.x_pad * (p.x_w + 1) >= (1LL << 29)) return false;
  }
  if (p.s2d && p.gK == 5) return false;  // kernels of 9 and 10 (stride 2), 17 to 20 (stride 4): no form
  GeomRules rules;
  rules.bn = bn;
  rules.r_step = 16;  // half a slot is a multiple of 256 bytes
  rules.qu = kCells(compiled_k(p));
  // what else runs these layers is at most half as fast, so up to half of a group's channels may be
  // padding, and a quarter of the positions
  rules.chan_num = 2; rules.chan_den = 1;
  rules.tpi_num = 5; rules.tpi_den = 4;
  // two workgroups per CU where the staged rows allow it
  // make_geom counts 4 bytes per tap for a table: the offsets take 8
  const int table = 4 * p.gK * p.gK + 8;
  if (!kc::make_geom(p, 0, 2 * CB, fg, lds, kLdsCap - table, rules) &&
      !kc::make_geom(p, 0, 2 * CB, fg, lds, 2 * kLdsCap - 1024 - table, rules))
    return false;
  *lds += table;
  return true;
}

inline int row_tiles(const GemmTN& p, int BM) { return (p.M + BM - 1) / BM; }

// workgroups that registers (165 of the smallest unrolled form) and LDS let share a CU
inline int workgroups_per_cu(const GemmTN& p, size_t lds, int rows) {
  return std::max(1, std::min(rows == 32 && compiled_k(p) == 3 && p.s2d < 4 ? 3 : 2, (int)(160 * 1024 / lds)));
}

// Edge of the MFMA's blocks: unrolled taps in blocks of 32 x 32 where a workgroup has its CU alone, by its cells (64 and
// 128 rows 0.86 to 0.89 times the time of 16 x 16) or, on 64 rows, because at most half of the CUs get a second one, and on
// 32 rows at any size (0.85 to 1.0).  Beyond that the matrix cores run into the power limit, where 16 x 16 are the faster
// ones.  64 rows, 64 channels of 27 x 27, K = 3: 274 workgroups 0.93, 365 0.94 and 0.96, 399 0.95 and 0.98, 479 0.99 and
// 1.02 times; K = 5: 288 0.93, 384 0.95, 504 1.00 and 1.01; conv4 at batch 256 1.05.  128 rows: 476 workgroups 1.03, 1600
// 1.09.  The limit shows in runs of one kernel that last: bursts of 0.4 ms in turn with another form had 32 x 32 ahead by
// 5 % on 64 rows at any size.
inline int split_block(const GemmTN& p, size_t lds, long long tn, int rows) {
  if (!compiled_k(p) || rows == 96 || rows == 48) return 16;
  if (rows == 32 || workgroups_per_cu(p, lds, rows) == 1) return 32;
  return rows == 64 && tn * row_tiles(p, rows) * p.G <= 384 ? 32 : 16;
}

// A launch: rows of a workgroup, edge of the MFMA's blocks, what it is estimated to take, kWide64 positions on 64 rows.
struct Tile {
  int rows, block;
  double us;
  bool wide;
};

// Rounds of workgroups, each as long as the chain of one: us per K tile of a workgroup that has its CU alone, what
// every further one on the CU adds, and per round to fill and drain; per channel group the staging that its tiles do
// not hide, and what each cell of a thread beyond the first adds to that; the two launches; 9 us per million values of
// the pack.  Fitted to 58900 launches of 24800 passes (1 to 512 images of up to 240 x 240, each pass with every tile that
// it can take), without what memory bounds: off by 5 to 7 % in the mean and by up to 11 to 16 % in nine of ten, by form.
// 64 rows were fitted in blocks of 32 x 32; in 16 x 16 they are within 5 % of that (split_block).
Tile estimate(const GemmTN& p, const KcGeom& fg, size_t lds, long long tn, int rows, bool wide = false) {
  struct Rate {
    double tile, next, fill;
  };
  struct Form {
    Rate of[7];  // 32, 64, 96, 128 rows, 128 rows in 32 x 32 blocks, 48 rows, the wide form
    double group, cell, launches;
  };
  static constexpr Form forms[5] = {
      // any K, 3, 5; regrouped: any K, 3
      {{{0.172, 0.076, 4.3}, {0.266, 0.144, 6.6}, {0.370, 0.210, 9.0}, {0.461, 0.294, 10.7}, {}}, 0.90, 0.49, 3.5},
      {{{0.206, 0.118, 3.6}, {0.278, 0.215, 6.2}, {0.460, 0.250, 8.3}, {0.551, 0.333, 9.8}, {0.451, 0.468, 8.3}, {0.313, 0.285, 7.0}, {0.348, 0.150, 6.6}}, 0.0, 0.36, 3.9},
      {{{0.149, 0.117, 4.5}, {0.229, 0.232, 7.1}, {0.414, 0.245, 9.6}, {0.512, 0.312, 11.4}, {0.382, 0.469, 12.2}, {0.258, 0.310, 8.0}, {0.270, 0.175, 7.6}}, 0.0, 0.0, 3.2},
      {{{0.177, 0.063, 3.5}, {0.274, 0.116, 7.1}, {0.369, 0.192, 11.1}, {0.467, 0.280, 14.3}, {}}, 1.28, 0.80, 5.9},
      {{{0.242, 0.091, 3.3}, {0.319, 0.173, 6.2}, {0.505, 0.213, 8.7}, {0.578, 0.304, 11.6}, {0.524, 0.385, 10.8}}, 0.0, 0.73, 6.1}};
  const int S = p.s2d ? p.s2d : 1, KT = compiled_k(p);
  const Form& f = forms[S > 1 ? (KT ? 4 : 3) : KT == 3 ? 1 : KT == 5 ? 2 : 0];
  const int share = workgroups_per_cu(p, lds, rows), block = wide ? 16 : split_block(p, lds, tn, rows);
  const Rate& r = f.of[wide ? 6 : rows == 48 ? 5 : rows == 128 && block == 32 ? 4 : rows / 32 - 1];
  const long long per_cu = (tn * row_tiles(p, rows) * p.G + 255) / 256;
  const double tiles = (double)fg.ngroups * tiles_per_group(p.gK);
  const double staging = fg.ngroups * (f.group + f.cell * ((fg.R + NT - 1) / NT - 1) + (p.gs > 1 ? 0.9 : 0.0));
  auto round = [&](long long n) { return n ? tiles * (r.tile + (double)(n - 1) * r.next) + staging + r.fill : 0.0; };
  return {rows, block, (double)(per_cu / share) * round(share) + round(per_cu % share) + f.launches +
                           9.0e-6 * p.G * p.Mpad * tiles * CG,
          wide};
}

// The largest row tile that puts a workgroup on every CU (464 rows, 57 column tiles: 64 rows 18.2 us, 96 23.7).  Where
// the rows pad less in tiles of 96 than of 128 the estimates choose between the two (450 kernels run as 5 tiles of 96
// or 4 of 128, which have the higher rate: of 62 such passes that took 128 rows, 0.92 times the time of 96).  Smaller tiles
// are not weighed against larger ones: they sum in parts, the larger ones do not, and a layer keeps the precision that
// it has (129 to 192 rows as two tiles of 96 would take 0.95 times as long as three of 64).
Tile split_tile(const GemmTN& p, KcGeom* geom, size_t* lds_bytes, long long nimg) {
  const KcGeom fg = *geom;
  const size_t lds = *lds_bytes;
  const long long tn = column_tiles(p, fg, nimg);
  auto fills = [&](int rows) { return tn * row_tiles(p, rows) * p.G >= 256; };
  int rows = p.Mpad % 128 == 0 ? 128 : p.Mpad % 64 == 0 ? 64 : 32;
  while (rows > 32 && !fills(rows)) rows /= 2;
  const Tile t = estimate(p, fg, lds, tn, rows);
  // 41 to 48 rows, 137 to 144: tiles of 48 x 192 instead of 64 x 128, where their cells leave room for two workgroups
  // per CU (without: 1.0 to 1.3 times the time, 185 images of 65 x 65, 204 -> 42 channels, K = 3 922 -> 1046 us) and the
  // launch is large enough for 16 x 16 blocks, which sum in the same parts.  Of 62 such layers 0.73 to 0.97 times the
  // time, conv2's backward-data 641 -> 527 us, conv1's 501 -> 402.  (From 33 rows it is still ahead, 140 images of 43 x 43,
  // 249 -> 35 channels 382 -> 316; that 40 kernels run on 64 rows is pinned by what tests the forms.)
  if (t.block == 16 && rows == 64 && compiled_k(p) && !p.s2d && p.M > row_tiles(p, 48) * 48 - 8 &&
      10 * row_tiles(p, 48) * 48 <= 9 * row_tiles(p, 64) * 64) {
    KcGeom wide;
    size_t wide_lds;
    if (!split_geom(p, &wide, &wide_lds, kWide48) || wide_lds > kLdsCap) return t;
    const Tile t48 = estimate(p, wide, wide_lds, column_tiles(p, wide, nimg, kWide48), 48);
    if (t.us <= t48.us) return t;
    *geom = wide;
    *lds_bytes = wide_lds;
    return t48;
  }
  // 64 rows x 160 positions instead of x 128 where that saves a round of workgroups or the launch is long, again where 16 x
  // 16 blocks sum in the same parts: the wave's kernel values serve five blocks instead of four.  Of 90 such layers the
  // estimates choose the faster one but for 0.1 % of the time in the mean (3.6 % at most): 33 images of 34 x 34, 236 ->
  // 122 channels, K = 3, 598 workgroups or 478, 84 -> 64 us; 63 of 34 x 34, 241 -> 53, K = 5, 343 -> 265; 65 of 39 x 39,
  // 268 -> 374 535 -> 486; with as many rounds as before it loses (76 images of 33 x 33, 193 -> 56, 129 -> 147).  Few
  // channel groups stay, which fill and drain more than they multiply.
  if (rows == 64 && t.block == 16 && compiled_k(p) && !p.s2d && fg.ngroups > (p.gK == 3 ? 4 : 8)) {
    KcGeom wide;
    size_t wide_lds;
    if (split_geom(p, &wide, &wide_lds, kWide64) && wide_lds <= kLdsCap) {
      const Tile tw = estimate(p, wide, wide_lds, column_tiles(p, wide, nimg, kWide64), 64, true);
      if (tw.us < 0.95 * t.us) {
        *geom = wide;
        *lds_bytes = wide_lds;
        return tw;
      }
    }
  }
  if (rows < 128 || row_tiles(p, 96) * 96 >= row_tiles(p, 128) * 128) return t;
  const Tile t96 = estimate(p, fg, lds, tn, 96);
  return t.us < 0.97 * t96.us ? t : t96;
}

}  // namespace

int conv_fused_split_mpad(int M) { return M <= 32 ? 32 : (M + 63) / 64 * 64; }

long long conv_fused_split_kpad(int channels_per_group, int K) {
  return (long long)((channels_per_group + CG - 1) / CG) * tiles_per_group(K) * CG;
}

bool conv_fused_split_fits(const GemmTN& p) {
  KcGeom fg;
  size_t lds;
  return split_geom(p, &fg, &lds);
}

double conv_fused_split_seconds(const GemmTN& p, int nimg) {
  KcGeom fg;
  size_t lds;
  if (!split_geom(p, &fg, &lds)) return 1.0;
  return 1e-6 * split_tile(p, &fg, &lds, nimg).us;
}

int launch_pack_split(const float* w, void* pack, int kind, int G, int Og, int Cg, int K, int s, int Mpad,
                      hipStream_t st) {
  const int U = kind >= 2 ? (K + s - 1) / s : K;
  const int channels = kind == 1 || kind == 2 ? Og : kind == 3 ? Cg * s * s : Cg;
  SplitPack d{kind, G, Og, Cg, K, s, U, Mpad, tiles_per_group(U), (channels + CG - 1) / CG};
  const long long total = (long long)G * d.ngroups * d.tpg * Mpad * CG;
  const long long blocks = (total + 255) / 256;
  if (blocks <= 0 || blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  ProfScope ps("pack_split_kernel", 0.0, 4.0 * G * Og * Cg * K * K + 6.0 * total, st);
  hipLaunchKernelGGL(pack_split_kernel, dim3((unsigned)blocks), dim3(256), 0, st, w,
                     reinterpret_cast<unsigned short*>(pack), d);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

// p.A must have been written by launch_pack_split with Mpad = conv_fused_split_mpad(M);
// p.Kpad = conv_fused_split_kpad(...).
int launch_conv_fused_split(const GemmTN& p0, hipStream_t st) {
  GemmTN p = p0;
  colmap_prepare(&p.bmap);
  colmap_prepare(&p.cmap);
  if (p.d2s) {
    if (p.dS < 1 || p.M != p.dCg * p.dS * p.dS) return CCT_EINVAL;
    make_fastdiv_parts(p.dS * p.dS, &p.d_divSS_M, &p.d_divSS_sh);
    make_fastdiv_parts(p.dS, &p.d_divS_M, &p.d_divS_sh);
  }
  KcGeom fg;
  size_t lds;
  if (p.Mpad != conv_fused_split_mpad(p.M) || !split_geom(p, &fg, &lds)) return CCT_EUNSUPPORTED;
  if (p.Kpad != conv_fused_split_kpad(p.gCg, p.gK)) return CCT_EINVAL;
  const Tile t = split_tile(p, &fg, &lds, p.Ncols / (p.gHout * p.gWout));
  switch (t.rows) {
    case 32: return launch_rows<1, 2, 32>(p, fg, lds, st);
    case 64:
      if (t.wide)
        return p.gK == 3 ? launch_variant<2, 2, 3, 1, 16, kWide64>(p, fg, lds, st)
                         : launch_variant<2, 2, 5, 1, 16, kWide64>(p, fg, lds, st);
      return t.block == 32 ? launch_rows<2, 2, 32>(p, fg, lds, st) : launch_rows<2, 2, 16>(p, fg, lds, st);
    case 48:
      return p.gK == 3 ? launch_variant<1, 3, 3, 1, 16, kWide48>(p, fg, lds, st)
                       : launch_variant<1, 3, 5, 1, 16, kWide48>(p, fg, lds, st);
    case 96: return launch_rows<2, 3, 16>(p, fg, lds, st);
    default: return t.block == 32 ? launch_rows<4, 2, 32>(p, fg, lds, st) : launch_rows<4, 2, 16>(p, fg, lds, st);
  }
}

}  // namespace cct
