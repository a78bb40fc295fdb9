// Matrix product C[m][col] = sum_k A(m, k) * B(k, col) (+ bias[m]) of fp32 operands as sums of three
// bf16 terms on the bf16 matrix cores (split_bf16.h), for products whose B is a tensor in place: x, w or
// dy of a fully connected layer, the planes of a layer with 1 x 1 kernels.
//
//   - A is the small operand.  It comes packed and split, [group][tile of 16 k][term][row][16]
//     (launch_pack_rows_split), and never passes through LDS: a lane loads the 16 bytes of its row and
//     term straight from the pack, one stage ahead.  The waves of a workgroup are stacked along the rows,
//     so that no two waves read the same rows where there are 128 of them.  DIRECT: up to 32 rows of a
//     k-contiguous fp32 matrix, which every lane splits itself (one launch less);
//   - B is staged: 128 columns x 16 or 32 k per stage, fetched two stages ahead into registers, split
//     there and written to LDS as granules of 8 k, [term][8 k][column], which lanes write and read side by
//     side (the planes are 64 bytes apart beyond their size, for the k-contiguous form's writes).  B is
//     read once per row tile; BT: it lies k-contiguous (w of a forward product), 16-byte loads, otherwise
//     column-contiguous through a column map, 4-byte loads;
//   - groups are channel groups or splits of the contraction.
// With 128 rows the matrix cores bound it: 48 MFMAs per stage and wave (1536 cycles) against about 110
// vector instructions of splitting; two waves per SIMD and the registers to read ahead.  With 64 or 32
// rows B's way from memory does: four waves per SIMD, stages of half the size, no reading ahead.
// Measured (before: fp32 matrix instructions): fc6 at batch 256, 19.3 GFLOP, forward 195 -> 117 us,
// backward-weights 192 -> 126; one image of fc6 (151 MB of w) 50 -> 36 us; 1 x 1 kernels, 128 images of
// 28 x 28, 256 -> 64 channels, 52 -> 41 us.
#include <algorithm>

#include "cct_internal.h"
#include "gemm_common.h"
#include "split_bf16.h"

namespace cct {
namespace {

constexpr int NT = 256;
constexpr int BN = 128;
constexpr int TK = 16;                      // k per tile of the pack
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes, dword aligned
constexpr int KPAD = 32;                    // the pack is padded to whole stages of any form
constexpr int PLANE = BN * 16 + 64;         // bytes of one (term, 8 k) plane in LDS

template <int WAVES_M, bool BT, bool DIRECT>
__global__ __launch_bounds__(NT, WAVES_M == 4 ? 2 : WAVES_M == 1 && !BT ? 6 : 4) void gemm_split(GemmTN p, int Ktotal, int tiles_m, int tiles_n) {
  constexpr int WAVES_N = 4 / WAVES_M;
  constexpr int WN = BN / (32 * WAVES_N);
  constexpr int BM = 32 * WAVES_M;
  constexpr int SK = WAVES_M == 4 ? 32 : 16;  // k per stage
  constexpr int TPS = SK / TK;                // tiles per stage
  constexpr int GPT = BN * (SK / 8) / NT;     // granules of 8 k per thread and stage
  constexpr int SLOT = 3 * (SK / 8) * PLANE;
  // 128 rows: two waves per SIMD, the next block's operands are read behind the current MFMAs; fewer:
  // four waves per SIMD hide each other's reads and the registers go there
  constexpr int NB = WAVES_M == 4 ? 2 : 1;

  __shared__ __attribute__((aligned(16))) unsigned char Bs[2 * SLOT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int lane_lo = lane & 31, lane_hi = lane >> 5;

  // every XCD gets a contiguous run of column tiles, the row tiles of one next to each other (they share B)
  int bid = blockIdx.x;
  {
    const int total = tiles_m * tiles_n;
    const int per = total >> 3, rem = total & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    bid = xcd * per + min(xcd, rem) + idx;
  }
  const int tile_n = bid / tiles_m, tile_m = bid - tile_n * tiles_m;
  const int g = blockIdx.y;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int kd = min(p.Kdim, Ktotal - g * p.Kdim);
  const int stages = (kd + SK - 1) / SK;
  const bool half = TPS == 2 && (kd - 1) % SK < TK;  // the last stage is one tile

  // ---- B: fixed columns (or column and k for BT) per thread, the stage enters through the base
  const float* Bg = reinterpret_cast<const float*>(p.B) + (long long)g * p.b_gs;
  const int n_f = BT ? 0 : fdiv_u(n0, p.bmap.divM, p.bmap.divsh);
  const float* Bt = BT ? Bg + (long long)n0 * p.b_ks : Bg + (long long)n_f * p.bmap.img_stride;
  unsigned voff[BT ? GPT : 1];
  unsigned dst[GPT];  // byte offset of the granule's first term in a slot
  if constexpr (BT) {
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      const int q = tid + u * NT, c = q / (SK / 8), kh = q % (SK / 8);
      voff[u] = (unsigned)((long long)(min(n0 + c, p.Ncols - 1) - n0) * p.b_ks + kh * 8) * 4u;
      dst[u] = kh * PLANE + c * 16;
    }
  } else {
    const int c = tid & 127;
    voff[0] = (unsigned)(col_offset(p.bmap, min(n0 + c, p.Ncols - 1)) - (long long)n_f * p.bmap.img_stride) * 4u;
#pragma unroll
    for (int u = 0; u < GPT; ++u) dst[u] = ((wave >> 1) + 2 * u) * PLANE + c * 16;
  }
  float stg[2][GPT][8];
  auto stage_load = [&](int set, int t) {
    const int k0 = t * SK;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Bt + (BT ? (long long)k0 : k0 * p.b_ks)), 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      if constexpr (BT) {
        if (k0 + SK > kd) {  // the last stage ends inside a row
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int kh = (tid + u * NT) % (SK / 8) * 8, k = min(kh + e, kd - 1 - k0);
            stg[set][u][e] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(voff[u] + (unsigned)(k - kh) * 4u), 0, 0));
          }
          continue;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff[u], h * 16, 0));
#pragma unroll
          for (int e = 0; e < 4; ++e) stg[set][u][h * 4 + e] = v[e];
        }
      } else {
        // k past the last one repeats it (A is zero there)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = min(((wave >> 1) + 2 * u) * 8 + e, kd - 1 - k0);
          stg[set][u][e] = __builtin_bit_cast(
              float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff[0], (int)((unsigned)k * (unsigned)p.b_ks * 4u), 0));
        }
      }
    }
  };
  auto stage_store = [&](int set, int slot, int u) {
    u32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned a, b, c;
      split_pair(stg[set][u][2 * e], stg[set][u][2 * e + 1], &a, &b, &c);
      h[e] = a;
      m[e] = b;
      l[e] = c;
    }
    unsigned char* d = Bs + slot * SLOT + dst[u];
    *reinterpret_cast<u32x4*>(d) = h;
    *reinterpret_cast<u32x4*>(d + (SK / 8) * PLANE) = m;
    *reinterpret_cast<u32x4*>(d + 2 * (SK / 8) * PLANE) = l;
  };

  // ---- A straight from the pack (L2), a stage (two tiles) ahead
  const unsigned short* Abase = reinterpret_cast<const unsigned short*>(p.A) +
                                ((long long)g * p.a_gs * 3 + (long long)(m0 + wave_m * 32) * TK);
  const __amdgpu_buffer_rsrc_t a_rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(Abase), 0, 0x7fffffff, 0x00020000);
  const int a_voff = (lane_lo * TK + lane_hi * 8) * 2;
  const unsigned term_b = (unsigned)p.Mpad * TK * 2u;
  const int ktiles = TPS * stages;
  u32x4 a[TPS][3];
  // DIRECT: A lies in fp32, k-contiguous rows a_ms apart, and a lane splits the 8 values it supplies
  const float* Ad = DIRECT ? reinterpret_cast<const float*>(p.A) + g * p.a_gs +
                                 (long long)min(m0 + wave_m * 32 + lane_lo, p.M - 1) * p.a_ms + lane_hi * 8
                           : nullptr;
  auto load_a = [&](int set, int t) {
    if constexpr (DIRECT) {
      const int k0 = min(t, ktiles - 1) * TK, left = kd - k0 - lane_hi * 8;
      float v[8];
      if (k0 + TK <= kd) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4u q = *reinterpret_cast<const f32x4u*>(Ad + k0 + h * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[h * 4 + e] = q[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = e < left ? Ad[k0 + e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        unsigned hh, mm, ll;
        split_pair(v[2 * e], v[2 * e + 1], &hh, &mm, &ll);
        a[set][0][e] = hh;
        a[set][1][e] = mm;
        a[set][2][e] = ll;
      }
      return;
    }
    const unsigned so = (unsigned)min(t, ktiles - 1) * (3u * term_b);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      a[set][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rs, a_voff, (int)(so + q * term_b), 0));
  };

  floatx16 acc_h[WN], acc_c[WN];  // h*h, and the corrections
#pragma unroll
  for (int j = 0; j < WN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_h[j][r] = acc_c[j][r] = 0.f;

  stage_load(0, 0);
  if (stages > 1) stage_load(1, 1);
#pragma unroll
  for (int e = 0; e < TPS; ++e) load_a(e, e);
#pragma unroll
  for (int u = 0; u < GPT; ++u) stage_store(0, 0, u);
  if (stages > 2) stage_load(0, 2);

  const int b_lds = lane_hi * PLANE + (wave_n * WN * 32 + lane_lo) * 16;
  u32x4 b[NB][3];
  auto read_b = [&](int set, int j, int base) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      b[set][q] = *reinterpret_cast<const u32x4*>(Bs + base + b_lds + j * 512 + q * (SK / 8) * PLANE);
  };
  auto mfma6 = [&](int set, int bs, int j) {
    __builtin_amdgcn_sched_barrier(0);
#define CCT_M(X, Y, ACC)                                                                \
  ACC = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[set][X]),   \
                                                __builtin_bit_cast(bf16x8, b[bs][Y]), ACC, 0, 0, 0)
    CCT_M(2, 0, acc_c[j]);
    CCT_M(0, 2, acc_c[j]);
    CCT_M(1, 1, acc_c[j]);
    CCT_M(1, 0, acc_c[j]);
    CCT_M(0, 1, acc_c[j]);
    CCT_M(0, 0, acc_h[j]);
#undef CCT_M
    __builtin_amdgcn_sched_barrier(0);
  };
  __syncthreads();  // slot 0 is visible
  if (NB == 2) read_b(0, 0, 0);

  // One stage: TPS tiles of WN blocks (NB = 2: block i + 1 is read while block i is multiplied).  The
  // values of stage t + 1 (set `nset`) are split into the other slot behind the first blocks, their
  // registers are loaded with stage t + 3; the workgroup meets before the next stage's first read.
  auto stage = [&](int t, int slot, int nset) {
    const bool more = t + 1 < stages;
    const int base = slot * SLOT, other = (slot ^ 1) * SLOT;
#pragma unroll
    for (int i = 0; i < TPS * WN; ++i) {
      const int tt = i / WN, j = i % WN;
      if (NB == 1) {
        read_b(0, j, base + tt * 2 * PLANE);
      } else if (i + 1 < TPS * WN) {
        read_b((i + 1) % NB, (i + 1) % WN, base + ((i + 1) / WN) * 2 * PLANE);
      } else if (more) {
        __syncthreads();
        read_b(0, 0, other);
      }
      if (tt == 0 || more || !half) mfma6(tt, i % NB, j);
      if (j == WN - 1) load_a(tt, TPS * (t + 1) + tt);
      if (more && i < GPT) {
        stage_store(nset, slot ^ 1, i);
        if (i == GPT - 1 && t + 3 < stages) stage_load(nset, t + 3);
      }
    }
    if (NB == 1) __syncthreads();
  };
  int t = 0;
  for (; t + 1 < stages; t += 2) {
    stage(t, 0, 1);
    stage(t + 1, 1, 0);
  }
  if (t < stages) stage(t, 0, 1);

  // ---- epilogue: accumulator register r is row 8*(r/4) + 4*(lane/32) + r%4 of the wave's rows
  const int mw = m0 + wave_m * 32;
  float* __restrict__ C = p.C + (long long)g * p.c_gs;
  const float* bias = p.bias ? p.bias + (p.bias_gs < 0 ? 0 : (long long)g * p.bias_gs) : nullptr;
  // NaN once a result is not finite: one instruction each (compares, whose answers are collected in scalar masks,
  // took 2 % of fc6's products and 4 % of a 4096 -> 1000 layer's)
  float check = 0.f;
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const int col = n0 + wave_n * WN * 32 + j * 32 + lane_lo;
    if (col >= p.Ncols) continue;
    float* __restrict__ cl = C + col_offset(p.cmap, col);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mw + (r >> 2) * 8 + lane_hi * 4 + (r & 3);
      if (m >= p.M) continue;
      float v = acc_h[j][r] + acc_c[j][r];
      check = fmaf(v, 0.f, check);
      v *= kSplitUnscale;
      if (bias) v += bias[p.bias_gs < 0 ? col : m];
      cl[(long long)m * p.c_ms] = v;
    }
  }
  if (!__any(check != check)) return;
  // blocks with results that are not finite: again in plain fp32 (split_bf16.h)
  const GemmTN& q = first_argument<GemmTN>();
  float* Cq = q.C + (long long)g * q.c_gs;
  const float* Bq = reinterpret_cast<const float*>(q.B) + (long long)g * q.b_gs;
  const float* bq = q.bias ? q.bias + (q.bias_gs < 0 ? 0 : (long long)g * q.bias_gs) : nullptr;
#pragma unroll 1
  for (int j = 0; j < WN; ++j) {
    const int col = n0 + wave_n * WN * 32 + j * 32 + lane_lo, c = min(col, q.Ncols - 1);
    float* cl = Cq + col_offset(q.cmap, c) + (long long)(mw + lane_hi * 4) * q.c_ms;
    unsigned todo = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = (r >> 2) * 8 + (r & 3);
      if (col < q.Ncols && mw + lane_hi * 4 + rr < q.M && !finite(cl[(long long)rr * q.c_ms])) todo |= 1u << r;
    }
    if (!__any(todo)) continue;
    const float* bc = Bq + (BT ? (long long)c * q.b_ks : col_offset(q.bmap, c));
    const int m = min(mw + lane_lo, q.M - 1);
    const floatx16 v = fp32_block(
        (kd + 1) / 2,
        [&](int s) {
          const int k = 2 * s + lane_hi;
          if (k >= kd) return 0.f;
          if constexpr (DIRECT) return reinterpret_cast<const float*>(q.A)[g * q.a_gs + m * q.a_ms + k];
          const unsigned short* ak = reinterpret_cast<const unsigned short*>(q.A) + (long long)g * q.a_gs * 3 +
                                     ((long long)(k / TK) * 3 * q.Mpad + m) * TK + k % TK;
          const long long term = (long long)q.Mpad * TK;
          return join_value(ak[0], ak[term], ak[2 * term]);
        },
        [&](int s) {
          const int k = 2 * s + lane_hi;
          return k < kd ? bc[BT ? (long long)k : k * q.b_ks] : 0.f;
        },
        [&](const floatx16& acc) { return numbers(acc, todo); });
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (!(todo >> r & 1)) continue;
      const int rr = (r >> 2) * 8 + (r & 3);
      float sum = v[r];
      if (bq) sum += bq[q.bias_gs < 0 ? col : mw + lane_hi * 4 + rr];
      cl[(long long)rr * q.c_ms] = sum;
    }
  }
}

// pack[g][tile][term][m][16] = the terms of src[g * sg + (m / taps) * sm + m % taps + k * sk], zero padded in
// m and k: k runs over min(Kdim, Ktotal - g * Kdim) indices.
struct RowsPack {
  int G, M, Mpad, Kpad, Kdim, Ktotal;
  long long sm, sk, sg;
  int taps;
};
__global__ __launch_bounds__(256) void pack_rows_split_kernel(const float* __restrict__ src,
                                                              unsigned short* __restrict__ pack, RowsPack d) {
  const long long per = (long long)d.Kpad / 8 * d.Mpad;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= per * d.G) return;
  const int g = (int)(t / per);
  const long long e = t - g * per;
  const int half = (int)(e & 1);
  const long long r = e >> 1;
  const int tile = (int)(r / d.Mpad), m = (int)(r - (long long)tile * d.Mpad);
  const int k0 = tile * TK + half * 8;
  const int kd = min(d.Kdim, d.Ktotal - g * d.Kdim);
  const int row = m / d.taps;
  const float* s = src + g * d.sg + row * d.sm + (m - row * d.taps) + k0 * d.sk;
  unsigned short h[8], mm[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float v = m < d.M && k0 + i < kd ? s[i * d.sk] : 0.f;
    split_value(v, &h[i], &mm[i], &l[i]);
  }
  unsigned short* dst = pack + (((long long)g * (d.Kpad / TK) + tile) * 3 * d.Mpad + m) * TK + half * 8;
  const long long term = (long long)d.Mpad * TK;
  auto put = [](unsigned short* to, const unsigned short (&v)[8]) {
    uint4 q;
    q.x = v[0] | ((unsigned)v[1] << 16);
    q.y = v[2] | ((unsigned)v[3] << 16);
    q.z = v[4] | ((unsigned)v[5] << 16);
    q.w = v[6] | ((unsigned)v[7] << 16);
    *reinterpret_cast<uint4*>(to) = q;
  };
  put(dst, h);
  put(dst + term, mm);
  put(dst + 2 * term, l);
}

template <int WAVES_M, bool BT, bool DIRECT = false>
int launch_variant(const GemmTN& p, int Ktotal, hipStream_t st) {
  const int tiles_m = p.Mpad / (32 * WAVES_M), tiles_n = (p.Ncols + BN - 1) / BN;
  const long long blocks = (long long)tiles_m * tiles_n;
  if (blocks <= 0 || blocks >= 2147483647LL || p.G < 1 || p.G > 65535) return CCT_EUNSUPPORTED;
  const double mk = (double)p.M * p.Kdim * p.G, kn = (double)p.Kdim * p.Ncols * p.G;
  ProfScope ps(2.0 * p.M * kn, 6.0 * mk + 4.0 * kn + 4.0 * (double)p.M * p.Ncols * p.G, st,
               "gemm_split<%d, %s>", 32 * WAVES_M, BT ? "k-contiguous" : "in place");
  hipLaunchKernelGGL((gemm_split<WAVES_M, BT, DIRECT>), dim3((unsigned)blocks, (unsigned)p.G), dim3(NT), 0, st, p, Ktotal,
                     tiles_m, tiles_n);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace

int gemm_split_mpad(int M) { return M <= 32 ? 32 : (M + 63) / 64 * 64; }
int gemm_split_kpad(int K) { return (K + KPAD - 1) / KPAD * KPAD; }

// 32-bit byte offsets: the pack of one group, B inside a stage of one column tile
bool gemm_split_fits(const GemmTN& p, bool bt) {
  if (p.bf16 || p.M < 1 || p.Ncols < 1 || p.Kdim < 1) return false;
  if ((long long)p.Mpad * p.Kpad * 6 >= (1LL << 31) || p.b_ks >= (1LL << 22)) return false;
  if (bt) return true;
  const long long T = (BN - 1) / p.bmap.P + 2;  // images that 128 columns can touch
  return p.bmap.P == 2147483647 ? (long long)p.Ncols < (1LL << 29)
                                : (T + 1) * p.bmap.img_stride < (1LL << 28);
}

// Row tile: the largest that divides the padded rows, smaller while the launch would not put a workgroup
// on every CU.  Up to 128 k a workgroup is mostly filling and draining: 64 rows put twice as many on a CU
// (118 images of 30 x 30, 41 -> 105 channels: 43 us with 128 rows, 32 with 64; at 256 k, fc6's
// backward-weights product, 135 against 149).
int gemm_split_bm(int Mpad, long long tiles_n, int K, int G) {
  int BM = Mpad % 128 == 0 && K > 128 ? 128 : Mpad % 64 == 0 ? 64 : 32;
  long long wgs = tiles_n * ((unsigned)Mpad / (unsigned)BM) * G;
  for (; BM > 32 && wgs < 256; BM /= 2) wgs *= 2;
  return BM;
}

// Rounds of workgroups (512 of 128 rows fit the chip, 1024 of fewer) times their stages at the measured
// rates, 4 us to fill and drain a round.  Where the fullest CU holds fewer of them than fit, each is faster,
// but a lone workgroup of 128 rows still takes two thirds as long as one of two.
double gemm_split_seconds(int Mpad, int K, long long cols, long long G) {
  const long long tiles_n = (cols + BN - 1) / BN;
  const int BM = gemm_split_bm(Mpad, tiles_n, K, (int)G);
  const int log_bm = BM == 128 ? 7 : BM == 64 ? 6 : 5, log_slots = BM == 128 ? 9 : 10;
  const unsigned long long wgs = (unsigned long long)tiles_n * (Mpad >> log_bm) * G, slots = 1ULL << log_slots;
  const double flops = BM == 128 ? 1.0 / 230.0e12 : BM == 64 ? 1.0 / 200.0e12 : 1.0 / 120.0e12;
  const double stage = 2.0 * BM * BN * 32 * flops * (double)slots;
  const double rounds = (double)((wgs + slots - 1) >> log_slots);
  const double share = std::min(1.0, 0.3 + 0.7 * (double)((wgs + 255) >> 8) * (256.0 / (double)slots));
  return rounds * ((K + 31) / 32 * stage * share + 4.0e-6);
}

int launch_gemm_split(const GemmTN& p0, int Ktotal, bool bt, hipStream_t st) {
  GemmTN p = p0;
  colmap_prepare(&p.bmap);
  colmap_prepare(&p.cmap);
  if (p.Mpad != gemm_split_mpad(p.M) || p.Kpad != gemm_split_kpad(p.Kdim)) return CCT_EINVAL;
  if (!gemm_split_fits(p, bt)) return CCT_EUNSUPPORTED;
  const int BM = gemm_split_bm(p.Mpad, (p.Ncols + BN - 1) / BN, p.Kdim, p.G);
  if (p.a_ms) return bt && p.M <= 32 ? launch_variant<1, true, true>(p, Ktotal, st) : CCT_EUNSUPPORTED;
  if (bt) {
    if (BM == 32) return launch_variant<1, true>(p, Ktotal, st);
    return BM == 64 ? launch_variant<2, true>(p, Ktotal, st) : launch_variant<4, true>(p, Ktotal, st);
  }
  if (BM == 32) return launch_variant<1, false>(p, Ktotal, st);
  return BM == 64 ? launch_variant<2, false>(p, Ktotal, st) : launch_variant<4, false>(p, Ktotal, st);
}

int launch_pack_rows_split(const float* src, void* pack, int G, int M, int Mpad, int Kpad, int Kdim, int Ktotal,
                           long long sm, long long sk, long long sg, hipStream_t st, int taps) {
  const RowsPack d{G, M, Mpad, Kpad, Kdim, Ktotal, sm, sk, sg, taps};
  const long long total = (long long)Kpad / 8 * Mpad * G, blocks = (total + 255) / 256;
  if (blocks <= 0 || blocks >= 2147483647LL) return CCT_EUNSUPPORTED;
  ProfScope ps("pack_rows_split_kernel", 0.0, 4.0 * M * (double)Ktotal + 48.0 * total, st);
  hipLaunchKernelGGL(pack_rows_split_kernel, dim3((unsigned)blocks), dim3(256), 0, st, src,
                     reinterpret_cast<unsigned short*>(pack), d);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

}  // namespace cct
