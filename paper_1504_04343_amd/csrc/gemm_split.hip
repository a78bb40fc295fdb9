// Matrix product C[m][col] = sum_k A(m, k) * B(k, col) (+ bias[m]) of fp32 operands as sums of three
// bf16 terms on the bf16 matrix cores (split_bf16.h), for products whose B is a tensor in place: x, w or
// dy of a fully connected layer, the planes of a layer with 1 x 1 kernels.
//
//   - a workgroup computes up to 144 rows x 128 columns with four waves; a wave owns all rows of 32 columns, blocks of
//     16 x 16 (v_mfma_f32_16x16x32_bf16), two accumulators each;
//   - B goes from memory into the registers of the one wave that multiplies it, which splits it there: no LDS, no
//     meeting of waves.  A lane supplies 8 k of two neighbouring columns per stage of 32 k.  The split of the next stage is
//     written between the MFMAs of this one, 3 or 4 instructions at a time (32 rows: behind them).  Columns are taken in
//     pairs (8-byte loads and stores), one by one (planes of a few pixels), or k-contiguous (w of a forward product,
//     16-byte loads);
//   - A is shared by the four waves through LDS: units of 16 rows and one term, in lane order, so that a read is 1 KiB
//     without conflicts.  128 and 144 rows: packed that way and split once per call (launch_pack_rows_split), moved to
//     LDS by loads that write it directly.  32 and 64 rows: fp32 values in place, any strides, split by the
//     workgroup on their way; a launch less, and no pack to wait for.  16 rows, and 32 of one stage: by every wave for itself,
//     without LDS;
//   - groups are channel groups or splits of the contraction.
// What bounds it (fc6 at batch 256, 19.3 GFLOP per product in 91 to 105 us): the MFMAs alone take 62 us, LDS reads add 2,
// splitting 9, waiting for memory 20.  Before, B went through LDS and A straight to registers in tiles of 128 and 64 rows,
// always behind a pack: forward 104 -> 91 us, the two gradients 128 -> 104 each; 144 rows x 512 k x 100352 columns, three
// tiles of 64 before, 126 -> 90; 256 images of 4096 -> 1000 features, forward, both gradients and what lies around them,
// 104 -> 87.
#include <algorithm>
#include <type_traits>

#include "cct_internal.h"
#include "gemm_common.h"
#include "split_bf16.h"

namespace cct {
namespace {

constexpr int NT = 256;
constexpr int BN = 128;
constexpr int SK = 32;  // k per stage
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));  // 8 bytes, dword aligned

// How the operands lie.
enum AForm { kPacked, kRows, kStrided };     // fp32: k-contiguous, or any strides
enum BForm { kColumns, kPairs, kContiguous };  // column-contiguous: one by one, in pairs; k-contiguous

// ALONE: every wave splits A's values itself, without LDS and without meeting; 1: a contraction of one stage.  In products
// of few rows, which wait for memory, fewer registers and more waves are worth it: one stage of 32 rows, 16 rows of any number
// (14 <- 9 channels, 540000 columns in two groups: 22.6 us as a pack and a product, 36.7 with LDS, 24 so).
template <int RB, BForm BF, AForm AF, int ALONE = 0>
__global__ __launch_bounds__(NT, RB >= 8 ? 2 : RB == 4 ? 3 : ALONE && (RB == 1 || ALONE == 1) ? 5 : 4) void gemm_split(GemmTN p, int Ktotal, int tiles_m, int tiles_n) {
  constexpr int BM = 16 * RB;
  constexpr bool DIRECT = AF != kPacked, BT = BF == kContiguous;
  constexpr int UNITS = 3 * RB;
  constexpr int SLOT = UNITS * 1024;
  constexpr int AP = ALONE ? RB : ((DIRECT ? RB : UNITS) + 3) / 4;  // what a wave moves of A per stage: rows of 16 or units
  // Stages of B in registers: as they were loaded, as many as there is room for, and split.  Two blocks of rows have one split
  // stage, made behind the MFMAs of the one before: two of them, made between the MFMAs, spilled, four waves per SIMD hide the
  // splitting as well, and it is memory that bounds them (2900 products of 8 to 32
  // rows: 0.92 times the time, 1.04 at most).
  constexpr int RAWS = RB == 8 ? 2 : 1, SPLITS = RB <= 2 ? 1 : 2;
  // Three slots for A: the workgroup meets in front of a stage's last block of rows, behind which the next stage's first
  // operands are read.  Two (fp32 values, whose registers come first; 9 blocks of rows): between the stages.
  constexpr bool EARLY = !DIRECT && RB % 2 == 0;
  constexpr int SLOTS = EARLY ? 3 : 2;

  __shared__ __attribute__((aligned(16))) unsigned char As[ALONE ? 16 : SLOTS * SLOT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = lane & 15, kg = lane >> 4;  // row / pair of columns, which 8 k of a stage

  // every XCD gets a contiguous run of tiles, 8 row tiles at a time next to each other: what runs at a time shares
  // both operands in its L2
  int idx = blockIdx.x;
  {
    const int total = tiles_m * tiles_n;
    const int per = total >> 3, rem = total & 7;
    const int xcd = idx & 7;
    idx = xcd * per + min(xcd, rem) + (idx >> 3);
  }
  const int strip = idx / (8 * tiles_n), inner = idx - strip * 8 * tiles_n, rows = min(8, tiles_m - strip * 8);
  const int tile_n = inner / rows, tile_m = strip * 8 + inner - tile_n * rows;
  const int g = blockIdx.y;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int kd = min(p.Kdim, Ktotal - g * p.Kdim);
  const int stages = (kd + SK - 1) / SK, last = stages - 1;

  // ---- B: a lane supplies two neighbouring columns, 8 k of each.  In pairs an image has an even number of columns: where
  // its plane is odd, the second of its last pair is no column (what it loads is not stored)
  const float* Bg = reinterpret_cast<const float*>(p.B) + (long long)g * p.b_gs;
  const int n_f = BT                ? 0
                  : BF == kColumns ? fdiv_u(n0, p.bmap.divM, p.bmap.divsh)
                  : p.pair_P       ? fdiv_u(n0, p.pair_M, p.pair_sh)
                                   : 0;
  const float* Bt = BT ? Bg + (long long)n0 * p.b_ks : Bg + (long long)n_f * p.bmap.img_stride;
  // which column of the matrix is column v of the tiles, and is it one?
  auto column = [&](int v, bool* live) {
    if constexpr (BF != kPairs) {
      *live = v < p.Ncols;
      return min(v, p.Ncols - 1);
    } else {
      const int c = min(v, p.pair_cols - 2 + (v & 1)), img = p.pair_P ? fdiv_u(c, p.pair_M, p.pair_sh) : 0;
      const int pix = c - img * p.pair_P;
      *live = v < p.pair_cols && pix < (p.pair_P ? p.bmap.P : p.Ncols);
      return p.pair_P ? img * p.bmap.P + min(pix, p.bmap.P - 1) : min(pix, p.Ncols - 1);
    }
  };
  unsigned voff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    bool live;
    const int col = column(n0 + wave * 32 + 2 * lo + j, &live);
    voff[j] = BT ? (unsigned)((long long)(col - n0) * p.b_ks + kg * 8) * 4u
                 : (unsigned)(col_offset(p.bmap, col) - (long long)n_f * p.bmap.img_stride + (long long)kg * 8 * p.b_ks) * 4u;
  }
  // k past the last one: the last one again (in a contraction of 35 reading on was half of what came from memory); k-contiguous
  // what lies there, or zero beyond the tensor's end.  A is zero there; an infinity only costs the recomputation.  The range is
  // checked against the vector offset alone: all of an address that may lie beyond goes there.  Stages past the last one have a
  // range of nothing: as many loads are in flight as ever, but none goes to memory (a contraction of one stage would read B
  // three times).
  const long long b_left = p.b_len - (Bt - reinterpret_cast<const float*>(p.B));
  auto range = [](long long left) { return left < 0 ? 0 : left >= 0x1fffffff ? 0x7fffffff : (int)left * 4; };
  float raw[RAWS][2][8];
  auto load_b = [&](int set, int t) {
    const int tt = min(t, last);
    const long long at = (long long)tt * SK * (BT ? 1 : p.b_ks);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Bt + at), 0, t > last ? 0 : range(b_left - at), 0x00020000);
    unsigned ks = BT ? 4u : (unsigned)p.b_ks * 4u;
    asm volatile("" : "+s"(ks));  // the sums below are not kept in registers between the stages
    unsigned end[2];  // the stage's last k
#pragma unroll
    for (int j = 0; j < 2; ++j) end[j] = voff[j] + (unsigned)(min(kd - tt * SK, SK) - 1 - kg * 8) * ks;
#pragma unroll
    for (int e = 0; e < (BT ? 2 : 8); ++e)
#pragma unroll
      for (int j = 0; j < (BF == kPairs ? 1 : 2); ++j) {
        if constexpr (BT) {
          const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(voff[j] + 4 * e * ks), 0, 0));
#pragma unroll
          for (int i = 0; i < 4; ++i) raw[set][j][e * 4 + i] = v[i];
        } else if constexpr (BF == kPairs) {
          const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)min(voff[0] + e * ks, end[0]), 0, 0));
          raw[set][0][e] = v[0];
          raw[set][1][e] = v[1];
        } else {
          raw[set][j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)min(voff[j] + e * ks, end[j]), 0, 0));
        }
      }
  };
  // The terms of a stage in b[t & 1].  The next stage's are made between the MFMAs of this one, a quarter of a
  // pair of values (3 or 4 instructions, less than an MFMA takes) at a time.
  u32x4 b[SPLITS][2][3];
  float ra = 0.f, rb = 0.f;
  auto split_step = [&](float (&v)[2][8], int set, int n) { split_quarter(v[n >> 4], b[set][n >> 4], n & 15, ra, rb); };

  // ---- A: through LDS.  Units of 16 rows and one term, 1 KiB, in lane order: packed ones are moved there directly,
  // fp32 values pass through registers
  float av[DIRECT ? AP : 1][8];
  unsigned a_voff[DIRECT ? AP : 1];
  const unsigned char* Ap = nullptr;
  const float* Ad = nullptr;
  const int last_unit = (p.Mpad - m0) / 16 * 3 - 1;
  if constexpr (DIRECT) {
    const int r0 = m0 / p.a_taps;
    Ad = reinterpret_cast<const float*>(p.A) + g * p.a_gs + (long long)r0 * p.a_ms;
#pragma unroll
    for (int u = 0; u < AP; ++u) {
      const int m = min(m0 + (ALONE ? u : wave + 4 * u) * 16 + lo, p.M - 1), r = m / p.a_taps;
      a_voff[u] = (unsigned)((r - r0) * p.a_ms + (m - r * p.a_taps) + kg * 8 * p.a_ks) * 4u;
    }
  } else {
    Ap = reinterpret_cast<const unsigned char*>(p.A) + (long long)g * p.a_gs * 6 + (long long)m0 / 16 * 3072;
  }
  auto move_a = [&](int t, int slot) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(Ap + (long long)min(t, last) * p.Mpad * 192), 0, t > last ? 0 : 0x7fffffff, 0x00020000);
#pragma unroll
    for (int u = 0; u < AP; ++u)
      if (4 * u + 4 <= UNITS || wave + 4 * u < UNITS)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(As + slot * SLOT + (wave + 4 * u) * 1024), 16, lane * 16,
                                                 min(wave + 4 * u, last_unit) * 1024, 0, 0);
  };
  const long long a_left = DIRECT ? p.a_len - (Ad - reinterpret_cast<const float*>(p.A)) : 0;
  auto load_a = [&](int t) {
    const long long at = (long long)min(t, last) * SK * (AF == kRows ? 1 : p.a_ks);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Ad + at), 0, t > last ? 0 : range(a_left - at), 0x00020000);
    unsigned ks = AF == kRows ? 4u : (unsigned)p.a_ks * 4u;
    asm volatile("" : "+s"(ks));
#pragma unroll
    for (int u = 0; u < AP; ++u) {
      if (!ALONE && 4 * u + 4 > RB && wave + 4 * u >= RB) continue;
      if constexpr (AF == kRows) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(a_voff[u] + 4 * h * ks), 0, 0));
#pragma unroll
          for (int e = 0; e < 4; ++e) av[u][h * 4 + e] = x[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          av[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
              rs, (int)(a_voff[u] + e * ks), 0, 0));
      }
    }
  };
  auto split_a = [&](int t, int u, u32x4 (&q)[3]) {
    const int over = kd - t * SK - kg * 8;  // a lane's values from here on are past the last k: zero
#pragma unroll
    for (int e = 0; e < 8; ++e) av[u][e] = e < over ? av[u][e] : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned h, m, l;
      split_pair(av[u][2 * e], av[u][2 * e + 1], &h, &m, &l);
      q[0][e] = h;
      q[1][e] = m;
      q[2][e] = l;
    }
  };
  auto store_a = [&](int t, int slot) {
#pragma unroll
    for (int u = 0; u < AP; ++u) {
      if (4 * u + 4 > RB && wave + 4 * u >= RB) continue;
      u32x4 q[3];
      split_a(t, u, q);
#pragma unroll
      for (int i = 0; i < 3; ++i)
        *reinterpret_cast<u32x4*>(As + slot * SLOT + ((wave + 4 * u) * 3 + i) * 1024 + lane * 16) = q[i];
    }
  };

  f32x4 acc_h[RB][2], acc_c[RB][2];  // h*h, and the corrections
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc_h[i][j][r] = acc_c[i][j][r] = 0.f;

  if constexpr (DIRECT) load_a(0); else move_a(0, 0);
  load_b(0, 0);
  if constexpr (DIRECT && !ALONE) {
    store_a(0, 0);
    load_a(1);
  }
  if constexpr (EARLY) move_a(1, 1);
  if (RAWS == 2) load_b(1, 1);
#pragma unroll
  for (int n = 0; n < 32; ++n) split_step(raw[0], 0, n);
  if constexpr (ALONE != 1) load_b(0, RAWS);
  if constexpr (!DIRECT) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)

  // Two sets of A's operands; where registers decide how many workgroups share a CU, one, read term by term
  constexpr int SETS = RB <= 2 ? 1 : 2;
  u32x4 a[SETS][3];
  auto read_a = [&](int i, int q, int at) {
    a[i % SETS][q] = *reinterpret_cast<const u32x4*>(As + at * SLOT + (i % RB * 3 + q) * 1024 + lane * 16);
  };
  auto meet = [&]() {
    if constexpr (DIRECT) {
      __syncthreads();
    } else {
      // nothing of this wave's is under way to LDS but what may be; __syncthreads() waits for that too
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Loads of B that may be in flight when A of the next stage has to be in place: the last ones
  constexpr int LEFT = RAWS == 2 && EARLY ? (BT ? 4 : BF == kPairs ? 8 : 16) : 0;
  int slot = 0;  // of A
  auto after = [&](int v) { return v == SLOTS - 1 ? 0 : v + 1; };
  // One stage.  A's operands of a block of rows are read behind the MFMAs of the block before; B's next ones are split
  // behind the last 36 MFMAs (of two blocks of rows: behind all), then their registers are loaded once more.  The last stage does
  // none of this for a next one (a layer of 256 -> 64 channels, 8 stages, 44.0 us with it and 42.1 without; fc6's three
  // products 357 and 352).  It stands once: behind a branch on the parity of the stages its accumulators would meet
  // in different registers and spill.
  auto stage = [&](int t, int set, auto more) {
    constexpr bool MORE = decltype(more)::value;
    const int next = after(slot);
    if constexpr (!EARLY && !ALONE) {
      meet();  // A of this stage is visible, nobody reads the other slot any more
      if constexpr (!DIRECT && MORE) move_a(t + 1, next);
#pragma unroll
      for (int q = 0; q < 3; ++q) read_a(0, 2 - q, slot);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      if (EARLY && MORE && i == RB - 1) {
        __builtin_amdgcn_s_waitcnt(0x0f70 | (LEFT & 15) | (LEFT >> 4 << 14));
        meet();  // A of the next stage is visible, nobody reads the slot before this one any more
        move_a(t + 2, after(next));
      }
      if constexpr (ALONE) {
        split_a(t, i, a[0]);
        if (MORE && i == RB - 1) load_a(t + 1);
      }
      auto read = [&](int q) {
        if (ALONE) return;
        if (i + 1 < RB) read_a(i + 1, q, slot);
        else if (EARLY && MORE) read_a(i + 1, q, next);
      };
      auto mfma = [&](int k, int x, int y, f32x4 (&acc)[2]) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i % SETS][x]),
                                                           __builtin_bit_cast(bf16x8, b[set % SPLITS][j][y]), acc[j], 0, 0, 0);
          const int n = i * 12 + k + j - (RB * 12 - 36);
          if (MORE && SPLITS == 2 && n >= 0 && n < 32) split_step(raw[RAWS == 2 ? set ^ 1 : 0], (set ^ 1) % SPLITS, n);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (SETS == 2) read(2);
      mfma(0, 2, 0, acc_c[i]);
      read(SETS == 2 ? 1 : 2);
      mfma(2, 1, 1, acc_c[i]);
      if (SETS == 2) read(0);
      mfma(4, 1, 0, acc_c[i]);
      if (SETS == 1) read(1);
      mfma(6, 0, 2, acc_c[i]);
      mfma(8, 0, 1, acc_c[i]);
      mfma(10, 0, 0, acc_h[i]);
      if (SETS == 1) read(0);
      if (DIRECT && !ALONE && MORE && i == (RB - 1) / 2) {
        store_a(min(t + 1, last), next);
        load_a(t + 2);
      }
    }
    if constexpr (!DIRECT && !EARLY && MORE) __builtin_amdgcn_s_waitcnt(0x0f70);  // A of the next stage is in place
    if (MORE && SPLITS == 1) {
#pragma unroll
      for (int n = 0; n < 32; ++n) split_step(raw[RAWS == 2 ? set ^ 1 : 0], 0, n);
    }
    if (MORE) load_b(RAWS == 2 ? set ^ 1 : 0, t + 1 + RAWS);
    slot = next;
  };
  if constexpr (EARLY) {
    meet();
#pragma unroll
    for (int q = 0; q < 3; ++q) read_a(0, 2 - q, 0);
  }
  constexpr std::true_type more;
  constexpr std::false_type end;
  int t = 0;
  if constexpr (ALONE) {
    if constexpr (ALONE != 1)
      for (; t < last; ++t) stage(t, 0, more);
  } else {
    for (; t + 2 < stages; t += 2) {
      stage(t, 0, more);
      stage(t + 1, 1, more);
    }
    if (t < last) {
      stage(t, 0, more);
      if constexpr (SPLITS == 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 3; ++q) b[0][j][q] = b[1][j][q];
      }
      ++t;
    }
  }
  stage(t, 0, end);
  if constexpr (!DIRECT) __builtin_amdgcn_s_waitcnt(0x0f70);  // nothing is moved into LDS after the end

  // ---- epilogue: a lane holds rows 16 i + 4 kg .. + 3 of its two columns
  const int mw = m0 + kg * 4;
  float* __restrict__ C = p.C + (long long)g * p.c_gs;
  const float* bias = p.bias ? p.bias + (p.bias_gs < 0 ? 0 : (long long)g * p.bias_gs) : nullptr;
  // NaN once a result is not finite: one instruction each (compares, whose answers are collected in scalar masks,
  // took 2 % of fc6's products and 4 % of a 4096 -> 1000 layer's)
  float check = 0.f;
  int first = n0 + wave * 32 + 2 * lo;
  if constexpr (!ALONE) asm volatile("" : "+v"(first));  // not kept from before
  bool live[2];
  int col[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) col[j] = column(first + j, &live[j]);
  const long long o0 = col_offset(p.cmap, col[0]), o1 = col_offset(p.cmap, col[1]);
  const bool both = __all(o1 == o0 + 1 && live[1]);
  float* __restrict__ cl0 = C + o0 + (long long)mw * p.c_ms;
  float* __restrict__ cl1 = C + o1 + (long long)mw * p.c_ms;
  const bool by_col = bias && p.bias_gs < 0;
  float cb[2] = {-0.f, -0.f};
  if (by_col) {
    cb[0] = bias[col[0]];
    cb[1] = bias[col[1]];
    asm volatile("" : "+v"(cb[0]), "+v"(cb[1]));  // waited for here, as in load_bias
  }
  float bv[RB * 4];
  load_bias(bv, by_col ? nullptr : bias, p.M - 1, [&](int r) { return mw + r / 4 * 16 + r % 4; });
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mw + i * 16 + r;
      float v[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        v[j] = acc_h[i][j][r] + acc_c[i][j][r];
        check = fmaf(v[j], 0.f, check);
        v[j] *= kSplitUnscale;
      }
      if (m >= p.M) continue;
      v[0] += by_col ? cb[0] : bv[i * 4 + r];
      v[1] += by_col ? cb[1] : bv[i * 4 + r];
      const long long row = (long long)(i * 16 + r) * p.c_ms;
      if (both) {
        *reinterpret_cast<f32x2u*>(cl0 + row) = f32x2u{v[0], v[1]};
      } else {
        if (live[0]) cl0[row] = v[0];
        if (live[1]) cl1[row] = v[1];
      }
    }
  if (!__any(check != check)) return;
  __threadfence_block();  // what the other lanes have stored is read below
  // blocks with results that are not finite: again in plain fp32 (split_bf16.h)
  const GemmTN& q = first_argument<GemmTN>();
  const int lane_lo = lane & 31, lane_hi = lane >> 5;
  float* Cq = q.C + (long long)g * q.c_gs;
  const float* Bq = reinterpret_cast<const float*>(q.B) + (long long)g * q.b_gs;
  const float* bq = q.bias ? q.bias + (q.bias_gs < 0 ? 0 : (long long)g * q.bias_gs) : nullptr;
  bool is_col;
  const int c = column(n0 + wave * 32 + lane_lo, &is_col);
  const float* bc = Bq + (BT ? (long long)c * q.b_ks : col_offset(q.bmap, c));
#pragma unroll 1
  for (int i = 0; i < (RB + 1) / 2; ++i) {  // 32 rows; the last ones may be the next tile's: not looked at
    const int mb = m0 + i * 32, m_end = min(m0 + BM, q.M);
    float* cl = Cq + col_offset(q.cmap, c) + (long long)(mb + lane_hi * 4) * q.c_ms;
    unsigned todo = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = (r >> 2) * 8 + (r & 3);
      if (is_col && mb + lane_hi * 4 + rr < m_end && !finite(cl[(long long)rr * q.c_ms])) todo |= 1u << r;
    }
    if (!__any(todo)) continue;
    const int m = min(mb + lane_lo, q.M - 1);
    const floatx16 v = fp32_block(
        (kd + 1) / 2,
        [&](int s) {
          const int k = 2 * s + lane_hi;
          if (k >= kd) return 0.f;
          if constexpr (DIRECT)
            return reinterpret_cast<const float*>(q.A)[g * q.a_gs + m / q.a_taps * q.a_ms + m % q.a_taps + k * q.a_ks];
          const unsigned short* ak = reinterpret_cast<const unsigned short*>(q.A) + (long long)g * q.a_gs * 3 +
                                     ((long long)(k / SK) * (q.Mpad / 16) + m / 16) * 1536 + (k % SK / 8 * 16 + m % 16) * 8 + k % 8;
          return join_value(ak[0], ak[512], ak[1024]);
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
      if (bq) sum += bq[q.bias_gs < 0 ? c : mb + lane_hi * 4 + rr];
      cl[(long long)rr * q.c_ms] = sum;
    }
  }
}

// pack[g][stage][block of 16 rows][term][lane][8] = the terms of src[g * sg + (m / taps) * sm + m % taps + k * sk], zero
// padded in m and k, where lane stands for row m = 16 block + lane % 16 and k = 32 stage + lane / 16 * 8 + 0 .. 7: k
// runs over min(Kdim, Ktotal - g * Kdim) indices.
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
  const int lane = (int)(e & 63);
  const long long r = e >> 6;
  const int blocks = d.Mpad / 16, stage = (int)(r / blocks), m = (int)(r - (long long)stage * blocks) * 16 + (lane & 15);
  const int k0 = stage * SK + (lane >> 4) * 8;
  const int kd = min(d.Kdim, d.Ktotal - g * d.Kdim);
  const int row = m / d.taps;
  const float* s = src + g * d.sg + row * d.sm + (m - row * d.taps) + k0 * d.sk;
  unsigned short h[8], mm[8], l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float v = m < d.M && k0 + i < kd ? s[i * d.sk] : 0.f;
    split_value(v, &h[i], &mm[i], &l[i]);
  }
  unsigned short* dst = pack + ((long long)g * d.Kpad * d.Mpad * 3) + r * 1536 + lane * 8;
  auto put = [](unsigned short* to, const unsigned short (&v)[8]) {
    uint4 q;
    q.x = v[0] | ((unsigned)v[1] << 16);
    q.y = v[2] | ((unsigned)v[3] << 16);
    q.z = v[4] | ((unsigned)v[5] << 16);
    q.w = v[6] | ((unsigned)v[7] << 16);
    *reinterpret_cast<uint4*>(to) = q;
  };
  put(dst, h);
  put(dst + 512, mm);
  put(dst + 1024, l);
}

}  // namespace

int gemm_split_mpad(int M) { return M <= 32 ? 32 : (M + 63) / 64 * 64; }
int gemm_split_kpad(int K) { return (K + SK - 1) / SK * SK; }

// 32-bit byte offsets: the pack of one group, B inside a stage of one column tile
bool gemm_split_fits(const GemmTN& p, bool bt) {
  if (p.bf16 || p.M < 1 || p.Ncols < 1 || p.Kdim < 1) return false;
  if ((long long)p.Mpad * p.Kpad * 6 >= (1LL << 31) || p.b_ks >= (1LL << 22)) return false;
  if (bt) return true;
  const long long T = (BN - 1) / p.bmap.P + 2;  // images that 128 columns can touch
  return p.bmap.P == 2147483647 ? (long long)p.Ncols < (1LL << 29)
                                : (T + 1) * p.bmap.img_stride < (1LL << 28);
}

namespace {
// The forms: tiles of 32 (16 where that is all) and 64 rows, which read A in place and split it themselves, and of 128 and
// 144, for which it is packed first.  A launch less is what counts where the chip is not full (33 to 512 images of fully connected layers,
// up to 2 GFLOP: 0.6 to 0.8 times the time of a pack and a product); large products split A once per column tile too often.

// 32-bit byte offsets in A in place, from a tile's first row and a stage's first k
bool in_place_fits(long long sm, long long sk, int taps) { return (64 / taps + 2) * sm + taps + 32 * sk < (1LL << 29); }

// What a launch takes, in us: rounds of workgroups, each as long as its stages take a workgroup that has its CU alone,
// what every further one on the CU adds per stage and to fill and drain; the launch; the pack (4.3 us and so many per
// million values).  Not less than its bytes at the rate the form streams at.  Fitted to 1160 products of 2 MFLOP to 200
// GFLOP, each with every form, inputs from memory: off by 3 to 10 % in the mean; the form with the lowest estimate takes
// 0.5 to 2 % longer than the best one in the mean.  Per stage of 32 k and workgroup: 64 rows alone 1.0, among three
// 0.68; 144 rows alone 1.36, among two 1.11 (its MFMAs: 0.75).
struct Form {
  int rb, share;  // workgroups that a CU holds
  struct Rate {
    double stage, next, fill, launch, pack, bytes, next_fill;
  } rate[2];  // B column-contiguous, k-contiguous
};
constexpr Form kForms[4] = {
    {2, 4, {{0.885, 0.322, 1.723, 2.504, 0.00, 3.34e6, 1.138}, {1.094, 0.372, 0.000, 3.194, 0.00, 2.79e6, 0.789}}},
    {4, 3, {{1.010, 0.517, 1.152, 3.516, 0.00, 3.74e6, 1.983}, {0.929, 0.680, 0.000, 4.514, 0.00, 4.13e6, 0.304}}},
    {8, 2, {{1.226, 0.773, 1.057, 4.257, 5.98, 2.48e6, 3.112}, {1.034, 0.967, 1.682, 3.886, 5.10, 3.15e6, 0.000}}},
    {9, 2, {{1.356, 0.867, 1.333, 3.711, 6.00, 2.75e6, 2.727}, {1.333, 1.106, 0.000, 4.913, 4.80, 3.02e6, 0.000}}}};

// One tile of up to 32 rows with B column-contiguous, which waves work on alone in most forms: fitted to 2870 products, off by
// 8 % in the mean, 17 % in nine of ten (with the rates of many such tiles: a quarter, by 1.55 too much for long
// contractions, which sent layers to kernels that took twice as long).
constexpr Form kFewRows = {2, 5, {{0.424, 0.147, 2.033, 3.420, 0.00, 5.36e6, 0.000}, {}}};

double form_us(const Form& f, bool bt, int M, int K, long long cols, long long G) {
  const Form::Rate& r = f.rate[bt];
  const unsigned long long tiles_m = ((unsigned)M + 16u * f.rb - 1) / (16u * f.rb);
  const unsigned long long per_cu = (tiles_m * ((cols + BN - 1) / BN) * G + 255) / 256, rounds = per_cu / f.share;
  const int rest = (int)(per_cu - rounds * f.share), stages = (int)(((unsigned)K + SK - 1) / SK);
  auto round = [&](int n) { return n ? stages * (r.stage + (n - 1) * r.next) + r.fill + (n - 1) * r.next_fill : 0.0; };
  double t = (double)rounds * round(f.share) + round(rest) + r.launch;
  if (f.rb > 4) t += 4.3 + r.pack * 1e-6 * (double)((M + 63) / 64 * 64) * (stages * (double)SK) * G;
  const double values = (double)G * ((double)K * cols + (double)M * cols + (double)M * K);
  return std::max(t, 4.0 * values / r.bytes + r.launch);
}

template <class Fits>
const Form* choose(bool bt, int M, int K, long long cols, long long G, Fits fits, double* us) {
  const Form* best = nullptr;
  for (const Form& f : kForms) {
    // (up to 32 rows 32 at a time, whatever the estimates say: 16 images of fc6 forward 45 us against 52 in tiles of 64)
    if (!fits(f) || (f.rb == 4 && M <= 32)) continue;
    const double t = form_us(f.rb == 2 && M <= 32 && !bt ? kFewRows : f, bt, M, K, cols, G);
    if (!best || t < *us) {
      best = &f;
      *us = t;
    }
  }
  return best;
}

template <int RB, BForm BF, AForm AF, int ALONE = 0>
int launch_variant(const GemmTN& p, int Ktotal, hipStream_t st) {
  const int tiles_m = (p.M + 16 * RB - 1) / (16 * RB), tiles_n = ((BF == kPairs ? p.pair_cols : p.Ncols) + BN - 1) / BN;
  const long long blocks = (long long)tiles_m * tiles_n;
  if (blocks <= 0 || blocks >= 2147483647LL || p.G < 1 || p.G > 65535) return CCT_EUNSUPPORTED;
  const double mk = (double)p.M * p.Kdim * p.G, kn = (double)p.Kdim * p.Ncols * p.G;
  ProfScope ps(2.0 * p.M * kn, (AF == kPacked ? 6.0 : 4.0) * mk + 4.0 * kn + 4.0 * (double)p.M * p.Ncols * p.G, st,
               "gemm_split<%d, %s>", 16 * RB, BF == kContiguous ? "k-contiguous" : "in place");
  hipLaunchKernelGGL((gemm_split<RB, BF, AF, ALONE>), dim3((unsigned)blocks, (unsigned)p.G), dim3(NT), 0, st, p, Ktotal,
                     tiles_m, tiles_n);
  CCT_CHECK_LAUNCH();
  return CCT_OK;
}

template <BForm BF, AForm AF>
int launch_in_place(const GemmTN& p, int Ktotal, hipStream_t st) {
  if (p.rb == 4) return launch_variant<4, BF, AF>(p, Ktotal, st);
  const bool one = p.Kdim <= SK;
  if (p.M <= 16) return one ? launch_variant<1, BF, AF, 1>(p, Ktotal, st) : launch_variant<1, BF, AF, 2>(p, Ktotal, st);
  return one ? launch_variant<2, BF, AF, 1>(p, Ktotal, st) : launch_variant<2, BF, AF>(p, Ktotal, st);
}

template <BForm BF>
int launch_columns(const GemmTN& p, int Ktotal, hipStream_t st) {
  if (!p.a_ms) return p.rb == 8 ? launch_variant<8, BF, kPacked>(p, Ktotal, st) : launch_variant<9, BF, kPacked>(p, Ktotal, st);
  if (p.a_ks == 1 && p.a_taps == 1) return launch_in_place<BF, kRows>(p, Ktotal, st);
  if constexpr (BF == kContiguous) return CCT_EUNSUPPORTED;
  else return launch_in_place<BF, kStrided>(p, Ktotal, st);
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
}  // namespace

// `pack`: there is room for it.
double gemm_split_seconds(bool bt, bool pack, int M, int K, long long cols, long long G) {
  double us = 0.0;
  choose(bt, M, K, cols, G, [&](const Form& f) { return pack || f.rb <= 4; }, &us);
  return 1e-6 * us;
}

int gemm_split_operand(GemmTN* p, bool bt, const float* src, void* pack, int Ktotal, long long sm, long long sk, long long sg,
                       int taps, hipStream_t st) {
  const bool in_place = in_place_fits(sm, sk, taps);
  double us;
  const Form* f = choose(bt, p->M, p->Kdim, p->Ncols, p->G, [&](const Form& v) { return v.rb <= 4 ? in_place : pack != nullptr; }, &us);
  if (!f) return CCT_EUNSUPPORTED;
  p->rb = f->rb;
  p->a_ms = 0;
  if (f->rb > 4) {
    p->A = pack;
    p->a_gs = (long long)p->Mpad * p->Kpad;
    return launch_pack_rows_split(src, pack, p->G, p->M, p->Mpad, p->Kpad, p->Kdim, Ktotal, sm, sk, sg, st, taps);
  }
  p->A = src;
  p->a_gs = sg; p->a_ms = sm; p->a_ks = sk; p->a_taps = taps;
  // elements of A from p->A on
  p->a_len = (p->G - 1) * sg + (p->M - 1) / taps * sm + taps - 1 + (Ktotal - (p->G - 1) * (long long)p->Kdim - 1) * sk + 1;
  return CCT_OK;
}

// Pairs, unless the planes are so small that the columns which make them even weigh, or these take the count past 32
// bits (an odd plane's is up to a fifteenth more than the tensor's columns, which may be up to 2^31 - 257).
int gemm_split_pair_columns(int P, int Ncols, int* pair_P) {
  *pair_P = 0;
  if (P == 2147483647) return (Ncols + 1) / 2 * 2;
  const long long even = P + P % 2, cols = Ncols / P * even;
  if ((P % 2 && P < 15) || cols > 2147483647LL - (BN - 1)) return 0;
  *pair_P = (int)even;
  return (int)cols;
}

int launch_gemm_split(const GemmTN& p0, int Ktotal, bool bt, hipStream_t st) {
  GemmTN p = p0;
  colmap_prepare(&p.bmap);
  colmap_prepare(&p.cmap);
  if (p.Mpad != gemm_split_mpad(p.M) || p.Kpad != gemm_split_kpad(p.Kdim)) return CCT_EINVAL;
  if (!gemm_split_fits(p, bt)) return CCT_EUNSUPPORTED;
  p.pair_P = p.pair_cols = 0;
  // elements of B from p.B on
  p.b_len = bt                        ? (long long)p.Ncols * p.b_ks
            : p.bmap.P == 2147483647 ? Ktotal * p.b_ks
                                     : (long long)(p.Ncols / p.bmap.P) * p.bmap.img_stride;
  if (bt) return launch_columns<kContiguous>(p, Ktotal, st);
  p.pair_cols = gemm_split_pair_columns(p.bmap.P, p.Ncols, &p.pair_P);
  if (p.pair_P) make_fastdiv_parts(p.pair_P, &p.pair_M, &p.pair_sh);
  return p.pair_cols ? launch_columns<kPairs>(p, Ktotal, st) : launch_columns<kColumns>(p, Ktotal, st);
}

}  // namespace cct
