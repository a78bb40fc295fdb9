// The matrix product of two operands that lie in memory as granules: 8 consecutive reduction indices of one
// row as 16 bytes of bf16, one term (bf16 operands) or three whose sum is the fp32 value (split_bf16.h).
// A column is the 8 reduction indices of a granule.
//
// A workgroup computes BM x 256 results with waves of up to 64 x 64.  A stage is SLOTS (column, term) pairs of
// both operands, moved from memory into LDS by buffer loads that write LDS directly: no registers, no vector
// instruction, no conversion in the loop.  Two stages alternate, one meeting of the workgroup per stage;
// operand reads are 16 consecutive granules of four columns, which do not conflict.
//
// Blocks of 16 x 16 (v_mfma_f32_16x16x32_bf16) and not of 32 x 32 (32x32x16): at the card's power limit, which large
// products run into, they are the faster ones (operands in registers, 2 waves per SIMD, random normals: 2200 against
// 1870 TFLOP/s; zeros: 2450 both), because an accumulator is read and written half as often per flop; the results round
// alike (2-norm against 64 bits the same to four digits).  Measured with three terms, 128 rows: conv2's
// backward-weights product (114.7 GFLOP) 604 -> 537 us, conv3's at batch 1024 (306 GFLOP) 1319 -> 1255.
// 32 x 32 where the results go straight to the output tensor (conv_granules), in rows of 128 bytes instead of 64: over
// 3400 bf16 layers in bursts of 0.4 ms forward 1 to 3 % faster, backward-data 2 to 5 % on 128 rows, and in runs of one
// pass that last 0.92 to 0.98 times the time on 128 rows, 0.98 to 1.03 on 64; partial products (conv_bwdw_img) 2 %
// slower.
//
// A wave of 64 x 64 reads 24 KiB of LDS for 96 MFMAs (1536 matrix-core cycles) per 32 reduction indices, three quarters
// of what LDS can deliver to four SIMDs, and a 128 x 256 workgroup fetches 72 KiB of L2 for 3072 cycles of its CU.
// With one term LDS and the matrix cores are equally busy.
#pragma once
#include <type_traits>

#include "cct_internal.h"
#include "gemm_common.h"
#include "split_bf16.h"

namespace cct {
namespace {

constexpr int kGran = 16;  // bytes of a granule
constexpr int BN = 256;    // columns of the result per workgroup

typedef __attribute__((address_space(3))) void* lds_ptr;

// waves of a workgroup
constexpr int granule_waves(int BM, int TERMS) { return TERMS == 3 ? 8 : BM / 16; }

__device__ __forceinline__ f32x4 granule_mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 granule_mfma(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// MB: rows and columns of a block of results, 16 or 32
template <int BM, int TERMS, int SLOTS, int MB>
struct GranuleProduct {
  static constexpr int JB = 64 / MB;  // blocks of a wave's 64 columns; columns that an MFMA takes
  using Acc = std::conditional_t<MB == 32, floatx16, f32x4>;
  static constexpr int NW = granule_waves(BM, TERMS);
  static constexpr int WAVES_N = BN / 64;
  static constexpr int NCOL = SLOTS / TERMS;  // columns per stage
  static_assert(SLOTS % TERMS == 0 && NCOL % 4 == 0, "an MFMA takes four columns");
  static constexpr int BMP = (BM + 63) / 64 * 64;  // rows as they are loaded
  static constexpr int STAGE = SLOTS * (BMP + BN) * kGran;
  static constexpr int LDS = 2 * STAGE;
  // A wave moves the granules of CPW columns, or a WPC-th of one column: one address per column.
  static constexpr int CPW = NCOL > NW ? NCOL / NW : 1, WPC = NW > NCOL ? NW / NCOL : 1;
  static constexpr int A_PARTS = BMP / 64, B_PARTS = BN / 64 / WPC;  // loads of 64 rows, per wave for B
  static constexpr int A_UNITS = TERMS * A_PARTS, A_PER = (A_UNITS + WPC - 1) / WPC;
  static_assert(CPW * NW == NCOL * WPC && WPC <= 2, "whole loads");

  // byte offsets of the rows a lane loads, from a column's granules: the same in every stage
  unsigned a_voff[A_PARTS], b_voff[B_PARTS];
  static constexpr int RB = BM / (MB * NW / WAVES_N);  // blocks of rows per wave
  // three terms: h*h alone in one accumulator, the corrections in the other
  Acc acc[RB][JB], acc_c[TERMS == 3 ? RB : 1][TERMS == 3 ? JB : 1];

  static __device__ __forceinline__ int wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
  // which 64 rows of B b_voff[u] stands for
  __device__ __forceinline__ int b_part(int u) const { return wave() % WPC * B_PARTS + u; }

  // Columns [c_begin, c_end): A's lie a_col apart, B's at b_at(column); terms lie a_term / b_term apart.
  template <class BAt>
  __device__ __forceinline__ void run(unsigned char* smem, int c_begin, int c_end, const unsigned char* A,
                                      long long a_col, int a_term, int b_term, BAt b_at) {
    const int lane = threadIdx.x & 63, w = wave(), sub = w % WPC;
    // columns past the end have an empty range: they load as zeros
    auto load_stage = [&](int buf, int c0) {
      unsigned char* As = smem + buf * STAGE;
      unsigned char* Bs = As + SLOTS * BMP * kGran;
#pragma unroll
      for (int v = 0; v < CPW; ++v) {
        const int cc = w / WPC + v * NW;
        const int col = c0 + cc, cl = min(col, c_end - 1), range = col < c_end ? 0x7fffffff : 0;
        const __amdgpu_buffer_rsrc_t ra =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(A + cl * a_col), 0, range, 0x00020000);
        const __amdgpu_buffer_rsrc_t rb =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(b_at(cl)), 0, range, 0x00020000);
#pragma unroll
        for (int k = 0; k < TERMS; ++k)
#pragma unroll
          for (int u = 0; u < B_PARTS; ++u)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rb, (lds_ptr)(Bs + ((cc * TERMS + k) * BN + (sub * B_PARTS + u) * 64) * kGran), 16, (int)b_voff[u],
                k * b_term, 0, 0);
#pragma unroll
        for (int k = 0; k < TERMS; ++k)
#pragma unroll
          for (int u = 0; u < A_PARTS; ++u)  // the first A_PER units are the first wave's
            if (WPC == 1 || (k * A_PARTS + u) / A_PER == sub)
              __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr)(As + ((cc * TERMS + k) * BMP + u * 64) * kGran),
                                                       16, (int)a_voff[u], k * a_term, 0, 0);
      }
    };
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int r = 0; r < MB * MB / 64; ++r) {
          acc[i][j][r] = 0.f;
          if constexpr (TERMS == 3) acc_c[i][j][r] = 0.f;
        }

    // operands read behind the MFMAs before them; one term has a single MFMA per block, which is too little to read
    // behind (1 to 4 % slower)
    constexpr bool AHEAD = TERMS == 3;
    const int stages = (c_end - c_begin + NCOL - 1) / NCOL;  // <= 0 for an empty range
    if (stages > 0) load_stage(0, c_begin);
    const int lo = lane % MB, kg = lane / MB;  // row of a block, which of the JB columns
    const int a_lds = (kg * TERMS * BMP + w / WAVES_N * (MB * RB) + lo) * kGran;
    const int b_lds = SLOTS * BMP * kGran + (kg * TERMS * BN + w % WAVES_N * 64 + lo) * kGran;
    for (int t = 0; t < stages; ++t) {
      // this stage's loads have landed and nobody reads the other buffer any more
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      __syncthreads();
      if (t + 1 < stages) load_stage((t + 1) & 1, c_begin + (t + 1) * NCOL);
      const unsigned char* st = smem + (t & 1) * STAGE;
#pragma unroll
      for (int kb = 0; kb < NCOL / JB; ++kb) {
        bf16x8 a[RB][TERMS], b[AHEAD ? 2 : JB][TERMS];
        auto read_a = [&](int i) {
#pragma unroll
          for (int k = 0; k < TERMS; ++k)
            a[i][k] = *reinterpret_cast<const bf16x8*>(st + a_lds + ((JB * kb * TERMS + k) * BMP + i * MB) * kGran);
        };
        auto read_b = [&](int set, int j) {
#pragma unroll
          for (int k = 0; k < TERMS; ++k)
            b[set][k] = *reinterpret_cast<const bf16x8*>(st + b_lds + ((JB * kb * TERMS + k) * BN + j * MB) * kGran);
        };
        if constexpr (AHEAD) {
          read_a(0);
          read_b(0, 0);
        } else {
#pragma unroll
          for (int i = 0; i < RB; ++i) read_a(i);
#pragma unroll
          for (int j = 0; j < JB; ++j) read_b(j, j);
        }
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            // the next operands behind these MFMAs: in the first column of blocks the rows, then the next column
            if (AHEAD && j == 0 && i + 1 < RB) read_a(i + 1);
            if (AHEAD && i == RB - 1 && j + 1 < JB) read_b((j + 1) & 1, j + 1);
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
#define CCT_M(X, Y, ACC) ACC[i][j] = granule_mfma(a[i][X], b[AHEAD ? j & 1 : j][Y], ACC[i][j])
            if constexpr (TERMS == 3) {
              CCT_M(2, 0, acc_c);
              CCT_M(0, 2, acc_c);
              CCT_M(1, 1, acc_c);
              CCT_M(1, 0, acc_c);
              CCT_M(0, 1, acc_c);
            }
            CCT_M(0, 0, acc);
#undef CCT_M
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
          }
      }
    }
  }

  // the row of result r of block row i, the column of block column j: relative to the workgroup's tile; four consecutive
  // rows per lane and quad of registers
  __device__ __forceinline__ int row(int i, int r) const {
    return wave() / WAVES_N * (MB * RB) + i * MB + r / 4 * 8 + ((int)threadIdx.x & 63) / MB * 4 + r % 4;
  }
  __device__ __forceinline__ int column(int j) const { return wave() % WAVES_N * 64 + j * MB + ((int)threadIdx.x & 63) % MB; }

  // f(row, column, value) for every result of the lane, relative to the workgroup's tile.  The first row and column are
  // worked out once: through row() and column() every result had its own, which are a quarter more instructions in all and
  // 2 us of a short launch (conv_bwdw_img<64, 1, 8>, 3 images of 15 x 18, 5.1 us against 6.9).
  template <class F>
  __device__ __forceinline__ void for_each(F f) const {
    const int lane = threadIdx.x & 63, w = wave();
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < MB * MB / 64; ++r) {
          float v = acc[i][j][r];
          if constexpr (TERMS == 3) v += acc_c[i][j][r];
          f(w / WAVES_N * (MB * RB) + i * MB + r / 4 * 8 + lane / MB * 4 + r % 4, w % WAVES_N * 64 + j * MB + lane % MB, v);
        }
  }
};

}  // namespace
}  // namespace cct
