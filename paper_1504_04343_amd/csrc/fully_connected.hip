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
// over O the same way (the splits run as the groups of one launch).  The products run on gemm_split; the
// fp32 kernels are for workspaces without room for its packed operand and for backward-weights passes
// over up to 32 images.
#include <algorithm>
#include <cstring>

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
  float acc = 0.0f;
  int s = 0;
  for (; s + 4 <= S; s += 4) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = src[(long long)(s + u) * total];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += v[u];
  }
  for (; s < S; ++s) acc += src[(long long)s * total];
  if (bias) {
    const int n = fdiv((int)t, divO);
    acc += bias[(int)t - n * divO.d];
  }
  y[t] = acc;
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
// cannot take, or a backward-weights pass over up to 32 images, whose product is one short stage of
// 32 images: the fp32 kernel wastes less there (fc6, one image: 36 us against 43).
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
  long long S = 1, least = 1;
  double best = 1e30, shortest = 1e30;
  *limited = false;
  auto each = [&](auto visit) {
    visit(1LL);
    for (int sp = 2; sp <= 64 && Kd >= (long long)sp * kFcMinSplitRows; sp += sp < 16 ? 1 : 4) visit((long long)sp);
  };
  if (!bwdw) {
    each([&](long long sp) {
      const long long n = count(sp);
      const double t = chain_seconds(p.Mpad, (cols + 127) / 128, (int)len(sp), n) + (n > 1 ? 2.0 * n * out / 6.0e12 : 0.0);
      if (t >= shortest) return;
      if (need(sp) <= cap) {
        shortest = t;
        least = sp;
      } else {
        *limited = true;
      }
    });
    S = least;
    each([&](long long sp) {
      if (sp < least || need(sp) > cap) return;
      const double t = seconds(sp);
      if (t >= best) return;
      best = t;
      S = sp;
    });
  }
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
