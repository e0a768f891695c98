// Pair kernels: the O(P^2) Gaussian blob-kernel sums of the particle scheme.
//
// One pass computes, for every row particle I and a column weight vector wh,
//   O_I[n] = sum_J e_IJ V_J[n],   V_J = (wh_J x_J, wh_J),
//   e_IJ   = exp2(t_IJ),  t_IJ = -kappa |x_I - x_J|^2,  kappa = log2(e) / 2h^2,
// over all J including J = I (eq. model_DeteParAppr and the two kernel sums of
// eq. model_DymRepPar).  The squared distance is expanded through augmented
// vectors so that t_IJ is one dot product:
//   Q_I = (x_I, -kappa |x_I|^2, 1),  K_J = (2 kappa x_J, 1, -kappa |x_J|^2),
//   t_IJ = Q_I . K_J.
// The FP32 forms below clamp e at one, the expanded |x_I - x_J|^2 at zero; the others
// leave t as it comes, which exceeds zero by its rounding only.
//
// Five implementations (vds.h), by the operand arrays that the prep kernel writes.  The
// default, FP32 by three BF16 parts, is described where it stands; the others:
//  * MFMA: each wavefront owns RB blocks of 16 rows; per 16-column chunk,
//    ceil((D+2)/4) v_mfma_f32_16x16x4_f32 form t for a 16x16 pair tile, the
//    VALU takes exp2, and four more MFMAs accumulate e V.  The accumulator
//    layout of the first product is already the A-operand layout of the second
//    once the chunk's columns are visited in the order 4k + i, which is how the
//    prep kernel stores V.  Operands are pre-swizzled so every lane reads
//    consecutive dwords.
//  * VALU: one thread per row pair, column tiles of 256 staged in LDS, FP32
//    FMAs, v_exp_f32.
//  * MFMA, FP16-split product: t as above on FP32 MFMA, then the e V product
//    on v_mfma_f32_16x16x32_f16 with both factors split into two halves,
//    e = e_hi + e_lo and V = V_hi + V_lo, and e V taken as
//    e_hi V_hi + e_hi V_lo + e_lo V_hi (the dropped e_lo V_lo is 2^-22 of it).
//    Half products are exact in the FP32 accumulator, so the product keeps
//    about 22 bits against 24 for FP32, at three MFMAs per 32 columns instead
//    of eight.  FP16 has a narrow exponent range, so e is computed as
//    2^(t + 15) (the shift enters through the accumulator of the t product)
//    and the column weights in V are divided by their maximum; with e spanning
//    2^15 down to the FP16 subnormals, pairs as weak as 1e-12 of the strongest
//    still count.  The shift and the weight maximum are taken out in FP64 at
//    the end.
//  * MFMA, FP16-split products throughout: as the previous one, and t too on
//    v_mfma_f32_16x16x32_f16 from split halves of sqrt(2 kappa) x, with the
//    squared norms kept in FP32 (layout at pair_rows_f16).
// Column ranges are split over blockIdx.y (the default form: over the runs of a balanced
// grid); every split writes its own partial sums, reduced later in a fixed order
// (deterministic, no float atomics).
//
// Accuracy: the drift needs x_I S_I - M_I, a difference of two sums whose
// magnitudes can exceed it by an order of magnitude (narrow kernels, isolated
// particles).  Plain FP32 accumulation over thousands of columns would leave
// errors of ~1e-6 relative to the sums, amplified by that ratio.  So the FP32
// accumulators are flushed into FP64 running sums every kFlush chunks (16
// columns each; kFlush3 of 32 in the default form), and the kernel itself forms, in FP64,
//   A_I[n] = x_I[n] O_I[D] - O_I[n]  (n < D),   O_I[D] = sum_J e_IJ wh_J,
// i.e. it writes sum_J e_IJ wh_J (x_I - x_J) and the weighted kernel sum.
// With exclude_self the J = I term is left out of both sums: it adds nothing to
// the difference sum, but for an isolated particle it dominates the kernel sum
// and would swamp its neighbours' contributions in FP32.  The caller adds the
// self weight back in FP64.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "bf3.h"
#include "vds_internal.h"

namespace vds {

constexpr int kFlush = 8;  // chunks per FP32 accumulation group

// One wavefront: row blocks rb0 .. rb0 + RB - 1 against column chunks [c0, c1),
// results into out[row][16].  No barriers: waves are independent.
template <int KK, int RB>
__device__ void pair_rows(const float *__restrict__ QB, int nrow_blocks, const float *__restrict__ KA,
                          const float4 *__restrict__ VB, int c0, int c1, const float *__restrict__ xc, int D,
                          int exclude_self, float *__restrict__ out, int rb0) {
  if (rb0 >= nrow_blocks) return;
  const int lane = threadIdx.x & 63;
  // position of the self pair inside a diagonal 16x16 tile, per element i
  const int diag_i = (lane & 15) - 4 * (lane >> 4);  // in 0..3 when this lane holds one

  float qv[RB][KK];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qv[r][kk] = (rb0 + r < nrow_blocks) ? QB[((int64_t)(rb0 + r) * KK + kk) * 64 + lane] : 0.f;

  double tot[RB][4];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) tot[r][i] = 0.0;

  float ka[KK];
  float4 vb;
  if (c0 < c1) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) ka[kk] = KA[((int64_t)c0 * KK + kk) * 64 + lane];
    vb = VB[(int64_t)c0 * 64 + lane];
  }
  for (int c = c0; c < c1;) {
    const int cg_end = min(c1, c + kFlush);
    floatx4 acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (; c < cg_end; ++c) {
      // prefetch the next chunk's operands while this one computes
      float kn[KK];
      float4 vn;
      const int cn = (c + 1 < c1) ? c + 1 : c;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kn[kk] = KA[((int64_t)cn * KK + kk) * 64 + lane];
      vn = VB[(int64_t)cn * 64 + lane];

#pragma unroll
      for (int r = 0; r < RB; ++r) {
        floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) t = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[kk], qv[r][kk], t, 0, 0, 0);
        // e = 2^t clamped to [0, 1] by the instruction's output clamp: the same as
        // clamping the expanded squared distance at zero
        float e0 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[0]), 0.f, 1.f);
        float e1 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[1]), 0.f, 1.f);
        float e2 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[2]), 0.f, 1.f);
        float e3 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[3]), 0.f, 1.f);
        if (exclude_self && c == rb0 + r) {  // scalar branch: the diagonal tile
          e0 = diag_i == 0 ? 0.f : e0;
          e1 = diag_i == 1 ? 0.f : e1;
          e2 = diag_i == 2 ? 0.f : e2;
          e3 = diag_i == 3 ? 0.f : e3;
        }
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(e0, vb.x, acc[r], 0, 0, 0);
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(e1, vb.y, acc[r], 0, 0, 0);
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(e2, vb.z, acc[r], 0, 0, 0);
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(e3, vb.w, acc[r], 0, 0, 0);
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) ka[kk] = kn[kk];
      vb = vn;
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[r][i] += (double)acc[r][i];
  }

  // lane holds O[row 4 (lane / 16) + i][column lane % 16] of each row block;
  // the weighted kernel sum O[.][D] sits in lane (lane & 48) + D
  const int n = lane & 15;
  const int src = (lane & 48) + D;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    if (rb0 + r >= nrow_blocks) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double s = __shfl(tot[r][i], src);
      const int64_t row = (int64_t)(rb0 + r) * 16 + 4 * (lane >> 4) + i;
      double v = 0.0;
      if (n < D) v = (double)xc[row * D + n] * s - tot[r][i];
      else if (n == D) v = s;
      out[row * 16 + n] = (float)v;
    }
  }
}

template <int KK, int RB>
__global__ __launch_bounds__(256) void k_pair_mfma(const float *__restrict__ QB, int nrow_blocks,
                                                   const float *__restrict__ KA, const float4 *__restrict__ VB,
                                                   int ncol_chunks, int chunks_per_split,
                                                   const float *__restrict__ xc, int D, int exclude_self,
                                                   float *__restrict__ partial, int64_t part_stride_rows,
                                                   const int *__restrict__ done) {
  if (done != nullptr && *done) return;
  // wave index as a scalar so that row-block tests compile to scalar branches
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb0 = ((int)blockIdx.x * 4 + wave) * RB;
  const int c0 = (int)blockIdx.y * chunks_per_split;
  const int c1 = min(ncol_chunks, c0 + chunks_per_split);
  pair_rows<KK, RB>(QB, nrow_blocks, KA, VB, c0, c1, xc, D, exclude_self,
                    partial + (int64_t)blockIdx.y * part_stride_rows * 16, rb0);
}

// ---- FP32 by three BF16 parts ------------------------------------------------
//
// The default form (VDS_PAIR_MFMA32).  On gfx950 an FP32 matrix instruction
// runs at a sixteenth of the BF16 rate and lets no vector instruction issue
// beside it, a BF16 one does.  An FP32 number is the exact sum of three BF16
// numbers (8 bits each), so both products are taken on
// v_mfma_f32_16x16x32_bf16, whose products are exact in FP32, from operands
// that hold all 24 bits:
//  * distances: with y = sqrt(2 kappa) x = yh + ym + yl, six products per
//    component (hh, mm, hm, mh, hl, lh; the dropped ml, lm, ll are below
//    2^-26 |y_I y_J|) and both norms -|y|^2 / 2 in three parts each give
//    t_IJ = y_I.y_J - |y_I|^2/2 - |y_J|^2/2 in 6 D + 6 slots of the
//    contraction (D = 9: two instructions per 16 x 16 pairs).  y and the norms
//    are split from FP64, and the norm is that of the parts, so t is the
//    distance of two slightly displaced points to within the accumulation's
//    rounding;
//  * kernel-weighted sums: e = 2^t is cut into three parts in registers: the
//    upper halves of the values are a BF16 operand as they stand, and what
//    they leave comes from a product with minus the identity (exact), which
//    takes it off the vector units.  The parts meet those of V, which sit side
//    by side as columns of B (D = 9: 30 of 32).
// The distance product leaves lane l with the row I = l % 16 and the columns
// J = 4 (l / 16) + v of two 16-column blocks: eight values, which are the
// A operand of the sums' instruction (row l % 16, k = 8 (l / 16) + i) when V is
// stored with its columns in the order J = 16 (i / 4) + 4 (l / 16) + i % 4.
// Eight waves of a workgroup take the same 32-column chunks, staged in LDS
// straight from memory (no registers), kStage3 chunks per barrier, double
// buffered.  Accumulation: FP32 within groups of kFlush3 chunks, then the
// three parts of a sum are added and go to FP64, and the difference sums are
// formed in FP64 as for the other forms.
//
// Bound: the matrix pipe and vector issue together, and the board's power (the
// clock falls from 2.39 to about 2.1 GHz).  Per 1024 pairs at D = 9: 26 matrix
// instructions (416 cycles), 16 exponentials and 24 packs (224), about 690
// cycles in all.  Measured, P = 20000, D = 9: 128 us per pass against 170 with
// FP32 instructions (32x32x2 distances, 4x4x1 sums); D = 15, P = 50000: 1.02
// against 1.57 ms; 32 batched ensembles (4.3e9 pairs) 1.35 against 1.87 ms.
// With dot products (v_dot2_f32_bf16) forming what a cut leaves, the pass took
// 157 us: they hold the matrix pipe; with and/subtract pairs, 153.

constexpr int kWaves3 = 8;   // waves per workgroup
constexpr int kStage3 = 2;   // 32-column chunks staged in LDS per barrier

// Row blocks of 16 per wave: rows_per_wave of the tuning, 1 or 2.  From D = 12
// on, two would not leave four waves a SIMD's registers (D = 15, P = 30000: 368
// against 538 us per pass), so one is taken.
constexpr int kMaxRB3 = 2;
constexpr int bf3_rb(int D, int rows_per_wave) { return D >= 12 ? 1 : rows_per_wave; }

// A single state of at most this many rows takes one as well: with runs of a few
// units, half the rows are half of what a workgroup loads before its first chunk and
// sums after its last, and 2048 waves' work divides more evenly.  Explicit step with
// two and with one, D = 9: P = 4100 49 and 41 us, 7000 67 and 60, 9200 84 and 82,
// 10240 93 and 93, 12200 116 and 120 (D = 3: 46 and 36, 56 and 49, 67 and 65, 73 and
// 74, 90 and 94), where each column's operands being read twice as often costs more.
constexpr int64_t kOneBlockRows3 = 9216;

template <int D>
struct Bf3Shape {
  static constexpr int NQ = bf3_slices(D);   // instructions of a 16x16 distance tile
  static constexpr int NT = bf3_tiles(D);    // 16-column tiles of the three parts of the D + 1 sums
  static constexpr int PC = 2 * NQ + NT;     // 1 KiB pieces (64 lanes x 16 bytes) of one 32-column chunk
};

// LDS of one workgroup: staged chunks (double buffered) and the FP64 running
// sums of its waves (one slot per lane and value, touched by its own lane only;
// held here they leave the registers to the arithmetic, so that four waves
// share a SIMD: 128 instead of 147 us per pass at D = 9, P = 20000).
template <int D>
struct Bf3Lds {
  uint4 buf[2][kStage3 * Bf3Shape<D>::PC * 64];
  double tot[kWaves3][4 * kMaxRB3][64];
};

// One segment: wave w of the workgroup takes the 16-row blocks
// (kWaves3 rg + w) RB .. + RB - 1 against the columns of chunks [c0, c1) and
// hands the partial sums of its rows to put(row, n, sum), self pairs
// left out.  Every thread of the workgroup calls it with the same arguments (it holds
// barriers).  With run_len > 0 the segment is part of a run of
// run_len chunk units of which done0 came before it, and every stage sets the
// waves' issue priority by the share of the run still to do (see k_pair_bf3).
template <int D, int RB, class Put>
__device__ __forceinline__ void bf3_segment(const uint4 *__restrict__ K3, const uint4 *__restrict__ V3,
                                            const float *__restrict__ xr, int rg, int c0,
                                            int c1, const Put &put, Bf3Lds<D> &lds,
                                            int64_t done0 = 0, int64_t run_len = 0) {
  using S = Bf3Shape<D>;
  constexpr int NQ = S::NQ, NT = S::NT, PC = S::PC;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb0 = (rg * kWaves3 + wave) * RB;
  // position of the self pair inside a diagonal 16x16 block, per element i
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  bf16x8 neg[2];
  minus_identity(lane, neg);

  // wave w brings in the pieces w, w + 8, ... of the stage that starts at
  // chunk c (chunk by chunk: distance operands, then V)
  auto stage = [&](int c, int buf) {
#pragma unroll
    for (int i = 0; i < (kStage3 * PC + kWaves3 - 1) / kWaves3; ++i) {
      const int pc = wave + kWaves3 * i;
      const int cc = pc / PC, w = pc % PC;
      if (pc < kStage3 * PC && c + cc < c1) {  // scalar
        const uint4 *src = w < 2 * NQ ? K3 + ((int64_t)(c + cc) * 2 * NQ + w) * 64
                                      : V3 + ((int64_t)(c + cc) * NT + (w - 2 * NQ)) * 64;
        piece_to_lds(src, &lds.buf[buf][pc * 64], lane);
      }
    }
  };
  stage(c0, 0);

  bf16x8 q[RB][NQ];
#pragma unroll
  for (int r = 0; r < RB; ++r) bf3_row_operand<D>(K3, rb0 + r, lane, q[r]);
  double (*tl)[64] = lds.tot[wave];
  floatx4 acc[RB][NT];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) tl[4 * r + i][lane] = 0.0;
#pragma unroll
    for (int T = 0; T < NT; ++T) acc[r][T] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  auto flush = [&] {
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      double t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = tl[4 * r + i][lane];
      bf3_flush<D>(acc[r], lane, t);
#pragma unroll
      for (int i = 0; i < 4; ++i) tl[4 * r + i][lane] = t[i];
    }
  };
  // one chunk of 32 columns; kDiag: it holds the wave's self pairs
  auto chunk = [&](int c, const uint4 *cb, auto diag) {
    constexpr bool kDiag = decltype(diag)::value;
    bf16x8 ka[2][NQ], va[NT];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int m = 0; m < NQ; ++m) ka[b][m] = as_bf8(cb[(b * NQ + m) * 64 + lane]);
#pragma unroll
    for (int T = 0; T < NT; ++T) va[T] = as_bf8(cb[(2 * NQ + T) * 64 + lane]);
    floatx4 e[RB][2];
#pragma unroll
    for (int m = 0; m < NQ; ++m)
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          if (m == 0) e[r][b] = floatx4{0.f, 0.f, 0.f, 0.f};
          e[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[b][m], q[r][m], e[r][b], 0, 0, 0);
        }
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // no clamp: t exceeds zero only by its rounding
#pragma unroll
        for (int i = 0; i < 4; ++i) e[r][b][i] = __builtin_amdgcn_exp2f(e[r][b][i]);
        if constexpr (kDiag)
          if (2 * c + b == rb0 + r) {
#pragma unroll
            for (int i = 0; i < 4; ++i) e[r][b][i] = diag_i == i ? 0.f : e[r][b][i];
          }
      }
    // e = e_0 + e_1 + e_2 in BF16; part p meets the columns of the parts
    // q <= 2 - p of V (the others are below 2^-24 of the product), rounded up
    // to whole tiles.  What a cut leaves is formed on the matrix cores.
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const int nt = ((3 - p) * (D + 1) + 15) / 16;
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const bf16x8 ep = upper_halves(e[r][0], e[r][1]);
        if (p < 2) {
#pragma unroll
          for (int b = 0; b < 2; ++b) e[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(neg[b], ep, e[r][b], 0, 0, 0);
        }
#pragma unroll
        for (int T = 0; T < nt; ++T) acc[r][T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ep, va[T], acc[r][T], 0, 0, 0);
      }
    }
  };

  for (int c = c0; c < c1; c += kStage3) {
    if (run_len > 0) {  // scalar: priority 3 while more than half the run is left, then 2, 1, 0 below 20 %, 5 %
      const int64_t rem = run_len - (done0 + (c - c0));
      if (20 * rem > 10 * run_len) __builtin_amdgcn_s_setprio(3);
      else if (20 * rem > 4 * run_len) __builtin_amdgcn_s_setprio(2);
      else if (20 * rem > run_len) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
    }
    const int buf = ((c - c0) / kStage3) & 1;
    // this stage's pieces are in LDS once every wave has waited for its own
    // and met the barrier, which also ends the reads of the buffer that the
    // next stage's pieces go to
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (c + kStage3 < c1) stage(c + kStage3, buf ^ 1);
    const uint4 *cb = lds.buf[buf];
    for (int cc = 0; cc < kStage3 && c + cc < c1; ++cc) {
      if (c + cc == rb0 >> 1)  // scalar branch
        chunk(c + cc, cb + cc * PC * 64, std::true_type{});
      else
        chunk(c + cc, cb + cc * PC * 64, std::false_type{});
    }
    if (((c - c0) / kStage3 + 1) % (kFlush3 / kStage3) == 0) flush();
  }
  flush();
  __syncthreads();  // the next segment may overwrite either buffer

  // lane holds O[row 4 (lane / 16) + i][n = lane % 16]; the weighted kernel sum
  // O[.][D] sits in lane (lane & 48) + D
  const int n = lane & 15;
  const int src = (lane & 48) + D;
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double s = tl[4 * r + i][src];
      const int64_t row = (int64_t)(rb0 + r) * 16 + 4 * (lane >> 4) + i;
      if (n < D) put(row, n, (double)xr[row * D + n] * s - tl[4 * r + i][lane]);
      else if (n == D) put(row, n, s);
    }
}

template <int D, int RB>
__global__ __launch_bounds__(kWaves3 * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_pair_bf3(
    const uint4 *__restrict__ K3, const uint4 *__restrict__ V3, const float *__restrict__ xr, SplitMap map, float *__restrict__ partial,
    int64_t part_stride_rows, const int *__restrict__ done) {
  __shared__ Bf3Lds<D> lds;
  if (done != nullptr && *done) return;  // the whole grid returns: no barrier is left waiting
  // workgroups go to the 8 XCDs round robin by linear id, and each XCD has its
  // own L2: with a multiple of 8 runs, XCD x takes the consecutive runs
  // x G / 8 .. (x + 1) G / 8 - 1, i.e. a band of row groups against all columns
  const int G = (int)gridDim.x;
  const int L = G % 8 == 0 ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const int64_t nch = map.nch;
  const int64_t u_beg = map.run_start(L), u_end = map.run_start(L + 1);
  // The workgroups of a compute unit share its SIMDs, which issue for the
  // oldest ready wave first: left alone, the first one placed runs ahead and
  // the last finishes with few waves to hide latency.  Each workgroup
  // therefore lowers its waves' priority as its run progresses, so that the
  // laggards are issued first and all finish together.
  // One segment per row group this run covers: chunks [c0, c1) of row group rg.
  for (int64_t u = u_beg; u < u_end;) {
    const int64_t rg = u / nch;
    const int c0 = (int)(u - rg * nch);
    const int c1 = (int)min(nch, u_end - rg * nch);
    const int slot = (int)(L - map.run_of(rg * nch));
    u = rg * nch + c1;
    float *out = partial + (int64_t)slot * part_stride_rows * (D + 1);
    bf3_segment<D, RB>(K3, V3, xr, (int)rg, c0, c1, [out](int64_t row, int n, double v) { out[row * (D + 1) + n] = (float)v; },
                       lds, rg * nch + c0 - u_beg, u_end - u_beg);
  }
}

// Batched form: a persistent grid walks the (ensemble, row group, column range)
// items, each a slot of partial sums in its rows.  The ranges are whole accumulation
// groups, their slots FP64 and rounded once when they are added, so that a row's sums
// are those of a whole ensemble but for the order in which FP64 adds the groups.
template <int D, int RB>
__global__ __launch_bounds__(kWaves3 * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_batch_pair_bf3(
    const int2 *__restrict__ items, int nitems, const EnsDesc *__restrict__ ens, const float *__restrict__ xc,
    const uint4 *__restrict__ K3, const uint4 *__restrict__ V3, float *__restrict__ partial) {
  using S = Bf3Shape<D>;
  __shared__ Bf3Lds<D> lds;
  // this workgroup's chunks over all its items, for the issue priority by
  // progress (see k_pair_bf3)
  int64_t total = 0;
  auto columns = [&](int2 item, int &c0, int &c1) {
    const EnsDesc &d = ens[item.x];
    const int nc = (int)((d.p.P + 31) / 32), ng = (nc + kFlush3 - 1) / kFlush3, k = item.y >> kItemTileBits;
    c0 = k * ng / d.splits * kFlush3;
    c1 = min(nc, (k + 1) * ng / d.splits * kFlush3);
  };
  int c0, c1;
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    columns(items[it], c0, c1);
    total += c1 - c0;
  }
  int64_t done = 0;
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int2 item = items[it];
    const EnsDesc &d = ens[item.x];
    const int64_t off = d.pad_off, slot = (item.y >> kItemTileBits) * d.p.Ppad;
    float *out = partial + d.part_off;
    columns(item, c0, c1);
    const uint4 *k3 = K3 + off / 16 * S::NQ * 64;
    const uint4 *v3 = V3 + off / 32 * S::NT * 64;
    const int rg = item.y & ((1 << kItemTileBits) - 1);
    if (d.splits == 1)
      bf3_segment<D, RB>(k3, v3, xc + off * D, rg, c0, c1,
                         [out](int64_t row, int n, double v) { out[row * 16 + n] = (float)v; }, lds, done, total);
    else
      bf3_segment<D, RB>(k3, v3, xc + off * D, rg, c0, c1,
                         [out, slot](int64_t row, int n, double v) {
                           reinterpret_cast<double *>(out)[(slot + row) * (D + 1) + n] = v;
                         },
                         lds, done, total);
    done += c1 - c0;
  }
}

// ---- FP16-split variant ----------------------------------------------------

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

constexpr float kF16Shift = 15.f;  // e = 2^(t + 15) <= 2^15 < FP16 max, t <= 0 up to rounding
constexpr int kFlushPairs = 4;     // chunk pairs (32 columns each) per FP32 group

// (a, b) -> hi = (a, b) rounded toward zero to FP16, lo = the remainders
// a - hi, b - hi (exact in FP32) rounded to nearest FP16.  `one` is 1.0 passed
// in at run time, so that the compiler keeps fma(-hi, one, a) and selects the
// mixed-precision FMA that reads the packed FP16 halves directly.
__device__ inline void split_pair(float a, float b, float one, half2v &hi, half2v &lo) {
  hi = __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(a, b));
  const float ra = __builtin_fmaf(-(float)hi.x, one, a);
  const float rb = __builtin_fmaf(-(float)hi.y, one, b);
  lo = half2v{(_Float16)ra, (_Float16)rb};
}

__device__ inline half8 as_half8(uint4 u) {
  half8 h;
  __builtin_memcpy(&h, &u, sizeof(h));
  return h;
}

// One wavefront: row blocks rb0 .. rb0 + RB - 1 against column chunk pairs
// [p0, p1).  VH[cp * 64 + lane] holds, for lane = n + 16 g, the FP16 highs of
// V_J[n] for the eight columns J = 32 cp + 16 s + 4 g + i (slot 4 s + i) and
// VH[lo_off + cp * 64 + lane] the lows.  out_scale multiplies every sum.
//
// t comes from FP32 MFMAs over the QB/KA operands (KQ = 0, KK slices), or
// (KQ > 0) from KQ FP16 MFMAs of 32 products each over the QH/KH operands:
// with c = sqrt(2 kappa) and y = c x split into FP16 halves, slot 3k + (0, 1, 2)
// holds (y_I,hi y_J,hi, y_I,hi y_J,lo, y_I,lo y_J,hi) for component k, and
// slots 3D, 3D + 1 hold 16 times the two halves of -kappa |x_J|^2 / 16.  The
// row norm -kappa |x_I|^2 (RN) enters exactly, in FP32, through the
// accumulator's initial value.
template <int KK, int KQ, int RB>
__device__ __forceinline__ void pair_rows_f16(const float *__restrict__ QB, const uint4 *__restrict__ QH,
                              const float *__restrict__ RN, int nrow_blocks, const float *__restrict__ KA,
                              const uint4 *__restrict__ KH, const uint4 *__restrict__ VH, int64_t lo_off, int p0,
                              int p1, const float *__restrict__ xc, int D, int exclude_self, double out_scale,
                              float one, float *__restrict__ out, int rb0) {
  constexpr bool kQ16 = KQ > 0;
  constexpr int NK = kQ16 ? 1 : KK;  // FP32 operand slices (unused with FP16 distances)
  constexpr int NQ = kQ16 ? KQ : 1;  // FP16 operand slices (unused with FP32 distances)
  if (rb0 >= nrow_blocks) return;
  const int lane = threadIdx.x & 63;
  const int diag_i = (lane & 15) - 4 * (lane >> 4);

  float qv[RB][NK];
  half8 qh[RB][NQ];
  float rinit[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const bool ok = rb0 + r < nrow_blocks;
    if constexpr (kQ16) {
#pragma unroll
      for (int m = 0; m < KQ; ++m)
        qh[r][m] = as_half8(ok ? QH[((int64_t)(rb0 + r) * KQ + m) * 64 + lane] : uint4{0, 0, 0, 0});
      rinit[r] = (ok ? RN[(int64_t)(rb0 + r) * 16 + (lane & 15)] : 0.f) + kF16Shift;
    } else {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) qv[r][kk] = ok ? QB[((int64_t)(rb0 + r) * KK + kk) * 64 + lane] : 0.f;
      rinit[r] = kF16Shift;
    }
  }

  double tot[RB][4];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) tot[r][i] = 0.0;

  // Operands of one chunk pair (32 columns): distance operands of its two
  // 16-column slices and the V highs and lows.  Two of them alternate so that
  // the loads of the next chunk pair overlap this one's arithmetic without
  // register copies; addresses are a wave-uniform base plus the lane offset.
  struct ColOps {
    float fa[2][NK];
    uint4 ha[2][NQ];
    uint4 h, l;
  };
  auto load_cols = [&](int cp, ColOps &o) {
    if constexpr (kQ16) {
      const uint4 *kb = KH + (int64_t)(2 * cp) * KQ * 64;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int m = 0; m < KQ; ++m) o.ha[s][m] = kb[(s * KQ + m) * 64 + lane];
    } else {
      const float *kb = KA + (int64_t)(2 * cp) * KK * 64;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) o.fa[s][kk] = kb[(s * KK + kk) * 64 + lane];
    }
    const uint4 *vb = VH + (int64_t)cp * 64;
    o.h = vb[lane];
    o.l = vb[lo_off + lane];
  };
  floatx4 acc[RB];
  auto compute = [&](int cp, const ColOps &o) {
    const half8 h8 = as_half8(o.h), l8 = as_half8(o.l);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      float e[8];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        floatx4 t = {rinit[r], rinit[r], rinit[r], rinit[r]};
        if constexpr (kQ16) {
#pragma unroll
          for (int m = 0; m < KQ; ++m)
            t = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(o.ha[s][m]), qh[r][m], t, 0, 0, 0);
        } else {
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) t = __builtin_amdgcn_mfma_f32_16x16x4f32(o.fa[s][kk], qv[r][kk], t, 0, 0, 0);
        }
        // no clamp: e exceeds 2^15 only by the rounding of t, and the RTZ
        // conversion of the split saturates at the FP16 maximum
#pragma unroll
        for (int i = 0; i < 4; ++i) e[4 * s + i] = __builtin_amdgcn_exp2f(t[i]);
      }
      if (exclude_self && (2 * cp == rb0 + r || 2 * cp + 1 == rb0 + r)) {  // scalar branch: diagonal tile
        // an empty volatile asm keeps this a branch: if-converted into
        // selects it would cost four VALU instructions on every tile
        asm volatile("" ::: "memory");
        const int sd = 2 * cp == rb0 + r ? 0 : 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) e[sd + i] = diag_i == i ? 0.f : e[sd + i];
      }
      half8 eh, el;
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        half2v h, l;
        split_pair(e[j], e[j + 1], one, h, l);
        eh[j] = h.x;
        eh[j + 1] = h.y;
        el[j] = l.x;
        el[j + 1] = l.y;
      }
      acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh, h8, acc[r], 0, 0, 0);
      acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh, l8, acc[r], 0, 0, 0);
      acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(el, h8, acc[r], 0, 0, 0);
    }
  };
  ColOps b0, b1;
  if (p0 < p1) load_cols(p0, b0);
  // groups of kFlushPairs (even) chunk pairs, so every group but the last
  // starts with its operands in b0; loads past the end re-read the last
  // chunk pair
  for (int cp = p0; cp < p1;) {
    const int g_end = min(p1, cp + kFlushPairs);
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (; cp < g_end; cp += 2) {
      load_cols(min(cp + 1, p1 - 1), b1);
      compute(cp, b0);
      if (cp + 1 < g_end) {
        load_cols(min(cp + 2, p1 - 1), b0);
        compute(cp + 1, b1);
      }
    }
    cp = g_end;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[r][i] += (double)acc[r][i];
  }

  const int n = lane & 15;
  const int src = (lane & 48) + D;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    if (rb0 + r >= nrow_blocks) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double s = __shfl(tot[r][i], src);
      const int64_t row = (int64_t)(rb0 + r) * 16 + 4 * (lane >> 4) + i;
      double v = 0.0;
      if (n < D) v = ((double)xc[row * D + n] * s - tot[r][i]) * out_scale;
      else if (n == D) v = s * out_scale;
      out[row * 16 + n] = (float)v;
    }
  }
}

// Operands of the FP16-split pair pass.
struct PairF16Ops {
  const float *QB, *KA;   // FP32 distance operands (FP32 distances)
  const uint4 *QH, *KH;   // FP16 distance operands (FP16 distances)
  const float *RN;        // row norms -kappa |x_I|^2 (FP16 distances)
  const uint4 *VH;        // V highs, then lows at lo_off
  int64_t lo_off;
};

template <int KK, int KQ, int RB>
__global__ __launch_bounds__(256, 4) void k_pair_mfma16(PairF16Ops ops, int nrow_blocks, int ncol_pairs,
                                                     int pairs_per_split, const float *__restrict__ xc, int D,
                                                     int exclude_self, const float *__restrict__ wscale, float one,
                                                     float *__restrict__ partial, int64_t part_stride_rows,
                                                     const int *__restrict__ done) {
  if (done != nullptr && *done) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb0 = ((int)blockIdx.x * 4 + wave) * RB;
  const int p0 = (int)blockIdx.y * pairs_per_split;
  const int p1 = min(ncol_pairs, p0 + pairs_per_split);
  const double scale = (wscale != nullptr ? (double)*wscale : 1.0) * 0x1p-15;
  pair_rows_f16<KK, KQ, RB>(ops.QB, ops.QH, ops.RN, nrow_blocks, ops.KA, ops.KH, ops.VH, ops.lo_off, p0, p1, xc, D,
                            exclude_self, scale, one, partial + (int64_t)blockIdx.y * part_stride_rows * 16, rb0);
}

// Batched ensembles: a persistent grid walks a static list of (ensemble, row
// tile) items, sorted by decreasing cost, each over all of its ensemble's
// columns (one split).  Operands of ensemble e start at padded particle
// ens[e].pad_off of the concatenated arrays.
template <int KK, int RB>
__global__ __launch_bounds__(256) void k_batch_pair(const int2 *__restrict__ items, int nitems,
                                                    const EnsDesc *__restrict__ ens, const float *__restrict__ QB,
                                                    const float *__restrict__ KA, const float4 *__restrict__ VB,
                                                    const float *__restrict__ xc, int D, float *__restrict__ partial) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int2 item = items[it];
    const int64_t off = ens[item.x].pad_off;
    const int64_t P = ens[item.x].p.P;
    const int nrb = (int)(ens[item.x].p.Ppad / 16);
    const int ncc = (int)((P + 15) / 16);
    const int rb0 = (item.y * 4 + wave) * RB;
    pair_rows<KK, RB>(QB + off * KK * 4, nrb, KA + off * KK * 4, VB + off * 4, 0, ncc, xc + off * D, D, 1,
                      partial + off * 16, rb0);
  }
}

// VALU variant.  D is the configuration dimension; the augmented length is D + 2.
// FP32 accumulation over 64 columns, then FP64 running sums (see above).
template <int D>
__global__ __launch_bounds__(256) void k_pair_valu(const float *__restrict__ QB, int64_t nrows,
                                                   const float *__restrict__ KA, const float *__restrict__ VB,
                                                   int64_t ncol_chunks, int64_t chunks_per_split, int exclude_self,
                                                   float *__restrict__ partial, int64_t part_stride_rows,
                                                   const int *__restrict__ done) {
  constexpr int KA_LEN = D + 2;
  constexpr int KK = (D + 2 + 3) / 4;
  constexpr int NV = D + 1;
  constexpr int RT = 2;
  __shared__ float sK[KA_LEN][256];
  __shared__ float sV[NV][256];
  if (done != nullptr && *done) return;

  const int tid = threadIdx.x;
  int64_t rows[RT];
  float q[RT][KA_LEN];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    rows[r] = (int64_t)blockIdx.x * (256 * RT) + r * 256 + tid;
    const int64_t I = rows[r] < nrows ? rows[r] : 0;
#pragma unroll
    for (int k = 0; k < KA_LEN; ++k)
      q[r][k] = QB[((I >> 4) * KK + (k >> 2)) * 64 + (I & 15) + 16 * (k & 3)];
  }
  double tot[RT][NV];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int n = 0; n < NV; ++n) tot[r][n] = 0.0;

  const int64_t c0 = (int64_t)blockIdx.y * chunks_per_split;
  const int64_t c1 = min(ncol_chunks, c0 + chunks_per_split);
  for (int64_t tile = c0; tile < c1; tile += 16) {
    const int64_t c = tile + (tid >> 4);
    const int jj = tid & 15;
    if (c < c1) {
#pragma unroll
      for (int k = 0; k < KA_LEN; ++k) sK[k][tid] = KA[(c * KK + (k >> 2)) * 64 + jj + 16 * (k & 3)];
#pragma unroll
      for (int n = 0; n < NV; ++n) sV[n][tid] = VB[(c * 64 + (jj >> 2) * 16 + n) * 4 + (jj & 3)];
    } else {
#pragma unroll
      for (int k = 0; k < KA_LEN; ++k) sK[k][tid] = 0.f;
#pragma unroll
      for (int n = 0; n < NV; ++n) sV[n][tid] = 0.f;
    }
    __syncthreads();
    for (int j0 = 0; j0 < 256; j0 += 64) {
      float acc[RT][NV];
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int n = 0; n < NV; ++n) acc[r][n] = 0.f;
      for (int j = j0; j < j0 + 64; ++j) {
        const int64_t col = tile * 16 + j;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          float t = 0.f;
#pragma unroll
          for (int k = 0; k < KA_LEN; ++k) t = fmaf(q[r][k], sK[k][j], t);
          float e = __builtin_amdgcn_exp2f(fminf(t, 0.f));
          if (exclude_self && col == rows[r]) e = 0.f;
#pragma unroll
          for (int n = 0; n < NV; ++n) acc[r][n] = fmaf(e, sV[n][j], acc[r][n]);
        }
      }
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int n = 0; n < NV; ++n) tot[r][n] += (double)acc[r][n];
    }
    __syncthreads();
  }
  float *out = partial + (int64_t)blockIdx.y * part_stride_rows * 16;
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    if (rows[r] >= nrows) continue;
    const double s = tot[r][D];
#pragma unroll
    for (int n = 0; n < D; ++n) out[rows[r] * 16 + n] = (float)((double)q[r][n] * s - tot[r][n]);
    out[rows[r] * 16 + D] = (float)s;
  }
}

// Batched FP16-split variant over the same work list.  Pass A's V holds the
// weights 1/P_e over their maximum 1/P_e, so its sums are scaled by 1/P_e.
template <int KK, int KQ, int RB>
__global__ __launch_bounds__(256) void k_batch_pair16(const int2 *__restrict__ items, int nitems,
                                                      const EnsDesc *__restrict__ ens, PairF16Ops ops, int pass_a,
                                                      const float *__restrict__ xc, int D, float one,
                                                      float *__restrict__ partial) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int2 item = items[it];
    const EnsDesc &d = ens[item.x];
    const int64_t off = d.pad_off;
    const int nrb = (int)(d.p.Ppad / 16);
    const int ncp = (int)((d.p.P + 31) / 32);
    const int rb0 = (item.y * 4 + wave) * RB;
    const double scale = (pass_a ? (double)d.p.uniform_w : 1.0) * 0x1p-15;
    const int64_t qoff = (off / 16) * KQ * 64;  // uint4 units of the distance operands
    pair_rows_f16<KK, KQ, RB>(ops.QB + off * KK * 4, ops.QH + qoff, ops.RN + off, nrb, ops.KA + off * KK * 4,
                              ops.KH + qoff, ops.VH + off * 4, d.p.Ppad * 2, 0, ncp, xc + off * D, D, 1, scale,
                              one, partial + off * 16, rb0);
  }
}

template <int KK, int KQ>
static void launch_batch16_k(int rb, int grid, const int2 *items, int nitems, const EnsDesc *ens,
                             const PairF16Ops &ops, int pass_a, const float *xc, int D, float *partial,
                             hipStream_t s) {
  switch (rb) {
    case 1: k_batch_pair16<KK, KQ, 1><<<grid, 256, 0, s>>>(items, nitems, ens, ops, pass_a, xc, D, 1.f, partial); break;
    case 2: k_batch_pair16<KK, KQ, 2><<<grid, 256, 0, s>>>(items, nitems, ens, ops, pass_a, xc, D, 1.f, partial); break;
    default: k_batch_pair16<KK, KQ, 4><<<grid, 256, 0, s>>>(items, nitems, ens, ops, pass_a, xc, D, 1.f, partial); break;
  }
}

template <int KK>
static void launch_batch_kk(int rb, int grid, const int2 *items, int nitems, const EnsDesc *ens, const float *QB,
                            const float *KA, const float *VB, const float *xc, int D, float *partial, hipStream_t s) {
  const float4 *vb = reinterpret_cast<const float4 *>(VB);
  switch (rb) {
    case 1: k_batch_pair<KK, 1><<<grid, 256, 0, s>>>(items, nitems, ens, QB, KA, vb, xc, D, partial); break;
    case 2: k_batch_pair<KK, 2><<<grid, 256, 0, s>>>(items, nitems, ens, QB, KA, vb, xc, D, partial); break;
    default: k_batch_pair<KK, 4><<<grid, 256, 0, s>>>(items, nitems, ens, QB, KA, vb, xc, D, partial); break;
  }
}

template <int D>
static void launch_batch_bf3_d(int rb, int grid, const int2 *items, int nitems, const EnsDesc *ens, const float *xc,
                               const void *K3, const float *V3, float *partial, hipStream_t s) {
  const uint4 *k3 = reinterpret_cast<const uint4 *>(K3), *v3 = reinterpret_cast<const uint4 *>(V3);
  if (bf3_rb(D, rb) == 1)
    k_batch_pair_bf3<D, 1><<<grid, kWaves3 * 64, 0, s>>>(items, nitems, ens, xc, k3, v3, partial);
  else
    k_batch_pair_bf3<D, bf3_rb(D, 2)><<<grid, kWaves3 * 64, 0, s>>>(items, nitems, ens, xc, k3, v3, partial);
}

void launch_batch_pair(int impl, int rb, int grid, int KK, int D, const int2 *items, int nitems, const EnsDesc *ens,
                       const float *QB, const float *KA, const float *VB, const F16Operands &f16, bool pass_a,
                       const float *xc, float *partial, hipStream_t s) {
  if (impl == VDS_PAIR_MFMA32) {
    switch (D) {
      case 3: launch_batch_bf3_d<3>(rb, grid, items, nitems, ens, xc, f16.QH, VB, partial, s); break;
      case 6: launch_batch_bf3_d<6>(rb, grid, items, nitems, ens, xc, f16.QH, VB, partial, s); break;
      case 9: launch_batch_bf3_d<9>(rb, grid, items, nitems, ens, xc, f16.QH, VB, partial, s); break;
      case 12: launch_batch_bf3_d<12>(rb, grid, items, nitems, ens, xc, f16.QH, VB, partial, s); break;
      default: launch_batch_bf3_d<15>(rb, grid, items, nitems, ens, xc, f16.QH, VB, partial, s); break;
    }
    return;
  }
  if (impl == VDS_PAIR_MFMA_F16X2 || impl == VDS_PAIR_MFMA_F16X2_ALL) {
    const PairF16Ops ops{QB, KA, reinterpret_cast<const uint4 *>(f16.QH), reinterpret_cast<const uint4 *>(f16.KH),
                         f16.RN, reinterpret_cast<const uint4 *>(VB), 0};
    const int pa = pass_a ? 1 : 0;
    if (impl == VDS_PAIR_MFMA_F16X2_ALL) {
      if (f16_slices(D) == 1) launch_batch16_k<0, 1>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s);
      else launch_batch16_k<0, 2>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s);
    } else {
      switch (KK) {
        case 2: launch_batch16_k<2, 0>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s); break;
        case 3: launch_batch16_k<3, 0>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s); break;
        case 4: launch_batch16_k<4, 0>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s); break;
        default: launch_batch16_k<5, 0>(rb, grid, items, nitems, ens, ops, pa, xc, D, partial, s); break;
      }
    }
    return;
  }
  switch (KK) {
    case 2: launch_batch_kk<2>(rb, grid, items, nitems, ens, QB, KA, VB, xc, D, partial, s); break;
    case 3: launch_batch_kk<3>(rb, grid, items, nitems, ens, QB, KA, VB, xc, D, partial, s); break;
    case 4: launch_batch_kk<4>(rb, grid, items, nitems, ens, QB, KA, VB, xc, D, partial, s); break;
    default: launch_batch_kk<5>(rb, grid, items, nitems, ens, QB, KA, VB, xc, D, partial, s); break;
  }
}

int pair_tile_rows(int impl, int rb, int D) {
  return impl == VDS_PAIR_MFMA32 ? kWaves3 * bf3_rb(D, rb) * 16 : 4 * rb * 16;
}

bool pair_shape_ok(const vds_tuning &t, int D) {
  if (D < 3 || D > kMaxD || D % 3 != 0) return false;
  if (t.col_splits < 1 || t.col_splits > kMaxSplits) return false;
  if (t.impl == VDS_PAIR_MFMA || t.impl == VDS_PAIR_MFMA_F16X2 || t.impl == VDS_PAIR_MFMA_F16X2_ALL)
    return t.rows_per_wave == 1 || t.rows_per_wave == 2 || t.rows_per_wave == 4;
  if (t.impl == VDS_PAIR_MFMA32) return t.rows_per_wave == 1 || t.rows_per_wave == 2;
  return t.impl == VDS_PAIR_VALU;
}

template <int KK>
static void launch_mfma_kk(int rb, dim3 grid, const float *QB, int nrb, const float *KA, const float *VB,
                           int ncc, int cps, const float *xc, int D, int ex, float *partial, int64_t stride,
                           const int *done, hipStream_t s) {
  const float4 *vb = reinterpret_cast<const float4 *>(VB);
  switch (rb) {
    case 1: k_pair_mfma<KK, 1><<<grid, 256, 0, s>>>(QB, nrb, KA, vb, ncc, cps, xc, D, ex, partial, stride, done); break;
    case 2: k_pair_mfma<KK, 2><<<grid, 256, 0, s>>>(QB, nrb, KA, vb, ncc, cps, xc, D, ex, partial, stride, done); break;
    default: k_pair_mfma<KK, 4><<<grid, 256, 0, s>>>(QB, nrb, KA, vb, ncc, cps, xc, D, ex, partial, stride, done); break;
  }
}

template <int KK, int KQ>
static void launch_mfma16_k(int rb, dim3 grid, const PairF16Ops &ops, int nrb, int ncp, int pps, const float *xc,
                            int D, int ex, const float *wscale, float *partial, int64_t stride, const int *done,
                            hipStream_t s) {
  switch (rb) {
    case 1: k_pair_mfma16<KK, KQ, 1><<<grid, 256, 0, s>>>(ops, nrb, ncp, pps, xc, D, ex, wscale, 1.f, partial, stride, done); break;
    case 2: k_pair_mfma16<KK, KQ, 2><<<grid, 256, 0, s>>>(ops, nrb, ncp, pps, xc, D, ex, wscale, 1.f, partial, stride, done); break;
    default: k_pair_mfma16<KK, KQ, 4><<<grid, 256, 0, s>>>(ops, nrb, ncp, pps, xc, D, ex, wscale, 1.f, partial, stride, done); break;
  }
}

template <int D>
static void launch_bf3_d(int rb, const void *K3, const float *V3, const float *xr, const SplitMap &map,
                         float *partial, int64_t stride, const int *done, hipStream_t s) {
  const uint4 *k3 = reinterpret_cast<const uint4 *>(K3), *v3 = reinterpret_cast<const uint4 *>(V3);
  const dim3 grid((unsigned)map.G), block(kWaves3 * 64);
  if (bf3_rb(D, rb) == 1)
    k_pair_bf3<D, 1><<<grid, block, 0, s>>>(k3, v3, xr, map, partial, stride, done);
  else
    k_pair_bf3<D, bf3_rb(D, 2)><<<grid, block, 0, s>>>(k3, v3, xr, map, partial, stride, done);
}

// Compute units of the current device (256 on MI355X), looked up once per
// device (host threads may race to fill a slot; they store the same value).
int device_cu_count() {
  constexpr int kDevs = 64;
  static std::atomic<int> cache[kDevs];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return 256;
  int n = cache[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    cache[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

SplitMap pair_split_map(const vds_tuning &t, int D, int64_t nrow_blocks, int64_t ncol_chunks) {
  SplitMap m;
  if (t.impl != VDS_PAIR_MFMA32) {
    m.splits = t.col_splits;
    return m;
  }
  m.width = D + 1;  // the compact layout
  // kWaves3 waves of RB 16-row blocks per row group (whole groups: the rows are
  // a multiple of 256); columns in chunks of 32
  const int rb = nrow_blocks * 16 <= kOneBlockRows3 ? 1 : bf3_rb(D, t.rows_per_wave);
  m.group_shift = pair_group_shift(rb);  // kWaves3 rb 16 rows
  static_assert(kWaves3 * 16 == 1 << pair_group_shift(1), "row groups of 128 or 256 rows");
  m.n_rg = (nrow_blocks + kWaves3 * rb - 1) / (kWaves3 * rb);
  m.nch = (ncol_chunks + 1) / 2;
  m.splits = kMaxSplits;
  // col_splits / 2 workgroups of eight waves per compute unit; runs of at least
  // qmin units, so that at most kMaxSplits runs meet in one row group
  const int64_t U = m.units();
  m.inv_units = 1.0 / (double)U;
  const int64_t qmin = (m.nch + kMaxSplits - 2) / (kMaxSplits - 1);
  int64_t G = std::min<int64_t>(std::max<int64_t>(1, (int64_t)t.col_splits * device_cu_count() / 2), U / qmin);
  if (G >= 8) G -= G % 8;
  m.G = (int)std::max<int64_t>(G, 1);
  return m;
}

void launch_pair_pass(const vds_tuning &t, int KK, int D, const float *QB, int64_t nrow_blocks, const float *KA,
                      const float *VB, int64_t ncol_chunks, int64_t ncol_pad, const float *xc, bool exclude_self,
                      const float *wscale, const F16Operands &f16, float *partial, int64_t part_stride_rows,
                      const int *done, hipStream_t s) {
  const int ex = exclude_self ? 1 : 0;
  const int splits = t.col_splits;
  const int64_t cps = (ncol_chunks + splits - 1) / splits;
  if (t.impl == VDS_PAIR_MFMA32) {
    // whole row groups (nrow_blocks counts 16-row blocks of a multiple of 256 rows); columns
    // in chunks of 32, the last inside the padding (ncol_pad is a multiple of 256 columns),
    // whose weights are zero
    const SplitMap map = pair_split_map(t, D, nrow_blocks, ncol_chunks);
    const int rb = (1 << map.group_shift) / (kWaves3 * 16);
    switch (D) {
      case 3: launch_bf3_d<3>(rb, f16.QH, VB, xc, map, partial, part_stride_rows, done, s); break;
      case 6: launch_bf3_d<6>(rb, f16.QH, VB, xc, map, partial, part_stride_rows, done, s); break;
      case 9: launch_bf3_d<9>(rb, f16.QH, VB, xc, map, partial, part_stride_rows, done, s); break;
      case 12: launch_bf3_d<12>(rb, f16.QH, VB, xc, map, partial, part_stride_rows, done, s); break;
      default: launch_bf3_d<15>(rb, f16.QH, VB, xc, map, partial, part_stride_rows, done, s); break;
    }
    return;
  }
  if (t.impl == VDS_PAIR_MFMA_F16X2 || t.impl == VDS_PAIR_MFMA_F16X2_ALL) {
    // chunk pairs; the second chunk of the last pair lies inside the padding
    // (ncol_pad is a multiple of 32 columns), whose V is zero
    const int64_t ncp = (ncol_chunks + 1) / 2;
    const int64_t pps = (ncp + splits - 1) / splits;
    PairF16Ops ops{QB, KA, reinterpret_cast<const uint4 *>(f16.QH), reinterpret_cast<const uint4 *>(f16.KH), f16.RN,
                   reinterpret_cast<const uint4 *>(VB), ncol_pad / 32 * 64};  // lows follow the highs
    const int rb = t.rows_per_wave;
    dim3 grid((unsigned)((nrow_blocks + 4 * rb - 1) / (4 * rb)), (unsigned)splits);
    const int nrb = (int)nrow_blocks, np = (int)ncp, pp = (int)pps;
    if (t.impl == VDS_PAIR_MFMA_F16X2_ALL) {
      if (f16_slices(D) == 1)
        launch_mfma16_k<0, 1>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s);
      else
        launch_mfma16_k<0, 2>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s);
    } else {
      switch (KK) {
        case 2: launch_mfma16_k<2, 0>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s); break;
        case 3: launch_mfma16_k<3, 0>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s); break;
        case 4: launch_mfma16_k<4, 0>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s); break;
        default: launch_mfma16_k<5, 0>(rb, grid, ops, nrb, np, pp, xc, D, ex, wscale, partial, part_stride_rows, done, s); break;
      }
    }
  } else if (t.impl == VDS_PAIR_MFMA) {
    const int rb = t.rows_per_wave;
    dim3 grid((unsigned)((nrow_blocks + 4 * rb - 1) / (4 * rb)), (unsigned)splits);
    switch (KK) {
      case 2: launch_mfma_kk<2>(rb, grid, QB, (int)nrow_blocks, KA, VB, (int)ncol_chunks, (int)cps, xc, D, ex, partial, part_stride_rows, done, s); break;
      case 3: launch_mfma_kk<3>(rb, grid, QB, (int)nrow_blocks, KA, VB, (int)ncol_chunks, (int)cps, xc, D, ex, partial, part_stride_rows, done, s); break;
      case 4: launch_mfma_kk<4>(rb, grid, QB, (int)nrow_blocks, KA, VB, (int)ncol_chunks, (int)cps, xc, D, ex, partial, part_stride_rows, done, s); break;
      default: launch_mfma_kk<5>(rb, grid, QB, (int)nrow_blocks, KA, VB, (int)ncol_chunks, (int)cps, xc, D, ex, partial, part_stride_rows, done, s); break;
    }
  } else {
    const int64_t nrows = nrow_blocks * 16;
    dim3 grid((unsigned)((nrows + 511) / 512), (unsigned)splits);
    switch (D) {
      case 3: k_pair_valu<3><<<grid, 256, 0, s>>>(QB, nrows, KA, VB, ncol_chunks, cps, ex, partial, part_stride_rows, done); break;
      case 6: k_pair_valu<6><<<grid, 256, 0, s>>>(QB, nrows, KA, VB, ncol_chunks, cps, ex, partial, part_stride_rows, done); break;
      case 9: k_pair_valu<9><<<grid, 256, 0, s>>>(QB, nrows, KA, VB, ncol_chunks, cps, ex, partial, part_stride_rows, done); break;
      case 12: k_pair_valu<12><<<grid, 256, 0, s>>>(QB, nrows, KA, VB, ncol_chunks, cps, ex, partial, part_stride_rows, done); break;
      default: k_pair_valu<15><<<grid, 256, 0, s>>>(QB, nrows, KA, VB, ncol_chunks, cps, ex, partial, part_stride_rows, done); break;
    }
  }
}

}  // namespace vds
