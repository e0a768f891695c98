// Galerkin reduced model of the particle scheme (C ABI of include/vds_pod.h).
//
// Per freeze: reconstruct q~ = U p, run the two kernel passes at q~ for
// S = Z w and T = Z (w/S), form Y = Z U_a (the default; [w U_a | (w/S) U_a] in the
// other forms) with the kernel matrix generated tile by tile on MFMA (never
// stored), then contract with the mode blocks into X^B1 and X^B2.  Between freezes a single workgroup takes the
// explicit Euler steps of the reduced equation.  Midpoint freezes add a second
// freeze per window, at the state half a window on.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include <rocblas/rocblas.h>

#include "bf3.h"
#include "vds_ctx.h"
#include "vds_linalg.h"
#include "vds_pod.h"

using namespace vds;

namespace {

constexpr int kMaxR = 1024;
constexpr int kNBG = 8;       // 16-column output blocks per workgroup of the kernel-GEMM
constexpr int kKgFlush = 8;   // chunks per FP32 accumulation group
constexpr int kKgWaves = 8;   // waves of a workgroup of the default kernel-GEMM
constexpr int kKgRows = 256;  // its rows: two 16-row blocks per wave
// floats of one (row group, column group) output tile with NB column tiles of 16
constexpr int kgemm_tile(int NB) { return kKgRows * 16 * NB; }

// The balanced grid of the default kernel-GEMM: the (column group, row group)
// items, column-group major, times the nch 32-column chunks of Z, cut into G
// equal runs, one workgroup each.
struct KgMap {
  int NB;       // column tiles of 16 per item: 4, 8 or 12
  int NCG, n_rg, nch, G;
  double inv_G, inv_units;  // a 64-bit division is some hundred instructions on the GPU
  __host__ __device__ int64_t items() const { return (int64_t)NCG * n_rg; }
  __host__ __device__ int64_t units() const { return items() * nch; }
  // floor(a / b) for a below 2^53, with inv = 1 / b
  __host__ __device__ static int64_t quotient(int64_t a, int64_t b, double inv) {
    int64_t q = (int64_t)((double)a * inv);
    const int64_t r = a - q * b;
    if (r < 0) --q;
    else if (r >= b) ++q;
    return q;
  }
  // first unit of run L, and the first run that starts after unit u
  __host__ __device__ int64_t run_start(int64_t L) const { return quotient(L * units(), G, inv_G); }
  __host__ __device__ int64_t run_after(int64_t u) const { return quotient((u + 1) * G - 1, units(), inv_units) + 1; }
};

// One workgroup per compute unit (its eight waves take a SIMD's registers two
// at a time), each with at least two chunks.  Column tiles per item by the
// matrix instructions a chunk costs: 12 per tile, and 16 for its part of Z; the
// padding of the last group counts (R = 180: 3 x 12 tiles for 34; R = 40: 8).
KgMap kgemm_map(int64_t P, int ncols) {
  KgMap m{};
  const int tiles = (ncols + 15) / 16;
  double best = 0.0;
  for (int nb : {12, 8, 4}) {
    const int g = (tiles + nb - 1) / nb;
    const double cost = (double)g * (12.0 * nb + 16.0);
    if (m.NB == 0 || cost < best) {
      m.NB = nb;
      m.NCG = g;
      best = cost;
    }
  }
  m.n_rg = (int)(round_up(P, kRowAlign) / kKgRows);
  m.nch = (int)((P + 31) / 32);
  int64_t G = std::min<int64_t>(device_cu_count(), m.units() / 2);
  if (G >= 8) G -= G % 8;
  m.G = (int)std::max<int64_t>(G, 1);
  m.inv_G = 1.0 / (double)m.G;
  m.inv_units = 1.0 / (double)m.units();
  return m;
}

// Row length of Y of the default kernel-GEMM.
int64_t rom_ldy3(int R) { return (3 * (int64_t)R + 15) / 16 * 16; }

struct RomLayout {
  size_t Ude, Mbig, XH, I1, XB1, XB2, XB, Bsw, Y, qt, T, invS, part, red, psave, pprev, total;
  int NB16;
  int64_t ldy, part_floats;
  KgMap kg;     // grid of the default kernel-GEMM (its continuation slots are sized for its runs)
};

RomLayout rom_layout(const vds_problem &p, int R) {
  RomLayout L{};
  const int64_t P = p.P, Ppad = round_up(P, kRowAlign);
  const int ncols = 2 * 3 * R;
  L.NB16 = (ncols + 15) / 16;
  L.ldy = (int64_t)L.NB16 * 16;
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off += (b + 255) / 256 * 256;
    return o;
  };
  L.Ude = take(sizeof(float) * 3 * (size_t)R * P);
  L.Mbig = take(sizeof(float) * 9 * (size_t)R * R);
  L.XH = take(sizeof(float) * R * R);
  L.I1 = take(sizeof(float) * R * R);
  L.XB1 = take(sizeof(float) * R * R);
  L.XB2 = take(sizeof(float) * R * R);
  L.XB = take(sizeof(float) * R * R);
  // B of the kernel-GEMM: the 16-column swizzled layout of 6 R columns, or the
  // BF16 thirds of 3 R columns (6 bytes each)
  L.kg = kgemm_map(P, 3 * R);
  L.Bsw = take(std::max(sizeof(float) * (size_t)Ppad * L.ldy,
                        sizeof(uint16_t) * 3 * (size_t)Ppad * 16 * L.kg.NB * L.kg.NCG));
  L.Y = take(sizeof(float) * (size_t)Ppad * L.ldy);  // Y of 6 R columns, or of 3 R
  L.qt = take(sizeof(float) * (size_t)p.nb * P * 3);
  L.T = take(sizeof(float) * Ppad);
  L.invS = take(sizeof(float) * Ppad);
  const int64_t m = 3 * P;
  // (the GEMMs' split partials, or the kernel-GEMM's continuation tiles: one per run)
  const size_t part = std::max({sizeof(float) * (size_t)gemm_splits(3 * R, 3 * R, P) * 9 * R * R,
                                sizeof(float) * (size_t)gemm_splits(R, R, P, 3) * R * R,
                                sizeof(float) * (size_t)m * p.nb,
                                sizeof(float) * (size_t)L.kg.G * kgemm_tile(L.kg.NB)});
  L.part = take(part);
  L.part_floats = (int64_t)(part / sizeof(float));
  L.red = take(sizeof(double) * 16);
  L.psave = take(sizeof(float) * (size_t)p.nb * R);
  L.pprev = take(sizeof(float) * (size_t)p.nb * R);
  L.total = off;
  return L;
}

// Splits of the two R x R x 3 P products of a reduced operator build: two
// workgroups per compute unit (one leaves each waiting for its own loads: 77 and
// 62 us at R = 180, P = 20000, two took 51 and 44), at least two rounds each, as many
// as the partial-sum buffer holds for both.
int rom_splits(const RomLayout &L, int R, int64_t P) {
  const int64_t t = (R + kGemmTile - 1) / kGemmTile, rounds = (P + kGemmSlab - 1) / kGemmSlab * 3;
  int64_t s = std::min<int64_t>({512 / (t * t), rounds / 2, L.part_floats / (2 * (int64_t)R * R)});
  if (s >= 8) s -= s % 8;
  return (int)std::max<int64_t>(s, 1);
}

// Ude[a][s][I] = U[s m + 3 I + a]: the mode blocks U_a, K-contiguous over I.
__global__ void k_deinterleave(const float *__restrict__ U, int64_t P, int R, float *__restrict__ Ude) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= 3 * (int64_t)R * P) return;
  const int64_t I = t % P;
  const int64_t rest = t / P;
  const int s = (int)(rest % R), a = (int)(rest / R);
  Ude[t] = U[(int64_t)s * 3 * P + 3 * I + a];
}

// X^H = sum_ab G_ab M_ab and I1 = sum_a M_aa from Mbig[(a R + s)][(b R + t)].
__global__ void k_hydro(const float *__restrict__ Mbig, int R, EvalParams p, float *__restrict__ XH,
                        float *__restrict__ I1) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)R * R) return;
  const int s = (int)(t / R), u = (int)(t % R);
  const int64_t ld = 3 * (int64_t)R;
  float h = 0.f, id = 0.f;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      const float m = Mbig[(a * (int64_t)R + s) * ld + b * R + u];
      h += p.G[3 * a + b] * m;
      if (a == b) id += m;
    }
  XH[t] = h;
  I1[t] = id;
}

// T_I = w_I / S_I + sum_{K != I} (w_K / S_K) e_IK from the pass-B partials, and 1/S.
__global__ void k_rom_scalars(const float *__restrict__ part, SplitMap splits, int64_t Ppad, int64_t P, int D,
                              const float *__restrict__ S, const float *__restrict__ wv, float *__restrict__ T,
                              float *__restrict__ invS) {
  const int64_t I = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (I >= Ppad) return;
  if (I >= P) {
    T[I] = 0.f;
    invS[I] = 0.f;
    return;
  }
  const double o = ordered_sum<double>(part + I * splits.width + D, splits.count(I), Ppad * splits.width);
  const double Si = (double)S[I];
  T[I] = (float)(o + (double)wv[I] / Si);
  invS[I] = (float)(1.0 / Si);
}

// Kernel-GEMM right operand B[J][col], col = h dR + a R + t:
// (h = 0: w_J, h = 1: w_J / S_J) * U_a[t][J], in the swizzled MFMA layout
// Bsw[((c NB16 + nbk) 64 + lane) 4 + i] = B[16 c + 4 (lane / 16) + i][16 nbk + lane % 16].
__global__ void k_rom_bsw(const float *__restrict__ Ude, const float *__restrict__ wv, const float *__restrict__ invS,
                          int64_t P, int64_t Ppad, int R, int NB16, float *__restrict__ Bsw) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t ldy = (int64_t)NB16 * 16;
  if (t >= Ppad * ldy) return;
  const int64_t J = t / ldy;
  const int col = (int)(t % ldy);
  const int dR = 3 * R;
  float v = 0.f;
  if (J < P && col < 2 * dR) {
    const int h = col / dR, rem = col % dR, a = rem / R, tt = rem % R;
    const float wgt = h == 0 ? wv[J] : wv[J] * invS[J];
    v = wgt * Ude[((int64_t)a * R + tt) * P + J];
  }
  const int64_t c = J >> 4;
  const int jj = (int)(J & 15);
  const int lane = 16 * (jj >> 2) + (col & 15);
  const int nbk = col >> 4;
  Bsw[((c * NB16 + nbk) * 64 + lane) * 4 + (jj & 3)] = v;
}

// Y[I][col] = sum_J Z_IJ B[J][col], Z_IJ = exp(-|x_I - x_J|^2 / 2h^2) (Z_II = 1),
// from the Q/K operands of the pair kernels.  One 16-row block per wavefront,
// kNBG 16-column output blocks per workgroup; FP32 accumulation flushed to FP64.
template <int KK>
__global__ __launch_bounds__(256) void k_kernel_gemm(const float *__restrict__ QB, const float *__restrict__ KA,
                                                     int nrow_blocks, int ncol_chunks,
                                                     const float4 *__restrict__ Bsw, int NB16,
                                                     float *__restrict__ Y, int64_t ldy) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = (int)blockIdx.x * 4 + wave;
  if (rb >= nrow_blocks) return;
  const int nb0 = (int)blockIdx.y * kNBG;
  const int nbn = min(kNBG, NB16 - nb0);
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  float qv[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qv[kk] = QB[((int64_t)rb * KK + kk) * 64 + lane];
  double tot[kNBG][4];
#pragma unroll
  for (int g = 0; g < kNBG; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) tot[g][i] = 0.0;

  for (int c = 0; c < ncol_chunks;) {
    const int cg_end = min(ncol_chunks, c + kKgFlush);
    floatx4 acc[kNBG];
#pragma unroll
    for (int g = 0; g < kNBG; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (; c < cg_end; ++c) {
      floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        t = __builtin_amdgcn_mfma_f32_16x16x4f32(KA[((int64_t)c * KK + kk) * 64 + lane], qv[kk], t, 0, 0, 0);
      float e0 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[0]), 0.f, 1.f);
      float e1 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[1]), 0.f, 1.f);
      float e2 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[2]), 0.f, 1.f);
      float e3 = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(t[3]), 0.f, 1.f);
      if (c == rb) {  // the self pair has Z_II = K_h(0) = 1 exactly
        e0 = diag_i == 0 ? 1.f : e0;
        e1 = diag_i == 1 ? 1.f : e1;
        e2 = diag_i == 2 ? 1.f : e2;
        e3 = diag_i == 3 ? 1.f : e3;
      }
      const float4 *bp = Bsw + ((int64_t)c * NB16 + nb0) * 64 + lane;
#pragma unroll
      for (int g = 0; g < kNBG; ++g) {
        if (g < nbn) {
          const float4 b = bp[(int64_t)g * 64];
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(e0, b.x, acc[g], 0, 0, 0);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(e1, b.y, acc[g], 0, 0, 0);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(e2, b.z, acc[g], 0, 0, 0);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(e3, b.w, acc[g], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < kNBG; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[g][i] += (double)acc[g][i];
  }
#pragma unroll
  for (int g = 0; g < kNBG; ++g) {
    if (g >= nbn) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = (int64_t)rb * 16 + 4 * (lane >> 4) + i;
      Y[row * ldy + (int64_t)(nb0 + g) * 16 + (lane & 15)] = (float)tot[g][i];
    }
  }
}

// ---- FP32 kernel-GEMM by three BF16 parts (the operands of VDS_PAIR_MFMA32) --
//
// Y[I][col] = sum_J Z_IJ U_a[t][J], col = a R + t < 3 R.  With the reduced
// model's uniform weights and Z symmetric, W = sum_a U_a^T diag(1/S) Y_a holds
// both operators' kernel terms: X^B1 needs w W, X^B2 needs
// w sum_a U_a^T Z diag(1/S) U_a = w W^T.  So B is the basis alone: half the
// columns of the weighted pair (w U_a, (w/S) U_a), and laid out once.
//
// A workgroup of eight waves owns 256 rows (32 per wave) and NB column tiles
// of 16.  Per 32-column chunk of Z each wave forms its 32 x 32 piece as the
// pair kernel does (pair_kernels.hip; Z_II = 1 set exactly), cut into three
// BF16 parts that are A operands as they stand, and multiplies them with the
// chunk's B parts from LDS: the six products hh, hm, mh, mm, hl, lh (the others
// are below 2^-24 of the product), FP32 accumulation over all of Z.  The piece
// of the next chunk is formed between this chunk's products.
//
// Bound: matrix pipe (144 of 160 instructions per chunk are the product's six
// parts) and the board's power.  P = 20000, R = 180: 8.2e11 FLOP of FP32 work
// were 7.1 ms on FP32 instructions (77 % of that peak) with both weighted
// column sets.
//
// B of (chunk c, column group cg): pieces (tile T, part p) of 64 lanes x 8
// values, value i of lane l being part p of U column 16 (NB cg + T) + l % 16
// at row J = 32 c + 16 (i / 4) + 4 (l / 16) + i % 4.

__global__ __launch_bounds__(256) void k_rom_b3(const float *__restrict__ Ude, int64_t P, int nch, int ncols, int tiles,
                                                uint4 *__restrict__ Bk) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = (int)(t & 63);
  const int64_t ct = t >> 6;  // c tiles + T
  if (ct >= (int64_t)nch * tiles) return;
  const int64_t c = ct / tiles;
  const int col = (int)(ct % tiles) * 16 + (lane & 15);
  uint32_t o[3][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    Bf3 v[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int i = 2 * j + k;
      const int64_t J = 32 * c + 16 * (i >> 2) + 4 * (lane >> 4) + (i & 3);
      v[k] = split_bf3(J < P && col < ncols ? (double)Ude[(int64_t)col * P + J] : 0.0);
    }
    o[0][j] = (uint32_t)v[0].h | ((uint32_t)v[1].h << 16);
    o[1][j] = (uint32_t)v[0].m | ((uint32_t)v[1].m << 16);
    o[2][j] = (uint32_t)v[0].l | ((uint32_t)v[1].l << 16);
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) Bk[(ct * 3 + p) * 64 + lane] = uint4{o[p][0], o[p][1], o[p][2], o[p][3]};
}

// A run's segment that starts an item writes the item's output tile to Y; one
// that continues an item (its run's first) writes to the run's slot,
// kgemm_tile(NB) floats, which k_kgemm_fixup adds to Y.  Consecutive runs share
// an XCD (and its L2's B blocks).
template <int D, int NB>
__global__ __launch_bounds__(kKgWaves * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_kernel_gemm_bf3(
    const uint4 *__restrict__ K3, const uint4 *__restrict__ Bk, KgMap map, int ncols, float *__restrict__ Y,
    int64_t ldy, float *__restrict__ slots) {
  constexpr int NQ = bf3_slices(D);
  constexpr int KP = 2 * NQ, BP = 3 * NB, PC = KP + BP;  // pieces: K of the next chunk, B of this one
  __shared__ uint4 buf[2][PC * 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = (int)gridDim.x;
  const int L = G % 8 == 0 ? (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
  const int64_t nch = map.nch;
  const int64_t u_beg = map.run_start(L), u_end = map.run_start(L + 1);
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  bf16x8 neg[2];
  minus_identity(lane, neg);
  // the segments that start an item first (every run's first segment then
  // starts at chunk 0, so the runs of a column group read its B blocks nearly
  // in step through their XCD's L2), a continued item's part last
  const int64_t i_first = u_beg / nch;
  const bool continued = u_beg > i_first * nch;
  const int64_t i_lo = continued ? i_first + 1 : i_first;
  const int64_t n_seg = (u_end - 1) / nch - i_lo + 1 + (continued ? 1 : 0);
  for (int64_t sgi = 0; sgi < n_seg; ++sgi) {
    const int64_t item = continued && sgi == n_seg - 1 ? i_first : i_lo + sgi;
    const int c0 = (int)(max(u_beg, item * nch) - item * nch);
    const int c1 = (int)(min(u_end, (item + 1) * nch) - item * nch);
    const int cg = (int)(item / map.n_rg);
    const int rb0 = (int)(item % map.n_rg) * (kKgWaves * 2) + wave * 2;  // this wave's two 16-row blocks
    auto stage = [&](int c, int b) {  // K of chunk c + 1 and B of chunk c
#pragma unroll
      for (int i = 0; i < (PC + kKgWaves - 1) / kKgWaves; ++i) {
        const int pc = wave + kKgWaves * i;
        if (pc < PC && (pc >= KP || c + 1 < c1)) {  // scalar
          const uint4 *src = pc < KP ? K3 + ((int64_t)(c + 1) * KP + pc) * 64
                                     : Bk + (((int64_t)c * map.NCG + cg) * BP + (pc - KP)) * 64;
          piece_to_lds(src, &buf[b][pc * 64], lane);
        }
      }
    };
    stage(c0, 0);
    bf16x8 q[2][NQ];
#pragma unroll
    for (int r = 0; r < 2; ++r) bf3_row_operand<D>(K3, rb0 + r, lane, q[r]);
    floatx4 e[2][2];
    bf16x8 ep[2][3];  // the parts of this chunk's piece of Z
    auto distances = [&](const uint4 *kb) {
#pragma unroll
      for (int m = 0; m < NQ; ++m)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const bf16x8 ka = as_bf8(kb[(b * NQ + m) * 64 + lane]);
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (m == 0) e[r][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            e[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, q[r][m], e[r][b], 0, 0, 0);
          }
        }
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) e[r][b][i] = __builtin_amdgcn_exp2f(e[r][b][i]);
    };
    auto self_pairs = [&](int c) {
      if (c == rb0 >> 1) {  // scalar branch: Z_II = K_h(0) = 1 exactly
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) e[r][r][i] = diag_i == i ? 1.f : e[r][r][i];
      }
    };
    auto cut = [&](bf16x8 (&o)[2][3]) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          o[r][p] = upper_halves(e[r][0], e[r][1]);
          if (p < 2) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
              e[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(neg[b], o[r][p], e[r][b], 0, 0, 0);
          }
        }
    };
    floatx4 acc[2][NB];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int T = 0; T < NB; ++T) acc[r][T] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto products = [&](const uint4 *bb, int T) {
      bf16x8 bv[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) bv[p] = as_bf8(bb[(T * 3 + p) * 64 + lane]);
      // the small products of the chunk among themselves first: added to the
      // sum over all of Z one by one, what is below half a unit of it would be
      // lost, and Z's lower parts are all positive
      constexpr int pe[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
      floatx4 low[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) low[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < 5; ++x)
#pragma unroll
        for (int r = 0; r < 2; ++r)
          low[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ep[r][pe[x]], bv[pb[x]], low[r], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        acc[r][T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ep[r][0], bv[0], acc[r][T], 0, 0, 0);
        acc[r][T] += low[r];
      }
    };
    distances(K3 + (int64_t)c0 * KP * 64);
    self_pairs(c0);
    cut(ep);
    for (int c = c0; c < c1; ++c) {
      const int b = (c - c0) & 1;
      // each wave waits for its own pieces and the barrier publishes them; it
      // also ends the reads of the buffer the next stage goes to
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (c + 1 < c1) stage(c + 1, b ^ 1);
      const uint4 *bb = buf[b] + KP * 64;
      distances(buf[b]);  // of chunk c + 1 (past the last chunk: not used)
#pragma unroll
      for (int T = 0; T < NB / 2; ++T) products(bb, T);
      self_pairs(c + 1);
      bf16x8 en[2][3];
      cut(en);
#pragma unroll
      for (int T = NB / 2; T < NB; ++T) products(bb, T);
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int p = 0; p < 3; ++p) ep[r][p] = en[r][p];
    }
    __syncthreads();  // the next segment may overwrite either buffer
    // lane holds row 4 (lane / 16) + i of each block, column 16 T + lane % 16
    const bool first = c0 == 0;
    float *o = first ? Y + (int64_t)rb0 * 16 * ldy + (int64_t)cg * 16 * NB
                     : slots + (int64_t)L * kgemm_tile(NB) + (wave * 32) * (16 * NB);
    const int64_t ld = first ? ldy : 16 * NB;
#pragma unroll
    for (int T = 0; T < NB; ++T) {
      if (first && cg * 16 * NB + 16 * T + (lane & 15) >= ncols) continue;
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[(16 * r + 4 * (lane >> 4) + i) * ld + 16 * T + (lane & 15)] = acc[r][T][i];
    }
  }
}

// Y += the slots of the runs that continue item blockIdx.y, in run order
// (block x: elements x 1024 .. of its tile, four per thread).
// Bound: memory (Y twice, the slots once).  P = 20000, R = 180: 21 us, 72 with
// one element per thread and 64-bit divisions for the runs.
__global__ __launch_bounds__(256) void k_kgemm_fixup(const float *__restrict__ slots, KgMap map, float *__restrict__ Y,
                                                     int64_t ldy) {
  const int item = (int)blockIdx.y;
  const int64_t u0 = (int64_t)item * map.nch, u1 = u0 + map.nch;
  const int64_t La = map.run_after(u0), Lb = min((int64_t)map.G, map.run_after(u1 - 1));
  if (La >= Lb) return;
  const int e = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;
  const int W = 16 * map.NB, r = e / W;
  const int col = item / map.n_rg * W + e % W;
  if (col >= ldy) return;
  float4 *y = reinterpret_cast<float4 *>(Y + ((int64_t)(item % map.n_rg) * kKgRows + r) * ldy + col);
  float4 v = *y;
  for (int64_t L = La; L < Lb; ++L) {
    const float4 c = *reinterpret_cast<const float4 *>(slots + L * kgemm_tile(map.NB) + e);
    v.x += c.x, v.y += c.y, v.z += c.z, v.w += c.w;
  }
  *y = v;
}

template <int D>
void launch_kgemm_bf3(const KgMap &m, const uint4 *K3, const uint4 *Bk, int ncols, float *Y, int64_t ldy, float *slots,
                      hipStream_t s) {
  const dim3 grid((unsigned)m.G), block(kKgWaves * 64);
  switch (m.NB) {
    case 4: k_kernel_gemm_bf3<D, 4><<<grid, block, 0, s>>>(K3, Bk, m, ncols, Y, ldy, slots); break;
    case 8: k_kernel_gemm_bf3<D, 8><<<grid, block, 0, s>>>(K3, Bk, m, ncols, Y, ldy, slots); break;
    default: k_kernel_gemm_bf3<D, 12><<<grid, block, 0, s>>>(K3, Bk, m, ncols, Y, ldy, slots); break;
  }
}

// X^B1 = (w W - I1) / h^2, X^B2 = (w W^T - G2) / h^2 and X^B their sum, straight
// from the split partials of W and of the symmetric G2 (whose entries below the
// diagonal are those above it).  A workgroup owns a 16 x 16 tile; its four groups
// of 256 threads take every fourth split of W's tile, of its mirror image and of
// G2's, FP64, fixed order.
// Bound: the latency of splits / 4 loads, then the partials' bytes.  P = 20000,
// R = 180: 18 us for 128 splits; two sums over 64 splits, one thread per entry, and
// an elementwise launch took 17 + 17 + 3.
__global__ __launch_bounds__(1024) void k_rom_assemble(GemmShape gw, GemmShape gg, const float *__restrict__ partW,
                                                       const float *__restrict__ partG, int splits,
                                                       const float *__restrict__ I1, int R, float w, float ih2,
                                                       float *__restrict__ XB1, float *__restrict__ XB2,
                                                       float *__restrict__ XB) {
  __shared__ double red[3][4][256];
  __shared__ float tot[3][16][17];
  const int ti = blockIdx.x, tj = blockIdx.y;
  const int sg = threadIdx.x >> 8, e = threadIdx.x & 255, r = e >> 4, c = e & 15;
  const int64_t RR = (int64_t)R * R;
  // tile (a, b) of the three matrices: W's (ti, tj) and (tj, ti), G2's on or above the diagonal
  const int ta[3] = {ti, tj, min(ti, tj)}, tb[3] = {tj, ti, max(ti, tj)};
  const float *src[3];
  bool in[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int i = 16 * ta[q] + r, j = 16 * tb[q] + c;
    in[q] = i < R && j < R;
    src[q] = (q < 2 ? partW : partG) + (in[q] ? (int64_t)i * R + j : 0);
  }
  double s3[3] = {0.0, 0.0, 0.0};
  for (int k0 = sg; k0 < splits; k0 += 32) {
    float v[3][8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) v[q][u] = src[q][min(k0 + 4 * u, splits - 1) * RR];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) s3[q] += k0 + 4 * u < splits ? (double)v[q][u] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) red[q][sg][e] = in[q] ? s3[q] : 0.0;
  __syncthreads();
  if (sg < 3) {
    const int i = 16 * ta[sg] + r, j = 16 * tb[sg] + c;
    double s = (red[sg][0][e] + red[sg][1][e]) + (red[sg][2][e] + red[sg][3][e]);
    if (s != s) s = (double)gemm_entry_fp32(sg < 2 ? gw : gg, i, j);
    tot[sg][r][c] = (float)s;
  }
  __syncthreads();
  const int i = 16 * ti + r, j = 16 * tj + c;
  if (sg != 0 || i >= R || j >= R) return;
  const int64_t t = (int64_t)i * R + j;
  const float g2 = i > j ? tot[2][c][r] : tot[2][r][c];
  const float a = ih2 * (w * tot[0][r][c] - I1[t]), b = ih2 * (w * tot[1][c][r] - g2);
  XB1[t] = a;
  XB2[t] = b;
  XB[t] = a + b;
}

// ---- FP16-split kernel-GEMM (used with the FP16-split pair kernels) ---------
//
// The same product with Z and B split into FP16 halves and taken on
// v_mfma_f32_16x16x32_f16 as Z_hi B_hi + Z_hi B_lo + Z_lo B_hi (about 22
// significant bits).  Z enters as 2^15 Z and B as 2^8 B' with B' = U_a for the
// w-weighted columns (uniform weights over their maximum) and (w/S) U_a for the
// others; the epilogue multiplies column col by scale0 (col < 3R) or scale1.

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
constexpr float kKgShift = 15.f;
constexpr float kKgBScale = 256.f;
constexpr int kKgFlushPairs = 4;

// BH[((cp NB16 + nbk) 64 + n + 16 g) 8 + 4 s + i] = high half of B[32 cp + 16 s + 4 g + i][16 nbk + n];
// the low halves follow after Ppad ldy halves.
__global__ void k_rom_bsw16(const float *__restrict__ Ude, const float *__restrict__ wv,
                            const float *__restrict__ invS, float wmax, int64_t P, int64_t Ppad, int R, int NB16,
                            _Float16 *__restrict__ BH) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t ldy = (int64_t)NB16 * 16;
  if (t >= Ppad * ldy) return;
  const int64_t J = t / ldy;
  const int col = (int)(t % ldy);
  const int dR = 3 * R;
  float v = 0.f;
  if (J < P && col < 2 * dR) {
    const int h = col / dR, rem = col % dR, a = rem / R, tt = rem % R;
    const float wgt = h == 0 ? wv[J] / wmax : wv[J] * invS[J];
    v = kKgBScale * wgt * Ude[((int64_t)a * R + tt) * P + J];
  }
  const int jl = (int)(J & 15);
  const int64_t idx = (((J >> 5) * NB16 + (col >> 4)) * 64 + (col & 15) + 16 * (jl >> 2)) * 8 + 4 * ((J >> 4) & 1) +
                      (jl & 3);
  const _Float16 hi = (_Float16)v;
  BH[idx] = hi;
  BH[idx + Ppad * ldy] = (_Float16)(v - (float)hi);
}

__device__ inline half8 as_half8(uint4 u) {
  half8 h;
  __builtin_memcpy(&h, &u, sizeof(h));
  return h;
}

template <int KK>
__global__ __launch_bounds__(256) void k_kernel_gemm16(const float *__restrict__ QB, const float *__restrict__ KA,
                                                       int nrow_blocks, int ncol_chunks,
                                                       const uint4 *__restrict__ BH, int64_t lo_off, int NB16,
                                                       int dR, double scale0, double scale1, float one,
                                                       float *__restrict__ Y, int64_t ldy) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = (int)blockIdx.x * 4 + wave;
  if (rb >= nrow_blocks) return;
  const int nb0 = (int)blockIdx.y * kNBG;
  const int nbn = min(kNBG, NB16 - nb0);
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  const int ncp = (ncol_chunks + 1) / 2;  // the last pair's second chunk lies in the zero padding
  float qv[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qv[kk] = QB[((int64_t)rb * KK + kk) * 64 + lane];
  double tot[kNBG][4];
#pragma unroll
  for (int g = 0; g < kNBG; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) tot[g][i] = 0.0;
  const floatx4 shift = {kKgShift, kKgShift, kKgShift, kKgShift};

  for (int cp = 0; cp < ncp;) {
    const int g_end = min(ncp, cp + kKgFlushPairs);
    floatx4 acc[kNBG];
#pragma unroll
    for (int g = 0; g < kNBG; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (; cp < g_end; ++cp) {
      float e[8];
#pragma unroll
      for (int sc = 0; sc < 2; ++sc) {
        const int c = 2 * cp + sc;
        floatx4 t = shift;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          t = __builtin_amdgcn_mfma_f32_16x16x4f32(KA[((int64_t)c * KK + kk) * 64 + lane], qv[kk], t, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) e[4 * sc + i] = fminf(__builtin_amdgcn_exp2f(t[i]), 32768.f);
        if (c == rb) {  // the self pair has Z_II = K_h(0) = 1 exactly
#pragma unroll
          for (int i = 0; i < 4; ++i) e[4 * sc + i] = diag_i == i ? 32768.f : e[4 * sc + i];
        }
      }
      half8 eh, el;
#pragma unroll
      for (int j = 0; j < 8; j += 2) {
        const half2v h = __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(e[j], e[j + 1]));
        const float ra = __builtin_fmaf(-(float)h.x, one, e[j]);
        const float rb2 = __builtin_fmaf(-(float)h.y, one, e[j + 1]);
        eh[j] = h.x;
        eh[j + 1] = h.y;
        el[j] = (_Float16)ra;
        el[j + 1] = (_Float16)rb2;
      }
      const uint4 *bp = BH + ((int64_t)cp * NB16 + nb0) * 64 + lane;
#pragma unroll
      for (int g = 0; g < kNBG; ++g) {
        if (g < nbn) {
          const half8 bh = as_half8(bp[(int64_t)g * 64]);
          const half8 bl = as_half8(bp[lo_off + (int64_t)g * 64]);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh, bh, acc[g], 0, 0, 0);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh, bl, acc[g], 0, 0, 0);
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(el, bh, acc[g], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < kNBG; ++g)
#pragma unroll
      for (int i = 0; i < 4; ++i) tot[g][i] += (double)acc[g][i];
  }
#pragma unroll
  for (int g = 0; g < kNBG; ++g) {
    if (g >= nbn) break;
    const int col = (nb0 + g) * 16 + (lane & 15);
    const double sc = col < dR ? scale0 : scale1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t row = (int64_t)rb * 16 + 4 * (lane >> 4) + i;
      Y[row * ldy + col] = (float)(tot[g][i] * sc);
    }
  }
}

// The same product with FP16-split distances (the pair kernels' QH/KH/RN
// operands), tiled for reuse: a workgroup of kLdsWaves waves owns
// kLdsWaves x 2 row blocks (256 rows) and kNBG column blocks (128 columns);
// per chunk pair (32 columns of Z) it stages the chunk's B highs and lows and
// its K-side distance operands in LDS once (double buffered, one barrier), and
// every wave generates its two 16 x 32 tiles of Z and multiplies them by all
// kNBG column blocks.  Each B element is thus read once per 256 rows instead
// of once per 16.  FP32 accumulation over all columns of Z (no FP64 flush: 64
// accumulators per lane already; the error stays ~1e-6 of the sums).
constexpr int kLdsWaves = 8;
constexpr int kLdsRB = 2;

// (at most 128 VGPRs, so that two workgroups share a CU: 2.5 instead of
// 3.0 ms per launch at P = 20000, 1080 columns)
template <int KQ>
__global__ __launch_bounds__(kLdsWaves * 64, 4) void k_kernel_gemm16_lds(
    const uint4 *__restrict__ QH, const uint4 *__restrict__ KH, const float *__restrict__ RN, int nrow_blocks,
    int ncp, const uint4 *__restrict__ BH, int64_t lo_off, int NB16, int dR, double scale0, double scale1,
    float one, float *__restrict__ Y, int64_t ldy) {
  __shared__ uint4 bsh[2][2 * kNBG * 64];
  __shared__ uint4 ksh[2][2 * KQ * 64];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rb0 = ((int)blockIdx.x * kLdsWaves + wave) * kLdsRB;
  const int nb0 = (int)blockIdx.y * kNBG;
  const int nbn = min(kNBG, NB16 - nb0);
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  half8 qh[kLdsRB][KQ];
  float rinit[kLdsRB];
#pragma unroll
  for (int r = 0; r < kLdsRB; ++r) {
    const bool ok = rb0 + r < nrow_blocks;
#pragma unroll
    for (int m = 0; m < KQ; ++m)
      qh[r][m] = as_half8(ok ? QH[((int64_t)(rb0 + r) * KQ + m) * 64 + lane] : uint4{0, 0, 0, 0});
    rinit[r] = (ok ? RN[(int64_t)(rb0 + r) * 16 + (lane & 15)] : 0.f) + kKgShift;
  }
  floatx4 acc[kLdsRB][kNBG];
#pragma unroll
  for (int r = 0; r < kLdsRB; ++r)
#pragma unroll
    for (int g = 0; g < kNBG; ++g) acc[r][g] = floatx4{0.f, 0.f, 0.f, 0.f};

  // tile loads: thread t < kNBG 64 takes B high and low element t of the
  // chunk's kNBG x 64 uint4 (zero past the last column block) and, for
  // t < 2 KQ 64, distance operand t
  const int gt = t >> 6;
  static_assert(kNBG <= kLdsWaves && 2 * 2 <= kLdsWaves, "one tile element per thread");
  auto load_tile = [&](int cp, uint4 &bh, uint4 &bl, uint4 &kh) {
    const int64_t bo = ((int64_t)cp * NB16 + nb0) * 64 + t;
    bh = gt < nbn ? BH[bo] : uint4{0, 0, 0, 0};
    bl = gt < nbn ? BH[lo_off + bo] : uint4{0, 0, 0, 0};
    if (t < 2 * KQ * 64) kh = KH[(int64_t)(2 * cp) * KQ * 64 + t];
  };
  auto store_tile = [&](int buf, const uint4 &bh, const uint4 &bl, const uint4 &kh) {
    if (gt < kNBG) {
      bsh[buf][t] = bh;
      bsh[buf][kNBG * 64 + t] = bl;
    }
    if (t < 2 * KQ * 64) ksh[buf][t] = kh;
  };
  uint4 nbh = uint4{0, 0, 0, 0}, nbl = uint4{0, 0, 0, 0}, nkh = uint4{0, 0, 0, 0};
  if (ncp > 0) {
    load_tile(0, nbh, nbl, nkh);
    store_tile(0, nbh, nbl, nkh);
  }
  __syncthreads();
  const bool active = rb0 < nrow_blocks;  // wave-uniform; every wave still stages tiles
  for (int cp = 0; cp < ncp; ++cp) {
    const int cur = cp & 1;
    if (cp + 1 < ncp) load_tile(cp + 1, nbh, nbl, nkh);
    if (active) {
      half8 eh[kLdsRB], el[kLdsRB];
#pragma unroll
      for (int r = 0; r < kLdsRB; ++r) {
        float e[8];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          floatx4 tt = {rinit[r], rinit[r], rinit[r], rinit[r]};
#pragma unroll
          for (int m = 0; m < KQ; ++m)
            tt = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(ksh[cur][(s2 * KQ + m) * 64 + lane]), qh[r][m], tt,
                                                        0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) e[4 * s2 + i] = __builtin_amdgcn_exp2f(tt[i]);
          if (2 * cp + s2 == rb0 + r) {  // the self pair has Z_II = K_h(0) = 1 exactly
#pragma unroll
            for (int i = 0; i < 4; ++i) e[4 * s2 + i] = diag_i == i ? 32768.f : e[4 * s2 + i];
          }
        }
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
          const half2v h = __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(e[j], e[j + 1]));
          const float ra = __builtin_fmaf(-(float)h.x, one, e[j]);
          const float rb2 = __builtin_fmaf(-(float)h.y, one, e[j + 1]);
          eh[r][j] = h.x;
          eh[r][j + 1] = h.y;
          el[r][j] = (_Float16)ra;
          el[r][j + 1] = (_Float16)rb2;
        }
      }
#pragma unroll
      for (int g = 0; g < kNBG; ++g) {
        const half8 bh = as_half8(bsh[cur][g * 64 + lane]);
        const half8 bl = as_half8(bsh[cur][kNBG * 64 + g * 64 + lane]);
#pragma unroll
        for (int r = 0; r < kLdsRB; ++r) {
          acc[r][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh[r], bh, acc[r][g], 0, 0, 0);
          acc[r][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(eh[r], bl, acc[r][g], 0, 0, 0);
          acc[r][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(el[r], bh, acc[r][g], 0, 0, 0);
        }
      }
    }
    if (cp + 1 < ncp) store_tile(cur ^ 1, nbh, nbl, nkh);
    __syncthreads();
  }
  if (!active) return;
#pragma unroll
  for (int r = 0; r < kLdsRB; ++r) {
    if (rb0 + r >= nrow_blocks) break;
#pragma unroll
    for (int g = 0; g < kNBG; ++g) {
      if (g >= nbn) break;
      const int col = (nb0 + g) * 16 + (lane & 15);
      const double sc = col < dR ? scale0 : scale1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = (int64_t)(rb0 + r) * 16 + 4 * (lane >> 4) + i;
        Y[row * ldy + col] = (float)((double)acc[r][g][i] * sc);
      }
    }
  }
}

__global__ void k_fill_scaled(const float *__restrict__ src, float a, int64_t n, float *__restrict__ dst) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) dst[t] = a * src[t];
}

__global__ void k_add(const float *__restrict__ a, const float *__restrict__ b, int64_t n, float *__restrict__ c) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) c[t] = a[t] + b[t];
}

// p <- p + a (p - prev), in place: the linear extrapolation of the reduced
// state from an earlier one
__global__ void k_extrapolate(float *__restrict__ p, const float *__restrict__ prev, float a, int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) p[t] = fmaf(a, p[t] - prev[t], p[t]);
}

// Lanes of each four exchanged by a DPP quad_perm control.
template <int kPerm>
__device__ __forceinline__ float quad_swap(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kPerm, 0xf, 0xf, true));
}

// Explicit Euler on the reduced state p[k][s] (eq. model_DymReduced):
// dp_k/dt = X^H p_k - (kT/zeta) sum_j A_kj X^B p_j - (1/zeta) sum_j A_kj H_j p_j.
// One workgroup; p in LDS; each wavefront takes whole rows of X^H / X^B.
__global__ __launch_bounds__(1024) void k_rom_steps(const float *__restrict__ XH, const float *__restrict__ XB,
                                                    float *__restrict__ p, int nb, int R, int nsteps, EvalParams ep) {
  __shared__ float ps[kMaxNb][kMaxR];
  __shared__ float y[kMaxNb][kMaxR];
  __shared__ float z[kMaxNb][kMaxR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  for (int t = tid; t < nb * R; t += blockDim.x) ps[t / R][t % R] = p[t];
  __syncthreads();
  const float ktz = ep.kT * ep.inv_zeta;
  for (int step = 0; step < nsteps; ++step) {
    for (int row = wave; row < 2 * R; row += nw) {
      const float *M = row < R ? XH + (int64_t)row * R : XB + (int64_t)(row - R) * R;
      float acc[kMaxNb];
#pragma unroll
      for (int k = 0; k < kMaxNb; ++k) acc[k] = 0.f;
      for (int u = lane; u < R; u += 64) {
        const float m = M[u];
#pragma unroll
        for (int k = 0; k < kMaxNb; ++k)
          if (k < nb) acc[k] = fmaf(m, ps[k][u], acc[k]);
      }
#pragma unroll
      for (int k = 0; k < kMaxNb; ++k) {
        float v = acc[k];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        acc[k] = v;
      }
      if (lane == 0) {
        for (int k = 0; k < nb; ++k) {
          if (row < R) y[k][row] = acc[k];
          else z[k][row - R] = acc[k];
        }
      }
    }
    __syncthreads();
    float pn[kMaxNb * kMaxR / 1024 + 1];
    int cnt = 0;
    for (int t = tid; t < nb * R; t += blockDim.x, ++cnt) {
      const int k = t / R, s = t % R;
      float az = 2.f * z[k][s], ah = 2.f * ep.H[k] * ps[k][s];
      if (k > 0) {
        az -= z[k - 1][s];
        ah -= ep.H[k - 1] * ps[k - 1][s];
      }
      if (k + 1 < nb) {
        az -= z[k + 1][s];
        ah -= ep.H[k + 1] * ps[k + 1][s];
      }
      pn[cnt] = ps[k][s] + ep.dt * (y[k][s] - ktz * az - ep.inv_zeta * ah);
    }
    __syncthreads();
    cnt = 0;
    for (int t = tid; t < nb * R; t += blockDim.x, ++cnt) ps[t / R][t % R] = pn[cnt];
    __syncthreads();
  }
  for (int t = tid; t < nb * R; t += blockDim.x) p[t] = ps[t / R][t % R];
}

// The same steps with both operators held in registers for the whole window:
// four lanes per matrix row s, each with the float4 column groups g, g + 4, ...
// of X^H and of X^B, so a step reads only the state, as float4 broadcasts from
// LDS.  The sums over the four lanes (DPP) give a row's y_k and z_k for every
// bond in the same lanes, which also keep the row's own state: the update needs
// no exchange, and with the state double-buffered in LDS a step is one barrier.
// Only as many waves as the rows need.  kQ: columns per lane (R <= 4 kQ, kQ a
// multiple of 4), NB = nb bonds known at compile time.
// Bound: one wave's chain of 2 NB kQ FMAs, the sums, the LDS read and the
// barrier; the register budget of exactly the waves there are lets the state's
// loads go out together (R = 64: 407 against 651 ns).  Measured per step, NB = 3:
// R = 16 0.20, 40 0.34, 64 0.41, 128 0.73, 180 1.3 us; two lanes per row of
// [X^H; X^B], 768 threads and an exchange through LDS took 0.65, 0.90, 0.91,
// 2.4, 2.1.
constexpr int kRegMaxR = 192;
template <int kQ, int NB>
__global__ __launch_bounds__(16 * kQ) __attribute__((amdgpu_waves_per_eu((kQ + 15) / 16, (kQ + 15) / 16))) void
k_rom_steps_reg(const float *__restrict__ XH, const float *__restrict__ XB, float *__restrict__ p, int R, int nsteps,
                EvalParams ep) {
  static_assert(kQ % 4 == 0 && 4 * kQ <= kRegMaxR, "columns are read as float4");
  constexpr int W = 4 * kQ, C4 = kQ / 4;
  __shared__ float4 ps[2][NB][W / 4];
  const int tid = threadIdx.x;
  const int row = tid >> 2, g = tid & 3;
  const bool active = row < R;
  float mh[kQ], mb[kQ];
#pragma unroll
  for (int j = 0; j < kQ; ++j) {
    const int u = 16 * (j / 4) + 4 * g + j % 4;
    const bool in = active && u < R;
    mh[j] = in ? XH[(int64_t)row * R + u] : 0.f;
    mb[j] = in ? XB[(int64_t)row * R + u] : 0.f;
  }
  float *ps0 = reinterpret_cast<float *>(&ps[0][0][0]);
  for (int t = tid; t < 2 * NB * W; t += blockDim.x) {  // zero padding: the unused columns meet zeros
    const int b = t / (NB * W), k = (t / W) % NB, s = t % W;
    ps0[t] = (b == 0 && s < R) ? p[k * R + s] : 0.f;
  }
  float own[NB], H[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    own[k] = active ? p[k * R + row] : 0.f;
    H[k] = ep.H[k];
  }
  const float ktz = ep.kT * ep.inv_zeta, inv_zeta = ep.inv_zeta, dt = ep.dt;
  __syncthreads();
  int cur = 0;
  for (int step = 0; step < nsteps; ++step) {
    float y[NB], z[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) y[k] = z[k] = 0.f;
#pragma unroll
    for (int c = 0; c < C4; ++c)
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const float4 v = ps[cur][k][4 * c + g];
        y[k] = fmaf(mh[4 * c], v.x, y[k]);
        z[k] = fmaf(mb[4 * c], v.x, z[k]);
        y[k] = fmaf(mh[4 * c + 1], v.y, y[k]);
        z[k] = fmaf(mb[4 * c + 1], v.y, z[k]);
        y[k] = fmaf(mh[4 * c + 2], v.z, y[k]);
        z[k] = fmaf(mb[4 * c + 2], v.z, z[k]);
        y[k] = fmaf(mh[4 * c + 3], v.w, y[k]);
        z[k] = fmaf(mb[4 * c + 3], v.w, z[k]);
      }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      y[k] += quad_swap<0x4e>(y[k]);  // lanes 2, 3, 0, 1 of each four
      z[k] += quad_swap<0x4e>(z[k]);
      y[k] += quad_swap<0xb1>(y[k]);  // lanes 1, 0, 3, 2
      z[k] += quad_swap<0xb1>(z[k]);
    }
    float nw[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      float az = 2.f * z[k], ah = 2.f * H[k] * own[k];
      if (k > 0) {
        az -= z[k - 1];
        ah -= H[k - 1] * own[k - 1];
      }
      if (k + 1 < NB) {
        az -= z[k + 1];
        ah -= H[k + 1] * own[k + 1];
      }
      nw[k] = own[k] + dt * (y[k] - ktz * az - inv_zeta * ah);
    }
    float *pn = reinterpret_cast<float *>(&ps[cur ^ 1][0][0]);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      own[k] = nw[k];
      if (active && g == k % 4) pn[k * W + row] = nw[k];
    }
    __syncthreads();
    cur ^= 1;
  }
#pragma unroll
  for (int k = 0; k < NB; ++k)
    if (active && g == k % 4) p[k * R + row] = own[k];
}

template <int kQ>
void launch_steps_reg(int nb, const float *XH, const float *XB, float *p, int R, int n, const EvalParams &ep,
                      hipStream_t s) {
  const int threads = (4 * R + 63) / 64 * 64;
  switch (nb) {
    case 1: k_rom_steps_reg<kQ, 1><<<1, threads, 0, s>>>(XH, XB, p, R, n, ep); break;
    case 2: k_rom_steps_reg<kQ, 2><<<1, threads, 0, s>>>(XH, XB, p, R, n, ep); break;
    case 3: k_rom_steps_reg<kQ, 3><<<1, threads, 0, s>>>(XH, XB, p, R, n, ep); break;
    case 4: k_rom_steps_reg<kQ, 4><<<1, threads, 0, s>>>(XH, XB, p, R, n, ep); break;
    default: k_rom_steps_reg<kQ, 5><<<1, threads, 0, s>>>(XH, XB, p, R, n, ep); break;
  }
}

// ---- exact integration of a frozen window --------------------------------
//
// Generator of eq. model_DymReduced on vec(p) (index i = k R + s), column-major:
// L[i + l n] with l = j R + u,
//   delta_kj X^H_su - (kT/zeta) A_kj X^B_su - (1/zeta) A_kj H_j delta_su.
__global__ void k_generator(const float *__restrict__ XH, const float *__restrict__ XB, int nb, int R,
                            EvalParams ep, double *__restrict__ Lm) {
  const int64_t n = (int64_t)nb * R;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= n * n) return;
  const int64_t i = t % n, l = t / n;
  const int k = (int)(i / R), s = (int)(i % R), j = (int)(l / R), u = (int)(l % R);
  const double A = k == j ? 2.0 : ((k - j == 1 || j - k == 1) ? -1.0 : 0.0);
  double v = -(double)ep.kT * (double)ep.inv_zeta * A * (double)XB[(int64_t)s * R + u];
  if (k == j) v += (double)XH[(int64_t)s * R + u];
  if (s == u) v -= (double)ep.inv_zeta * A * (double)ep.H[j];
  Lm[t] = v;
}

// Largest absolute column sum of a column-major n x n matrix, per column.
__global__ void k_colabs(const double *__restrict__ Lm, int64_t n, double *__restrict__ cs) {
  const int64_t l = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (l >= n) return;
  double a = 0.0;
  for (int64_t i = 0; i < n; ++i) a += fabs(Lm[i + l * n]);
  cs[l] = a;
}

__global__ void k_scale64(const double *__restrict__ a, double f, int64_t n, double *__restrict__ b) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) b[t] = f * a[t];
}

__global__ void k_identity64(int64_t n, double *__restrict__ M) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n * n) M[t] = (t % n == t / n) ? 1.0 : 0.0;
}

__global__ void k_f64_to_f32(const double *__restrict__ a, int64_t n, float *__restrict__ b) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) b[t] = (float)a[t];
}

// tau_ab = (n / P) sum_k H_k p_k^T M_ab p_k (uniform weights), FP64 sums: a
// workgroup per ab, its waves over the rows, lanes over the columns.
__global__ __launch_bounds__(1024) void k_rom_stress(const float *__restrict__ Mbig, const float *__restrict__ p, int nb,
                                                     int R, EvalParams ep, double *__restrict__ out) {
  __shared__ double sm[16];
  const int ab = blockIdx.x;  // 0..8
  const int a = ab / 3, b = ab % 3, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t ld = 3 * (int64_t)R;
  const float *M = Mbig + (int64_t)a * R * ld + (int64_t)b * R;
  double acc = 0.0;
  for (int u = lane; u < R; u += 64)
#pragma unroll 4
    for (int s = wave; s < R; s += 16) {
      const double m = M[s * ld + u];
      double pp = 0.0;
#pragma unroll
      for (int k = 0; k < kMaxNb; ++k)
        if (k < nb) pp += (double)ep.H[k] * (double)p[k * R + s] * (double)p[k * R + u];
      acc += m * pp;
    }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d);
  if (lane == 0) sm[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int v = 0; v < 16; ++v) t += sm[v];
    out[ab] = t * (double)ep.n / (double)ep.P;
  }
}

inline unsigned nblk256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

struct vds_rom_s {
  vds_ctx ctx = nullptr;
  const float *U = nullptr;
  int R = 0;
  RomLayout L{};
  char *ws = nullptr;
  bool b3_ready = false;  // Bsw holds the basis as the default kernel-GEMM reads it
  float *Ude, *Mbig, *XH, *I1, *XB1, *XB2, *XB, *Bsw, *Y, *qt, *T, *invS, *part, *psave, *pprev;
  double *red;
  HostSlot host;  // kHostTau stresses
};

namespace {

constexpr int kHostTau = 56;  // 72 bytes each in one block

vds_status rom_gemm(vds_rom r, GemmShape g, double flops) {
  timed(r->ctx, VDS_TIMER_GEMM, flops, [&] { launch_gemm(g, r->part, r->ctx->stream); });
  return VDS_OK;
}

// Stresses of reduced states (from the M_ab), in stream order into tau[9],
// tau[9] + 9, ...: the kernel writes them to pinned memory, which is emptied
// when it is full and at the end.
struct StressOut {
  vds_rom r;
  double *tau;
  int queued = 0;
  vds_status add(const float *p) {
    vds_ctx c = r->ctx;
    double *host = static_cast<double *>(r->host.take(sizeof(double) * 9 * kHostTau));
    k_rom_stress<<<9, 1024, 0, c->stream>>>(r->Mbig, p, c->prob.nb, r->R, c->ep, host ? host + 9 * queued : r->red);
    if (host != nullptr) {
      vds_status st = hip_check(c, hipGetLastError(), "stress");
      return st == VDS_OK && ++queued == kHostTau ? finish() : st;
    }
    vds_status st = hip_check(c, hipMemcpyAsync(tau, r->red, sizeof(double) * 9, hipMemcpyDeviceToHost, c->stream),
                              "copy stress");
    tau += 9;
    return st;
  }
  vds_status finish() {  // synchronises
    vds_status st = hip_check(r->ctx, hipStreamSynchronize(r->ctx->stream), "synchronise");
    if (st != VDS_OK) return st;
    if (queued > 0) std::memcpy(tau, r->host.p, sizeof(double) * 9 * queued);
    r->host.read();
    tau += 9 * queued;
    queued = 0;
    return VDS_OK;
  }
};

// q~ = U p into r->qt.
void reconstruct_qt(vds_rom r, const float *p) {
  vds_ctx c = r->ctx;
  const int64_t m = 3 * c->prob.P;
  timed(c, VDS_TIMER_PROJ, 4.0 * m * r->R,
        [&] { launch_pod_reconstruct(r->U, m, r->R, c->prob.nb, p, r->qt, c->stream); });
}

// The basis as the B operand of the default kernel-GEMM, laid out once.
void prepare_b3(vds_rom r) {
  const vds_ctx c = r->ctx;
  const KgMap &m = r->L.kg;
  const int tiles = m.NB * m.NCG;
  k_rom_b3<<<nblk256((int64_t)m.nch * tiles * 64), 256, 0, c->stream>>>(r->Ude, c->prob.P, m.nch, 3 * r->R, tiles,
                                                                        reinterpret_cast<uint4 *>(r->Bsw));
  r->b3_ready = true;
}

// X^B1, X^B2 and X^B from the pair operands, S and T at q~ with the default
// kernel-GEMM (uniform weights: see there).
vds_status operators_bf3(vds_rom r) {
  vds_ctx c = r->ctx;
  const int R = r->R;
  const int64_t P = c->prob.P, RR = (int64_t)R * R;
  const RomLayout &L = r->L;
  hipStream_t s = c->stream;
  if (!r->b3_ready) prepare_b3(r);
  const int ncols = 3 * R;
  const int64_t ldy = rom_ldy3(R);
  timed(c, VDS_TIMER_KGEMM, 2.0 * (double)P * P * ncols, [&] {
    const uint4 *k3 = static_cast<const uint4 *>(c->f16.QH), *bk = reinterpret_cast<const uint4 *>(r->Bsw);
    switch (c->ep.D) {
      case 3: launch_kgemm_bf3<3>(L.kg, k3, bk, ncols, r->Y, ldy, r->part, s); break;
      case 6: launch_kgemm_bf3<6>(L.kg, k3, bk, ncols, r->Y, ldy, r->part, s); break;
      case 9: launch_kgemm_bf3<9>(L.kg, k3, bk, ncols, r->Y, ldy, r->part, s); break;
      case 12: launch_kgemm_bf3<12>(L.kg, k3, bk, ncols, r->Y, ldy, r->part, s); break;
      default: launch_kgemm_bf3<15>(L.kg, k3, bk, ncols, r->Y, ldy, r->part, s); break;
    }
    k_kgemm_fixup<<<dim3((unsigned)(kgemm_tile(L.kg.NB) / 1024), (unsigned)L.kg.items()), 256, 0, s>>>(r->part, L.kg,
                                                                                                       r->Y, ldy);
  });
  GemmShape g;
  g.M = R;
  g.N = R;
  g.K = P;
  g.nbatch = 3;
  g.A = r->Ude;
  g.lda = P;
  g.sA = (int64_t)R * P;
  g.B = r->Y;  // W = sum_a U_a^T diag(1/S) Y_a
  g.ldb = ldy;
  g.sB = R;
  g.b_mn = true;
  g.scale = r->invS;
  g.splits = rom_splits(L, R, P);
  float *partG = r->part + (int64_t)g.splits * RR;
  timed(c, VDS_TIMER_GEMM, 2.0 * 3 * RR * P, [&] { launch_gemm_parts(g, r->part, s); });
  GemmShape g2 = g;
  g2.B = r->Ude;  // G2 = sum_a U_a^T diag(T) U_a
  g2.ldb = P;
  g2.sB = (int64_t)R * P;
  g2.b_mn = false;
  g2.scale = r->T;
  g2.symmetric = true;
  timed(c, VDS_TIMER_GEMM, 2.0 * 3 * RR * P, [&] {
    launch_gemm_parts(g2, partG, s);
    const unsigned t16 = (unsigned)((R + 15) / 16);
    k_rom_assemble<<<dim3(t16, t16), 1024, 0, s>>>(g, g2, r->part, partG, g.splits, r->I1, R, c->ep.uniform_w,
                                                   c->ep.inv_h2, r->XB1, r->XB2, r->XB);
  });
  return hip_check(c, hipGetLastError(), "reduced operators");
}

vds_status freeze(vds_rom r, const float *p) {
  vds_ctx c = r->ctx;
  const int R = r->R;
  const int64_t P = c->prob.P, Ppad = c->ep.Ppad;
  const RomLayout &L = r->L;
  hipStream_t s = c->stream;
  reconstruct_qt(r, p);
  // S and T at q~ (uniform weights), Q/K operands for Z
  eval_pass_a(c, r->qt, nullptr, nullptr);
  if (rows_path(c)) {
    pass_b(c, MODE_SUMS, false, nullptr, nullptr, r->T, r->invS, nullptr, 0, nullptr, nullptr);
  } else {
    eval_pass_b(c, nullptr);
    k_rom_scalars<<<nblk256(Ppad), 256, 0, s>>>(c->part, c->smap, Ppad, P, c->ep.D, c->S, c->wv, r->T, r->invS);
  }
  if (c->ep.bf3) return operators_bf3(r);
  r->b3_ready = false;  // the forms below lay their weighted columns out in Bsw
  // Y = Z B, in the FP16-split form when the context's pair kernels use it
  if (c->ep.vhalf) {
    const float wmax = c->ep.uniform_w;  // the reduced model runs with uniform weights
    k_rom_bsw16<<<nblk256(Ppad * L.ldy), 256, 0, s>>>(r->Ude, c->wv, r->invS, wmax, P, Ppad, R, L.NB16,
                                                      reinterpret_cast<_Float16 *>(r->Bsw));
    const int nrb = (int)(Ppad / 16), ncc = (int)((P + 15) / 16);
    dim3 grid((unsigned)((nrb + 3) / 4), (unsigned)((L.NB16 + kNBG - 1) / kNBG));
    const uint4 *bh = reinterpret_cast<const uint4 *>(r->Bsw);
    const int64_t lo_off = Ppad * L.ldy / 8;  // uint4 units
    const double unscale = 1.0 / ((double)kKgBScale * 32768.0);
    const double s0 = (double)wmax * unscale, s1 = unscale;
    const double flops = 2.0 * (double)P * P * 2 * 3 * R;
    if (c->ep.qhalf) {
      const uint4 *qh = reinterpret_cast<const uint4 *>(c->f16.QH), *kh = reinterpret_cast<const uint4 *>(c->f16.KH);
      const int ncp = (ncc + 1) / 2;
      dim3 g2((unsigned)((nrb + kLdsWaves * kLdsRB - 1) / (kLdsWaves * kLdsRB)), (unsigned)((L.NB16 + kNBG - 1) / kNBG));
      timed(c, VDS_TIMER_KGEMM, flops, [&] {
        if (c->ep.KQ == 1)
          k_kernel_gemm16_lds<1><<<g2, kLdsWaves * 64, 0, s>>>(qh, kh, c->f16.RN, nrb, ncp, bh, lo_off, L.NB16, 3 * R,
                                                               s0, s1, 1.f, r->Y, L.ldy);
        else
          k_kernel_gemm16_lds<2><<<g2, kLdsWaves * 64, 0, s>>>(qh, kh, c->f16.RN, nrb, ncp, bh, lo_off, L.NB16, 3 * R,
                                                               s0, s1, 1.f, r->Y, L.ldy);
      });
    } else timed(c, VDS_TIMER_KGEMM, flops, [&] {
      switch (c->ep.KK) {
        case 2: k_kernel_gemm16<2><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, bh, lo_off, L.NB16, 3 * R, s0, s1, 1.f, r->Y, L.ldy); break;
        case 3: k_kernel_gemm16<3><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, bh, lo_off, L.NB16, 3 * R, s0, s1, 1.f, r->Y, L.ldy); break;
        case 4: k_kernel_gemm16<4><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, bh, lo_off, L.NB16, 3 * R, s0, s1, 1.f, r->Y, L.ldy); break;
        default: k_kernel_gemm16<5><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, bh, lo_off, L.NB16, 3 * R, s0, s1, 1.f, r->Y, L.ldy); break;
      }
    });
  } else {
    // the 16x16 FP32 forms (VDS_PAIR_MFMA, VDS_PAIR_VALU) read the 16-row operand layout
    k_rom_bsw<<<nblk256(Ppad * L.ldy), 256, 0, s>>>(r->Ude, c->wv, r->invS, P, Ppad, R, L.NB16, r->Bsw);
    const int nrb = (int)(Ppad / 16), ncc = (int)((P + 15) / 16);
    dim3 grid((unsigned)((nrb + 3) / 4), (unsigned)((L.NB16 + kNBG - 1) / kNBG));
    const float4 *b4 = reinterpret_cast<const float4 *>(r->Bsw);
    const double flops = 2.0 * (double)P * P * 2 * 3 * R;
    timed(c, VDS_TIMER_KGEMM, flops, [&] {
      switch (c->ep.KK) {
        case 2: k_kernel_gemm<2><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, b4, L.NB16, r->Y, L.ldy); break;
        case 3: k_kernel_gemm<3><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, b4, L.NB16, r->Y, L.ldy); break;
        case 4: k_kernel_gemm<4><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, b4, L.NB16, r->Y, L.ldy); break;
        default: k_kernel_gemm<5><<<grid, 256, 0, s>>>(c->QB, c->KA, nrb, ncc, b4, L.NB16, r->Y, L.ldy); break;
      }
    });
  }
  const float ih2 = c->ep.inv_h2;
  const int64_t RR = (int64_t)R * R;
  // X^B1 = -(1/h^2) I1 + (1/h^2) sum_a U_a^T diag(1/S) Y1_a
  k_fill_scaled<<<nblk256(RR), 256, 0, s>>>(r->I1, -ih2, RR, r->XB1);
  {
    GemmShape g;
    g.M = R;
    g.N = R;
    g.K = P;
    g.nbatch = 3;
    g.A = r->Ude;
    g.lda = P;
    g.sA = (int64_t)R * P;
    g.B = r->Y;
    g.ldb = L.ldy;
    g.sB = R;
    g.b_mn = true;
    g.scale = r->invS;
    g.alpha = ih2;
    g.C = r->XB1;
    g.ldc = R;
    g.accumulate = true;
    g.splits = gemm_splits(R, R, P, 3);
    rom_gemm(r, g, 2.0 * 3 * RR * P);
  }
  // X^B2 = -(1/h^2) sum_a U_a^T diag(T) U_a + (1/h^2) sum_a U_a^T Y2_a
  {
    GemmShape g;
    g.M = R;
    g.N = R;
    g.K = P;
    g.nbatch = 3;
    g.A = r->Ude;
    g.lda = P;
    g.sA = (int64_t)R * P;
    g.B = r->Ude;
    g.ldb = P;
    g.sB = (int64_t)R * P;
    g.scale = r->T;
    g.alpha = -ih2;
    g.C = r->XB2;
    g.ldc = R;
    g.splits = gemm_splits(R, R, P, 3);
    rom_gemm(r, g, 2.0 * 3 * RR * P);
    g.B = r->Y + 3 * R;
    g.ldb = L.ldy;
    g.sB = R;
    g.b_mn = true;
    g.scale = nullptr;
    g.alpha = ih2;
    g.accumulate = true;
    rom_gemm(r, g, 2.0 * 3 * RR * P);
  }
  k_add<<<nblk256(RR), 256, 0, s>>>(r->XB1, r->XB2, RR, r->XB);
  return hip_check(c, hipGetLastError(), "reduced operators");
}

}  // namespace

extern "C" {

size_t vds_rom_workspace_bytes(const vds_problem *prob, int32_t R) {
  if (prob == nullptr || prob->P < 1 || prob->nb < 1 || R < 1 || R > kMaxR || R > 3 * prob->P) return 0;
  return rom_layout(*prob, R).total;
}

vds_status vds_rom_create(vds_ctx c, const float *U, int32_t R, void *ws, size_t bytes, vds_rom *out) {
  vds_status st = ready(c);
  if (st != VDS_OK) return st;
  if (!U || !ws || !out || R < 1 || R > kMaxR || R > 3 * c->prob.P)
    return set_err(c, VDS_ERR_ARG, "bad arguments (1 <= R <= min(1024, 3P))");
  if (c->prob.potential != VDS_HOOKEAN)
    return set_err(c, VDS_ERR_ARG, "the reduced spring term is exact only for Hookean springs");
  const RomLayout L = rom_layout(c->prob, R);
  if (bytes < L.total) return set_err(c, VDS_ERR_NOMEM, "reduced-model workspace too small");
  vds_rom r = new (std::nothrow) vds_rom_s();
  if (r == nullptr) return set_err(c, VDS_ERR_NOMEM, "host allocation failed");
  r->ctx = c;
  r->U = U;
  r->R = R;
  r->L = L;
  r->ws = static_cast<char *>(ws);
  auto f = [&](size_t o) { return reinterpret_cast<float *>(r->ws + o); };
  r->Ude = f(L.Ude);
  r->Mbig = f(L.Mbig);
  r->XH = f(L.XH);
  r->I1 = f(L.I1);
  r->XB1 = f(L.XB1);
  r->XB2 = f(L.XB2);
  r->XB = f(L.XB);
  r->Bsw = f(L.Bsw);
  r->Y = f(L.Y);
  r->qt = f(L.qt);
  r->T = f(L.T);
  r->invS = f(L.invS);
  r->part = f(L.part);
  r->red = reinterpret_cast<double *>(r->ws + L.red);
  r->psave = f(L.psave);
  r->pprev = f(L.pprev);
  const int64_t P = c->prob.P;
  hipStream_t s = c->stream;
  k_deinterleave<<<nblk256(3 * (int64_t)R * P), 256, 0, s>>>(U, P, R, r->Ude);
  GemmShape g;
  g.M = 3 * R;
  g.N = 3 * R;
  g.K = P;
  g.A = r->Ude;
  g.lda = P;
  g.B = r->Ude;
  g.ldb = P;
  g.C = r->Mbig;
  g.ldc = 3 * R;
  g.splits = gemm_splits(3 * R, 3 * R, P);
  rom_gemm(r, g, 2.0 * 9.0 * R * R * P);
  k_hydro<<<nblk256((int64_t)R * R), 256, 0, s>>>(r->Mbig, R, c->ep, r->XH, r->I1);
  if (c->ep.bf3) prepare_b3(r);
  st = hip_check(c, hipGetLastError(), "reduced model setup");
  if (st != VDS_OK) {
    delete r;
    return st;
  }
  *out = r;
  return VDS_OK;
}

void vds_rom_destroy(vds_rom r) { delete r; }

vds_status vds_rom_operators(vds_rom r, const float *p, float *XH, float *XB1, float *XB2) {
  if (r == nullptr) return VDS_ERR_ARG;
  vds_ctx c = r->ctx;
  if (!p) return set_err(c, VDS_ERR_ARG, "null p");
  vds_status st = freeze(r, p);
  if (st != VDS_OK) return st;
  const size_t b = sizeof(float) * r->R * r->R;
  if (XH) st = hip_check(c, hipMemcpyAsync(XH, r->XH, b, hipMemcpyDeviceToDevice, c->stream), "copy");
  if (XB1 && st == VDS_OK) st = hip_check(c, hipMemcpyAsync(XB1, r->XB1, b, hipMemcpyDeviceToDevice, c->stream), "copy");
  if (XB2 && st == VDS_OK) st = hip_check(c, hipMemcpyAsync(XB2, r->XB2, b, hipMemcpyDeviceToDevice, c->stream), "copy");
  return st;
}

vds_status vds_rom_stress(vds_rom r, const float *p, double *tau) {
  if (r == nullptr) return VDS_ERR_ARG;
  vds_ctx c = r->ctx;
  if (!p || !tau) return set_err(c, VDS_ERR_ARG, "null argument");
  StressOut out{r, tau};
  vds_status st = out.add(p);
  return st == VDS_OK ? out.finish() : st;
}

size_t vds_rom_exact_workspace_bytes(const vds_problem *prob, int32_t R) {
  if (prob == nullptr || R < 1 || prob->nb < 1) return 0;
  const size_t n = (size_t)prob->nb * R;
  return sizeof(double) * (4 * n * n + 4 * n) + 8 * 256;
}

vds_status vds_rom_run_exact(vds_rom r, float *p, int32_t nsteps, int32_t freeze_every, int32_t adaptive,
                             double energy_tol, double *windows_host, int32_t max_windows, void *ws,
                             size_t ws_bytes, double *tau, vds_rom_window_stats *stats) {
  if (r == nullptr) return VDS_ERR_ARG;
  vds_ctx c = r->ctx;
  if (!p || nsteps < 0 || freeze_every < 1 || !ws || (windows_host == nullptr) != (max_windows <= 0) ||
      (adaptive && !(energy_tol > 0.0)))
    return set_err(c, VDS_ERR_ARG, "bad arguments");
  const int nb = c->prob.nb, R = r->R;
  const int64_t n = (int64_t)nb * R;
  if (ws_bytes < vds_rom_exact_workspace_bytes(&c->prob, R)) return set_err(c, VDS_ERR_NOMEM, "workspace too small");
  hipStream_t s = c->stream;
  // workspace: generator, B = scaled generator, two Horner / squaring buffers, vectors
  auto take = [&, off = size_t(0)](size_t bytes) mutable {
    char *q = static_cast<char *>(ws) + off;
    off += (bytes + 255) / 256 * 256;
    return reinterpret_cast<double *>(q);
  };
  double *Lm = take(sizeof(double) * n * n), *Bm = take(sizeof(double) * n * n);
  double *Tm = take(sizeof(double) * n * n), *Cm = take(sizeof(double) * n * n);
  double *pv = take(sizeof(double) * n), *pw = take(sizeof(double) * n), *cs = take(sizeof(double) * n);
  float *ptrial = reinterpret_cast<float *>(take(sizeof(float) * n));  // trial state of an adaptive window
  rocblas_handle hb = static_cast<rocblas_handle>(blas_handle(c));
  if (hb == nullptr) return VDS_ERR_HIP;
  rocblas_set_pointer_mode(hb, rocblas_pointer_mode_host);
  vds_status st = VDS_OK;
  const unsigned nn_blocks = (unsigned)nblk256(n * n);
  std::vector<double> hcs(n);

  // p <- exp(tw L) p with the generator L frozen at the window start (in Lm)
  auto advance = [&](double tw, float *pout) -> vds_status {
    k_colabs<<<(unsigned)nblk256(n), 256, 0, s>>>(Lm, n, cs);
    vds_status e = hip_check(c, hipMemcpyAsync(hcs.data(), cs, sizeof(double) * n, hipMemcpyDeviceToHost, s), "copy");
    if (e == VDS_OK) e = hip_check(c, hipStreamSynchronize(s), "synchronise");
    if (e != VDS_OK) return e;
    const double norm = tw * *std::max_element(hcs.begin(), hcs.end());
    // scaling: |B|_1 <= 1/2, where the degree-12 Taylor remainder is below 2e-14
    int sq = 0;
    while (norm / std::ldexp(1.0, sq) > 0.5) ++sq;
    k_scale64<<<nn_blocks, 256, 0, s>>>(Lm, tw / std::ldexp(1.0, sq), n * n, Bm);
    k_identity64<<<nn_blocks, 256, 0, s>>>(n, Tm);
    double *T = Tm, *C = Cm;
    const double one = 1.0, zero = 0.0;
    for (int k = 12; k >= 1; --k) {  // Horner: T <- I + B T / k
      k_identity64<<<nn_blocks, 256, 0, s>>>(n, C);
      const double a = 1.0 / k;
      if (rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, (int)n, (int)n, (int)n, &a, Bm, (int)n,
                        T, (int)n, &one, C, (int)n) != rocblas_status_success)
        return set_err(c, VDS_ERR_HIP, "rocblas_dgemm");
      std::swap(T, C);
    }
    for (int i = 0; i < sq; ++i) {  // squaring: T <- T T
      if (rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, (int)n, (int)n, (int)n, &one, T, (int)n,
                        T, (int)n, &zero, C, (int)n) != rocblas_status_success)
        return set_err(c, VDS_ERR_HIP, "rocblas_dgemm");
      std::swap(T, C);
    }
    launch_f32_to_f64(p, pv, n, s);
    if (rocblas_dgemv(hb, rocblas_operation_none, (int)n, (int)n, &one, T, (int)n, pv, 1, &zero, pw, 1) !=
        rocblas_status_success)
      return set_err(c, VDS_ERR_HIP, "rocblas_dgemv");
    k_f64_to_f32<<<(unsigned)nblk256(n), 256, 0, s>>>(pw, n, pout);
    return hip_check(c, hipGetLastError(), "window");
  };
  // F, dissipation, work of the reconstructed state q~ = U p
  auto energy = [&](const float *pp, double *F, double *Dg, double *W) {
    reconstruct_qt(r, pp);
    return vds_energy(c, r->qt, nullptr, F, Dg, W);
  };

  const double dt = c->prob.dt, t_total = nsteps * dt, tw_max = freeze_every * dt;
  double t = 0.0, tw = tw_max, max_gap = 0.0;
  int windows = 0, rejected = 0, recorded = 0, truncated = 0;
  double F0 = 0, D0 = 0, W0 = 0;
  if (adaptive && nsteps > 0) st = energy(p, &F0, &D0, &W0);
  while (st == VDS_OK && t < t_total - 0.5 * dt) {
    tw = std::min(tw, t_total - t);
    st = freeze(r, p);
    if (st != VDS_OK) break;
    k_generator<<<nn_blocks, 256, 0, s>>>(r->XH, r->XB, nb, R, c->ep, Lm);
    double gap = 0.0;
    for (;;) {
      st = advance(tw, adaptive ? ptrial : p);
      if (st != VDS_OK || !adaptive) break;
      double F1, D1, W1;
      st = energy(ptrial, &F1, &D1, &W1);
      if (st != VDS_OK) break;
      const double bound = energy_tol * tw * 0.5 * (std::fabs(W0) + D0 + std::fabs(W1) + D1);
      gap = std::fabs(F1 - F0 - tw * 0.5 * ((W0 - D0) + (W1 - D1)));
      if (gap <= bound || tw <= dt * (1.0 + 1e-9)) {
        if (gap > bound) ++truncated;  // accepted at the smallest window
        st = hip_check(c, hipMemcpyAsync(p, ptrial, sizeof(float) * n, hipMemcpyDeviceToDevice, s), "copy");
        max_gap = std::max(max_gap, bound > 0 ? gap / bound * energy_tol : gap);
        F0 = F1;
        D0 = D1;
        W0 = W1;
        break;
      }
      ++rejected;
      tw = std::max(dt, 0.5 * tw);
    }
    if (st != VDS_OK) break;
    t += tw;
    ++windows;
    if (windows_host && recorded < max_windows) windows_host[recorded++] = tw;
    if (adaptive) {
      const double bound = energy_tol * tw * 0.5 * (std::fabs(W0) + D0);
      if (gap < 0.25 * bound) tw = std::min(2.0 * tw, tw_max);  // grows back, up to the requested interval
    }
  }

  if (st != VDS_OK) return st;
  if (stats) {
    stats->windows = windows;
    stats->rejected = rejected;
    stats->truncated = truncated;
    stats->recorded = recorded;
    stats->t_reached = t;
    stats->max_energy_gap = max_gap;
  }
  st = hip_check(c, hipGetLastError(), "exact windows");
  if (st != VDS_OK) return st;
  if (tau) return vds_rom_stress(r, p, tau);
  return hip_check(c, hipStreamSynchronize(s), "synchronise");
}

}  // extern "C"

namespace {

// n reduced explicit Euler steps of p with the current operators (one launch).
void rom_steps(vds_rom r, float *p, int n) {
  vds_ctx c = r->ctx;
  const int nb = c->prob.nb, R = r->R;
  auto reg = [&](auto q) { launch_steps_reg<decltype(q)::value>(nb, r->XH, r->XB, p, R, n, c->ep, c->stream); };
  if (R <= 16) reg(std::integral_constant<int, 4>{});
  else if (R <= 32) reg(std::integral_constant<int, 8>{});
  else if (R <= 48) reg(std::integral_constant<int, 12>{});
  else if (R <= 64) reg(std::integral_constant<int, 16>{});
  else if (R <= 96) reg(std::integral_constant<int, 24>{});
  else if (R <= 128) reg(std::integral_constant<int, 32>{});
  else if (R <= kRegMaxR) reg(std::integral_constant<int, 48>{});
  else
    k_rom_steps<<<1, 1024, 0, c->stream>>>(r->XH, r->XB, p, nb, R, n, c->ep);
}

// The windows of vds_rom_run / vds_rom_run_midpoint.
// Operators frozen per window of freeze_every reduced steps.  FREEZE_START:
// at the window's start state.  FREEZE_MIDPOINT: at the state half a window
// on, predicted by reduced steps with the start's operators (two operator
// builds per window).  FREEZE_EXTRAPOLATED: at the midpoint state extrapolated
// linearly from this and the previous window's start states (one build per
// window; the first window predicts as FREEZE_MIDPOINT does).  Both midpoint
// forms predict the midpoint state to O(L^2) in the window length L, so the
// frozen operators are O(L^2) from those at the true midpoint.
enum FreezeAt { FREEZE_START = 0, FREEZE_MIDPOINT = 1, FREEZE_EXTRAPOLATED = 2 };

// With output_every >= 1 the stress after steps output_every, 2 output_every,
// ... and after the last step goes to tau[9 i ...]; with output_every == 0 only
// the stress after the last step (tau may be NULL).
vds_status rom_windows(vds_rom r, float *p, int nsteps, int freeze_every, FreezeAt at, double *tau,
                       int output_every = 0) {
  vds_ctx c = r->ctx;
  StressOut out{r, tau};
  // steps [k, k + n) of the run, split at the output steps
  auto steps_out = [&](int k, int n) -> vds_status {
    while (n > 0) {
      const int m = output_every > 0 ? std::min(n, output_every - k % output_every) : n;
      rom_steps(r, p, m);
      k += m;
      n -= m;
      if (tau != nullptr && ((output_every > 0 && k % output_every == 0) || k == nsteps)) {
        vds_status st = out.add(p);
        if (st != VDS_OK) return st;
      }
    }
    return VDS_OK;
  };
  const int64_t np = (int64_t)c->prob.nb * r->R;
  const size_t pbytes = sizeof(float) * (size_t)np;
  auto copy = [&](float *dst, const float *src) {
    return hip_check(c, hipMemcpyAsync(dst, src, pbytes, hipMemcpyDeviceToDevice, c->stream), "copy");
  };
  int nprev = 0;  // length of the previous window (0: none yet)
  for (int s0 = 0; s0 < nsteps; s0 += freeze_every) {
    const int n = std::min(freeze_every, nsteps - s0), half = n / 2;
    vds_status st = VDS_OK;
    if (at == FREEZE_EXTRAPOLATED && nprev > 0 && half > 0) {
      // the midpoint state from the last two window starts; back to the start
      st = copy(r->psave, p);
      if (st != VDS_OK) return st;
      k_extrapolate<<<(unsigned)((np + 255) / 256), 256, 0, c->stream>>>(p, r->pprev, (float)half / (float)nprev, np);
      st = freeze(r, p);
      if (st == VDS_OK) st = copy(p, r->psave);
      if (st != VDS_OK) return st;
    } else {
      st = freeze(r, p);
      if (st != VDS_OK) return st;
      if (at != FREEZE_START && half > 0) {
        // operators at the state half a window on, predicted with the start's
        st = copy(r->psave, p);
        if (st != VDS_OK) return st;
        rom_steps(r, p, half);
        st = freeze(r, p);
        if (st == VDS_OK) st = copy(p, r->psave);
        if (st != VDS_OK) return st;
      }
    }
    if (at == FREEZE_EXTRAPOLATED) {
      st = copy(r->pprev, p);
      if (st != VDS_OK) return st;
      nprev = n;
    }
    vds_status so = steps_out(s0, n);
    if (so != VDS_OK) return so;
  }
  vds_status st = hip_check(c, hipGetLastError(), "reduced steps");
  if (st != VDS_OK) return st;
  if (tau != nullptr && nsteps == 0) st = out.add(p);
  return st == VDS_OK ? out.finish() : st;
}

}  // namespace

extern "C" {

vds_status vds_rom_run(vds_rom r, float *p, int32_t nsteps, int32_t freeze_every, int32_t output_every,
                       double *tau_hist) {
  if (r == nullptr) return VDS_ERR_ARG;
  if (!p || nsteps < 0 || freeze_every < 1 || output_every < 0) return set_err(r->ctx, VDS_ERR_ARG, "bad arguments");
  return rom_windows(r, p, nsteps, freeze_every, FREEZE_START, tau_hist, output_every);
}

vds_status vds_rom_run_midpoint(vds_rom r, float *p, int32_t nsteps, int32_t freeze_every, double *tau) {
  if (r == nullptr) return VDS_ERR_ARG;
  if (!p || nsteps < 0 || freeze_every < 1) return set_err(r->ctx, VDS_ERR_ARG, "bad arguments");
  return rom_windows(r, p, nsteps, freeze_every, FREEZE_MIDPOINT, tau);
}

vds_status vds_rom_run_extrapolated(vds_rom r, float *p, int32_t nsteps, int32_t freeze_every, double *tau) {
  if (r == nullptr) return VDS_ERR_ARG;
  if (!p || nsteps < 0 || freeze_every < 1) return set_err(r->ctx, VDS_ERR_ARG, "bad arguments");
  return rom_windows(r, p, nsteps, freeze_every, FREEZE_EXTRAPOLATED, tau);
}

}  // extern "C"
