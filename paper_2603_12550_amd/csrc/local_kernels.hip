// O(P D) kernels around the pair passes: centring and operand packing, the
// two finalisations (term1 and the pass-B weights; term2, drift and update,
// with the packing of the next state's operands), the implicit-iteration
// control, the FENE domain flag, and FP64 reductions of stress, energy,
// dissipation and work.  All reductions are two-stage (per-block partials in
// a fixed tree, then a fixed-order sum), so results are bitwise reproducible.
#include "bf3.h"
#include "vds_internal.h"

namespace vds {

// Lane movements inside a row of 16 as data-parallel-primitive controls: a few
// cycles each, where a shuffle goes through the LDS crossbar and back (some hundred
// in a chain).  0x100 + i: from lane n + i, 0x110 + i: from lane n - i (zeros from
// outside the row), 0x120 + i: rotated, 0x150 + i: lane i to all.
template <int kCtrl>
__device__ __forceinline__ float row_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kCtrl, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ __forceinline__ double row_move(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// Fixed-order tree sum over the first 256 threads of a block for NS values each
// (every thread of the block calls it).
template <int NS>
__device__ void block_sum(double (&v)[NS], double (*sm)[kRedBlock / 64]) {
  const int t = threadIdx.x;
  if (t < kRedBlock) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      double x = v[s];
      x += row_move<0x128>(x);
      x += row_move<0x124>(x);
      x += row_move<0x122>(x);
      x += row_move<0x121>(x);
      x += __shfl_xor(x, 16);
      x += __shfl_xor(x, 32);
      if ((t & 63) == 0) sm[s][t >> 6] = x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < NS; ++s) v[s] = (sm[s][0] + sm[s][1]) + (sm[s][2] + sm[s][3]);
}

// The dimension known at compile time, so that the per-particle bodies' index
// arithmetic folds (assumed, not stored: a changed copy of the parameters would
// put their arrays, which are indexed per lane, into scratch memory).
template <int D>
__device__ __forceinline__ void assume_dimension(const EvalParams &p) {
  __builtin_assume(p.D == D);
  __builtin_assume(p.nb == D / 3);
  __builtin_assume(p.KK == (D + 5) / 4);
}

__device__ inline float load_weight(const float *w, int64_t I, float uniform_w) {
  return w != nullptr ? w[I] : uniform_w;
}

// Swizzled operand positions (see pair_kernels.hip):
//   QB/KA: element k of the augmented vector of particle I at
//          [((I / 16) * KK + k / 4) * 64 + (I % 16) + 16 (k % 4)]
//   VB:    element n of V_J at [((J / 16) * 64 + ((J % 16) / 4) * 16 + n) * 4 + (J % 4)]
__device__ inline int64_t qk_index(int64_t I, int k, int KK) {
  return ((I >> 4) * KK + (k >> 2)) * 64 + (I & 15) + 16 * (k & 3);
}
__device__ inline int64_t v_index(int64_t J, int n) {
  return ((J >> 4) * 64 + ((J & 15) >> 2) * 16 + n) * 4 + (J & 3);
}
//   V as FP16 halves (VDS_PAIR_MFMA_F16X2): the high half of element n of V_J
//          at [((J / 32) * 64 + n + 16 ((J % 16) / 4)) * 8 + 4 ((J / 16) % 2) + J % 4]
//          and the low half Ppad * 16 halves further on.
__device__ inline int64_t vh_index(int64_t J, int n) {
  return ((J >> 5) * 64 + n + 16 * ((J & 15) >> 2)) * 8 + 4 * ((J >> 4) & 1) + (J & 3);
}
//   QH/KH: FP16 distance slot s (0 <= s < 32 KQ) of particle I at
//          [(((I / 16) * KQ + s / 32) * 64 + I % 16 + 16 ((s % 32) / 8)) * 8 + s % 8]
__device__ inline int64_t dh_index(int64_t I, int s, int KQ) {
  return ((((I >> 4) * KQ + (s >> 5)) * 64 + (I & 15) + 16 * ((s & 31) >> 3)) << 3) + (s & 7);
}
// Row-side and column-side values of FP16 distance slot s, given the component
// y_k = cs x_k for k = s / 3 and the norm term -kappa |x|^2 (see pair_kernels.hip).
__device__ inline void dh_slot(const EvalParams &p, int s, float yk, float nterm, _Float16 &qv, _Float16 &kv) {
  const _Float16 z = (_Float16)0.f;
  qv = z;
  kv = z;
  if (s < 3 * p.D) {
    const int ty = s % 3;
    const _Float16 hi = (_Float16)yk;
    const _Float16 lo = (_Float16)(yk - (float)hi);
    qv = ty == 2 ? lo : hi;
    kv = ty == 1 ? lo : hi;
  } else if (s < 3 * p.D + 2) {
    const float v = nterm * 0.0625f;
    const _Float16 hi = (_Float16)v;
    qv = (_Float16)16.f;
    kv = s == 3 * p.D ? hi : (_Float16)(v - (float)hi);
  }
}
__device__ inline void store_v(const EvalParams &p, float *V, int64_t J, int n, float v) {
  if (p.vhalf) {
    _Float16 *h = reinterpret_cast<_Float16 *>(V);
    const _Float16 hi = (_Float16)v;
    const int64_t i = vh_index(J, n);
    h[i] = hi;
    h[i + p.Ppad * 16] = (_Float16)(v - (float)hi);
  } else {
    V[v_index(J, n)] = v;
  }
}

// Lane n of particle J writes element n of V_J = (wx, w) (0 past the
// particles) in the format of the pair implementation; w_x is this lane's
// weighted coordinate or weight.
__device__ inline void store_v3(const EvalParams &p, float *V, int64_t J, int n, double v) {
  if (n > p.D) return;
  uint16_t *V3 = reinterpret_cast<uint16_t *>(V);
  const int NT = bf3_tiles(p.D);
  const Bf3 s = split_bf3(v);
  V3[v3_index(J, n, NT)] = s.h;
  V3[v3_index(J, p.D + 1 + n, NT)] = s.m;
  V3[v3_index(J, 2 * (p.D + 1) + n, NT)] = s.l;
}

// Partial sums of w_I x_I (FP64) per block of 256 particles, for the weighted
// centring, and in slot 15 the block's largest weight: lane n of group r of 16
// takes component n of particles r, r + 16, ... (all loads in flight), then the
// sixteen groups in order.
// Bodies take the block index `lb` within the problem (one ensemble) so that
// the batched step can run them per ensemble.
__device__ void mean_partials_body(const EvalParams &p, int64_t lb, const float *__restrict__ q,
                                   const float *__restrict__ w, double *__restrict__ meanp) {
  __shared__ double part[16][17];
  const int r = threadIdx.x >> 4, n = threadIdx.x & 15;
  constexpr int N = kRedBlock / 16;
  // (past the particles or the components: the last one's values, not counted)
  const float *src = q + (int64_t)(min(n, p.D - 1) / 3) * p.P * 3 + min(n, p.D - 1) % 3;
  float x[N], wi[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t I = min(lb * kRedBlock + 16 * i + r, p.P - 1);
    x[i] = src[3 * I];
    wi[i] = load_weight(w, I, p.uniform_w);
  }
  double v = 0.0;
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool real = lb * kRedBlock + 16 * i + r < p.P;
    v += real && n < p.D ? (double)wi[i] * (double)x[i] : 0.0;
    m = fmaxf(m, real ? wi[i] : 0.f);
  }
  part[r][n] = n == 15 ? (double)m : v;
  __syncthreads();
  if (threadIdx.x < 16) {
    double o = part[0][n];
    for (int i = 1; i < 16; ++i) o = n == 15 ? fmax(o, part[i][n]) : o + part[i][n];
    meanp[lb * 16 + n] = o;
  }
}

__global__ __launch_bounds__(kRedBlock) void k_mean_partials(EvalParams p, const float *__restrict__ q,
                                                             const float *__restrict__ w, double *__restrict__ meanp,
                                                             const int *done, Ctrl *begin) {
  if (done != nullptr && *done) return;
  if (begin != nullptr) {
    // opens a queued implicit step (no other block of this launch reads
    // the fields that block 0 clears)
    if (begin->halted) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      begin->done = 0;
      begin->conv_iter = -1;
      begin->checked = 0;
    }
  }
  mean_partials_body(p, blockIdx.x, q, w, meanp);
}

// Sum of the centring partials (mean_sh[0..D)) and the largest weight
// (mean_sh[15]), computed identically by every block: thread (c, j) = (t % 16,
// t / 16) folds the partials of blocks j, j + 16, ... of slot c, then one
// thread per slot combines the sixteen results in order.
__device__ void load_mean(const EvalParams &p, const double *meanp, int nmeanp, float *mean_sh) {
  __shared__ double part[16][17];
  const int c = threadIdx.x & 15, j = threadIdx.x >> 4;  // blockDim.x == 256
  double v = 0.0;
  const int nj = strided_count(j, nmeanp, 16);
  if (c == 15) v = strided_max(meanp + (int64_t)j * 16 + 15, nj, 256, 0.0);
  else if (c < p.D) v = ordered_sum<double>(meanp + (int64_t)j * 16 + c, nj, 256);
  part[c][j] = v;
  __syncthreads();
  if (threadIdx.x < 16 && (threadIdx.x < p.D || threadIdx.x == 15)) {
    double r = 0.0;
    for (int i = 0; i < 16; ++i) r = threadIdx.x == 15 ? fmax(r, part[threadIdx.x][i]) : r + part[threadIdx.x][i];
    mean_sh[threadIdx.x] = (float)r;
  }
  __syncthreads();
}

// The per-particle kernels below use 16 lanes per particle: lane n owns
// component n of the configuration vector (n < D <= 15), so loads and stores
// of a wave cover four particles' contiguous records and P/16 blocks fill the
// chip.  Cross-component terms (norms, the 3x3 flow, bond neighbours) are
// 16-wide shuffles.
__device__ inline int64_t group_particle(int64_t lb) { return (lb * kRedBlock + threadIdx.x) >> 4; }
__device__ inline int group_lane() { return threadIdx.x & 15; }
__device__ inline float gshfl(float v, int n) { return __shfl(v, n, 16); }
// Lane D of the row to all its lanes.
__device__ __forceinline__ double row_lane_d(int D, double v) {
  switch (D) {
    case 3: return row_move<0x150 + 3>(v);
    case 6: return row_move<0x150 + 6>(v);
    case 9: return row_move<0x150 + 9>(v);
    case 12: return row_move<0x150 + 12>(v);
    default: return row_move<0x150 + 15>(v);
  }
}
// The three components of this lane's bond (al = lane % 3).
struct Bond {
  float c0, c1, c2;
};
__device__ __forceinline__ Bond row_bond(float v, int al) {
  const float l1 = row_move<0x111>(v), l2 = row_move<0x112>(v), r1 = row_move<0x101>(v), r2 = row_move<0x102>(v);
  return Bond{al == 0 ? v : al == 1 ? l1 : l2, al == 0 ? r1 : al == 1 ? v : l1, al == 0 ? r2 : al == 1 ? r1 : v};
}
// The largest value of the wave, in every lane.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_move<0x128>(v));
  v = fmaxf(v, row_move<0x124>(v));
  v = fmaxf(v, row_move<0x122>(v));
  v = fmaxf(v, row_move<0x121>(v));
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}
__device__ inline float gsum(float v) {
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 16);
  return v;
}

// Convergence test of fixed-point iteration chk.iter from the combine kernel's
// block maxima of |dx| and |x|: max|dx| <= rtol * max(1, max|x|).  Every block
// of the calling launch evaluates it (the maxima are the previous kernel's
// output, so the launch boundary orders them) and gets the same answer;
// *resid receives max|dx|.
__device__ bool picard_converged(const PicardCheck &chk, const float *__restrict__ blockmax, int nblk,
                                 float *resid) {
  __shared__ float sr[kRedBlock / 64], sx[kRedBlock / 64];
  __shared__ int conv;
  __shared__ float rr;
  // (blocks of more threads: the first 256 take the maxima)
  const int nt = threadIdx.x < kRedBlock ? strided_count(threadIdx.x, nblk, kRedBlock) : 0;
  float r = strided_max(blockmax + 2 * threadIdx.x, nt, 2 * kRedBlock, 0.f);
  float x = strided_max(blockmax + 2 * threadIdx.x + 1, nt, 2 * kRedBlock, 0.f);
  r = wave_max(r);
  x = wave_max(x);
  if ((threadIdx.x & 63) == 0 && threadIdx.x < kRedBlock) {
    sr[threadIdx.x >> 6] = r;
    sx[threadIdx.x >> 6] = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kRedBlock / 64; ++i) {
      r = fmaxf(r, sr[i]);
      x = fmaxf(x, sx[i]);
    }
    rr = r;
    conv = r <= chk.rtol * fmaxf(1.f, x) ? 1 : 0;
  }
  __syncthreads();
  *resid = rr;
  return conv != 0;
}

// Column operand K3 of particle I from its centred coordinate x (lane n;
// zeros past the particles, when not real): see vds_internal.h.  kPoint: x is a point of
// a density, whose norm stays an FP32 number: at 1e19 h and further the density is zero.
template <bool kPoint = false>
__device__ inline void store_k3(const EvalParams &p, bool real, uint32_t *__restrict__ K3, int64_t I, int n, float x) {
  const int NQ = bf3_slices(p.D);
  const Bf3 y = split_bf3(n < p.D ? p.cs * (double)x : 0.0);
  const double ys = bf16_value(y.h) + bf16_value(y.m) + bf16_value(y.l);
  double nrm = ys * ys;
  nrm += row_move<0x128>(nrm);
  nrm += row_move<0x124>(nrm);
  nrm += row_move<0x122>(nrm);
  nrm += row_move<0x121>(nrm);
  // lane n holds dwords 3n .. 3n + 2: component n, the norm (n = D) or zeros
  uint32_t d[3] = {0u, 0u, 0u};
  if (real && n < p.D) {
    d[0] = d[1] = (uint32_t)y.h | ((uint32_t)y.m << 16);
    d[2] = (uint32_t)y.h | ((uint32_t)y.l << 16);
  } else if (real && n == p.D) {
    const Bf3 r = split_bf3(kPoint ? fmax(-0.5 * nrm, -1e38) : -0.5 * nrm);
    d[0] = (uint32_t)r.h | ((uint32_t)r.m << 16);
    d[1] = (uint32_t)r.l | 0x3f800000u;
    d[2] = 0x3f803f80u;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (3 * n + j < 16 * NQ) K3[bf3_index(I, 3 * n + j, NQ)] = d[j];
}

// Centre, pack Q/K operands and the pass-A V operand (weights w; over their
// maximum, which goes to *wscale, when V is written in FP16 halves).
// Lane n of particle I's raw coordinate (0 past the particles or D).
__device__ inline float prep_coord(const EvalParams &p, const float *__restrict__ q, int64_t I, int n) {
  return (I < p.P && n < p.D) ? q[((int64_t)(n / 3) * p.P + I) * 3 + (n % 3)] : 0.f;
}

// Operand packing of particle I (lane n) from its centred coordinate x and
// weight wi; mean_sh[15] is the largest weight.
__device__ void prep_write(const EvalParams &p, int64_t I, int n, float x, float wi, const float *mean_sh,
                           float *__restrict__ xc, float *__restrict__ wv, float *__restrict__ QB,
                           float *__restrict__ KA, float *__restrict__ VA, F16Operands f16) {
  const bool real = I < p.P;
  const float nrm = gsum(x * x);
  if (n == 0) wv[I] = wi;
  if (n < p.D) xc[I * p.D + n] = x;
  // the FP32 distance operands are read only by the FP32-distance pair forms
  if (p.bf3) store_k3(p, real, reinterpret_cast<uint32_t *>(f16.QH), I, n, x);
  for (int k = n; k < ((p.qhalf || p.bf3) ? 0 : 4 * p.KK); k += 16) {
    float qa = 0.f, ka = 0.f;
    if (real) {
      if (k < p.D) {
        qa = x;
        ka = 2.f * p.kappa * x;
      } else if (k == p.D) {
        qa = -p.kappa * nrm;
        ka = 1.f;
      } else if (k == p.D + 1) {
        qa = 1.f;
        ka = -p.kappa * nrm;
      }
    }
    QB[qk_index(I, k, p.KK)] = qa;
    KA[qk_index(I, k, p.KK)] = ka;
  }
  if (p.qhalf) {
    // slots 2 m and 2 m + 1 are adjacent: one 32-bit store each for QH and KH
    uint32_t *qh = reinterpret_cast<uint32_t *>(f16.QH);
    uint32_t *kh = reinterpret_cast<uint32_t *>(f16.KH);
    const float y = p.cs * x;
    const float nt = real ? -p.kappa * nrm : 0.f;
    for (int sp = n; sp < 16 * p.KQ; sp += 16) {  // the same trip count on every lane
      const int s0 = 2 * sp, k0 = s0 / 3, k1 = (s0 + 1) / 3;
      const float y0 = gshfl(y, k0 < 16 ? k0 : 0), y1 = gshfl(y, k1 < 16 ? k1 : 0);
      _Float16 q0, c0, q1, c1;
      dh_slot(p, s0, y0, nt, q0, c0);
      dh_slot(p, s0 + 1, y1, nt, q1, c1);
      const int64_t di = dh_index(I, s0, p.KQ) >> 1;
      qh[di] = (uint32_t)__builtin_bit_cast(uint16_t, q0) | ((uint32_t)__builtin_bit_cast(uint16_t, q1) << 16);
      kh[di] = (uint32_t)__builtin_bit_cast(uint16_t, c0) | ((uint32_t)__builtin_bit_cast(uint16_t, c1) << 16);
    }
    if (n == 0) f16.RN[I] = nt;
  }
  if (p.bf3) {
    store_v3(p, VA, I, n, n < p.D ? (double)wi * (double)x : (double)wi);
    return;
  }
  const float wn = p.vhalf ? (real ? wi / mean_sh[15] : 0.f) : wi;
  float v = 0.f;
  if (n < p.D) v = wn * x;
  else if (n == p.D) v = wn;
  store_v(p, VA, I, n, v);
}

// kGroups groups of 16 particles per block.
template <int kGroups>
__device__ void prep_body(const EvalParams &p, int64_t lb, const float *__restrict__ q, const float *__restrict__ w,
                          const double *__restrict__ meanp, int nmeanp, float *__restrict__ xc,
                          float *__restrict__ wv, float *__restrict__ QB, float *__restrict__ KA,
                          float *__restrict__ VA, float *__restrict__ wscale, F16Operands f16,
                          float *__restrict__ cmean = nullptr) {
  __shared__ float mean_sh[16];
  const int n = group_lane();
  float x[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) x[g] = prep_coord(p, q, group_particle(lb * kGroups + g), n);
  load_mean(p, meanp, nmeanp, mean_sh);
  if (p.vhalf && wscale != nullptr && lb == 0 && threadIdx.x == 0) *wscale = mean_sh[15];
  if (cmean != nullptr && lb == 0 && threadIdx.x < 16) cmean[threadIdx.x] = mean_sh[threadIdx.x];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int64_t I = group_particle(lb * kGroups + g);
    if (I >= p.Ppad) return;
    const float wi = I < p.P ? load_weight(w, I, p.uniform_w) : 0.f;
    prep_write(p, I, n, I < p.P && n < p.D ? x[g] - mean_sh[n] : 0.f, wi, mean_sh, xc, wv, QB, KA, VA, f16);
  }
}

template <int D>
__global__ __launch_bounds__(kRedBlock) void k_prep(EvalParams p, const float *__restrict__ q,
                                                    const float *__restrict__ w, const double *__restrict__ meanp,
                                                    int nmeanp, float *__restrict__ xc, float *__restrict__ wv,
                                                    float *__restrict__ QB, float *__restrict__ KA,
                                                    float *__restrict__ VA, float *__restrict__ wscale,
                                                    F16Operands f16, const int *done, float *__restrict__ cmean,
                                                    Ctrl *begin) {
  if (begin != nullptr) {
    // opens a queued implicit step (no other block of this launch reads the
    // fields that block 0 clears)
    if (begin->halted) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      begin->done = 0;
      begin->conv_iter = -1;
      begin->checked = 0;
    }
  } else if (done != nullptr && *done) {
    return;
  }
  assume_dimension<D>(p);
  prep_body<1>(p, blockIdx.x, q, w, meanp, nmeanp, xc, wv, QB, KA, VA, wscale, f16, cmean);
}

// Component n of row I summed over its partial-sum slots in slot order, in FP64.
__device__ inline double sum_splits(const EvalParams &p, const float *__restrict__ partial, const SplitMap &splits,
                                    int64_t I, int n) {
  return ordered_sum<double>(partial + I * splits.width + n, splits.count(I), p.Ppad * splits.width);
}
// The same for an ensemble of a batch.  (FP64 slots of column ranges: rounded once, as
// the slot of a whole ensemble is.)
__device__ inline double sum_splits(const EvalParams &p, const float *__restrict__ partial, const EnsDesc &d,
                                    int64_t I, int n) {
  const float *part = partial + d.part_off;
  if (d.splits == 1) return (double)part[I * 16 + n];
  const int W = p.D + 1;
  return (double)(float)ordered_sum<double>(reinterpret_cast<const double *>(part) + I * W + n, d.splits, p.Ppad * W);
}

// Pass-A finalisation: S_I = w_I + sum_{J != I} w_J e_IJ,
// term1_I = -(1/h^2) sum_J w_J e_IJ (x_I - x_J) / S_I, and the pass-B operand
// with weights w_J / S_J.  o is lane n's sum of particle I: the difference sum's
// component n < D, the weighted kernel sum at n = D.
// x and w are lane n's centred coordinate and the particle's weight, loaded
// ahead of the sums.
__device__ void finalize_a_row(const EvalParams &p, int64_t I, int n, double o, float x, float w,
                               float *__restrict__ S, float *__restrict__ t1, float *__restrict__ VB) {
  const bool real = I < p.P;  // padding columns carry zero weight in pass B too
  const double wI = (double)w;
  const double Si = row_lane_d(p.D, o) + wI;  // the pass left out the self term w_I e_II = w_I
  const double rS = 1.0 / Si, wd = real ? wI * rS : 0.0;
  const float wb = (float)wd;
  float v = 0.f;
  if (n < p.D) {
    if (real) t1[I * p.D + n] = (float)(-(double)p.inv_h2 * o * rS);
    v = wb * x;
  } else if (n == p.D) {
    if (real) S[I] = (float)Si;
    v = wb;
  }
  if (p.bf3) store_v3(p, VB, I, n, !real ? 0.0 : n < p.D ? wd * (double)x : wd);
  else store_v(p, VB, I, n, real ? v : 0.f);  // wb <= 1, so the FP16 form needs no normalisation
}

// Slots: the SplitMap of a single state, or the EnsDesc of an ensemble.
template <class Slots>
__device__ void finalize_a_body(const EvalParams &p, int64_t lb, const float *__restrict__ partial, const Slots &splits,
                                const float *__restrict__ xc, const float *__restrict__ wv, float *__restrict__ S,
                                float *__restrict__ t1, float *__restrict__ VB) {
  const int64_t I = group_particle(lb);
  const int n = group_lane();
  if (I >= p.Ppad) return;
  const float x = n < p.D ? xc[I * p.D + n] : 0.f, w = wv[I];
  const double o = I < p.P && n <= p.D ? sum_splits(p, partial, splits, I, n) : 0.0;
  finalize_a_row(p, I, n, o, x, w, S, t1, VB);
}

template <int D>
__global__ __launch_bounds__(kRedBlock) void k_finalize_a(EvalParams p, const float *__restrict__ partial, SplitMap splits,
                                                          const float *__restrict__ xc, const float *__restrict__ wv,
                                                          float *__restrict__ S, float *__restrict__ t1,
                                                          float *__restrict__ VB, const int *__restrict__ done) {
  if (done != nullptr && *done) return;
  assume_dimension<D>(p);
  finalize_a_body(p, blockIdx.x, partial, splits, xc, wv, S, t1, VB);
}

// Pass-B finalisation and everything local: term2, b = term1 + term2,
// g = kT b + grad Psi, u = -(1/zeta)(A (x) I) g, flow G q, and by mode the
// terms, the velocity, an explicit update or a fixed-point update (whose flow
// term is taken at the step's start state qs).  With `obs` it also
// accumulates F_h, dissipation, work and stress in FP64.  With pack.VA set
// (fixed-point or explicit mode) it packs the new iterate's or state's pair
// operands as the prep kernel would: the same lanes hold the same coordinates
// there.
// Lane n's inputs of particle I beside the pass-B sum, loaded ahead of it.
struct CombineIn {
  float t1, q, qs, w, S;
};
__device__ inline CombineIn combine_load(const EvalParams &p, int64_t lb, int mode, int obs, bool act,
                                         const float *__restrict__ t1, const float *__restrict__ S, const float *wv,
                                         const float *qin, const float *__restrict__ qs) {
  const int64_t I = group_particle(lb);
  const int n = group_lane();
  const bool real = act && I < p.P, comp = real && n < p.D;
  const int64_t idx = ((int64_t)(n / 3) * p.P + I) * 3 + n % 3;
  CombineIn c;
  c.t1 = comp ? t1[I * p.D + n] : 0.f;
  c.q = comp && mode != MODE_TERMS ? qin[idx] : 0.f;
  c.qs = comp && mode == MODE_PICARD ? qs[idx] : 0.f;
  c.w = real ? wv[I] : 0.f;
  c.S = real && obs ? S[I] : 1.f;
  return c;
}

// The block's first 256 threads hold its particles (act), all threads call it;
// o is lane n's pass-B sum of particle I, as in finalize_a_row, and in its other
// inputs (combine_load).
__device__ void combine_rows(const EvalParams &p, int64_t lb, int mode, int obs, bool act, double o,
                             const CombineIn &in, float *out, float *out2, double *__restrict__ redp,
                             float *__restrict__ blockmax, const PackOps &pack, int *fene_out) {
  __shared__ double sm[12][kRedBlock / 64];
  const int64_t I = group_particle(lb);
  const int n = group_lane();
  const bool real = act && I < p.P;   // uniform over the 16 lanes of a particle
  const bool comp = real && n < p.D;  // this lane owns a component
  const int k = n / 3, al = n % 3;
  const int64_t idx = ((int64_t)k * p.P + I) * 3 + al;
  double red[12];
#pragma unroll
  for (int s = 0; s < 12; ++s) red[s] = 0.0;
  float resid = 0.f, xmax = 0.f, xnew = 0.f;

  const float t2v = comp ? (float)(-(double)p.inv_h2 * o) : 0.f;
  const float t1v = in.t1;
  const float b = t1v + t2v;
  if (mode == MODE_TERMS) {
    if (comp) {
      out[idx] = t1v;
      out2[idx] = t2v;
    }
  } else {
    const float qv = in.q;
    // the three components of this lane's bond
    const auto [q0, q1, q2] = row_bond(qv, al);
    const float r2 = q0 * q0 + q1 * q1 + q2 * q2;
    // this lane's spring constant and row of G, by selects of uniform values: an
    // index that differs per lane would read the kernel arguments as vector loads
    float H = 0.f, G0 = p.G[6], G1 = p.G[7], G2 = p.G[8];
#pragma unroll
    for (int j = 0; j < kMaxNb; ++j) H = j == k && j < p.nb ? p.H[j] : H;
    if (al == 0) G0 = p.G[0], G1 = p.G[1], G2 = p.G[2];
    if (al == 1) G0 = p.G[3], G1 = p.G[4], G2 = p.G[5];
    float fac = H, psi = 0.f;
    if (p.potential == VDS_FENE) {
      const float sb = 1.f - r2 / p.b_max;
      // outside the domain (or not finite): every such lane stores the same flag
      if (fene_out != nullptr && comp && !(sb > 0.f)) *fene_out = 1;
      fac = H / sb;
      psi = comp && al == 0 ? -0.5f * H * p.b_max * logf(sb) : 0.f;
    } else {
      psi = comp && al == 0 ? 0.5f * H * r2 : 0.f;
    }
    const float gp = comp ? fac * qv : 0.f;
    const float g = comp ? p.kT * b + gp : 0.f;
    // (A (x) I) g with A = tridiag(-1, 2, -1) over bonds
    const float gm = row_move<0x113>(g), gpl = row_move<0x103>(g);
    float Ag = 2.f * g;
    if (k > 0) Ag -= gm;
    if (k + 1 < p.nb) Ag -= gpl;
    const float flow = G0 * q0 + G1 * q1 + G2 * q2;
    float qstart = 0.f, flow0 = 0.f;
    if (mode == MODE_PICARD) {
      qstart = in.qs;
      const auto [s0, s1, s2] = row_bond(qstart, al);
      flow0 = G0 * s0 + G1 * s1 + G2 * s2;
    }
    const float u = -p.inv_zeta * Ag;
    if (comp) {
      if (mode == MODE_VELOCITY) {
        out[idx] = flow + u;
      } else if (mode == MODE_EXPLICIT) {
        xnew = qv + p.dt * (flow + u);
        out[idx] = xnew;
      } else if (mode == MODE_PICARD) {
        const float xn = qstart + p.dt * (flow0 + u);
        out[idx] = xn;
        resid = fabsf(xn - qv);
        xmax = fabsf(xn);
        xnew = xn;
      }
    }
    if (act && (mode == MODE_PICARD || mode == MODE_EXPLICIT) && pack.VA != nullptr) {
      // the prep kernel's work for the new iterate or state: wv already holds
      // the weights (zero past the particles)
      const float x = comp ? xnew - pack.cmean[n] : 0.f;
      const float wi = in.w;
      prep_write(p, I, n, x, wi, pack.cmean, pack.xc, pack.wv, pack.QB, pack.KA, pack.VA, pack.f16);
    }
    if (obs) {
      // stress column beta needs grad Psi of this bond's component beta
      const auto [gp0, gp1, gp2] = row_bond(gp, al);
      if (comp) {
        const double wi = (double)in.w;
        red[RED_DISS] = wi * (double)g * (double)Ag * (double)p.inv_zeta;
        red[RED_WORK] = wi * (double)g * (double)flow;
        red[RED_TAU + 3 * al + 0] = (double)p.n * wi * (double)qv * (double)gp0;
        red[RED_TAU + 3 * al + 1] = (double)p.n * wi * (double)qv * (double)gp1;
        red[RED_TAU + 3 * al + 2] = (double)p.n * wi * (double)qv * (double)gp2;
        red[RED_F] = wi * (double)psi;
        if (n == 0) red[RED_F] += wi * (double)p.kT * (log((double)in.S) - (double)p.log_norm);
      }
    }
  }
  if (obs) {
    block_sum<12>(red, sm);
    if (threadIdx.x < 12 && lb * 16 < p.P) redp[lb * 16 + threadIdx.x] = red[threadIdx.x];
  }
  if (mode == MODE_PICARD) {
    // block maxima of |dx| and |x| into per-block slots; the check kernel
    // takes the max over blocks (no contended atomics)
    __shared__ float smax[2][kRedBlock / 64];
    resid = wave_max(resid);
    xmax = wave_max(xmax);
    if (act && (threadIdx.x & 63) == 0) {
      smax[0][threadIdx.x >> 6] = resid;
      smax[1][threadIdx.x >> 6] = xmax;
    }
    __syncthreads();
    if (threadIdx.x == 0 && lb * 16 < p.P) {
      float r = 0.f, x = 0.f;
      for (int i = 0; i < kRedBlock / 64; ++i) {
        r = fmaxf(r, smax[0][i]);
        x = fmaxf(x, smax[1][i]);
      }
      blockmax[2 * lb] = r;
      blockmax[2 * lb + 1] = x;
    }
  }
}

template <class Slots>
__device__ void combine_body(const EvalParams &p, int64_t lb, int mode, int obs, const float *__restrict__ partial,
                             const Slots &splits, const float *__restrict__ t1, const float *__restrict__ S,
                             const float *wv, const float *qin, const float *__restrict__ qs, float *out, float *out2,
                             double *__restrict__ redp, float *__restrict__ blockmax, const PackOps &pack,
                             int *fene_out) {
  const int64_t I = group_particle(lb);
  const CombineIn in = combine_load(p, lb, mode, obs, true, t1, S, wv, qin, qs);
  const double o = I < p.P && group_lane() < p.D ? sum_splits(p, partial, splits, I, group_lane()) : 0.0;
  combine_rows(p, lb, mode, obs, true, o, in, out, out2, redp, blockmax, pack, fene_out);
}

template <int D>
__global__ __launch_bounds__(kRedBlock) void k_combine(EvalParams p, int mode, int obs,
                                                       const float *__restrict__ partial, SplitMap splits,
                                                       const float *xc, const float *__restrict__ t1,
                                                       const float *__restrict__ S, const float *wv,
                                                       const float *qin, const float *__restrict__ qs,
                                                       float *out, float *out2, double *__restrict__ redp,
                                                       float *__restrict__ blockmax, const int *__restrict__ done,
                                                       PackOps pack, int *fene_out) {
  if (done != nullptr && *done) return;
  assume_dimension<D>(p);
  combine_body(p, blockIdx.x, mode, obs, partial, splits, t1, S, wv, qin, qs, out, out2, redp, blockmax, pack,
               fene_out);
}

// Sum over blocks of the FP64 block partials, slot by slot: wave s takes slot s,
// lane l folds blocks l, l + 64, ... in order, then a fixed butterfly over the
// wave (deterministic; the latency is that of nblk / 64 loads, not nblk).
__global__ __launch_bounds__(1024) void k_reduce_final(const double *__restrict__ redp, int nblk, int nslots,
                                                       double *__restrict__ out, const Ctrl *__restrict__ ctrl,
                                                       Ctrl *__restrict__ ctrl_out) {
  const int s = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (ctrl_out != nullptr && threadIdx.x == 1023) *ctrl_out = *ctrl;
  if (s >= nslots) return;
  double a0 = 0.0, a1 = 0.0;
  int b = lane;
  for (; b + 64 < nblk; b += 128) {
    a0 += redp[(int64_t)b * 16 + s];
    a1 += redp[(int64_t)(b + 64) * 16 + s];
  }
  if (b < nblk) a0 += redp[(int64_t)b * 16 + s];
  double acc = a0 + a1;
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) out[s] = acc;
}

// Stand-alone convergence test: between the fixed-point iterations of a
// queued step (after a combine that packed the next iterate) and in the
// host-driven iterations.
__global__ __launch_bounds__(kRedBlock) void k_picard_check(PicardCheck chk, const float *__restrict__ blockmax,
                                                            int nblk_chk) {
  Ctrl *ctrl = chk.ctrl;
  // the flag and the block maxima are loaded together (one block: nothing
  // else writes the flag during this launch)
  const int done = ctrl->done;
  float r;
  const bool conv = picard_converged(chk, blockmax, nblk_chk, &r);
  if (done || threadIdx.x != 0) return;
  ctrl->last_resid = r;
  ctrl->checked = chk.iter + 1;
  if (conv) {
    ctrl->conv_iter = chk.iter;
    ctrl->done = 1;
  }
}

__global__ void k_ctrl_reset(Ctrl *ctrl) {
  if (threadIdx.x != 0) return;
  ctrl->done = 0;
  ctrl->conv_iter = -1;
  ctrl->last_resid = 0.f;
  ctrl->checked = 0;
  ctrl->halted = 0;
  ctrl->steps_done = 0;
  ctrl->last_iters = 0;
  ctrl->total_iters = 0;
  ctrl->fene_out = 0;
}

// End of a queued implicit step (see launch_step_end), one thread per
// particle.  Only block 0 writes *ctrl.  If another block sees its `halted` or
// `done` of this launch, the step did not converge (conv_iter is still -1
// then) and it returns as block 0 does.
__global__ __launch_bounds__(kRedBlock) void k_step_end(EvalParams p, Ctrl *ctrl, PicardCheck chk,
                                                        const float *__restrict__ blockmax, int nblk_chk,
                                                        const float *__restrict__ xb0, const float *__restrict__ xb1,
                                                        float *__restrict__ q, float *__restrict__ xpred,
                                                        const float *__restrict__ w, double *__restrict__ meanp) {
  // block 0 may set `halted` and `done` during this launch: one read per
  // block keeps the block's waves together
  __shared__ int st[3];
  if (threadIdx.x == 0) {
    st[0] = ctrl->halted;
    st[1] = ctrl->done;
    st[2] = ctrl->conv_iter;
  }
  // the copy's loads for the tested iteration (the usual outcome) go out
  // before the test, so that their latency overlaps it
  const int64_t I = (int64_t)blockIdx.x * kRedBlock + threadIdx.x;
  const bool real = I < p.P;
  float qn[kMaxD], qo[kMaxD];
  auto at = [&](int a) { return ((int64_t)(a / 3) * p.P + I) * 3 + a % 3; };
  const float *src = (chk.iter & 1) ? xb1 : xb0;
#pragma unroll
  for (int a = 0; a < kMaxD; ++a) {
    qn[a] = 0.f;
    qo[a] = 0.f;
    if (real && a < p.D) {
      qn[a] = src[at(a)];
      if (xpred != nullptr) qo[a] = q[at(a)];
    }
  }
  __syncthreads();
  if (st[0]) return;
  int it;
  if (st[1]) {
    it = st[2];  // converged at an earlier test of this step
    if (it < 0) return;
    if ((it ^ chk.iter) & 1) {
      const float *alt = (it & 1) ? xb1 : xb0;
#pragma unroll
      for (int a = 0; a < kMaxD; ++a)
        if (real && a < p.D) qn[a] = alt[at(a)];
    }
  } else {
    float r;
    const bool conv = picard_converged(chk, blockmax, nblk_chk, &r);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctrl->last_resid = r;
      ctrl->checked = chk.iter + 1;
      if (!conv) {
        ctrl->halted = 1;
        ctrl->done = 1;
      }
    }
    if (!conv) return;
    it = chk.iter;
  }
#pragma unroll
  for (int a = 0; a < kMaxD; ++a) {
    if (real && a < p.D) {
      if (xpred != nullptr) xpred[at(a)] = 2.f * qn[a] - qo[a];
      q[at(a)] = qn[a];
    }
  }
  // the next step's centring partials from the new state, as k_mean_partials
  // computes them (of the block's own particles, written above)
  if (meanp != nullptr) {
    __syncthreads();
    mean_partials_body(p, blockIdx.x, q, w, meanp);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->steps_done += 1;
    ctrl->last_iters = it + 1;
    ctrl->total_iters += it + 1;
  }
}

__device__ void stress_body(const EvalParams &p, int64_t lb, const float *__restrict__ q, const float *__restrict__ w,
                            double *__restrict__ redp) {
  __shared__ double sm[9][kRedBlock / 64];
  const int64_t I = lb * kRedBlock + threadIdx.x;
  double t[9];
#pragma unroll
  for (int s = 0; s < 9; ++s) t[s] = 0.0;
  if (I < p.P) {
    const double wi = (double)load_weight(w, I, p.uniform_w) * (double)p.n;
    for (int k = 0; k < p.nb; ++k) {
      const float *qk = q + ((int64_t)k * p.P + I) * 3;
      const float r2 = qk[0] * qk[0] + qk[1] * qk[1] + qk[2] * qk[2];
      const float fac = p.potential == VDS_FENE ? p.H[k] / (1.f - r2 / p.b_max) : p.H[k];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) t[3 * a + b] += wi * (double)qk[a] * (double)(fac * qk[b]);
    }
  }
  block_sum<9>(t, sm);
  if (threadIdx.x < 9) redp[lb * 16 + threadIdx.x] = t[threadIdx.x];
}

__global__ __launch_bounds__(kRedBlock) void k_stress(EvalParams p, const float *__restrict__ q,
                                                      const float *__restrict__ w, double *__restrict__ redp) {
  stress_body(p, blockIdx.x, q, w, redp);
}

// Foreign rows y[ny][D] (particle-major) as Q operands, centred like the particles.
__global__ __launch_bounds__(kRedBlock) void k_density_rows(EvalParams p, const float *__restrict__ y, int64_t ny,
                                                            const double *__restrict__ meanp, int nmeanp,
                                                            float *__restrict__ QB, F16Operands f16,
                                                            int64_t nrows_pad) {
  __shared__ float mean_sh[16];
  load_mean(p, meanp, nmeanp, mean_sh);
  const int64_t I = (int64_t)blockIdx.x * kRedBlock + threadIdx.x;
  if (I >= nrows_pad) return;
  float x[kMaxD];
  float nrm = 0.f;
  for (int a = 0; a < p.D; ++a) {
    x[a] = I < ny ? y[I * p.D + a] - mean_sh[a] : 0.f;
    nrm = fmaf(x[a], x[a], nrm);
  }
  for (int k = 0; k < 4 * p.KK; ++k) {
    float qa = 0.f;
    if (I < ny) {
      if (k < p.D) qa = x[k];
      else if (k == p.D) qa = -p.kappa * nrm;
      else if (k == p.D + 1) qa = 1.f;
    }
    QB[qk_index(I, k, p.KK)] = qa;
  }
  if (p.qhalf) {
    _Float16 *qh = reinterpret_cast<_Float16 *>(f16.QH);
    for (int sl = 0; sl < 32 * p.KQ; ++sl) {
      const int k = sl / 3;
      _Float16 qv, kv;
      dh_slot(p, sl, I < ny && k < p.D ? p.cs * x[k] : 0.f, 0.f, qv, kv);
      qh[dh_index(I, sl, p.KQ)] = qv;
    }
    f16.RN[I] = I < ny ? -p.kappa * nrm : 0.f;
  }
}

__global__ __launch_bounds__(kRedBlock) void k_density_out(const float *__restrict__ partial, SplitMap splits,
                                                           int64_t stride_rows, int64_t ny, int D, float norm,
                                                           float *__restrict__ f) {
  const int64_t I = (int64_t)blockIdx.x * kRedBlock + threadIdx.x;
  if (I >= ny) return;
  f[I] = ordered_sum<float>(partial + I * splits.width + D, splits.count(I), stride_rows * splits.width) * norm;
}

// ---- batched ensembles: the same bodies, per ensemble ----

__global__ __launch_bounds__(kRedBlock) void k_batch_mean(BatchView b, const float *__restrict__ q,
                                                          double *__restrict__ meanp) {
  const EnsDesc &d = b.ens[b.blk256_ens[blockIdx.x]];
  mean_partials_body(d.p, blockIdx.x - d.blk256, q + d.q_off, nullptr, meanp + (int64_t)d.blk256 * 16);
}

// Ensemble d's slice of the concatenated FP16 distance operands, or of K3 in
// their place.
__device__ inline F16Operands batch_f16(const BatchView &b, const EnsDesc &d) {
  if (d.p.bf3)
    return F16Operands{reinterpret_cast<uint32_t *>(b.f16.QH) + d.pad_off * 16 * bf3_slices(d.p.D), nullptr, nullptr};
  if (!d.p.qhalf) return F16Operands{nullptr, nullptr, nullptr};
  const int64_t halves = d.pad_off * 32 * d.p.KQ;
  return F16Operands{reinterpret_cast<_Float16 *>(b.f16.QH) + halves, reinterpret_cast<_Float16 *>(b.f16.KH) + halves,
                     b.f16.RN + d.pad_off};
}

// Four groups of 16 particles per block (an ensemble is padded to 256): every block
// sums its ensemble's centring partials.  Bound: the operands' FP64 splits.  Measured over
// 269000 particles, D = 9: 54 us, 70 with one group (and D not known at compile time).
constexpr int kBatchGroups = 4;
template <int D>
__global__ __launch_bounds__(kRedBlock) void k_batch_prep(BatchView b, const float *__restrict__ q,
                                                          const double *__restrict__ meanp, float *__restrict__ xc,
                                                          float *__restrict__ wv, float *__restrict__ QB,
                                                          float *__restrict__ KA, float *__restrict__ VA) {
  const EnsDesc &d = b.ens[b.blk16_ens[blockIdx.x * kBatchGroups]];
  const int64_t o = d.pad_off;
  assume_dimension<D>(d.p);
  prep_body<kBatchGroups>(d.p, blockIdx.x - d.blk16 / kBatchGroups, q + d.q_off, nullptr,
                          meanp + (int64_t)d.blk256 * 16, (int)(d.p.Ppad / kRedBlock), xc + o * b.D, wv + o,
                          QB + o * b.KK * 4, KA + o * b.KK * 4, VA + o * b.vw, nullptr, batch_f16(b, d));
}

template <int D>
__global__ __launch_bounds__(kRedBlock) void k_batch_finalize_a(BatchView b, const float *__restrict__ partial,
                                                                const float *__restrict__ xc,
                                                                const float *__restrict__ wv, float *__restrict__ S,
                                                                float *__restrict__ t1, float *__restrict__ VB) {
  const EnsDesc &d = b.ens[b.blk16_ens[blockIdx.x]];
  const int64_t o = d.pad_off;
  assume_dimension<D>(d.p);
  finalize_a_body(d.p, blockIdx.x - d.blk16, partial, d, xc + o * b.D, wv + o, S + o, t1 + o * b.D,
                  VB + o * b.vw);
}

template <int D>
__global__ __launch_bounds__(kRedBlock) void k_batch_explicit(BatchView b, const float *__restrict__ partial,
                                                              const float *__restrict__ xc,
                                                              const float *__restrict__ t1,
                                                              const float *__restrict__ S,
                                                              const float *__restrict__ wv, float *q) {
  const EnsDesc &d = b.ens[b.blk16_ens[blockIdx.x]];
  const int64_t o = d.pad_off;
  assume_dimension<D>(d.p);
  combine_body(d.p, blockIdx.x - d.blk16, MODE_EXPLICIT, 0, partial, d, t1 + o * b.D, S + o,
               wv + o, q + d.q_off, nullptr, q + d.q_off, nullptr, nullptr, nullptr, PackOps{}, nullptr);
}

__global__ __launch_bounds__(kRedBlock) void k_batch_stress(BatchView b, const float *__restrict__ q,
                                                            double *__restrict__ redp) {
  const EnsDesc &d = b.ens[b.blk256_ens[blockIdx.x]];
  stress_body(d.p, blockIdx.x - d.blk256, q + d.q_off, nullptr, redp + (int64_t)d.blk256 * 16);
}

// A workgroup per ensemble, a wave per component: lane l folds blocks l, l + 64,
// ..., then the wave (one thread per component took 18 us at 63 blocks).
__global__ __launch_bounds__(576) void k_batch_stress_sum(const EnsDesc *__restrict__ ens,
                                                          const double *__restrict__ redp, double *__restrict__ tau) {
  const EnsDesc &d = ens[blockIdx.x];
  const int s = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nb = (int)(d.p.Ppad / kRedBlock);
  double acc = 0.0;
  for (int i = lane; i < nb; i += 64) acc += redp[((int64_t)d.blk256 + i) * 16 + s];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) tau[(int64_t)blockIdx.x * 9 + s] = acc;
}

// ---- small problems: a pass and what follows it in one launch ----------------
//
// Below kRowsMaxP particles a pass is a few microseconds of work and the launch
// that sums its partials costs as much again, most of it a chain of dependent
// loads.  Here a workgroup of sixteen waves owns 16 rows: wave w takes the
// 32-column chunks w, w + 16, ... (operands straight from memory, the next
// chunk's in flight), the waves' FP64 sums meet in LDS in wave order, and the
// first 256 threads, sixteen lanes per particle as everywhere, finish the rows:
// pass A with S, term1 and the pass-B operand, pass B with drift, update and the
// next state's operands.  Those go to a second K3 buffer, since other
// workgroups still read this one.
// Bound: latency (launch, row operand, first chunk, sums), and from some 3000
// particles on every workgroup's reading of all columns through L2.  The line lies
// where the workgroups fill the compute units once, 4096 particles: beyond it a few
// units take a second workgroup.  An explicit step in two launches and (in four), in us:
// D = 9 16.5 (38.0) at P = 2500, 23.0 (37.5) at 4000, 37.9 (40.4) at 4100, 45.1 (43.9) at
// 5000, 50.7 (50.2) at 6000; D = 15 29.2 (40.4) at 4000, 48.8 (44.9) at 4100, 58.5 (49.0)
// at 5000; D = 3 17.4 (34.1) at 4000, and above the line still 29.0 (36.0) at 4100 and 47.2
// (53.0) at 8000: one line serves all dimensions.

constexpr int kRowsWaves = 16;

template <int D>
struct RowsLds {
  double red[kRowsWaves][16][16];
};

// Sum of lane (particle 16 blockIdx.x + t / 16, n = t % 16) for the first 256
// threads: the difference sum's component n < D, the kernel sum at n = D.
template <int D>
__device__ double rows_pass(const uint4 *__restrict__ K3, const uint4 *__restrict__ V3, float x, int nch,
                            const int *__restrict__ done, RowsLds<D> &lds, bool &stopped) {
  constexpr int NQ = bf3_slices(D), NT = bf3_tiles(D);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = (int)blockIdx.x;
  const int diag_i = (lane & 15) - 4 * (lane >> 4);
  bf16x8 neg[2], q[NQ];
  uint4 kv[2 * NQ], vv[NT];
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < 2 * NQ; ++i) kv[i] = K3[((int64_t)c * 2 * NQ + i) * 64 + lane];
#pragma unroll
    for (int T = 0; T < NT; ++T) vv[T] = V3[((int64_t)c * NT + T) * 64 + lane];
  };
  // the flag, the row operand and the first chunk travel together (waves past
  // the chunks load chunk 0)
  const int dn = done != nullptr ? *done : 0;
  load(wave < nch ? wave : 0);
  bf3_row_operand<D>(K3, rb, lane, q);
  asm volatile("" : "+v"(kv[0].x), "+v"(vv[0].x));  // keeps the loads ahead of the test
  stopped = dn != 0;
  if (stopped) return 0.0;
  minus_identity(lane, neg);
  floatx4 acc[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T) acc[T] = floatx4{0.f, 0.f, 0.f, 0.f};
  double tot[4] = {0.0, 0.0, 0.0, 0.0};
  int count = 0;
  for (int c = wave; c < nch; c += kRowsWaves) {
    floatx4 e[2];
    bf16x8 va[NT];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      e[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < NQ; ++m)
        e[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(kv[b * NQ + m]), q[m], e[b], 0, 0, 0);
    }
#pragma unroll
    for (int T = 0; T < NT; ++T) va[T] = as_bf8(vv[T]);
    if (c + kRowsWaves < nch) load(c + kRowsWaves);
    bf3_accumulate<D>(e, va, neg, c == rb >> 1, rb & 1, diag_i, acc);
    if (++count % kFlush3 == 0) bf3_flush<D>(acc, lane, tot);
  }
  bf3_flush<D>(acc, lane, tot);
#pragma unroll
  for (int i = 0; i < 4; ++i) lds.red[wave][4 * (lane >> 4) + i][lane & 15] = tot[i];
  __syncthreads();
  double o = 0.0;
  if (threadIdx.x < kRedBlock) {
    const int r = threadIdx.x >> 4, n = threadIdx.x & 15;
    for (int w = 0; w < kRowsWaves; ++w) o += lds.red[w][r][n];
    const double s = row_move<0x150 + D>(o);
    if (n < D) o = (double)x * s - o;
  }
  return o;
}

// Pass A, S, term1 and the pass-B operand.  With chk.ctrl the launch first tests
// the fixed-point iteration before it (k_picard_check's work): every workgroup
// takes the test from the same block maxima, the first one records it.
template <int D>
__global__ __launch_bounds__(kRowsWaves * 64) void k_rows_a(EvalParams p, const uint4 *__restrict__ K3,
                                                            const uint4 *__restrict__ VA, const float *__restrict__ xc,
                                                            const float *__restrict__ wv, float *__restrict__ S,
                                                            float *__restrict__ t1, float *__restrict__ VB, int nch,
                                                            const int *__restrict__ done, PicardCheck chk,
                                                            const float *__restrict__ blockmax, int nblk_chk) {
  __shared__ RowsLds<D> lds;
  __shared__ int stop;
  assume_dimension<D>(p);
  __builtin_assume(p.bf3 == 1 && p.vhalf == 0 && p.qhalf == 0);
  const int64_t I = group_particle(blockIdx.x);
  const int n = group_lane();
  const bool act = threadIdx.x < kRedBlock;
  const float x = act && n < D ? xc[I * D + n] : 0.f, w = act ? wv[I] : 0.f;
  if (chk.ctrl != nullptr) {
    // the flag once per block: the first block may set it during this launch
    if (threadIdx.x == 0) stop = *done;
    float r;
    const bool conv = picard_converged(chk, blockmax, nblk_chk, &r);  // (holds barriers)
    const bool was = stop != 0;
    if (!was && blockIdx.x == 0 && threadIdx.x == 0) {
      chk.ctrl->last_resid = r;
      chk.ctrl->checked = chk.iter + 1;
      if (conv) {
        chk.ctrl->conv_iter = chk.iter;
        chk.ctrl->done = 1;
      }
    }
    if (was || conv) return;
  }
  bool stopped;
  const double o = rows_pass<D>(K3, VA, x, nch, chk.ctrl != nullptr ? nullptr : done, lds, stopped);
  if (!stopped && act) finalize_a_row(p, I, n, o, x, w, S, t1, VB);
}

// Pass B and the combination (modes of k_combine), or with MODE_SUMS the row
// scalars of the reduced model: out = sum_K (w_K / S_K) e_IK (K = I included),
// out2 = 1 / S_I.
template <int D>
__global__ __launch_bounds__(kRowsWaves * 64) void k_rows_b(EvalParams p, int mode, int obs,
                                                            const uint4 *__restrict__ K3, const uint4 *__restrict__ VB,
                                                            int nch, const float *xc, const float *__restrict__ t1,
                                                            const float *__restrict__ S, const float *wv,
                                                            const float *qin, const float *__restrict__ qs, float *out,
                                                            float *out2, double *__restrict__ redp,
                                                            float *__restrict__ blockmax, const int *__restrict__ done,
                                                            PackOps pack, int *fene_out) {
  __shared__ RowsLds<D> lds;
  assume_dimension<D>(p);
  __builtin_assume(p.bf3 == 1 && p.vhalf == 0 && p.qhalf == 0);
  const int64_t I = group_particle(blockIdx.x);
  const int n = group_lane();
  const bool act = threadIdx.x < kRedBlock;
  const float x = act && n < D ? xc[I * D + n] : 0.f;
  CombineIn in{};
  if (mode == MODE_SUMS) {
    if (act && I < p.P) in.S = S[I], in.w = wv[I];
  } else {
    in = combine_load(p, blockIdx.x, mode, obs, act, t1, S, wv, qin, qs);
  }
  bool stopped;
  const double o = rows_pass<D>(K3, VB, x, nch, done, lds, stopped);
  if (stopped) return;
  if (mode == MODE_SUMS) {
    if (act && I < p.P && n == D) {
      const double Si = (double)in.S;
      out[I] = (float)(o + (double)in.w / Si);
      out2[I] = (float)(1.0 / Si);
    }
    return;
  }
  combine_rows(p, blockIdx.x, mode, obs, act, o, in, out, out2, redp, blockmax, pack, fene_out);
}

// ---- density at given points, VDS_PAIR_MFMA32 ---------------------------------
//
// f(y_I) = norm sum_J w_J e_IJ: no difference sums, so a pair is its exponent
// (matrix cores), one exp2 and one FP32 FMA with the weight, and only 16 RB row
// sums leave a workgroup.  It packs its rows' operands itself (into LDS), its
// eight waves take the 32-column chunks c, c + 8, ... of the workgroup's columns
// with the next chunk's operands in flight, FP32 sums of at most 16 terms go to
// FP64 in fixed order.
// Bound: exp2 (a quarter of the vector rate) and the columns' operands through
// L2, 4 KB per chunk at D = 9 for 16 RB rows.  Measured, D = 9, P = 5000, 19683
// points: 23 us (the same in blocks of P rows through the pair pass: 27 + 5.3 +
// 5.5 us in each of four blocks).
constexpr int kDensityWaves = 8;

template <int D, int RB>
__global__ __launch_bounds__(kDensityWaves * 64) void k_density_bf3(EvalParams p, const float *__restrict__ y,
                                                                    int64_t ny, const float *__restrict__ cmean,
                                                                    const uint4 *__restrict__ K3,
                                                                    const float *__restrict__ wv, int nch, float norm,
                                                                    float *__restrict__ f, double *__restrict__ part) {
  constexpr int NQ = bf3_slices(D);
  __shared__ uint4 rows[RB * NQ * 64];
  __shared__ double red[kDensityWaves][16 * RB];
  assume_dimension<D>(p);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = long_block() * (16 * RB);
  if (i0 >= ny) return;
  const int cps = (nch + (int)gridDim.z - 1) / (int)gridDim.z;
  const int c0 = (int)blockIdx.z * cps, c1 = min(nch, c0 + cps);
  uint4 kv[2 * NQ];
  float4 wj[2];
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < 2 * NQ; ++i) kv[i] = K3[((int64_t)c * 2 * NQ + i) * 64 + lane];
#pragma unroll
    for (int b = 0; b < 2; ++b)
      wj[b] = *reinterpret_cast<const float4 *>(wv + (int64_t)c * 32 + 16 * b + 4 * (lane >> 4));
  };
  if (c0 + wave < c1) load(c0 + wave);
  for (int t = threadIdx.x; t < 256 * RB; t += kDensityWaves * 64) {
    const int r = t >> 4, n = t & 15;
    const bool real = i0 + r < ny;
    store_k3<true>(p, real, reinterpret_cast<uint32_t *>(rows), r, n, real && n < D ? y[(i0 + r) * D + n] - cmean[n] : 0.f);
  }
  __syncthreads();
  bf16x8 q[RB][NQ];
#pragma unroll
  for (int r = 0; r < RB; ++r) bf3_row_operand<D>(rows, r, lane, q[r]);
  float acc[RB][4];
  double tot[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    tot[r] = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[r][i] = 0.f;
  }
  auto flush = [&] {
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      tot[r] += ((double)acc[r][0] + (double)acc[r][1]) + ((double)acc[r][2] + (double)acc[r][3]);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[r][i] = 0.f;
    }
  };
  int count = 0;
  for (int c = c0 + wave; c < c1; c += kDensityWaves) {
    floatx4 e[RB][2];
    const float4 wc[2] = {wj[0], wj[1]};
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < RB; ++r) e[r][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < NQ; ++m)
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          e[r][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(kv[b * NQ + m]), q[r][m], e[r][b], 0, 0, 0);
    if (c + kDensityWaves < c1) load(c + kDensityWaves);
    // lane: columns 4 (lane / 16) + i of block b, row lane % 16
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float wb[4] = {wc[b].x, wc[b].y, wc[b].z, wc[b].w};
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][i] = fmaf(wb[i], __builtin_amdgcn_exp2f(e[r][b][i]), acc[r][i]);
    }
    if (++count % kFlush3 == 0) flush();
  }
  flush();
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    double t = tot[r];
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    if (lane < 16) red[wave][16 * r + lane] = t;
  }
  __syncthreads();
  if (threadIdx.x < 16 * RB && i0 + threadIdx.x < ny) {
    double t = 0.0;
    for (int v = 0; v < kDensityWaves; ++v) t += red[v][threadIdx.x];
    if (part != nullptr) part[(int64_t)blockIdx.z * ny + i0 + threadIdx.x] = t;
    else f[i0 + threadIdx.x] = (float)t * norm;
  }
}

__global__ __launch_bounds__(kRedBlock) void k_density_sum(const double *__restrict__ part, int splits, int64_t ny,
                                                           float norm, float *__restrict__ f) {
  const int64_t I = (int64_t)blockIdx.x * kRedBlock + threadIdx.x;
  if (I >= ny) return;
  double t = 0.0;
  for (int s = 0; s < splits; ++s) t += part[s * ny + I];
  f[I] = (float)t * norm;
}

// ---- launchers ----

static inline unsigned nblocks(int64_t n) { return (unsigned)((n + kRedBlock - 1) / kRedBlock); }

void launch_mean_partials(const EvalParams &p, const float *q, const float *w, double *meanp, const int *done,
                          Ctrl *begin, hipStream_t s) {
  k_mean_partials<<<nblocks(p.P), kRedBlock, 0, s>>>(p, q, w, meanp, done, begin);
}
void launch_prep(const EvalParams &p, const float *q, const float *w, const double *meanp, int nmeanp, float *xc,
                 float *wv, float *QB, float *KA, float *VA, float *wscale, const F16Operands *f16, const int *done,
                 hipStream_t s, float *cmean, Ctrl *begin) {
  const F16Operands ops = f16 != nullptr ? *f16 : F16Operands{nullptr, nullptr, nullptr};
  by_dimension(p.D, [&](auto d) {
    k_prep<decltype(d)::value><<<nblocks(p.Ppad * 16), kRedBlock, 0, s>>>(p, q, w, meanp, nmeanp, xc, wv, QB, KA, VA,
                                                                          wscale, ops, done, cmean, begin);
  });
}
void launch_finalize_a(const EvalParams &p, const float *partial, const SplitMap &splits, const float *xc, const float *wv,
                       float *S, float *t1, float *VB, const int *done, hipStream_t s) {
  by_dimension(p.D, [&](auto d) {
    k_finalize_a<decltype(d)::value>
        <<<nblocks(p.Ppad * 16), kRedBlock, 0, s>>>(p, partial, splits, xc, wv, S, t1, VB, done);
  });
}
void launch_combine(const EvalParams &p, int mode, bool obs, const float *partial, const SplitMap &splits, const float *xc,
                    const float *t1, const float *S, const float *wv, const float *qin, const float *q0,
                    float *out, float *out2, double *redp, float *blockmax, const int *done, hipStream_t s,
                    const PackOps *pack, int *fene_out) {
  const PackOps pk = pack != nullptr ? *pack : PackOps{};
  by_dimension(p.D, [&](auto d) {
    k_combine<decltype(d)::value><<<nblocks(p.P * 16), kRedBlock, 0, s>>>(p, mode, obs ? 1 : 0, partial, splits, xc, t1,
                                                                          S, wv, qin, q0, out, out2, redp, blockmax,
                                                                          done, pk, fene_out);
  });
}
// (particles up to the last chunk's end: their operands are written as zeros)
static unsigned rows_grid(const EvalParams &p) { return (unsigned)(round_up(p.P, 32) / 16); }
void launch_rows_a(const EvalParams &p, const void *K3, const float *VA, const float *xc, const float *wv, float *S,
                   float *t1, float *VB, const int *done, const PicardCheck *chk, const float *blockmax, int nblk_chk,
                   hipStream_t s) {
  const PicardCheck ck = chk != nullptr ? *chk : PicardCheck{nullptr, 0.f, 0};
  const int nch = (int)((p.P + 31) / 32);
  auto go = [&](auto d) {
    k_rows_a<decltype(d)::value><<<rows_grid(p), kRowsWaves * 64, 0, s>>>(
        p, static_cast<const uint4 *>(K3), reinterpret_cast<const uint4 *>(VA), xc, wv, S, t1, VB, nch, done, ck,
        blockmax, nblk_chk);
  };
  by_dimension(p.D, go);
}
void launch_rows_b(const EvalParams &p, int mode, bool obs, const void *K3, const float *VB, const float *xc,
                   const float *t1, const float *S, const float *wv, const float *qin, const float *q0, float *out,
                   float *out2, double *redp, float *blockmax, const int *done, hipStream_t s, const PackOps *pack,
                   int *fene_out) {
  const PackOps pk = pack != nullptr ? *pack : PackOps{};
  const int nch = (int)((p.P + 31) / 32);
  auto go = [&](auto d) {
    k_rows_b<decltype(d)::value><<<rows_grid(p), kRowsWaves * 64, 0, s>>>(
        p, mode, obs ? 1 : 0, static_cast<const uint4 *>(K3), reinterpret_cast<const uint4 *>(VB), nch, xc, t1, S, wv,
        qin, q0, out, out2, redp, blockmax, done, pk, fene_out);
  };
  by_dimension(p.D, go);
}
void launch_reduce_final(const double *redp, int nblk, int nslots, double *out, hipStream_t s, const Ctrl *ctrl,
                         Ctrl *ctrl_out) {
  k_reduce_final<<<1, 1024, 0, s>>>(redp, nblk, nslots, out, ctrl, ctrl_out);
}
void launch_ctrl_reset(Ctrl *ctrl, hipStream_t s) { k_ctrl_reset<<<1, 64, 0, s>>>(ctrl); }
void launch_step_end(const EvalParams &p, Ctrl *ctrl, const PicardCheck &chk, const float *blockmax, int nblk_chk,
                     const float *xb0, const float *xb1, float *q, float *xpred, const float *w, double *meanp,
                     hipStream_t s) {
  k_step_end<<<nblocks(p.P), kRedBlock, 0, s>>>(p, ctrl, chk, blockmax, nblk_chk, xb0, xb1, q, xpred, w, meanp);
}
void launch_picard_check(const PicardCheck &chk, const float *blockmax, int nblk_chk, hipStream_t s) {
  k_picard_check<<<1, kRedBlock, 0, s>>>(chk, blockmax, nblk_chk);
}
void launch_stress(const EvalParams &p, const float *q, const float *w, double *redp, hipStream_t s) {
  k_stress<<<nblocks(p.P), kRedBlock, 0, s>>>(p, q, w, redp);
}
void launch_density_rows(const EvalParams &p, const float *y, int64_t ny, const double *meanp, int nmeanp,
                         float *QB, const F16Operands *f16, hipStream_t s) {
  const F16Operands ops = f16 != nullptr ? *f16 : F16Operands{nullptr, nullptr, nullptr};
  // rows are padded to a multiple of 256 within the Ppad-row operand buffer
  const int64_t nrows_pad = round_up(ny, kRowAlign);
  k_density_rows<<<nblocks(nrows_pad), kRedBlock, 0, s>>>(p, y, ny, meanp, nmeanp, QB, ops, nrows_pad);
}
void launch_density_out(const EvalParams &p, const float *partial, const SplitMap &splits, int64_t ny, float norm, float *f,
                        hipStream_t s) {
  k_density_out<<<nblocks(ny), kRedBlock, 0, s>>>(partial, splits, p.Ppad, ny, p.D, norm, f);
}

// Row blocks per wave.  A compute unit takes ceil(workgroups / 256) of them one
// after the other (or at once, at a share of its speed), each a time of about
// RB + 1 (RB blocks of arithmetic, one of operand traffic).  P = 10000, D = 9,
// 19683 points: RB 1 to 5 take 93, 68, 58, 75, 52 us for the whole call (model
// 10, 9, 8, 10, 6); 40000 points at P = 20000: 280, 168, 165, 178, 146 (20, 15,
// 16, 15, 12); 8192 points: 77, 72, 74, 80, 84 (4, 3, 4, 5, 6).
static int density_row_blocks(int64_t ny) {
  int best = 1;
  int64_t cost = INT64_MAX;
  const int64_t cu = device_cu_count();
  for (int rb = 1; rb <= 5; ++rb) {
    const int64_t wgs = (ny + 16 * rb - 1) / (16 * rb);
    const int64_t t = (wgs + cu - 1) / cu * (rb + 1);
    if (t < cost) best = rb, cost = t;
  }
  return best;
}
// With at most 256 workgroups of 16 rows the columns are split too, but only into
// parts of at least 8 chunks a wave, about what the second launch costs
// (P = 20000, one point: 25 us for the call; 37 unsplit, 64 by the general pair
// pass).
int density_splits(int64_t P, int64_t ny) {
  const int64_t groups = (ny + 15) / 16, nch = (P + 31) / 32;
  return (int)std::max<int64_t>(1, std::min<int64_t>(512 / groups, nch / (8 * kDensityWaves)));
}
void launch_density(const EvalParams &p, const float *y, int64_t ny, const float *cmean, const void *K3,
                    const float *wv, float norm, float *f, void *part, hipStream_t s) {
  const int splits = density_splits(p.P, ny), nch = (int)((p.P + 31) / 32);
  double *pt = splits > 1 ? static_cast<double *>(part) : nullptr;
  const uint4 *k3 = static_cast<const uint4 *>(K3);
  by_dimension(p.D, [&](auto d) {
    constexpr int D = decltype(d)::value;
    auto go = [&](auto rc) {
      constexpr int RB = decltype(rc)::value;
      dim3 grid = long_grid((ny + 16 * RB - 1) / (16 * RB));
      grid.z = (unsigned)splits;
      k_density_bf3<D, RB><<<grid, kDensityWaves * 64, 0, s>>>(p, y, ny, cmean, k3, wv, nch, norm, f, pt);
    };
    switch (density_row_blocks(ny)) {
      case 1: go(std::integral_constant<int, 1>{}); break;
      case 2: go(std::integral_constant<int, 2>{}); break;
      case 3: go(std::integral_constant<int, 3>{}); break;
      case 4: go(std::integral_constant<int, 4>{}); break;
      default: go(std::integral_constant<int, 5>{}); break;
    }
  });
  if (splits > 1) k_density_sum<<<nblocks(ny), kRedBlock, 0, s>>>(pt, splits, ny, norm, f);
}

void launch_batch_mean(const BatchView &b, const float *q, double *meanp, hipStream_t s) {
  k_batch_mean<<<b.nblk256, kRedBlock, 0, s>>>(b, q, meanp);
}
void launch_batch_prep(const BatchView &b, const float *q, const double *meanp, float *xc, float *wv, float *QB,
                       float *KA, float *VA, hipStream_t s) {
  by_dimension(b.D, [&](auto d) {
    k_batch_prep<decltype(d)::value>
        <<<b.nblk16 / kBatchGroups, kRedBlock, 0, s>>>(b, q, meanp, xc, wv, QB, KA, VA);
  });
}
void launch_batch_finalize_a(const BatchView &b, const float *partial, const float *xc, const float *wv, float *S,
                             float *t1, float *VB, hipStream_t s) {
  by_dimension(b.D, [&](auto d) {
    k_batch_finalize_a<decltype(d)::value><<<b.nblk16, kRedBlock, 0, s>>>(b, partial, xc, wv, S, t1, VB);
  });
}
void launch_batch_explicit(const BatchView &b, const float *partial, const float *xc, const float *t1,
                           const float *S, const float *wv, float *q, hipStream_t s) {
  by_dimension(b.D, [&](auto d) {
    k_batch_explicit<decltype(d)::value><<<b.nblk16, kRedBlock, 0, s>>>(b, partial, xc, t1, S, wv, q);
  });
}
void launch_batch_stress(const BatchView &b, const float *q, double *redp, hipStream_t s) {
  k_batch_stress<<<b.nblk256, kRedBlock, 0, s>>>(b, q, redp);
}
void launch_batch_stress_sum(const EnsDesc *ens, int nens, const double *redp, double *tau, hipStream_t s) {
  k_batch_stress_sum<<<nens, 576, 0, s>>>(ens, redp, tau);
}

}  // namespace vds
