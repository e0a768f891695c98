// Learned reduced step (C ABI of include/vds_mlp.h): MLP training kernels
// (FP32 MFMA products with SiLU and MSE epilogues, Adam), BF16 MFMA inference, and the
// rollout that checks the network against the particle scheme and falls back.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "vds_ctx.h"
#include "vds_mlp.h"
#include "vds_pod.h"

using namespace vds;

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

thread_local std::string g_mlp_create_error;

struct MlpLayout {
  size_t params, grads, adam_m, adam_v, wbf, wpk, Z1, A1, Z2, A2, Y, dY, dZ1, dZ2, xs, xsc, ys, ysc, xin, tin, lossp, total;
};

// Resident learned steps (k_learned_steps_reg): one workgroup of 1024 threads
// keeps the BF16 weights on chip for a whole window of steps, layers 1 and 2
// in registers and layer 3 in LDS (gfx950 gives a workgroup 160 KiB).  Layer l
// splits a row over G_l consecutive lanes, each taking CK_l consecutive
// inputs; layer 3 has up to kNout3 * G3 row chunks ("slots"), slot s for
// thread s % 1024.  Shapes that fit: nin <= 8 * 68, width <= 128, nout <= 576.
constexpr int kRegThreads = 1024;
constexpr int kG1 = 8, kCK1 = 68, kG2 = 8, kCK2 = 16, kG3 = 4, kCK3 = 32, kNout3 = 576;
constexpr int kSlots3 = kNout3 * kG3;
constexpr int kS3 = (kSlots3 + kRegThreads - 1) / kRegThreads;
constexpr int64_t kPk1 = (int64_t)kRegThreads * kCK1, kPk2 = (int64_t)kRegThreads * kCK2,
                  kPk3 = (int64_t)kSlots3 * kCK3;  // BF16 elements
bool reg_steps_fit(int nin, int w, int nout) {
  return nin <= kG1 * kCK1 && w <= kRegThreads / kG1 && w <= kG2 * kCK2 && w <= kG3 * kCK3 && nout <= kNout3;
}

int64_t nparams(int nin, int w, int nout) {
  return (int64_t)w * nin + w + (int64_t)w * w + w + (int64_t)nout * w + nout;
}

// Output tiles of tb x tb blocks of 16 x 16.
__host__ __device__ constexpr int64_t mlp_tiles(int64_t M, int64_t N, int tb) {
  return ((M + 16 * tb - 1) / (16 * tb)) * ((N + 16 * tb - 1) / (16 * tb));
}

MlpLayout mlp_layout(int nin, int w, int nout, int B) {
  MlpLayout L{};
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off += (b + 255) / 256 * 256;
    return o;
  };
  const int64_t np = nparams(nin, w, nout);
  const int64_t Bp = (B + 15) / 16 * 16;
  L.params = take(sizeof(float) * np);
  L.grads = take(sizeof(float) * np);
  L.adam_m = take(sizeof(float) * np);
  L.adam_v = take(sizeof(float) * np);
  L.wbf = take(sizeof(uint16_t) * np);
  L.wpk = take(sizeof(uint16_t) * (kPk1 + kPk2 + kPk3));
  L.Z1 = take(sizeof(float) * Bp * w);
  L.A1 = take(sizeof(float) * Bp * w);
  L.Z2 = take(sizeof(float) * Bp * w);
  L.A2 = take(sizeof(float) * Bp * w);
  L.Y = take(sizeof(float) * Bp * nout);
  L.dY = take(sizeof(float) * Bp * nout);
  L.dZ1 = take(sizeof(float) * Bp * w);
  L.dZ2 = take(sizeof(float) * Bp * w);
  L.xs = take(sizeof(float) * nin);
  L.xsc = take(sizeof(float) * nin);
  L.ys = take(sizeof(float) * nout);
  L.ysc = take(sizeof(float) * nout);
  L.xin = take(sizeof(float) * Bp * nin);
  L.tin = take(sizeof(float) * Bp * nout);
  L.lossp = take(sizeof(double) * (mlp_tiles(B, nout, 1) + 2));
  L.total = off;
  return L;
}

__device__ inline short f2bf(float f) {
  const unsigned u = __float_as_uint(f);
  return (short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);  // round to nearest even
}
__device__ inline float silu(float z) { return z / (1.f + __expf(-z)); }
__device__ inline float silu_grad(float z) {
  const float s = 1.f / (1.f + __expf(-z));
  return s * (1.f + z * (1.f - s));
}

__global__ void k_to_bf16(const float *__restrict__ a, short *__restrict__ b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = f2bf(a[i]);
}

// ---- training products ----
//
// A minibatch is six launches, one per link of the chain
//   Z1 -> Z2 -> Y, loss -> {dZ2, dW3, db3} -> {dZ1, dW2, db2} -> {dW1, db1, loss}
// with bias, SiLU, the loss gradient and SiLU's derivative in the products'
// epilogues.  At the learned step's own shape (541-128-128-540, 64 rows: 62
// MFLOP, 1 MB) only latency counts, so an output tile is one 16 x 16 block, K
// goes over the eight waves of a workgroup (the block's wave sums meet in LDS)
// and the operands come straight from memory, four rounds of 16 in flight per
// wave.
// Bound: the chain of launches (3.3 to 4.9 us each, one or two memory latencies
// and the wave sum; 24 us together, 33 with the loss on the host).  25 launches
// of 64 x 64-tile products (each with its own sum over K splits), elementwise
// passes and one-thread column sums took 250 and 270 us.
enum MlpEpi { kEpiHidden, kEpiOutput, kEpiInputGrad, kEpiWeightGrad };

// C (M x N) = A B^T over K, FP32 MFMA.
struct MlpOp {
  int M, N, K;
  int epi;
  int64_t tiles;           // of the launch's tile edge
  const float *A, *B;
  int64_t lda, ldb;
  const float *aux;        // bias; in kEpiInputGrad Z of the layer below
  const float *T;          // kEpiOutput: targets, or null for the forward pass alone
  float *C;                // Z or Y; dZ; dW
  float *C2;               // hidden: A = silu(Z); output: dY
  double *lossp;           // output: one partial sum of (Y - T)^2 per tile
};

// db[j] = sum_i dZ[i][j] (N columns, n rows), in FP64.
struct MlpColsum {
  const float *dZ;
  int64_t n;
  int N;
  float *db;
};

// *out = (add ? *out : 0) + scale * sum of np partial sums.
struct MlpLoss {
  const double *lossp;
  int64_t np;
  double scale;
  int add;
  double *out;
};

typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// k indices k .. k+3 of one row (MN: of one column at stride ld) of an operand.
template <bool MN>
__device__ inline floatx4 mlp_load(const float *__restrict__ p, int64_t ld, int k) {
  if constexpr (MN) {
    const float *q = p + k * ld;
    return floatx4{q[0], q[ld], q[2 * ld], q[3 * ld]};
  } else {
    return *reinterpret_cast<const float4u *>(p + k);
  }
}

// The same at the end of K: what lies beyond counts as zero.
template <bool MN>
__device__ inline floatx4 mlp_load_tail(const float *__restrict__ p, int64_t ld, int k, int K) {
  floatx4 v;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t kk = min(k + t, K - 1);
    const float x = p[MN ? kk * ld : kk];
    v[t] = k + t < K ? x : 0.f;
  }
  return v;
}

constexpr int kMlpWaves = 8;

// Rows that a workgroup of a weight gradient, whose K is the batch (up to 2^20), sums in
// FP32: 256 per wave, 16 rounds of 16 k.  With more (LONG) a wave takes each such group's
// sum out of the accumulators: to FP64, or for tiles 64 wide, whose FP64 sums would take
// 128 registers more than there are, to an FP32 sum in LDS, of at most 512 groups.
// The waves' sums of more than 32 rows are added in FP64.  Relative error of dW1 with one FP32 sum per wave (and
// of the eight in FP32) and so: 541-128-128-540, 16384 rows 3.3e-7 and 1.1e-7, 65536 rows
// 5.2e-7 and 6.3e-8; 64-16-16-16, 262144 rows 9.8e-7 and 3.2e-8.  The time: 16384 rows 649
// and 612 us, 64-16-16-16 5.2 and 5.1 ms; in tiles 64 wide the longer loop holds fewer loads
// in flight (2049-2048-2048-2048, 4096 rows 3.35 and 3.44 ms).
constexpr int kMlpGroup = 16 * 16 * kMlpWaves;

// Where lane and wave keep element t of block (a, b) of a tile in LDS: [wave][row][column].
template <int TB>
__device__ inline int mlp_slot(int wave, int lane, int a, int b, int t) {
  return wave * (256 * TB * TB) + (16 * a + 4 * (lane >> 4) + t) * (16 * TB) + 16 * b + (lane & 15);
}

// This wave's share of tile (ti, tj): rounds of 16 k, wave, wave + 8, ...  Lane
// l holds k 4 (l / 16) .. + 3 of a round in row l % 16 of each block, one step
// of the matrix unit taking one k from each group of four.  red: the tile's LDS.
template <int TB, bool A_MN, bool B_MN, bool LONG>
__device__ inline void mlp_product(const MlpOp &o, int64_t ti, int64_t tj, int lane, int wave,
                                   floatx4 (&acc)[TB][TB], float *red) {
  constexpr int U = TB == 1 ? 4 : 1;
  const int m = lane & 15, k0 = (lane >> 4) * 4;
  const float *pa[TB], *pb[TB];
#pragma unroll
  for (int a = 0; a < TB; ++a) {
    const int64_t ra = min(ti * (16 * TB) + 16 * a + m, (int64_t)o.M - 1);
    const int64_t rb = min(tj * (16 * TB) + 16 * a + m, (int64_t)o.N - 1);
    pa[a] = o.A + (A_MN ? ra : ra * o.lda);
    pb[a] = o.B + (B_MN ? rb : rb * o.ldb);
  }
  auto products = [&](const floatx4(&va)[TB], const floatx4(&vb)[TB]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int a = 0; a < TB; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[a][t], vb[b][t], acc[a][b], 0, 0, 0);
  };
  const int full = o.K / 16;
  int r = wave;
  auto rounds = [&](int end) {
    for (; r + (U - 1) * kMlpWaves < end; r += U * kMlpWaves) {
      floatx4 va[U][TB], vb[U][TB];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int a = 0; a < TB; ++a) {
          const int k = 16 * (r + u * kMlpWaves) + k0;
          va[u][a] = mlp_load<A_MN>(pa[a], o.lda, k);
          vb[u][a] = mlp_load<B_MN>(pb[a], o.ldb, k);
        }
#pragma unroll
      for (int u = 0; u < U; ++u) products(va[u], vb[u]);
    }
  };
  constexpr bool kLong = LONG && A_MN && B_MN, kInLds = TB > 2;
  double tot[kLong && !kInLds ? TB : 1][TB][4];
  auto each = [&](auto &&f) {
#pragma unroll
    for (int a = 0; a < TB; ++a)
#pragma unroll
      for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) f(a, b, t);
  };
  auto slot = [&](int a, int b, int t) -> float & { return red[mlp_slot<TB>(wave, lane, a, b, t)]; };
  bool groups = false;  // a group has been taken out of acc
  if constexpr (kLong) {
    for (int end = kMlpGroup / 16; end < full; end += kMlpGroup / 16) {
      rounds(end);
      each([&](int a, int b, int t) {
        if constexpr (kInLds) slot(a, b, t) = groups ? slot(a, b, t) + acc[a][b][t] : acc[a][b][t];
        else tot[a][b][t] = groups ? tot[a][b][t] + (double)acc[a][b][t] : (double)acc[a][b][t];
        acc[a][b][t] = 0.f;
      });
      groups = true;
    }
  }
  rounds(full);
  for (; r <= full; r += kMlpWaves) {
    if (r == full && o.K % 16 == 0) break;
    floatx4 va[TB], vb[TB];
    const int k = 16 * r + k0;
#pragma unroll
    for (int a = 0; a < TB; ++a) {
      va[a] = r < full ? mlp_load<A_MN>(pa[a], o.lda, k) : mlp_load_tail<A_MN>(pa[a], o.lda, k, o.K);
      vb[a] = r < full ? mlp_load<B_MN>(pb[a], o.ldb, k) : mlp_load_tail<B_MN>(pb[a], o.ldb, k, o.K);
    }
    products(va, vb);
  }
  if constexpr (kLong) {
    if (groups)
      each([&](int a, int b, int t) {
        if constexpr (kInLds) acc[a][b][t] += slot(a, b, t);
        else acc[a][b][t] = (float)(tot[a][b][t] + (double)acc[a][b][t]);
      });
  }
}

// Sum of v over the workgroup's 512 threads, in thread 0, fixed order.
__device__ inline double mlp_block_sum(double v, int tid) {
  __shared__ double wsum[kMlpWaves];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d);
  if ((tid & 63) == 0) wsum[tid >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (tid == 0)
    for (int i = 0; i < kMlpWaves; ++i) s += wsum[i];
  return s;
}

template <int TB, bool LONG>
__device__ inline void mlp_tile(const MlpOp &o, int64_t tile, float *red, int tid) {
  constexpr int E = 16 * TB, NE = E * E;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t tm = (o.M + E - 1) / E, ti = tile % tm, tj = tile / tm;
  floatx4 acc[TB][TB];
#pragma unroll
  for (int a = 0; a < TB; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (o.epi == kEpiInputGrad)
    mlp_product<TB, false, true, LONG>(o, ti, tj, lane, wave, acc, red);
  else if (o.epi == kEpiWeightGrad)
    mlp_product<TB, true, true, LONG>(o, ti, tj, lane, wave, acc, red);
  else
    mlp_product<TB, false, false, LONG>(o, ti, tj, lane, wave, acc, red);
#pragma unroll
  for (int a = 0; a < TB; ++a)
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        red[mlp_slot<TB>(wave, lane, a, b, t)] = acc[a][b][t];
  __syncthreads();
  double e2 = 0.0;
  for (int e = tid; e < NE; e += kMlpWaves * 64) {
    const int64_t i = ti * E + e / E;
    const int j = (int)(tj * E) + e % E;
    if (i >= o.M || j >= o.N) continue;
    float c = 0.f;
    if (o.epi == kEpiWeightGrad && o.K > kMlpWaves * 32) {
      double d = 0.0;
#pragma unroll
      for (int v = 0; v < kMlpWaves; ++v) d += (double)red[v * NE + e];
      c = (float)d;
    } else {
#pragma unroll
      for (int v = 0; v < kMlpWaves; ++v) c += red[v * NE + e];
    }
    const int64_t at = i * o.N + j;
    if (o.epi == kEpiHidden) {
      const float z = c + o.aux[j];
      o.C[at] = z;
      o.C2[at] = silu(z);
    } else if (o.epi == kEpiOutput) {
      const float y = c + o.aux[j];
      o.C[at] = y;
      if (o.T) {
        const float d = y - o.T[at];
        o.C2[at] = 2.f * d / ((float)o.M * (float)o.N);
        e2 += (double)d * (double)d;
      }
    } else if (o.epi == kEpiInputGrad) {
      o.C[at] = c * silu_grad(o.aux[at]);
    } else {
      o.C[at] = c;
    }
  }
  if (o.epi == kEpiOutput && o.T) {
    e2 = mlp_block_sum(e2, tid);
    if (tid == 0) o.lossp[tile] = e2;
  }
}

// One launch: the tiles of two products, then 64 columns of a column sum per
// workgroup (eight groups of rows), then the loss.  LONG: batches of more than kMlpGroup
// rows, and any launch of 2^20 workgroups and more.
template <int TB, bool LONG>
__global__ __launch_bounds__(kMlpWaves * 64) void k_mlp(MlpOp o0, MlpOp o1, MlpColsum cs, MlpLoss ls) {
  __shared__ float red[kMlpWaves * 256 * TB * TB];
  const int tid = threadIdx.x;
  int64_t b = LONG ? long_block() : blockIdx.x;
  if (b < o0.tiles) return mlp_tile<TB, LONG>(o0, b, red, tid);
  b -= o0.tiles;
  if (b < o1.tiles) return mlp_tile<TB, LONG>(o1, b, red, tid);
  b -= o1.tiles;
  if (b < (cs.N + 63) / 64) {
    double *sums = reinterpret_cast<double *>(red);
    const int64_t j = b * 64 + (tid & 63);
    double s = 0.0;
    if (j < cs.N) {
      const float *p = cs.dZ + j;
      int64_t i = tid >> 6;
      for (; i + 7 * kMlpWaves < cs.n; i += 8 * kMlpWaves) {  // eight rows in flight
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(i + u * kMlpWaves) * cs.N];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (double)v[u];
      }
      for (; i < cs.n; i += kMlpWaves) s += (double)p[i * cs.N];
    }
    sums[tid] = s;
    __syncthreads();
    if (tid < 64 && j < cs.N) {
      for (int v = 1; v < kMlpWaves; ++v) s += sums[v * 64 + tid];
      cs.db[j] = (float)s;
    }
    return;
  }
  if (LONG && (b > (cs.N + 63) / 64 || ls.out == nullptr)) return;  // past the grid's last
  double s = 0.0;
  for (int64_t i = tid; i < ls.np; i += kMlpWaves * 64) s += ls.lossp[i];
  s = mlp_block_sum(s, tid);
  if (tid == 0) *ls.out = (ls.add ? *ls.out : 0.0) + s * ls.scale;
}

__global__ void k_adam(float *__restrict__ th, const float *__restrict__ g, float *__restrict__ m1,
                       float *__restrict__ m2, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + (1.f - b1) * gi;
  const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
  m1[i] = a;
  m2[i] = b;
  th[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// Y[i][j] = act(sum_k X[i][k] W[j][k] + bias[j]) with W in BF16 and X rounded to
// BF16 (FP32 accumulation): one wavefront per 16 x 16 output tile.
__global__ __launch_bounds__(64) void k_dense_bf16(const float *__restrict__ X, int n, int K,
                                                   const short *__restrict__ W, const float *__restrict__ bias,
                                                   int N, int act, float *__restrict__ Y) {
  const int lane = threadIdx.x;
  const int i0 = blockIdx.x * 16, j0 = blockIdx.y * 16;
  const int r = lane & 15, g = lane >> 4;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += 16) {
    shortx4 a, b;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + 4 * g + j;
      const int i = i0 + r, c = j0 + r;
      a[j] = (i < n && k < K) ? f2bf(X[(int64_t)i * K + k]) : (short)0;
      b[j] = (c < N && k < K) ? W[(int64_t)c * K + k] : (short)0;
    }
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 4 * g + q, c = j0 + r;
    if (i < n && c < N) {
      const float z = acc[q] + bias[c];
      Y[(int64_t)i * N + c] = act ? silu(z) : z;
    }
  }
}

// x = ((p, log_rate) - shift) / scale
__global__ void k_rollout_input(const float *__restrict__ p, int np_, float log_rate, const float *__restrict__ xs,
                                const float *__restrict__ xsc, float *__restrict__ x) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i > np_) return;
  const float v = i < np_ ? p[i] : log_rate;
  x[i] = (v - xs[i]) / xsc[i];
}

// p += y * scale + shift (or dp = that, when dp != NULL)
__global__ void k_rollout_update(float *__restrict__ p, const float *__restrict__ y, int np_,
                                 const float *__restrict__ ys, const float *__restrict__ ysc, float *__restrict__ dp) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= np_) return;
  const float d = y[i] * ysc[i] + ys[i];
  if (dp) dp[i] = d;
  else p[i] += d;
}

// ---- fused learned steps: one workgroup runs whole windows of steps ----

constexpr int kFusedThreads = 1024;
constexpr int kFusedMaxLdsFloats = 16384;  // 64 KiB of LDS per workgroup

__device__ inline float bf2f(short b) { return __uint_as_float((unsigned)(unsigned short)b << 16); }
__device__ inline float bf_round(float f) { return bf2f(f2bf(f)); }

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// out[j] = act(sum_k W[j][k] x[k] + bias[j]) for j < N: W in BF16 (row-major,
// N x K), x in LDS already rounded to BF16, FP32 sums (each lane takes
// k = lane, lane + 64, ..., then a butterfly over the wave); wave w of the
// block takes rows w, w + nw, ...  With `round_out` the result is stored
// rounded to BF16 (it is the next layer's input).
__device__ void gemv_bf16(const short *__restrict__ W, int N, int K, const float *x, const float *__restrict__ bias,
                          int act, bool round_out, float *out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = kFusedThreads / 64;
  for (int j0 = wave; j0 < N; j0 += 2 * nw) {
    const int j1 = j0 + nw;
    const short *r0 = W + (int64_t)j0 * K;
    const short *r1 = W + (int64_t)(j1 < N ? j1 : j0) * K;
    float s0 = 0.f, s1 = 0.f;
    for (int k = lane; k < K; k += 64) {
      const float xk = x[k];
      s0 = fmaf(bf2f(r0[k]), xk, s0);
      s1 = fmaf(bf2f(r1[k]), xk, s1);
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if (lane == 0) {
      float z = s0 + bias[j0];
      z = act ? silu(z) : z;
      out[j0] = round_out ? bf_round(z) : z;
      if (j1 < N) {
        z = s1 + bias[j1];
        z = act ? silu(z) : z;
        out[j1] = round_out ? bf_round(z) : z;
      }
    }
  }
}

// nsteps learned steps p += y * ysc + ys with y = network(((p, log_rate) - xs)
// / xsc), the same arithmetic as the BF16 inference path (inputs and hidden
// activations rounded to BF16, BF16 weights, FP32 sums and biases).  With dp
// non-null one increment is written there and p is left unchanged.  One
// workgroup of kFusedThreads; LDS holds x, both hidden layers and p.
__global__ __launch_bounds__(kFusedThreads) void k_rollout_fused(float *__restrict__ p, float *__restrict__ dp,
                                                                int np_, int w, float log_rate, int nsteps,
                                                                const short *__restrict__ W1,
                                                                const float *__restrict__ b1,
                                                                const short *__restrict__ W2,
                                                                const float *__restrict__ b2,
                                                                const short *__restrict__ W3,
                                                                const float *__restrict__ b3,
                                                                const float *__restrict__ xs,
                                                                const float *__restrict__ xsc,
                                                                const float *__restrict__ ys,
                                                                const float *__restrict__ ysc) {
  extern __shared__ float lds[];
  const int nin = np_ + 1;
  float *x = lds, *h1 = x + nin, *h2 = h1 + w, *ps = h2 + w, *y = ps + np_;
  for (int i = threadIdx.x; i < np_; i += kFusedThreads) ps[i] = p[i];
  __syncthreads();
  for (int step = 0; step < nsteps; ++step) {
    for (int i = threadIdx.x; i < nin; i += kFusedThreads) x[i] = bf_round(((i < np_ ? ps[i] : log_rate) - xs[i]) / xsc[i]);
    __syncthreads();
    gemv_bf16(W1, w, nin, x, b1, 1, true, h1);
    __syncthreads();
    gemv_bf16(W2, w, w, h1, b2, 1, true, h2);
    __syncthreads();
    gemv_bf16(W3, np_, w, h2, b3, 0, false, y);
    __syncthreads();
    for (int i = threadIdx.x; i < np_; i += kFusedThreads) {
      const float d = y[i] * ysc[i] + ys[i];
      if (dp != nullptr) dp[i] = d;
      else ps[i] += d;
    }
    __syncthreads();
  }
  if (dp == nullptr)
    for (int i = threadIdx.x; i < np_; i += kFusedThreads) p[i] = ps[i];
}

// Packing of the BF16 weights for k_learned_steps_reg.  Layers 1 and 2:
// thread t's chunk is contiguous, element kk = W_l[row][chunk * CK_l + kk]
// with (row, chunk) = (t / G_l, t % G_l).  Layer 3, as it sits in LDS: eight
// BF16 of slot s, group j (elements 8 j .. 8 j + 7 of its chunk) at uint4
// j * kSlots3 + s, so that neighbouring lanes read neighbouring 16 bytes.
// Zero outside the matrices.  One thread per packed element.
__global__ void k_pack_infer(const float *__restrict__ W1, const float *__restrict__ W2, const float *__restrict__ W3,
                             int nin, int w, int nout, short *__restrict__ pk) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= kPk1 + kPk2 + kPk3) return;
  const float *W;
  int G, CK, N, K;
  int64_t slot, kk;
  if (e < kPk1) {
    W = W1, G = kG1, CK = kCK1, N = w, K = nin, slot = e / kCK1, kk = e % kCK1;
  } else if (e < kPk1 + kPk2) {
    W = W2, G = kG2, CK = kCK2, N = w, K = w, slot = (e - kPk1) / kCK2, kk = (e - kPk1) % kCK2;
  } else {
    const int64_t f = e - kPk1 - kPk2, j = f / (8 * kSlots3);
    W = W3, G = kG3, CK = kCK3, N = nout, K = w, slot = (f / 8) % kSlots3, kk = 8 * j + f % 8;
  }
  const int64_t row = slot / G, k = (slot % G) * CK + kk;
  pk[e] = (row < N && k < K) ? f2bf(W[row * K + k]) : (short)0;
}

// Dot product of CK packed BF16 weights (registers) with CK floats of LDS.
template <int CK>
__device__ inline float dot_bf16(const uint2 (&wr)[CK / 4], const float *x) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < CK / 4; ++j) {
    const float4 xv = *reinterpret_cast<const float4 *>(x + 4 * j);
    s = fmaf(__uint_as_float(wr[j].x << 16), xv.x, s);
    s = fmaf(__uint_as_float(wr[j].x & 0xffff0000u), xv.y, s);
    s = fmaf(__uint_as_float(wr[j].y << 16), xv.z, s);
    s = fmaf(__uint_as_float(wr[j].y & 0xffff0000u), xv.w, s);
  }
  return s;
}

template <int G>
__device__ inline float group_sum(float v) {
#pragma unroll
  for (int off = G / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// nsteps learned steps with the weights on chip (layout of k_pack_infer), the
// arithmetic of the BF16 inference path: inputs and hidden activations
// rounded to BF16, FP32 products and sums (each lane sums its chunk in order,
// then a fixed butterfly over the row's lanes), FP32 biases.  With dp non-null
// one increment goes to dp and p is unchanged.
__global__ __launch_bounds__(kRegThreads) void k_learned_steps_reg(float *__restrict__ p, float *__restrict__ dp,
                                                                  int np_, int w, float log_rate, int nsteps,
                                                                  const short *__restrict__ pk,
                                                                  const float *__restrict__ b1,
                                                                  const float *__restrict__ b2,
                                                                  const float *__restrict__ b3,
                                                                  const float *__restrict__ xs,
                                                                  const float *__restrict__ xsc,
                                                                  const float *__restrict__ ys,
                                                                  const float *__restrict__ ysc) {
  __shared__ uint4 w3[kCK3 / 8 * kSlots3];
  __shared__ __align__(16) float x[kG1 * kCK1];
  __shared__ __align__(16) float h1[kG2 * kCK2];
  __shared__ __align__(16) float h2[kG3 * kCK3];
  __shared__ float ps[kNout3];
  __shared__ float y[kNout3];
  const int t = threadIdx.x, nin = np_ + 1;
  uint2 w1[kCK1 / 4], w2[kCK2 / 4];
  {
    const uint2 *q1 = reinterpret_cast<const uint2 *>(pk) + (int64_t)t * (kCK1 / 4);
    const uint2 *q2 = reinterpret_cast<const uint2 *>(pk + kPk1) + (int64_t)t * (kCK2 / 4);
#pragma unroll
    for (int j = 0; j < kCK1 / 4; ++j) w1[j] = q1[j];
#pragma unroll
    for (int j = 0; j < kCK2 / 4; ++j) w2[j] = q2[j];
    const uint4 *q3 = reinterpret_cast<const uint4 *>(pk + kPk1 + kPk2);
    for (int i = t; i < kCK3 / 8 * kSlots3; i += kRegThreads) w3[i] = q3[i];
  }
  const int r1 = t / kG1, c1 = t % kG1, c3 = t % kG3;
  for (int i = t; i < np_; i += kRegThreads) ps[i] = p[i];
  // padding of the layer inputs stays zero
  for (int i = t; i < kG1 * kCK1; i += kRegThreads) x[i] = 0.f;
  for (int i = t; i < kG2 * kCK2; i += kRegThreads) h1[i] = 0.f;
  for (int i = t; i < kG3 * kCK3; i += kRegThreads) h2[i] = 0.f;
  __syncthreads();
  for (int step = 0; step < nsteps; ++step) {
    // the packed weights stay packed: without this the BF16-to-FP32 unpacking
    // is hoisted out of the step loop and needs twice the registers
#pragma unroll
    for (int j = 0; j < kCK1 / 4; ++j) asm volatile("" : "+v"(w1[j].x), "+v"(w1[j].y));
#pragma unroll
    for (int j = 0; j < kCK2 / 4; ++j) asm volatile("" : "+v"(w2[j].x), "+v"(w2[j].y));
    for (int i = t; i < nin; i += kRegThreads) x[i] = bf_round(((i < np_ ? ps[i] : log_rate) - xs[i]) / xsc[i]);
    __syncthreads();
    float a = group_sum<kG1>(dot_bf16<kCK1>(w1, x + c1 * kCK1));
    if (c1 == 0 && r1 < w) h1[r1] = bf_round(silu(a + b1[r1]));
    __syncthreads();
    a = group_sum<kG2>(dot_bf16<kCK2>(w2, h1 + c1 * kCK2));
    if (c1 == 0 && r1 < w) h2[r1] = bf_round(silu(a + b2[r1]));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kS3; ++i) {
      const int slot = t + kRegThreads * i;  // uniform over each group of kG3 lanes
      if (slot < kSlots3) {
        const float *hx = h2 + c3 * kCK3;
        float s3 = 0.f;
#pragma unroll
        for (int j = 0; j < kCK3 / 8; ++j) {
          const uint4 wv = w3[j * kSlots3 + slot];
          const float4 xa = *reinterpret_cast<const float4 *>(hx + 8 * j);
          const float4 xb = *reinterpret_cast<const float4 *>(hx + 8 * j + 4);
          s3 = fmaf(__uint_as_float(wv.x << 16), xa.x, s3);
          s3 = fmaf(__uint_as_float(wv.x & 0xffff0000u), xa.y, s3);
          s3 = fmaf(__uint_as_float(wv.y << 16), xa.z, s3);
          s3 = fmaf(__uint_as_float(wv.y & 0xffff0000u), xa.w, s3);
          s3 = fmaf(__uint_as_float(wv.z << 16), xb.x, s3);
          s3 = fmaf(__uint_as_float(wv.z & 0xffff0000u), xb.y, s3);
          s3 = fmaf(__uint_as_float(wv.w << 16), xb.z, s3);
          s3 = fmaf(__uint_as_float(wv.w & 0xffff0000u), xb.w, s3);
        }
        a = group_sum<kG3>(s3);
        const int row = slot / kG3;
        if (c3 == 0 && row < np_) y[row] = a + b3[row];
      }
    }
    __syncthreads();
    for (int i = t; i < np_; i += kRegThreads) {
      const float d = y[i] * ysc[i] + ys[i];
      if (dp != nullptr) dp[i] = d;
      else ps[i] += d;
    }
    __syncthreads();
  }
  if (dp == nullptr)
    for (int i = t; i < np_; i += kRegThreads) p[i] = ps[i];
}

// SplitMix64 (Steele, Lea and Flood 2014): a counter-based stream of 64-bit
// values; one call per draw.
__device__ inline uint64_t splitmix64(uint64_t z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}
// Standard normal draw number `ctr` of stream `seed` by the Box-Muller
// transform of two SplitMix64 uniforms in (0, 1].
__device__ inline float normal_draw(uint64_t seed, uint64_t ctr) {
  const uint64_t a = splitmix64(seed ^ splitmix64(2 * ctr)), b = splitmix64(seed ^ splitmix64(2 * ctr + 1));
  const double u1 = ((double)(a >> 11) + 1.0) * 0x1.0p-53, u2 = (double)(b >> 11) * 0x1.0p-53;
  return (float)(sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}

// Minibatch rows i < nb: xin[i] = (X[order[i0 + i]] - xs) / xsc, tin likewise.
// With noise > 0 (learned steps, nin = nout + 1) input c < nout also gets
// noise * (ysc[c] / xsc[c]) * xi, xi standard normal from (seed, draw_base +
// row * nin + c): a perturbation of the state coefficient by `noise` standard
// deviations of its increment, the target unchanged.
__global__ void k_gather_scaled(const float *__restrict__ X, const float *__restrict__ T,
                                const int *__restrict__ order, int i0, int nb, int nin, int nout,
                                const float *__restrict__ xs, const float *__restrict__ xsc,
                                const float *__restrict__ ys, const float *__restrict__ ysc, float *__restrict__ xin,
                                float *__restrict__ tin, float noise, uint64_t seed, uint64_t draw_base) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row_len = nin + nout;
  if (t >= (int64_t)nb * row_len) return;
  const int i = (int)(t / row_len), c = (int)(t % row_len);
  const int64_t src = order ? order[i0 + i] : i0 + i;
  if (c < nin) {
    float x = (X[src * nin + c] - xs[c]) / xsc[c];
    if (noise > 0.f && c < nout)
      x += noise * (ysc[c] / xsc[c]) * normal_draw(seed, draw_base + (uint64_t)i * nin + c);
    xin[(int64_t)i * nin + c] = x;
  } else {
    tin[(int64_t)i * nout + (c - nin)] = (T[src * nout + (c - nin)] - ys[c - nin]) / ysc[c - nin];
  }
}

// Column mean and standard deviation of A[n][m] (FP64 sums); zero spread -> 1.
__global__ void k_col_stats(const float *__restrict__ A, int n, int m, float *__restrict__ mean,
                            float *__restrict__ sd) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= m) return;
  double s = 0.0, s2 = 0.0;
  for (int i = 0; i < n; ++i) {
    const double v = (double)A[(int64_t)i * m + j];
    s += v;
    s2 += v * v;
  }
  const double mu = s / n;
  const double var = fmax(s2 / n - mu * mu, 0.0);
  const double sdv = sqrt(var);
  mean[j] = (float)mu;
  sd[j] = (float)(sdv > 1e-30 * fmax(1.0, fabs(mu)) ? sdv : 1.0);
}

__global__ void k_make_pairs(const float *__restrict__ traj, int nt, int nout, float log_rate,
                             float *__restrict__ X, float *__restrict__ T) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)(nt - 1) * (nout + 1)) return;
  const int i = (int)(t / (nout + 1)), c = (int)(t % (nout + 1));
  if (c < nout) {
    const float a = traj[(int64_t)i * nout + c];
    X[(int64_t)i * (nout + 1) + c] = a;
    T[(int64_t)i * nout + c] = traj[(int64_t)(i + 1) * nout + c] - a;
  } else {
    X[(int64_t)i * (nout + 1) + c] = log_rate;
  }
}

inline unsigned nb256(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

struct vds_mlp_s {
  int nin, w, nout, B;
  int64_t np;
  hipStream_t s = nullptr;
  MlpLayout L{};
  char *ws = nullptr;
  float *params, *grads, *am, *av, *Z1, *A1, *Z2, *A2, *Y, *dY, *dZ1, *dZ2, *xs, *xsc, *ys, *ysc, *xin, *tin;
  short *wbf, *wpk;
  double *lossp;
  double *loss_out;  // one slot after the per-tile partials
  HostSlot host;  // a loss
  int t = 0;
  bool bf_stale = true;
  float noise = 0.f;          // training input noise (vds_mlp_set_input_noise)
  uint64_t noise_seed = 0, noise_draws = 0;
  std::string err;
  // parameter block views
  float *W1() { return params; }
  float *b1() { return params + (int64_t)w * nin; }
  float *W2() { return b1() + w; }
  float *b2() { return W2() + (int64_t)w * w; }
  float *W3() { return b2() + w; }
  float *b3() { return W3() + (int64_t)nout * w; }
};

namespace {

vds_status merr(vds_mlp m, vds_status st, const std::string &msg) {
  if (m) m->err = msg;
  return st;
}
vds_status mhip(vds_mlp m, hipError_t e, const char *what) {
  if (e == hipSuccess) return VDS_OK;
  return merr(m, VDS_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Tile edge of a launch in blocks of 16: wider tiles read less, but each product
// needs enough of them, since a tile's K is not split further than over its
// workgroup.  32 wide from 512 tiles on (two workgroups per compute unit): a
// minibatch of 2048 at 541-128-128-540 takes 112 us so and 121 with 16; 64 wide
// from 1024 on: 2049-2048-2048-2048 with 2048 rows 1.72 ms, 2.08 with 32 and
// 3.29 with 16.  By the smaller of the two products: 16384 rows at
// 541-128-128-540 take 0.78 ms with 16 and 1.19 when the many rows of one
// product choose 64 for both.
int mlp_edge(const MlpOp &a, const MlpOp &b) {
  auto tiles = [&](int tb) {
    const int64_t ta = mlp_tiles(a.M, a.N, tb);
    return b.M ? std::min(ta, mlp_tiles(b.M, b.N, tb)) : ta;
  };
  return tiles(4) >= 1024 ? 4 : tiles(2) >= 512 ? 2 : 1;
}

// Returns the tiles of the first product.
int64_t launch_mlp(vds_mlp m, MlpOp a, MlpOp b = MlpOp{}, const MlpColsum &cs = MlpColsum{},
                   const MlpLoss &ls = MlpLoss{}) {
  const int tb = mlp_edge(a, b);
  a.tiles = mlp_tiles(a.M, a.N, tb);
  b.tiles = mlp_tiles(b.M, b.N, tb);
  const int64_t n = a.tiles + b.tiles + (cs.N + 63) / 64 + (ls.out ? 1 : 0);
  const bool lng = (a.epi == kEpiWeightGrad && a.K > kMlpGroup) || (b.epi == kEpiWeightGrad && b.K > kMlpGroup) ||
                   n >= 1 << 20;
  auto go = [&](auto edge) {
    constexpr int TB = decltype(edge)::value;
    if (lng) k_mlp<TB, true><<<long_grid(n), kMlpWaves * 64, 0, m->s>>>(a, b, cs, ls);
    else k_mlp<TB, false><<<(unsigned)n, kMlpWaves * 64, 0, m->s>>>(a, b, cs, ls);
  };
  if (tb == 4) go(std::integral_constant<int, 4>{});
  else if (tb == 2) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 1>{});
  return a.tiles;
}

// Z (n x N) = X W^T + bias, X: n x K, W: N x K, and A = silu(Z); in the last
// layer (A null) with targets T also dY and the loss partials.
MlpOp dense(const float *X, int n, int K, const float *W, const float *bias, int N, float *Z, float *A) {
  MlpOp o{};
  o.M = n, o.N = N, o.K = K;
  o.epi = A ? kEpiHidden : kEpiOutput;
  o.A = X, o.lda = K;
  o.B = W, o.ldb = K;
  o.aux = bias;
  o.C = Z, o.C2 = A;
  return o;
}

// dZ of the layer below (n x K) = (dZ W) silu'(Z), dZ: n x N, W: N x K
MlpOp input_grad(const float *dZ, int n, int N, const float *W, int K, const float *Z, float *out) {
  MlpOp o{};
  o.M = n, o.N = K, o.K = N;
  o.epi = kEpiInputGrad;
  o.A = dZ, o.lda = N;
  o.B = W, o.ldb = K;
  o.aux = Z;
  o.C = out;
  return o;
}

// dW (N x K) = dZ^T A, dZ: n x N, A: n x K
MlpOp weight_grad(const float *dZ, int n, int N, const float *A, int K, float *dW) {
  MlpOp o{};
  o.M = N, o.N = K, o.K = n;
  o.epi = kEpiWeightGrad;
  o.A = dZ, o.lda = N;
  o.B = A, o.ldb = K;
  o.C = dW;
  return o;
}

// Y (n x nout); with targets T also dY, the loss partials and their number.
int64_t forward_fp32(vds_mlp m, const float *X, int n, float *Y, const float *T = nullptr) {
  launch_mlp(m, dense(X, n, m->nin, m->W1(), m->b1(), m->w, m->Z1, m->A1));
  launch_mlp(m, dense(m->A1, n, m->w, m->W2(), m->b2(), m->w, m->Z2, m->A2));
  MlpOp out = dense(m->A2, n, m->w, m->W3(), m->b3(), m->nout, Y, nullptr);
  out.T = T;
  out.C2 = m->dY;
  out.lossp = m->lossp;
  return launch_mlp(m, out);
}

// Gradients and loss of one minibatch; the loss is added to *loss or put there.
void loss_grad_fp32(vds_mlp m, const float *X, const float *T, int n, double *loss, bool add_loss) {
  const int w = m->w, nin = m->nin, nout = m->nout;
  float *gW1 = m->grads, *gb1 = gW1 + (int64_t)w * nin, *gW2 = gb1 + w, *gb2 = gW2 + (int64_t)w * w,
        *gW3 = gb2 + w, *gb3 = gW3 + (int64_t)nout * w;
  const int64_t np = forward_fp32(m, X, n, m->Y, T);
  launch_mlp(m, input_grad(m->dY, n, nout, m->W3(), w, m->Z2, m->dZ2), weight_grad(m->dY, n, nout, m->A2, w, gW3),
             MlpColsum{m->dY, n, nout, gb3});
  launch_mlp(m, input_grad(m->dZ2, n, w, m->W2(), w, m->Z1, m->dZ1), weight_grad(m->dZ2, n, w, m->A1, w, gW2),
             MlpColsum{m->dZ2, n, w, gb2});
  launch_mlp(m, weight_grad(m->dZ1, n, w, X, nin, gW1), MlpOp{}, MlpColsum{m->dZ1, n, w, gb1},
             MlpLoss{m->lossp, np, 1.0 / ((double)n * nout), add_loss, loss});
}

void refresh_bf16(vds_mlp m) {
  if (!m->bf_stale) return;
  k_to_bf16<<<nb256(m->np), 256, 0, m->s>>>(m->params, m->wbf, m->np);
  if (reg_steps_fit(m->nin, m->w, m->nout))
    k_pack_infer<<<nb256(kPk1 + kPk2 + kPk3), 256, 0, m->s>>>(m->W1(), m->W2(), m->W3(), m->nin, m->w, m->nout,
                                                              m->wpk);
  m->bf_stale = false;
}

// LDS floats of the fused step kernel: x, two hidden layers, p and the output.
int64_t fused_lds_floats(vds_mlp m) { return (int64_t)m->nin + 2 * m->w + 2 * (int64_t)m->nout; }

// nsteps learned steps on p (or one increment into dp): the kernel with the
// weights on chip, or the one streaming them, or the layer-by-layer BF16
// kernels step by step.
void learned_steps(vds_mlp m, float *p, float *dp, float log_rate, int nsteps);

void forward_bf16(vds_mlp m, const float *X, int n, float *Y) {
  refresh_bf16(m);
  const int w = m->w;
  const short *W1 = m->wbf, *W2 = W1 + (int64_t)w * m->nin + w, *W3 = W2 + (int64_t)w * w + w;
  dim3 g1((n + 15) / 16, (w + 15) / 16), g3((n + 15) / 16, (m->nout + 15) / 16);
  k_dense_bf16<<<g1, 64, 0, m->s>>>(X, n, m->nin, W1, m->b1(), w, 1, m->A1);
  k_dense_bf16<<<g1, 64, 0, m->s>>>(m->A1, n, w, W2, m->b2(), w, 1, m->A2);
  k_dense_bf16<<<g3, 64, 0, m->s>>>(m->A2, n, w, W3, m->b3(), m->nout, 0, Y);
}

void learned_steps(vds_mlp m, float *p, float *dp, float log_rate, int nsteps) {
  const int np_ = m->nout;
  refresh_bf16(m);
  if (reg_steps_fit(m->nin, m->w, m->nout)) {
    k_learned_steps_reg<<<1, kRegThreads, 0, m->s>>>(p, dp, np_, m->w, log_rate, dp != nullptr ? 1 : nsteps, m->wpk,
                                                     m->b1(), m->b2(), m->b3(), m->xs, m->xsc, m->ys, m->ysc);
    return;
  }
  if (fused_lds_floats(m) <= kFusedMaxLdsFloats) {
    const int w = m->w;
    const short *W1 = m->wbf, *W2 = W1 + (int64_t)w * m->nin + w, *W3 = W2 + (int64_t)w * w + w;
    const size_t lds = sizeof(float) * (size_t)fused_lds_floats(m);
    k_rollout_fused<<<1, kFusedThreads, lds, m->s>>>(p, dp, np_, w, log_rate, dp != nullptr ? 1 : nsteps, W1, m->b1(),
                                                     W2, m->b2(), W3, m->b3(), m->xs, m->xsc, m->ys, m->ysc);
    return;
  }
  float *xb = m->xin, *yb = m->Y;
  for (int i = 0; i < (dp != nullptr ? 1 : nsteps); ++i) {
    k_rollout_input<<<nb256(np_ + 1), 256, 0, m->s>>>(p, np_, log_rate, m->xs, m->xsc, xb);
    forward_bf16(m, xb, 1, yb);
    k_rollout_update<<<nb256(np_), 256, 0, m->s>>>(dp != nullptr ? nullptr : p, yb, np_, m->ys, m->ysc, dp);
  }
}

}  // namespace

extern "C" {

size_t vds_mlp_workspace_bytes(int32_t nin, int32_t w, int32_t nout, int32_t B) {
  if (nin < 1 || w < 1 || nout < 1 || B < 1 || nin > 65536 || w > 65536 || nout > 65536 || B > (1 << 20)) return 0;
  return mlp_layout(nin, w, nout, B).total;
}

vds_status vds_mlp_create(int32_t nin, int32_t w, int32_t nout, int32_t B, void *stream, vds_mlp *out) {
  if (out == nullptr) {
    g_mlp_create_error = "out is NULL";
    return VDS_ERR_ARG;
  }
  *out = nullptr;
  if (vds_mlp_workspace_bytes(nin, w, nout, B) == 0) {
    g_mlp_create_error = "invalid sizes";
    return VDS_ERR_ARG;
  }
  vds_mlp m = new (std::nothrow) vds_mlp_s();
  if (!m) {
    g_mlp_create_error = "host allocation failed";
    return VDS_ERR_NOMEM;
  }
  m->nin = nin;
  m->w = w;
  m->nout = nout;
  m->B = B;
  m->np = nparams(nin, w, nout);
  m->s = reinterpret_cast<hipStream_t>(stream);
  m->L = mlp_layout(nin, w, nout, B);
  *out = m;
  return VDS_OK;
}

vds_status vds_mlp_bind_workspace(vds_mlp m, void *ws, size_t bytes) {
  if (!m) return VDS_ERR_ARG;
  if (!ws || reinterpret_cast<uintptr_t>(ws) % 256) return merr(m, VDS_ERR_ARG, "workspace must be 256-byte aligned");
  if (bytes < m->L.total) return merr(m, VDS_ERR_NOMEM, "workspace too small");
  m->ws = static_cast<char *>(ws);
  const MlpLayout &L = m->L;
  auto f = [&](size_t o) { return reinterpret_cast<float *>(m->ws + o); };
  m->params = f(L.params);
  m->grads = f(L.grads);
  m->am = f(L.adam_m);
  m->av = f(L.adam_v);
  m->wbf = reinterpret_cast<short *>(m->ws + L.wbf);
  m->wpk = reinterpret_cast<short *>(m->ws + L.wpk);
  m->Z1 = f(L.Z1);
  m->A1 = f(L.A1);
  m->Z2 = f(L.Z2);
  m->A2 = f(L.A2);
  m->Y = f(L.Y);
  m->dY = f(L.dY);
  m->dZ1 = f(L.dZ1);
  m->dZ2 = f(L.dZ2);
  m->xs = f(L.xs);
  m->xsc = f(L.xsc);
  m->ys = f(L.ys);
  m->ysc = f(L.ysc);
  m->xin = f(L.xin);
  m->tin = f(L.tin);
  m->lossp = reinterpret_cast<double *>(m->ws + L.lossp);
  m->loss_out = m->lossp + mlp_tiles(m->B, m->nout, 1);
  // identity scaling until set
  std::vector<float> zx(m->nin, 0.f), ox(m->nin, 1.f), zy(m->nout, 0.f), oy(m->nout, 1.f);
  vds_status st = mhip(m, hipMemcpyAsync(m->xs, zx.data(), 4 * m->nin, hipMemcpyHostToDevice, m->s), "init");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->xsc, ox.data(), 4 * m->nin, hipMemcpyHostToDevice, m->s), "init");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->ys, zy.data(), 4 * m->nout, hipMemcpyHostToDevice, m->s), "init");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->ysc, oy.data(), 4 * m->nout, hipMemcpyHostToDevice, m->s), "init");
  if (st == VDS_OK) st = mhip(m, hipStreamSynchronize(m->s), "synchronise");
  return st;
}

void vds_mlp_destroy(vds_mlp m) { delete m; }
const char *vds_mlp_last_error(vds_mlp m) { return m ? m->err.c_str() : g_mlp_create_error.c_str(); }
int64_t vds_mlp_param_count(vds_mlp m) { return m ? m->np : -1; }

vds_status vds_mlp_set_params(vds_mlp m, const float *p) {
  if (!m || !p) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  vds_status st = mhip(m, hipMemcpyAsync(m->params, p, 4 * m->np, hipMemcpyDeviceToDevice, m->s), "copy");
  if (st == VDS_OK) st = mhip(m, hipMemsetAsync(m->am, 0, 4 * m->np, m->s), "clear");
  if (st == VDS_OK) st = mhip(m, hipMemsetAsync(m->av, 0, 4 * m->np, m->s), "clear");
  m->t = 0;
  m->bf_stale = true;
  return st;
}

vds_status vds_mlp_get_params(vds_mlp m, float *p) {
  if (!m || !p) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  return mhip(m, hipMemcpyAsync(p, m->params, 4 * m->np, hipMemcpyDeviceToDevice, m->s), "copy");
}

vds_status vds_mlp_get_grads(vds_mlp m, float *g) {
  if (!m || !g) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  return mhip(m, hipMemcpyAsync(g, m->grads, 4 * m->np, hipMemcpyDeviceToDevice, m->s), "copy");
}

vds_status vds_mlp_forward(vds_mlp m, const float *X, int32_t n, float *Y, int32_t bf16) {
  if (!m || !X || !Y) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  if (n < 1 || n > m->B) return merr(m, VDS_ERR_ARG, "batch size out of range");
  if (bf16) {
    forward_bf16(m, X, n, Y);
  } else {
    forward_fp32(m, X, n, Y);
  }
  return mhip(m, hipGetLastError(), "forward");
}

vds_status vds_mlp_set_input_noise(vds_mlp m, float sigma, uint64_t seed) {
  if (!m) return VDS_ERR_ARG;
  if (!(sigma >= 0.f) || !std::isfinite(sigma)) return merr(m, VDS_ERR_ARG, "noise must be finite and >= 0");
  if (sigma > 0.f && m->nin != m->nout + 1) return merr(m, VDS_ERR_ARG, "input noise needs nin = nout + 1");
  m->noise = sigma;
  m->noise_seed = seed;
  m->noise_draws = 0;
  return VDS_OK;
}

vds_status vds_mlp_predict_steps(vds_mlp m, float *p, float log_rate, int32_t nsteps) {
  if (!m || !p) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  if (m->nin != m->nout + 1) return merr(m, VDS_ERR_ARG, "learned steps need nin = nout + 1");
  if (nsteps < 0) return merr(m, VDS_ERR_ARG, "nsteps < 0");
  if (nsteps > 0) learned_steps(m, p, nullptr, log_rate, nsteps);
  return mhip(m, hipGetLastError(), "learned steps");
}

vds_status vds_mlp_loss_grad(vds_mlp m, const float *X, const float *T, int32_t n, double *loss) {
  if (!m || !X || !T) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  if (n < 1 || n > m->B) return merr(m, VDS_ERR_ARG, "batch size out of range");
  double *host = loss != nullptr ? static_cast<double *>(m->host.take(sizeof(double))) : nullptr;
  loss_grad_fp32(m, X, T, n, host != nullptr ? host : m->loss_out, false);
  vds_status st = mhip(m, hipGetLastError(), "loss_grad");
  if (st != VDS_OK || loss == nullptr) return st;
  if (host == nullptr)
    st = mhip(m, hipMemcpyAsync(loss, m->loss_out, sizeof(double), hipMemcpyDeviceToHost, m->s), "copy loss");
  if (st == VDS_OK) st = mhip(m, hipStreamSynchronize(m->s), "synchronise");
  if (st == VDS_OK && host != nullptr) {
    *loss = *host;
    m->host.read();
  }
  return st;
}

vds_status vds_mlp_adam_step(vds_mlp m, float lr, float b1, float b2, float eps) {
  if (!m) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  m->t += 1;
  const float c1 = 1.f - std::pow(b1, (float)m->t), c2 = 1.f - std::pow(b2, (float)m->t);
  k_adam<<<nb256(m->np), 256, 0, m->s>>>(m->params, m->grads, m->am, m->av, m->np, lr, b1, b2, eps, c1, c2);
  m->bf_stale = true;
  return mhip(m, hipGetLastError(), "adam");
}

vds_status vds_mlp_train_epoch(vds_mlp m, const float *X, const float *T, int32_t n, int32_t batch, float lr,
                               const int32_t *order, double *loss) {
  if (!m || !X || !T) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  if (batch < 1 || batch > m->B || n < batch) return merr(m, VDS_ERR_ARG, "bad batch size");
  const int nbatch = n / batch;
  double acc = 0.0;
  for (int bi = 0; bi < nbatch; ++bi) {
    k_gather_scaled<<<nb256((int64_t)batch * (m->nin + m->nout)), 256, 0, m->s>>>(
        X, T, order, bi * batch, batch, m->nin, m->nout, m->xs, m->xsc, m->ys, m->ysc, m->xin, m->tin, m->noise,
        m->noise_seed, m->noise_draws);
    m->noise_draws += (uint64_t)batch * m->nin;
    loss_grad_fp32(m, m->xin, m->tin, batch, m->loss_out, bi > 0);
    // (takes the launch errors of the whole minibatch)
    vds_status st = vds_mlp_adam_step(m, lr, 0.9f, 0.999f, 1e-8f);
    if (st != VDS_OK) return st;
  }
  vds_status st = VDS_OK;
  if (loss)
    st = mhip(m, hipMemcpyAsync(&acc, m->loss_out, sizeof(double), hipMemcpyDeviceToHost, m->s), "copy");
  if (st == VDS_OK) st = mhip(m, hipStreamSynchronize(m->s), "synchronise");
  if (st == VDS_OK && loss) *loss = acc / nbatch;
  return st;
}

vds_status vds_mlp_fit_scaling(vds_mlp m, const float *X, const float *T, int32_t n) {
  if (!m || !X || !T || n < 1) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  k_col_stats<<<nb256(m->nin), 256, 0, m->s>>>(X, n, m->nin, m->xs, m->xsc);
  k_col_stats<<<nb256(m->nout), 256, 0, m->s>>>(T, n, m->nout, m->ys, m->ysc);
  return mhip(m, hipGetLastError(), "fit scaling");
}

vds_status vds_mlp_make_pairs(vds_mlp m, const float *traj, int32_t nt, float log_rate, float *X, float *T) {
  if (!m || !traj || !X || !T || nt < 2) return VDS_ERR_ARG;
  if (m->nin != m->nout + 1) return merr(m, VDS_ERR_ARG, "pairs need nin = nout + 1");
  k_make_pairs<<<nb256((int64_t)(nt - 1) * (m->nout + 1)), 256, 0, m->s>>>(traj, nt, m->nout, log_rate, X, T);
  return mhip(m, hipGetLastError(), "make pairs");
}

vds_status vds_mlp_set_scaling(vds_mlp m, const float *xs, const float *xsc, const float *ys, const float *ysc) {
  if (!m || !xs || !xsc || !ys || !ysc) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  vds_status st = mhip(m, hipMemcpyAsync(m->xs, xs, 4 * m->nin, hipMemcpyDeviceToDevice, m->s), "copy");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->xsc, xsc, 4 * m->nin, hipMemcpyDeviceToDevice, m->s), "copy");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->ys, ys, 4 * m->nout, hipMemcpyDeviceToDevice, m->s), "copy");
  if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(m->ysc, ysc, 4 * m->nout, hipMemcpyDeviceToDevice, m->s), "copy");
  return st;
}

size_t vds_mlp_rollout_workspace_bytes(const vds_problem *prob, int32_t R) {
  if (!prob || prob->P < 1 || prob->nb < 1 || R < 1) return 0;
  const size_t q = sizeof(float) * 3 * (size_t)prob->P * prob->nb;
  const size_t pr = sizeof(float) * (size_t)prob->nb * R;
  const size_t mapw = vds_pod_map_workspace_bytes(prob, R);
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  return 2 * up(q) + 4 * up(pr) + up(mapw) + up(sizeof(float) * 16 * (prob->nb * R + 1));
}

vds_status vds_mlp_rollout_run(vds_mlp m, vds_ctx ctx, const float *U, int32_t R, float *p, float log_rate,
                               int32_t nsteps, int32_t K, double resid_tol, double energy_tol, void *ws,
                               size_t bytes, vds_mlp_rollout *stats) {
  if (!m || !ctx || !U || !p || !ws) return VDS_ERR_ARG;
  if (!m->ws) return merr(m, VDS_ERR_STATE, "no workspace bound");
  const vds_problem &pr = ctx->prob;
  const int np_ = pr.nb * R;
  if (m->nin != np_ + 1 || m->nout != np_) return merr(m, VDS_ERR_ARG, "network sizes do not match nb R");
  if (nsteps < 0 || K < 1) return merr(m, VDS_ERR_ARG, "bad step counts");
  if (bytes < vds_mlp_rollout_workspace_bytes(&pr, R)) return merr(m, VDS_ERR_NOMEM, "rollout workspace too small");
  if (ctx->stream != m->s) return merr(m, VDS_ERR_ARG, "context and network must share a stream");
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  char *w = static_cast<char *>(ws);
  const size_t qb = up(sizeof(float) * 3 * (size_t)pr.P * pr.nb), pb = up(sizeof(float) * np_);
  float *qt = reinterpret_cast<float *>(w);
  float *v = reinterpret_cast<float *>(w + qb);
  float *p_acc = reinterpret_cast<float *>(w + 2 * qb);
  float *dp_vds = reinterpret_cast<float *>(w + 2 * qb + pb);
  float *dp_net = reinterpret_cast<float *>(w + 2 * qb + 2 * pb);
  const size_t mapw = vds_pod_map_workspace_bytes(&pr, R);
  void *mws = w + 2 * qb + 4 * pb;

  vds_mlp_rollout S{};
  // energy at the reconstructed state, and the plain scheme's velocity there
  auto observe = [&](const float *pin, vds_diag *d) -> vds_status {
    vds_status st = vds_pod_reconstruct(ctx, U, R, pin, qt, mws, mapw);
    if (st == VDS_OK) st = vds_velocity(ctx, qt, nullptr, v, d);
    return st;
  };
  vds_diag d0{}, d1{};
  vds_status st = observe(p, &d0);
  if (st != VDS_OK) return st;
  const double dt = pr.dt;
  std::vector<float> a((size_t)np_), b((size_t)np_);
  for (int s0 = 0; s0 < nsteps; s0 += K) {
    const int n = std::min(K, nsteps - s0);
    st = mhip(m, hipMemcpyAsync(p_acc, p, 4 * np_, hipMemcpyDeviceToDevice, m->s), "copy");
    if (st != VDS_OK) return st;
    learned_steps(m, p, nullptr, log_rate, n);
    st = observe(p, &d1);
    // a reconstructed FENE bond outside the spring's domain fails the window
    const bool outside = st == VDS_ERR_ARG && pr.potential == VDS_FENE;
    if (outside) st = VDS_OK;
    if (st != VDS_OK) return st;
    double resid = HUGE_VAL, egap = HUGE_VAL;
    if (!outside) {
      // full-step residual at the window's end state
      learned_steps(m, p, dp_net, log_rate, 1);
      st = vds_pod_project(ctx, U, R, v, dp_vds, mws, mapw);
      if (st != VDS_OK) return st;
      st = mhip(m, hipMemcpyAsync(a.data(), dp_net, 4 * np_, hipMemcpyDeviceToHost, m->s), "copy");
      if (st == VDS_OK) st = mhip(m, hipMemcpyAsync(b.data(), dp_vds, 4 * np_, hipMemcpyDeviceToHost, m->s), "copy");
      if (st == VDS_OK) st = mhip(m, hipStreamSynchronize(m->s), "synchronise");
      if (st != VDS_OK) return st;
      double num = 0.0, den = 0.0;
      for (int i = 0; i < np_; ++i) {
        const double ref = dt * (double)b[i];
        num += ((double)a[i] - ref) * ((double)a[i] - ref);
        den += ref * ref;
      }
      resid = std::sqrt(num / std::max(den, 1e-300));
      const double rate0 = d0.work - d0.dissipation, rate1 = d1.work - d1.dissipation;
      const double gap = std::fabs(d1.F - d0.F - 0.5 * dt * n * (rate0 + rate1));
      const double scale =
          0.5 * dt * n * (std::fabs(d0.work) + d0.dissipation + std::fabs(d1.work) + d1.dissipation);
      egap = gap / std::max(scale, 1e-300);
      S.max_resid = std::max(S.max_resid, resid);
      S.max_energy_gap = std::max(S.max_energy_gap, egap);
    }
    S.checks += 1;
    if (outside || !(resid <= resid_tol) || !(egap <= energy_tol)) {
      // redo the window with the plain scheme from its start
      st = vds_pod_reconstruct(ctx, U, R, p_acc, qt, mws, mapw);
      if (st == VDS_OK) st = vds_step(ctx, qt, nullptr, n, nullptr);
      if (st == VDS_OK) st = vds_pod_project(ctx, U, R, qt, p, mws, mapw);
      if (st == VDS_OK) st = observe(p, &d1);
      if (st != VDS_OK) return st;
      S.fallbacks += 1;
    }
    d0 = d1;
    S.steps += n;
  }
  std::memcpy(S.tau, d0.tau, sizeof(S.tau));
  if (stats) *stats = S;
  return VDS_OK;
}

}  // extern "C"
