// Dense linear algebra for the POD offline phase and the reduced operators:
//  * GEMMs  C = alpha * sum_b A_b diag(s) B_b^T  (split-K partials, reduced in a
//    fixed order), operands K-contiguous or MN-contiguous, on BF16 matrix cores
//    from three BF16 parts per factor;
//  * single-workgroup FP64 kernels for small dense matrices (Cholesky factor
//    and triangular inverse, conversions).
#include <type_traits>

#include "bf3.h"
#include "vds_internal.h"
#include "vds_linalg.h"

namespace vds {

// ---- large products from three BF16 parts ------------------------------------
//
// One workgroup: a 96 x 96 output tile over the rounds of its split, 32 k each;
// wave w owns the 48 x 48 quadrant (w / 2, w % 2), 3 x 3 blocks of 16.  Lane l
// works on row l % 16 of each block and on k 4 g .. + 3 and 16 + 4 g .. + 3
// (g = l / 16; the order of k inside a round does not matter as long as both
// operands share it), cuts its eight values into three BF16 parts (gemm_cut) and
// takes the six products hh, hm, mh, mm, hl, lh of each block (the others are
// below 2^-26: the parts are rounded to nearest, so what is left out has no sign).
// K-contiguous operands come through LDS in FP32, a round ahead, by loads that go
// there directly; MN-contiguous ones straight into registers, where a wave's
// sixteen rows are contiguous (K-contiguous ones would take 64 address cycles per
// load instead of 16: only adjacent lanes are merged).  Two waves cut the same
// rows: with the parts in LDS instead of the values, a round's 37 KB of writes and
// 74 KB of reads at 32 and 64 bytes a cycle took 2300 cycles against 864 of matrix
// instructions.
// 96 wide: 540, 180 and 900 columns waste 7 to 14 % of a row of tiles, and a wave's
// sums leave room for three workgroups per compute unit (192 wide spills).
// XCD x runs consecutive (split, tile), so that a split's tiles read the same
// rounds through one L2.
// Bound: matrix pipe, 78 instructions of 16 cycles per round and wave (62 % busy).
// Measured: Gram of 60000 x 900 0.37 ms (0.52 with parts cut once and kept in LDS;
// 0.43 with the remainders formed by vector instructions, which a SIMD issues one
// every four cycles; 1.48 with FP32 matrix instructions); the two 180 x 180 x 60000
// products of a reduced operator build 38 and 37 us (44 and 51; 123 and 140).
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// Eight values of a lane into three operands, each the values so far rounded to
// nearest BF16; what that leaves is formed on the matrix cores (minus the identity
// times the part, added to the values, which sit as a tile of the accumulator's
// layout): 12 vector and 4 matrix instructions against 44 vector ones, of which a
// SIMD issues one every four cycles.
__device__ __forceinline__ void gemm_cut(float (&v)[8], const bf16x8 (&neg)[2], bf16x8 (&f)[3]) {
  floatx4 e[2] = {{v[0], v[1], v[2], v[3]}, {v[4], v[5], v[6], v[7]}};
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    // (conversions, not assembly: the compiler has to see who reads a matrix result)
#pragma unroll
    for (int i = 0; i < 8; ++i) f[p][i] = (__bf16)e[i / 4][i % 4];
    if (p < 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) e[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(neg[b], f[p], e[b], 0, 0, 0);
    }
  }
}

// VEC: every row of the K-contiguous operands starts on 16 bytes.
template <bool A_MN, bool B_MN, bool SCALE, bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(VEC && !A_MN && !B_MN && !SCALE ? 3 : 2))) void k_gemm_bf3(
    GemmShape g, int tn, int ntile, float *__restrict__ part) {
  constexpr int NB = kGemmTile / 32;  // 16-row blocks of a wave, each way
  // staged pieces of 8 rows x 128 bytes of each operand's round
  constexpr int kPiecesA = A_MN ? 0 : kGemmTile / 8, kPiecesB = B_MN ? 0 : kGemmTile / 8;
  constexpr int kLds = (kPiecesA + kPiecesB) * 64;
  static_assert(kLds > 0, "at most one operand is MN-contiguous");
  __shared__ float4 lds[2][kLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the grid is a multiple of eight: XCD x takes a run of consecutive (split, tile)
  const int id = (int)(blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8);
  if (id >= ntile * g.splits) return;
  const int split = id / ntile, tile = id % ntile;
  int ti, tj;
  if (g.symmetric) {  // tiles ti <= tj, row by row
    ti = 0;
    int left = tile;
    while (left >= tn - ti) left -= tn - ti, ++ti;
    tj = ti + left;
  } else {
    ti = tile / tn;
    tj = tile % tn;
  }
  const int wi = (wave >> 1) * 16 * NB, wj = (wave & 1) * 16 * NB;
  const int i0 = ti * kGemmTile + wi, j0 = tj * kGemmTile + wj;
  const int m = lane & 15, kl = 4 * (lane >> 4);

  // rows past the operand's read its last row (their outputs are not written)
  const float *pa[NB], *pb[NB];
#pragma unroll
  for (int a = 0; a < NB; ++a) {
    const int64_t r = min(i0 + 16 * a + m, g.M - 1);
    pa[a] = g.A + (A_MN ? r + kl * g.lda : r * g.lda + kl);
  }
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const int64_t r = min(j0 + 16 * c + m, g.N - 1);
    pb[c] = g.B + (B_MN ? r + kl * g.ldb : r * g.ldb + kl);
  }
  float va[NB][8], vb[NB][8], sc[8];
  auto read = [&](auto mn, const float *p, int64_t ld, float (&v)[8]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (decltype(mn)::value) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * h + e] = p[(16 * h + e) * ld];
      } else {
        const float4u f = *reinterpret_cast<const float4u *>(p + 16 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * h + e] = f[e];
      }
    }
  };
  // the same where the round passes K: n = K - k0 values are there
  auto read_end = [&](auto mn, const float *p, int64_t ld, int n, float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 16 * (e / 4) + e % 4;
      v[e] = kl + k < n ? p[decltype(mn)::value ? k * ld : k] : 0.f;
    }
  };
  using amn = std::integral_constant<bool, A_MN>;
  using bmn = std::integral_constant<bool, B_MN>;

  // the upper parts' products, and the others apart: added to a long sum one by
  // one, what is below half a unit of it would be lost (on a Gram's diagonal,
  // where the mm products are all positive, 5e-7 to 2e-6 of the entry)
  floatx4 acc[NB][NB], low[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = low[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[NB][3], fb[3], neg[2];
  minus_identity(lane, neg);
  auto products = [&](int c) {
    constexpr int xa[6] = {2, 0, 1, 1, 0, 0}, xb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int x = 0; x < 6; ++x)
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        floatx4 &t = x < 5 ? low[a][c] : acc[a][c];
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a][xa[x]], fb[xb[x]], t, 0, 0, 0);
      }
  };
  auto cut_b = [&](int c) {
    if constexpr (SCALE) {
#pragma unroll
      for (int e = 0; e < 8; ++e) vb[c][e] *= sc[e];
    }
    gemm_cut(vb[c], neg, fb);
  };

  // A staged row's eight 16-byte groups of k are exchanged by its row: group c sits
  // at c ^ (row / 2), so that sixteen rows' reads of one group cover all banks.
  // This thread's share of a round of an operand whose pieces follow piece p0: 16
  // bytes of row 8 piece + lane / 8 per piece and lane, straight to LDS, or with
  // rows off 16 bytes into registers first (put).
  float4u hold[VEC ? 1 : (kPiecesA + kPiecesB) / 4 + 1];
  auto stage = [&](auto npieces, const float *src, int64_t ld, int row0, int nrows, int p0, int b) {
#pragma unroll
    for (int i = 0; i < decltype(npieces)::value / 4; ++i) {
      const int pc = wave + 4 * i, row = 8 * pc + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
      const float *q = src + (int64_t)min(row0 + row, nrows - 1) * ld + 4 * c;
      if constexpr (VEC)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)q,
                                         (__attribute__((address_space(3))) void *)&lds[b][(p0 + pc) * 64], 16, 0, 0);
      else hold[p0 / 4 + i] = *reinterpret_cast<const float4u *>(q);
    }
  };
  auto put = [&](int b) {
    if constexpr (!VEC) {
#pragma unroll
      for (int i = 0; i < (kPiecesA + kPiecesB) / 4; ++i)
        *reinterpret_cast<floatx4 *>(&lds[b][(wave + 4 * i) * 64 + lane]) = hold[i];
    }
  };
  auto staged = [&](int p0, int b, int block, float (&v)[8]) {
    const float4 *src = &lds[b][p0 * 64 + block * 128 + m * 8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 f = src[(4 * h + (lane >> 4)) ^ (m >> 1)];
      v[4 * h] = f.x, v[4 * h + 1] = f.y, v[4 * h + 2] = f.z, v[4 * h + 3] = f.w;
    }
  };
  // full rounds [u, u_end) of all batches end to end; offsets of round u
  const int64_t per = g.K / kGemmSlab;
  int64_t u = per * g.nbatch * split / g.splits;
  const int64_t u_end = per * g.nbatch * (split + 1) / g.splits;
  int64_t bt = per > 0 ? u / per : 0, kr = u - bt * per;
  const float *ps = SCALE ? g.scale + kl : nullptr;
  int64_t oa = 0, ob = 0, os = 0;
  auto offsets = [&] {
    const int64_t k0 = kr * kGemmSlab;
    oa = bt * g.sA + (A_MN ? k0 * g.lda : k0);
    ob = bt * g.sB + (B_MN ? k0 * g.ldb : k0);
    os = bt * g.sS + k0;
  };
  auto stage_round = [&](int b) {
    if constexpr (!A_MN)
      stage(std::integral_constant<int, kPiecesA>{}, g.A + oa, g.lda, ti * kGemmTile, g.M, 0, b);
    if constexpr (!B_MN) stage(std::integral_constant<int, kPiecesB>{}, g.B + ob, g.ldb, tj * kGemmTile, g.N, kPiecesA, b);
  };
  auto read_scale = [&] {
    if constexpr (SCALE) read(std::false_type{}, ps + os, 0, sc);
  };
  offsets();
  if (u < u_end) {
    stage_round(0);
    if constexpr (A_MN) {
#pragma unroll
      for (int a = 0; a < NB; ++a) read(amn{}, pa[a] + oa, g.lda, va[a]);
    }
    if constexpr (B_MN) {
#pragma unroll
      for (int c = 0; c < NB; ++c) read(bmn{}, pb[c] + ob, g.ldb, vb[c]);
    }
    read_scale();
    put(0);
  }
  int buf = 0;
  while (u < u_end) {
    ++u;
    const bool more = u < u_end;
    if (more && ++kr == per) kr = 0, ++bt;
    offsets();  // of the next round (of this one again behind the last)
    // this round's values are in LDS once every wave has waited for its own and
    // met the barrier, which also ends the reads of the other buffer
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (more) stage_round(buf ^ 1);
#pragma unroll
    for (int a = 0; a < NB; ++a) {
      if constexpr (!A_MN) staged(0, buf, (wi >> 4) + a, va[a]);
      gemm_cut(va[a], neg, fa[a]);
    }
    if constexpr (A_MN) {
#pragma unroll
      for (int a = 0; a < NB; ++a) read(amn{}, pa[a] + oa, g.lda, va[a]);
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      if constexpr (!B_MN) staged(kPiecesA, buf, (wj >> 4) + c, vb[c]);
      cut_b(c);
      if constexpr (B_MN) read(bmn{}, pb[c] + ob, g.ldb, vb[c]);
      products(c);
    }
    read_scale();
    if (more) put(buf ^ 1);
    buf ^= 1;
  }
  // what is left of K in each batch
  const int n = (int)(g.K - per * kGemmSlab);
  if (n > 0)
    for (int b = split; b < g.nbatch; b += g.splits) {
      const int64_t k0 = per * kGemmSlab;
      const int64_t qa = b * g.sA + (A_MN ? k0 * g.lda : k0), qb = b * g.sB + (B_MN ? k0 * g.ldb : k0);
      if constexpr (SCALE) read_end(std::false_type{}, ps + b * g.sS + k0, 0, n, sc);
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        read_end(amn{}, pa[a] + qa, g.lda, n, va[a]);
        gemm_cut(va[a], neg, fa[a]);
      }
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        read_end(bmn{}, pb[c] + qb, g.ldb, n, vb[c]);
        cut_b(c);
        products(c);
      }
    }
  // lane holds C[row 4 (lane / 16) + r][col lane % 16] of each 16x16 block
  float *out = part + (int64_t)split * g.M * g.N;
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + 16 * a + 4 * (lane >> 4) + r;
        const int j = j0 + 16 * c + (lane & 15);
        if (i < g.M && j < g.N) out[(int64_t)i * g.N + j] = acc[a][c][r] + low[a][c][r];
      }
}

// C = alpha * sum_splits part (+ C if accumulate), fixed summation order.
__global__ __launch_bounds__(256) void k_gemm_reduce(GemmShape g, const float *__restrict__ part) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)g.M * g.N) return;
  const int i = (int)(t / g.N), j = (int)(t % g.N);
  double s = ordered_sum<double>(part + t, g.splits, (int64_t)g.M * g.N);
  if (s != s) s = (double)gemm_entry_fp32(g, i, j);
  float *dst = g.c_colmajor ? &g.C[(int64_t)j * g.ldc + i] : &g.C[(int64_t)i * g.ldc + j];
  const float v = (float)((double)g.alpha * s);
  *dst = g.accumulate ? *dst + v : v;
}

// The same for a symmetric product: a workgroup sums the 32 x 32 block (bi, bj),
// bi <= bj, and writes it and its mirror image (inside a tile on the diagonal the
// two differ in the order of their parts: the entries above it count).
// Bound: the partials' latency.  900 x 900, 13 splits: 9.7 us; 29 (8 splits) with each
// entry below the diagonal read at its mirror image, a line per lane.
__global__ __launch_bounds__(1024) void k_gemm_reduce_sym(GemmShape g, const float *__restrict__ part) {
  __shared__ float tile[32][33];
  int bi = 0, left = (int)blockIdx.x;
  const int nb = (g.N + 31) / 32;
  while (left >= nb - bi) left -= nb - bi, ++bi;
  const int bj = bi + left;
  const int c = threadIdx.x & 31, r = threadIdx.x >> 5;
  auto put = [&](int i, int j, float v) {
    float *dst = g.c_colmajor ? &g.C[(int64_t)j * g.ldc + i] : &g.C[(int64_t)i * g.ldc + j];
    *dst = g.accumulate ? *dst + v : v;
  };
  const int i = 32 * bi + r, j = 32 * bj + c;
  if (i < g.M && j < g.N && i <= j) {
    double s = ordered_sum<double>(part + (int64_t)i * g.N + j, g.splits, (int64_t)g.M * g.N);
    if (s != s) s = (double)gemm_entry_fp32(g, i, j);
    const float v = (float)((double)g.alpha * s);
    tile[r][c] = v;
    put(i, j, v);
  }
  __syncthreads();
  const int it = 32 * bj + r, jt = 32 * bi + c;  // below the diagonal
  if (it < g.M && jt < g.N && it > jt) put(it, jt, tile[c][r]);
}

static void launch_reduce(const GemmShape &g, const float *part, hipStream_t s) {
  if (g.symmetric) {
    const int64_t nb = (g.N + 31) / 32;
    k_gemm_reduce_sym<<<(unsigned)(nb * (nb + 1) / 2), 1024, 0, s>>>(g, part);
    return;
  }
  const int64_t n = (int64_t)g.M * g.N;
  k_gemm_reduce<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(g, part);
}

void launch_gemm_parts(const GemmShape &g, float *part, hipStream_t s) {
  const int tm = (g.M + kGemmTile - 1) / kGemmTile, tn = (g.N + kGemmTile - 1) / kGemmTile;
  const int ntile = g.symmetric ? tm * (tm + 1) / 2 : tm * tn;
  const dim3 grid((unsigned)round_up((int64_t)ntile * g.splits, 8));
  // loads of 16 bytes where every row starts on 16 bytes
  auto aligned = [](const float *p, int64_t ld, int64_t batch) {
    return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0 && batch % 4 == 0;
  };
  const bool vec = (g.a_mn || aligned(g.A, g.lda, g.sA)) && (g.b_mn || aligned(g.B, g.ldb, g.sB));
  auto run = [&](auto amn, auto bmn, auto scale) {
    constexpr bool A = decltype(amn)::value, B = decltype(bmn)::value, S = decltype(scale)::value;
    if (vec) k_gemm_bf3<A, B, S, true><<<grid, 256, 0, s>>>(g, tn, ntile, part);
    else k_gemm_bf3<A, B, S, false><<<grid, 256, 0, s>>>(g, tn, ntile, part);
  };
  auto go = [&](auto bmn) {
    if (g.scale != nullptr) run(std::false_type{}, bmn, std::true_type{});
    else run(std::false_type{}, bmn, std::false_type{});
  };
  if (g.a_mn) run(std::true_type{}, std::false_type{}, std::false_type{});
  else if (g.b_mn) go(std::true_type{});
  else go(std::false_type{});
}

void launch_gemm(const GemmShape &g, float *part, hipStream_t s) {
  launch_gemm_parts(g, part, s);
  launch_reduce(g, part, s);
}

// ---- small dense FP64 kernels (one workgroup) ----

// In place: A (n x n, row-major, FP64, symmetric) -> lower Cholesky factor L
// of A + shift I (upper part zeroed).  info = 0, or k + 1 if the pivot at k
// is not positive.
__global__ __launch_bounds__(256) void k_cholesky(double *A, int n, double shift, int *info) {
  __shared__ double piv;
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) A[(int64_t)i * n + i] += shift;
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    if (threadIdx.x == 0) {
      const double d = A[(int64_t)k * n + k];
      if (!(d > 0.0) && bad == 0) bad = k + 1;
      piv = d > 0.0 ? sqrt(d) : 1.0;
      A[(int64_t)k * n + k] = piv;
    }
    __syncthreads();
    for (int i = k + 1 + threadIdx.x; i < n; i += blockDim.x) A[(int64_t)i * n + k] /= piv;
    __syncthreads();
    // trailing update of the lower triangle, one row per thread stride
    for (int i = k + 1 + threadIdx.x; i < n; i += blockDim.x) {
      const double lik = A[(int64_t)i * n + k];
      for (int j = k + 1; j <= i; ++j) A[(int64_t)i * n + j] -= lik * A[(int64_t)j * n + k];
    }
    __syncthreads();
  }
  for (int t = threadIdx.x; t < n * n; t += blockDim.x) {
    const int i = t / n, j = t % n;
    if (j > i) A[t] = 0.0;
  }
  if (threadIdx.x == 0) *info = bad;
}

// Linv (n x n, row-major, FP32 out) = L^{-1} for lower-triangular L (FP64),
// one column of the inverse per thread by forward substitution.
__global__ __launch_bounds__(256) void k_tri_inverse(const double *L, int n, double *work, float *Linv) {
  for (int c = threadIdx.x; c < n; c += blockDim.x) {
    double *x = work + (int64_t)c * n;  // column c of L^{-1}
    for (int i = 0; i < n; ++i) {
      double s = (i == c) ? 1.0 : 0.0;
      for (int j = c; j < i; ++j) s -= L[(int64_t)i * n + j] * x[j];
      x[i] = i < c ? 0.0 : s / L[(int64_t)i * n + i];
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < n * n; t += blockDim.x) {
    const int i = t / n, j = t % n;
    Linv[t] = (float)work[(int64_t)j * n + i];  // Linv[i][j] = column j, entry i
  }
}

__global__ void k_f32_to_f64(const float *__restrict__ a, double *__restrict__ b, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) b[i] = (double)a[i];
}

void launch_cholesky(double *A, int n, double shift, int *info, hipStream_t s) {
  k_cholesky<<<1, 256, 0, s>>>(A, n, shift, info);
}
void launch_tri_inverse(const double *L, int n, double *work, float *Linv, hipStream_t s) {
  k_tri_inverse<<<1, 256, 0, s>>>(L, n, work, Linv);
}
void launch_f32_to_f64(const float *a, double *b, int64_t n, hipStream_t s) {
  k_f32_to_f64<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(a, b, n);
}

}  // namespace vds
