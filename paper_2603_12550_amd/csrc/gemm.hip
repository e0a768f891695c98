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
// One workgroup: a 96 x 96 output tile over the rounds of its split.  Each round
// brings 32 k of both operands from memory into registers (while the matrix
// cores work on the round before), cuts every value into three BF16 parts and
// writes them to LDS as 16-row operands (lane row % 16 + 16 (k / 8), eight k);
// wave w owns the 48 x 48 quadrant (w / 2, w % 2), 3 x 3 blocks of 16, and takes
// the six products hh, hm, mh, mm, hl, lh of each (the others are below 2^-26:
// the parts are rounded to nearest, so what is left out has no sign).
// 96 wide: 540, 180 and 900 columns waste 7 to 14 % of a row of tiles, six
// tasks of four values per thread, and two workgroups share a compute unit.
// With at least eight splits, split s runs on XCD s % 8, so that its tiles read
// the same rounds through one L2.
// Bound: matrix pipe and the cutting (11 vector instructions per two values).
// Measured: Gram of 60000 x 900 0.57 ms against 1.48 with FP32 instructions on
// 64 x 64 tiles; the two 180 x 180 x 60000 products of a reduced operator build
// 62 and 77 against 123 and 140 us.

constexpr int kOperandU4 = (kGemmTile / 16) * 3 * 64;  // LDS uint4s of one operand

// VEC: every row of the K-contiguous operands starts on 16 bytes.
template <bool A_MN, bool B_MN, bool SCALE, bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_bf3(
    GemmShape g, int tn, int ntile, float *__restrict__ part) {
  __shared__ uint4 lds[2][2 * kOperandU4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int id = (int)blockIdx.x;
  const bool xcd = g.splits % 8 == 0;
  const int split = xcd ? id % 8 + 8 * (id / (8 * ntile)) : id / ntile;
  const int tile = xcd ? (id / 8) % ntile : id % ntile;
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
  const int i0 = ti * kGemmTile, j0 = tj * kGemmTile;
  const int64_t per = (g.K + kGemmSlab - 1) / kGemmSlab;  // rounds of one batch
  const int64_t rounds = per * g.nbatch;
  const int64_t r_beg = rounds * split / g.splits, r_end = rounds * (split + 1) / g.splits;

  // task t + 256 x of the round (x < 3: operand A, else B) is four k of a row.
  // K-contiguous: eight lanes take the 32 k of a row, 16 bytes each;
  // MN-contiguous: lanes along the rows.  Either way a wave's loads are
  // contiguous (32 bytes per lane instead took 64 address cycles per load and
  // 10000 cycles per round).  Rows past the operand's read its last row (their
  // outputs are not written), so a full round's loads have no condition.
  float v[6][4], sc[3][4];
  auto load = [&](int64_t round) {
    const int64_t bt = round / per, k0 = (round - bt * per) * kGemmSlab;
    const bool full = k0 + kGemmSlab <= g.K;  // scalar
#pragma unroll
    for (int x = 0; x < 6; ++x) {
      const bool isA = x < 3;
      const int u = tid + 256 * (x % 3);
      const bool mn = isA ? A_MN : B_MN;
      const int row = mn ? u % kGemmTile : u >> 3, k4 = mn ? u / kGemmTile : u & 7;
      const int64_t ld = isA ? g.lda : g.ldb;
      const int64_t idx = min((isA ? i0 : j0) + row, (isA ? g.M : g.N) - 1);
      const int64_t k = k0 + 4 * k4;
      const float *p = (isA ? g.A + bt * g.sA : g.B + bt * g.sB) + (mn ? k * ld + idx : idx * ld + k);
      const int64_t step = mn ? ld : 1;
      if (VEC && full && !mn) {  // scalar
        const float4 f = *reinterpret_cast<const float4 *>(p);
        v[x][0] = f.x, v[x][1] = f.y, v[x][2] = f.z, v[x][3] = f.w;
      } else if (full) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[x][e] = p[e * step];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[x][e] = k + e < g.K ? p[e * step] : 0.f;
      }
      if constexpr (SCALE) {
        if (!isA) {
          const float *q = g.scale + bt * g.sS + k;
#pragma unroll
          for (int e = 0; e < 4; ++e) sc[x % 3][e] = full || k + e < g.K ? q[e] : 0.f;
        }
      }
    }
  };
  // slot of (row, k / 8) in a 16-row operand: the rows of odd k groups are
  // exchanged in halves, so that eight rows' writes cover all banks
  auto store = [&](int b) {
#pragma unroll
    for (int x = 0; x < 6; ++x) {
      const bool isA = x < 3;
      const int u = tid + 256 * (x % 3);
      const bool mn = isA ? A_MN : B_MN;
      const int row = mn ? u % kGemmTile : u >> 3, k4 = mn ? u / kGemmTile : u & 7;
      if constexpr (SCALE) {
        if (!isA) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[x][e] *= sc[x % 3][e];
        }
      }
      uint32_t o[2][3];
      split_pair_bf3(v[x][0], v[x][1], o[0]);
      split_pair_bf3(v[x][2], v[x][3], o[1]);
      const int kg = k4 >> 1, slot = 16 * kg + ((row & 15) ^ (8 * (kg & 1)));
      uint2 *dst = reinterpret_cast<uint2 *>(lds[b] + (isA ? 0 : kOperandU4) + (row >> 4) * 3 * 64 + slot) + (k4 & 1);
#pragma unroll
      for (int p = 0; p < 3; ++p) dst[p * 128] = uint2{o[0][p], o[1][p]};
    }
  };

  // the upper parts' products, and the others apart: added to a long sum one by
  // one, what is below half a unit of it would be lost (on a Gram's diagonal,
  // where the mm products are all positive, 5e-7 to 2e-6 of the entry)
  floatx4 acc[3][3], low[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) acc[a][b] = low[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int wa = (wave >> 1) * 3, wb = (wave & 1) * 3;
  const int fl = lane ^ (8 * ((lane >> 4) & 1));
  if (r_beg < r_end) load(r_beg);
  for (int64_t r = r_beg; r < r_end; ++r) {
    const int b = (int)(r - r_beg) & 1;
    store(b);
    __syncthreads();  // (the other buffer's readers passed this barrier a round ago)
    if (r + 1 < r_end) load(r + 1);
    bf16x8 fa[3][3], fb[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        fa[a][p] = as_bf8(lds[b][((wa + a) * 3 + p) * 64 + fl]);
        fb[a][p] = as_bf8(lds[b][kOperandU4 + ((wb + a) * 3 + p) * 64 + fl]);
      }
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int x = 0; x < 6; ++x)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          floatx4 &t = x < 5 ? low[a][c] : acc[a][c];
          t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a][pa[x]], fb[c][pb[x]], t, 0, 0, 0);
        }
  }
  // lane holds C[row 4 (lane / 16) + r][col lane % 16] of each 16x16 block
  float *out = part + (int64_t)split * g.M * g.N;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + 16 * (wa + a) + 4 * (lane >> 4) + r;
        const int j = j0 + 16 * (wb + c) + (lane & 15);
        if (i < g.M && j < g.N) out[(int64_t)i * g.N + j] = acc[a][c][r] + low[a][c][r];
      }
}

// C = alpha * sum_splits part (+ C if accumulate), fixed summation order.  A
// symmetric product takes the entries below the diagonal from their mirror
// images (inside a diagonal tile the two differ in the order of their parts).
__global__ __launch_bounds__(256) void k_gemm_reduce(GemmShape g, const float *__restrict__ part) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)g.M * g.N) return;
  const int i = (int)(t / g.N), j = (int)(t % g.N);
  const int64_t src = (g.symmetric && i > j) ? (int64_t)j * g.N + i : t;
  double s = ordered_sum<double>(part + src, g.splits, (int64_t)g.M * g.N);
  if (s != s) s = (double)gemm_entry_fp32(g, i, j);
  float *dst = g.c_colmajor ? &g.C[(int64_t)j * g.ldc + i] : &g.C[(int64_t)i * g.ldc + j];
  const float v = (float)((double)g.alpha * s);
  *dst = g.accumulate ? *dst + v : v;
}

static void launch_reduce(const GemmShape &g, const float *part, hipStream_t s) {
  const int64_t n = (int64_t)g.M * g.N;
  k_gemm_reduce<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(g, part);
}

void launch_gemm_parts(const GemmShape &g, float *part, hipStream_t s) {
  const int tm = (g.M + kGemmTile - 1) / kGemmTile, tn = (g.N + kGemmTile - 1) / kGemmTile;
  const int ntile = g.symmetric ? tm * (tm + 1) / 2 : tm * tn;
  // 16-byte loads where every row starts on 16 bytes
  auto vec = [](const float *p, int64_t ld, int64_t batch) {
    return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0 && batch % 4 == 0;
  };
  const bool v16 = (g.a_mn || vec(g.A, g.lda, g.sA)) && (g.b_mn || vec(g.B, g.ldb, g.sB));
  const dim3 grid((unsigned)((int64_t)ntile * g.splits));
  auto run = [&](auto amn, auto bmn, auto scale, auto al) {
    k_gemm_bf3<decltype(amn)::value, decltype(bmn)::value, decltype(scale)::value, decltype(al)::value>
        <<<grid, 256, 0, s>>>(g, tn, ntile, part);
  };
  auto go = [&](auto amn, auto bmn) {
    using std::false_type, std::true_type;
    if (g.scale != nullptr) {
      if (v16) run(amn, bmn, true_type{}, true_type{});
      else run(amn, bmn, true_type{}, false_type{});
    } else {
      if (v16) run(amn, bmn, false_type{}, true_type{});
      else run(amn, bmn, false_type{}, false_type{});
    }
  };
  if (!g.a_mn && !g.b_mn) go(std::false_type{}, std::false_type{});
  else if (g.a_mn && !g.b_mn) go(std::true_type{}, std::false_type{});
  else if (!g.a_mn && g.b_mn) go(std::false_type{}, std::true_type{});
  else go(std::true_type{}, std::true_type{});
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
