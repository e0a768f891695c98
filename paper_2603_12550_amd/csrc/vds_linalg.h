// Dense linear-algebra helpers shared by the POD and reduced-model code.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace vds {

// C = alpha * sum_{b < nbatch} A_b diag(scale_b) B_b^T (+ C when accumulate), where
// A_b is M x K and B_b is N x K.  Element (i, k) of A_b is A[b*sA + k*lda + i]
// when a_mn, else A[b*sA + i*lda + k]; likewise B with b_mn.  An MN-contiguous A has
// a K-contiguous B and no scale beside it (no other form is asked for).  The output is
// row-major (C[i*ldc + j]) or column-major (C[j*ldc + i]).  K is split over
// `splits` workgroup layers whose partial tiles are summed in a fixed order.
struct GemmShape {
  int M = 0, N = 0;
  int64_t K = 0;
  int nbatch = 1;
  const float *A = nullptr;
  int64_t lda = 0, sA = 0;
  bool a_mn = false;
  const float *B = nullptr;
  int64_t ldb = 0, sB = 0;
  bool b_mn = false;
  const float *scale = nullptr;
  int64_t sS = 0;
  float alpha = 1.f;
  float *C = nullptr;
  int64_t ldc = 0;
  bool c_colmajor = false;
  bool accumulate = false;
  int splits = 1;
  // C = A A^T (A and B the same matrix, M = N): only tiles on and above the
  // diagonal are computed, the others are mirrored in the reduction
  bool symmetric = false;
};

// BF16 matrix cores, three BF16 parts per FP32 factor.  Sums
// within a split in FP32, over the splits in FP64.
void launch_gemm(const GemmShape &g, float *part, hipStream_t s);
// The same without the sum: part[split][i][j], M x N per split (symmetric: the
// entries of tiles on and above the diagonal).
void launch_gemm_parts(const GemmShape &g, float *part, hipStream_t s);

// Entry (i, j) in FP32, term by term: for entries that are not numbers in the
// three-part product (an infinite factor, or one past the BF16 range, has no
// parts), so that they are what FP32 arithmetic makes of the inputs.  No further
// once the sum is not a number, which it then stays (looked at every 64 terms: at each
// one, the loads no longer run ahead): a Gram matrix of 60000 x 900 NaN takes 0.45 ms
// like any other (55 with every entry summed to its end), one with a single infinite
// factor, whose row of entries runs over all terms, 7.7.
__device__ inline float gemm_entry_fp32(const GemmShape &g, int i, int j) {
  float s = 0.f;
  for (int b = 0; b < g.nbatch; ++b)
    for (int64_t k0 = 0; k0 < g.K && s == s; k0 += 64)
      for (int64_t k = k0; k < min(g.K, k0 + 64); ++k) {
        const float x = g.A[b * g.sA + (g.a_mn ? k * g.lda + i : (int64_t)i * g.lda + k)];
        float y = g.B[b * g.sB + (g.b_mn ? k * g.ldb + j : (int64_t)j * g.ldb + k)];
        if (g.scale != nullptr) y *= g.scale[b * g.sS + k];
        s = fmaf(x, y, s);
      }
  return s;
}

void launch_cholesky(double *A, int n, double shift, int *info, hipStream_t s);
void launch_tri_inverse(const double *L, int n, double *work, float *Linv, hipStream_t s);
void launch_f32_to_f64(const float *a, double *b, int64_t n, hipStream_t s);

constexpr int kGemmTile = 96;  // output tile edge of launch_gemm
constexpr int kGemmSlab = 32;  // k-depth of one round

// Splits of launch_gemm's K (all batches end to end, in rounds of 32): up to three
// workgroups per compute unit, at least four rounds each, and at most 64 so that
// the sum over the splits stays small.
inline int gemm_splits(int M, int N, int64_t K, int nbatch = 1, bool symmetric = false) {
  const int64_t tm = (M + kGemmTile - 1) / kGemmTile, tn = (N + kGemmTile - 1) / kGemmTile;
  // a symmetric product runs only the tiles on and above the diagonal
  const int64_t tiles = symmetric ? tm * (tm + 1) / 2 : tm * tn;
  const int64_t rounds = (K + kGemmSlab - 1) / kGemmSlab * nbatch;
  int64_t s = 768 / tiles;
  if (s > rounds / 4) s = rounds / 4;
  if (s > 64) s = 64;
  return (int)(s < 1 ? 1 : s);
}

}  // namespace vds
