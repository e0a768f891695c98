// POD offline phase and POD maps (C ABI of include/vds_pod.h).
//
// Gram matrix X^T X by the three-part GEMM, symmetric eigensolve in FP64 by
// rocSOLVER (dsyevd), U = X V_R L_R^{-1/2} by the GEMM, then Cholesky-QR
// re-orthonormalisation (the FP32 Gram resolves eigenvalues only down to
// ~1e-7 of the largest, so the trailing columns need it).  Projection and
// reconstruction are skinny products that read U once (HBM bound).
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "bf3.h"
#include "vds_ctx.h"
#include "vds_linalg.h"
#include "vds_pod.h"

using namespace vds;

namespace {

// Both maps read U once from memory and little else, so what counts is enough
// loads in flight: 43 MB at P = 20000, R = 180.

// f(std::integral_constant<int, NB>) for the number of bonds.
template <class F>
void by_bonds(int nb, F &&f) {
  switch (nb) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 5>{}); break;
  }
}

// q_k = U p_k for the bonds k.  A workgroup owns 64 positions; its four waves
// take a quarter of the columns each, sixteen in flight, and add up in LDS
// (one position per thread over all columns left one wave per SIMD waiting).
// Bound: reading U.  Measured, P = 20000, R = 180, calls in a row: 10.6 us (4.1 TB/s; a
// large copy reaches 4.9) with the same U, which the last-level cache then holds, 11.9
// (3.6 TB/s) with sixteen in turn, which it does not; 17.4 and 19.9 with one wave per SIMD.
constexpr int kReconWaves = 4;
constexpr int kReconInFlight = 16;

template <int NB>
__global__ __launch_bounds__(kReconWaves * 64) void k_pod_reconstruct(const float *__restrict__ U, int64_t m, int R,
                                                                      const float *__restrict__ p,
                                                                      float *__restrict__ q) {
  __shared__ float red[kReconWaves][NB][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const int per = (R + kReconWaves - 1) / kReconWaves;
  const int r0 = wave * per, r1 = min(R, r0 + per);
  const float *u = U + min(i, m - 1);
  float acc[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) acc[k] = 0.f;
  for (int r = r0; r < r1; r += kReconInFlight) {
    float uv[kReconInFlight];
#pragma unroll
    for (int j = 0; j < kReconInFlight; ++j) uv[j] = u[(int64_t)min(r + j, r1 - 1) * m];
#pragma unroll
    for (int j = 0; j < kReconInFlight; ++j)
      if (r + j < r1) {  // scalar
#pragma unroll
        for (int k = 0; k < NB; ++k) acc[k] = fmaf(uv[j], p[(int64_t)k * R + r + j], acc[k]);
      }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) red[wave][k][lane] = acc[k];
  __syncthreads();
  for (int k = wave; k < NB; k += kReconWaves)
    if (i < m) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < kReconWaves; ++w) v += red[w][k][lane];
      q[(int64_t)k * m + i] = v;
    }
}

constexpr int kProjThreads = 256;
constexpr int kProjChunks = 32;  // the workspace holds at least this many partial sums per coefficient
constexpr int kProjRows = 8;

// First stage of p_k[r] = U_r . q_k: block (g, c) takes the rows
// r = 8 g .. 8 g + 7 of U against chunk c of the positions; a thread reads
// q_k[i] once for all eight rows and two positions at a time, so U is read once
// and q once per eight rows.  Then sums over rows of 16 lanes by DPP and over
// the block in LDS, in fixed order, into part[k R + r][c].
// Bound: reading U.  Measured, P = 20000, R = 180, with the sum over chunks, calls in a
// row: 11.9 us (this kernel alone 9.9, 4.4 TB/s) with the same U, which the last-level
// cache then holds, 13.4 with sixteen in turn, which it does not; 20.3 and 21.8 with one
// position at a time and cross-lane sums of all five possible bonds.
template <int NB>
__global__ __launch_bounds__(kProjThreads) void k_pod_project(const float *__restrict__ U, int64_t m, int R,
                                                              int64_t len, const float *__restrict__ q,
                                                              float *__restrict__ part) {
  constexpr int kGroups = kProjThreads / 16;
  __shared__ float red[kProjRows * NB][kGroups + 1];
  const int r0 = (int)blockIdx.x * kProjRows, c = (int)blockIdx.y;
  const int nr = min(kProjRows, R - r0);
  const int64_t i0 = c * len, i1 = min(m, i0 + len);
  float acc[kProjRows][NB];
#pragma unroll
  for (int j = 0; j < kProjRows; ++j)
#pragma unroll
    for (int k = 0; k < NB; ++k) acc[j][k] = 0.f;
  const float *u[kProjRows];
#pragma unroll
  for (int j = 0; j < kProjRows; ++j) u[j] = U + (int64_t)(r0 + min(j, nr - 1)) * m;  // rows past R repeat the last
  auto body = [&](auto nc, int64_t i) {
    constexpr int N = decltype(nc)::value;
    float qv[N][NB], uv[N][kProjRows];
#pragma unroll
    for (int t = 0; t < N; ++t) {
#pragma unroll
      for (int k = 0; k < NB; ++k) qv[t][k] = q[(int64_t)k * m + i + t * kProjThreads];
#pragma unroll
      for (int j = 0; j < kProjRows; ++j) uv[t][j] = u[j][i + t * kProjThreads];
    }
#pragma unroll
    for (int t = 0; t < N; ++t)
#pragma unroll
      for (int j = 0; j < kProjRows; ++j)
#pragma unroll
        for (int k = 0; k < NB; ++k) acc[j][k] = fmaf(uv[t][j], qv[t][k], acc[j][k]);
  };
  int64_t i = i0 + threadIdx.x;
  for (; i + kProjThreads < i1; i += 2 * kProjThreads) body(std::integral_constant<int, 2>{}, i);
  if (i < i1) body(std::integral_constant<int, 1>{}, i);
#pragma unroll
  for (int j = 0; j < kProjRows; ++j)
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      float v = acc[j][k];
      v += row_rotate<8>(v);
      v += row_rotate<4>(v);
      v += row_rotate<2>(v);
      v += row_rotate<1>(v);
      if ((threadIdx.x & 15) == 0) red[j * NB + k][threadIdx.x >> 4] = v;
    }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < kProjRows * NB) {
    const int j = t / NB, k = t % NB;
    if (j < nr) {
      float v = 0.f;
      for (int w = 0; w < kGroups; ++w) v += red[t][w];
      part[((int64_t)k * R + r0 + j) * gridDim.y + c] = v;
    }
  }
}

// Second stage: p[k R + r] = sum over the chunks, a wave per coefficient, FP64.
__global__ __launch_bounds__(256) void k_pod_project_sum(const float *__restrict__ part, int n, int nch,
                                                         float *__restrict__ p) {
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (e >= n) return;
  double v = 0.0;
  for (int c = lane; c < nch; c += 64) v += (double)part[(int64_t)e * nch + c];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  if (lane == 0) p[e] = (float)v;
}

// The whole projection in one launch for few and short rows: a workgroup per row of
// U, a thread takes every 1024th position, eight in flight; sums over rows of 16
// lanes by DPP and over the block in FP64.
// Bound: the launch, from some 50000 numbers per workgroup on its loads.  Measured
// against the two launches, calls in a row / alone: P = 2000, R = 60, nb = 3: 8.2 /
// 19.1 us, 11.1 / 21.3.
//
// The line: a workgroup reads (nb + 1) m numbers, which alone costs more than the
// launch saved from about 90000 on (P = 6000: nb = 3 20.9 and 21.4 us, nb = 5 22.2
// and 21.4), and more rows than compute units read q again where the groups of 8
// rows read it once (nb = 3, P = 6000: R = 256 21.9 and 22.3, R = 300 24.1 and 22.6).
constexpr int kProjOneThreads = 1024;
constexpr int kProjOneAhead = 8;
constexpr int kProjOneRows = 256;
constexpr int64_t kProjOneReads = 9 * kProjOneAhead * kProjOneThreads;

template <int NB>
__global__ __launch_bounds__(kProjOneThreads) void k_pod_project_one(const float *__restrict__ U, int64_t m, int R,
                                                                     const float *__restrict__ q,
                                                                     float *__restrict__ p) {
  __shared__ float red[NB][kProjOneThreads / 16];
  const int r = (int)blockIdx.x;
  const float *u = U + (int64_t)r * m;
  float acc[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) acc[k] = 0.f;
  for (int64_t i = threadIdx.x; i < m; i += kProjOneAhead * kProjOneThreads) {
    float uv[kProjOneAhead], qv[kProjOneAhead][NB];
#pragma unroll
    for (int t = 0; t < kProjOneAhead; ++t) {
      const int64_t at = min(i + t * kProjOneThreads, m - 1);
      uv[t] = u[at];
#pragma unroll
      for (int k = 0; k < NB; ++k) qv[t][k] = q[(int64_t)k * m + at];
    }
#pragma unroll
    for (int t = 0; t < kProjOneAhead; ++t)
      if (i + t * kProjOneThreads < m) {
#pragma unroll
        for (int k = 0; k < NB; ++k) acc[k] = fmaf(uv[t], qv[t][k], acc[k]);
      }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    float v = acc[k];
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    v += row_rotate<1>(v);
    if ((threadIdx.x & 15) == 0) red[k][threadIdx.x >> 4] = v;
  }
  __syncthreads();
  const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (k >= NB) return;
  double v = (double)red[k][lane];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  if (lane == 0) p[(int64_t)k * R + r] = (float)v;
}

}  // namespace

namespace vds {
void launch_pod_reconstruct(const float *U, int64_t m, int R, int nb, const float *p, float *q, hipStream_t s) {
  by_bonds(nb, [&](auto n) {
    k_pod_reconstruct<decltype(n)::value><<<(unsigned)((m + 63) / 64), kReconWaves * 64, 0, s>>>(U, m, R, p, q);
  });
}
}  // namespace vds

namespace {

struct PodLayout {
  size_t gram, gram64, eig, offd, info, Wt, U2, GU, GU64, Linv, work64, part, total;
};

PodLayout pod_layout(int64_t m, int32_t n, int32_t R) {
  PodLayout L{};
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off += (b + 255) / 256 * 256;
    return o;
  };
  L.gram = take(sizeof(float) * n * n);
  L.gram64 = take(sizeof(double) * n * n);
  L.eig = take(sizeof(double) * n);
  L.offd = take(sizeof(double) * n);
  L.info = take(sizeof(int) * 4);
  L.Wt = take(sizeof(float) * (size_t)R * n);
  L.U2 = take(sizeof(float) * (size_t)m * R);
  L.GU = take(sizeof(float) * R * R);
  L.GU64 = take(sizeof(double) * R * R);
  L.Linv = take(sizeof(float) * R * R);
  L.work64 = take(sizeof(double) * R * R);
  const int sg = gemm_splits(n, n, m, 1, true), su = gemm_splits(R, R, m);
  const size_t part = std::max({sizeof(float) * (size_t)sg * n * n, sizeof(float) * (size_t)su * R * R,
                                sizeof(float) * (size_t)m * R});
  L.part = take(part);
  L.total = off;
  return L;
}

// Wt[s][c] = V[c][n-1-s] / sqrt(max(lambda_{n-1-s}, floor)): the R leading
// eigenvectors (eigenvalues ascending in `eig`), scaled.
__global__ void k_scaled_modes(const double *V, const double *eig, int n, int R, double floor_, float *Wt) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)R * n) return;
  const int s = (int)(t / n), c = (int)(t % n);
  const int col = n - 1 - s;
  const double lam = fmax(eig[col], floor_);
  Wt[t] = (float)(V[(int64_t)col * n + c] / sqrt(lam));
}

vds_status gram_into(vds_ctx c, const float *X, int64_t m, int n, float *gram, float *part) {
  GemmShape g;
  g.M = n;
  g.N = n;
  g.K = m;
  g.A = X;
  g.lda = m;
  g.B = X;
  g.ldb = m;
  g.C = gram;
  g.ldc = n;
  g.symmetric = true;
  g.splits = gemm_splits(n, n, m, 1, true);
  // the symmetric product's own work: n (n + 1) / 2 entries of 2 m FLOP
  timed(c, VDS_TIMER_GEMM, (double)n * (n + 1) * (double)m, [&] { launch_gemm(g, part, c->stream); });
  return hip_check(c, hipGetLastError(), "gram");
}

// dst (m x R col-major) = src (m x R col-major) * B^T where B[j][k] = Bt[j*ldb + k] (R x kdim)
void times_small(vds_ctx c, const float *src, int64_t m, int kdim, const float *Bt, int R, float *dst, float *part) {
  GemmShape g;
  g.M = (int)m;
  g.N = R;
  g.K = kdim;
  g.A = src;
  g.lda = m;
  g.a_mn = true;
  g.B = Bt;
  g.ldb = kdim;
  g.C = dst;
  g.ldc = m;
  g.c_colmajor = true;
  g.splits = 1;
  timed(c, VDS_TIMER_GEMM, 2.0 * m * (double)R * kdim, [&] { launch_gemm(g, part, c->stream); });
}

}  // namespace

extern "C" {

size_t vds_pod_workspace_bytes(int64_t m, int32_t ncols, int32_t R) {
  if (m < 1 || ncols < 1 || R < 1 || R > ncols || R > m) return 0;
  return pod_layout(m, ncols, R).total;
}

vds_status vds_pod_gram(vds_ctx c, const float *X, int64_t m, int32_t n, float *gram, void *ws, size_t bytes) {
  if (c == nullptr) return VDS_ERR_ARG;
  if (!X || !gram || !ws || m < 1 || n < 1) return set_err(c, VDS_ERR_ARG, "bad arguments");
  const PodLayout L = pod_layout(m, n, 1);
  if (bytes < L.total) return set_err(c, VDS_ERR_NOMEM, "POD workspace too small");
  char *w = static_cast<char *>(ws);
  return gram_into(c, X, m, n, gram, reinterpret_cast<float *>(w + L.part));
}

vds_status vds_pod_basis(vds_ctx c, const float *X, int64_t m, int32_t n, int32_t R, float *U, double *eig_host,
                         void *ws, size_t bytes) {
  if (c == nullptr) return VDS_ERR_ARG;
  if (!X || !U || !ws || m < 1 || n < 1 || R < 1 || R > n || R > m)
    return set_err(c, VDS_ERR_ARG, "bad arguments (need 1 <= R <= min(m, ncols))");
  const PodLayout L = pod_layout(m, n, R);
  if (bytes < L.total) return set_err(c, VDS_ERR_NOMEM, "POD workspace too small");
  char *w = static_cast<char *>(ws);
  float *gram = reinterpret_cast<float *>(w + L.gram);
  double *gram64 = reinterpret_cast<double *>(w + L.gram64);
  double *eig = reinterpret_cast<double *>(w + L.eig);
  double *offd = reinterpret_cast<double *>(w + L.offd);
  int *info = reinterpret_cast<int *>(w + L.info);
  float *Wt = reinterpret_cast<float *>(w + L.Wt);
  float *U2 = reinterpret_cast<float *>(w + L.U2);
  float *GU = reinterpret_cast<float *>(w + L.GU);
  double *GU64 = reinterpret_cast<double *>(w + L.GU64);
  float *Linv = reinterpret_cast<float *>(w + L.Linv);
  double *work64 = reinterpret_cast<double *>(w + L.work64);
  float *part = reinterpret_cast<float *>(w + L.part);

  vds_status st = gram_into(c, X, m, n, gram, part);
  if (st != VDS_OK) return st;
  launch_f32_to_f64(gram, gram64, (int64_t)n * n, c->stream);

  rocblas_handle h = static_cast<rocblas_handle>(blas_handle(c));
  if (h == nullptr) return VDS_ERR_HIP;
  const rocblas_status rs =
      rocsolver_dsyevd(h, rocblas_evect_original, rocblas_fill_upper, n, gram64, n, eig, offd, info);
  if (rs != rocblas_status_success) return set_err(c, VDS_ERR_HIP, "rocsolver_dsyevd failed");

  std::vector<double> lam(n);
  int hinfo[4] = {0, 0, 0, 0};
  st = hip_check(c, hipMemcpyAsync(lam.data(), eig, sizeof(double) * n, hipMemcpyDeviceToHost, c->stream), "eig");
  if (st == VDS_OK) st = hip_check(c, hipMemcpyAsync(hinfo, info, sizeof(int), hipMemcpyDeviceToHost, c->stream), "info");
  if (st == VDS_OK) st = hip_check(c, hipStreamSynchronize(c->stream), "synchronise");
  if (st != VDS_OK) return st;
  if (hinfo[0] != 0) return set_err(c, VDS_ERR_HIP, "symmetric eigensolve did not converge");
  if (eig_host)
    for (int i = 0; i < n; ++i) eig_host[i] = lam[n - 1 - i];
  // FP32 Gram resolves eigenvalues to ~1e-7 of the largest; floor the rest
  const double floor_ = std::max(lam[n - 1], 1e-300) * 1e-12;
  k_scaled_modes<<<(unsigned)(((int64_t)R * n + 255) / 256), 256, 0, c->stream>>>(gram64, eig, n, R, floor_, Wt);
  // U2 = X Wt^T  (m x R)
  times_small(c, X, m, n, Wt, R, U2, part);

  // three Cholesky-QR passes: U <- U L^{-T}, L L^T = U^T U (+ shift on the first)
  float *src = U2, *dst = U;
  for (int pass = 0; pass < 3; ++pass) {
    GemmShape g;
    g.M = R;
    g.N = R;
    g.K = m;
    g.A = src;
    g.lda = m;
    g.B = src;
    g.ldb = m;
    g.C = GU;
    g.ldc = R;
    g.splits = gemm_splits(R, R, m);
    timed(c, VDS_TIMER_GEMM, 2.0 * R * (double)R * m, [&] { launch_gemm(g, part, c->stream); });
    launch_f32_to_f64(GU, GU64, (int64_t)R * R, c->stream);
    double shift = 0.0;
    if (pass == 0) {
      // shift ~ 1e-6 of the mean squared column norm
      double tr = 0.0;
      std::vector<float> gh((size_t)R * R);
      st = hip_check(c, hipMemcpyAsync(gh.data(), GU, sizeof(float) * R * R, hipMemcpyDeviceToHost, c->stream), "gu");
      if (st == VDS_OK) st = hip_check(c, hipStreamSynchronize(c->stream), "synchronise");
      if (st != VDS_OK) return st;
      for (int i = 0; i < R; ++i) tr += gh[(size_t)i * R + i];
      shift = 1e-6 * tr / R;
    }
    launch_cholesky(GU64, R, shift, info + 1, c->stream);
    launch_tri_inverse(GU64, R, work64, Linv, c->stream);
    // dst = src * Linv^T  (B[j][k] = Linv[j][k])
    times_small(c, src, m, R, Linv, R, dst, part);
    st = hip_check(c, hipMemcpyAsync(hinfo + 1, info + 1, sizeof(int), hipMemcpyDeviceToHost, c->stream), "info");
    if (st == VDS_OK) st = hip_check(c, hipStreamSynchronize(c->stream), "synchronise");
    if (st != VDS_OK) return st;
    if (hinfo[1] != 0) return set_err(c, VDS_ERR_ARG, "basis is numerically rank deficient (R exceeds the snapshots' rank)");
    std::swap(src, dst);
  }
  // the last pass wrote into what is now `src`
  if (src != U)
    st = hip_check(c, hipMemcpyAsync(U, src, sizeof(float) * m * R, hipMemcpyDeviceToDevice, c->stream), "copy U");
  if (st == VDS_OK) st = hip_check(c, hipStreamSynchronize(c->stream), "synchronise");
  return st;
}

size_t vds_pod_map_workspace_bytes(const vds_problem *prob, int32_t R) {
  if (prob == nullptr || prob->P < 1 || prob->nb < 1 || R < 1) return 0;
  const int64_t m = 3 * prob->P;
  // partial sums of the projection; never less than the positions of all bonds
  const int64_t tiles = (R + 63) / 64;
  const int64_t chunks = std::max<int64_t>(kProjChunks, std::min<int64_t>({64, (m + 255) / 256,
                                                                             (2048 + tiles - 1) / tiles}));
  return (sizeof(float) * (size_t)prob->nb * (size_t)std::max<int64_t>(chunks * R, m) + 255) / 256 * 256;
}

vds_status vds_pod_project(vds_ctx c, const float *U, int32_t R, const float *q, float *p, void *ws, size_t bytes) {
  if (c == nullptr) return VDS_ERR_ARG;
  if (!U || !q || !p || !ws || R < 1) return set_err(c, VDS_ERR_ARG, "bad arguments");
  if (bytes < vds_pod_map_workspace_bytes(&c->prob, R)) return set_err(c, VDS_ERR_NOMEM, "workspace too small");
  const int64_t m = 3 * c->prob.P;
  const int nb = c->prob.nb;
  if (R <= kProjOneRows && (nb + 1) * m <= kProjOneReads) {
    timed(c, VDS_TIMER_PROJ, 4.0 * m * R, [&] {
      by_bonds(nb, [&](auto n) {
        k_pod_project_one<decltype(n)::value><<<(unsigned)R, kProjOneThreads, 0, c->stream>>>(U, m, R, q, p);
      });
    });
    return hip_check(c, hipGetLastError(), "project");
  }
  float *part = static_cast<float *>(ws);
  // about four workgroups per compute unit over the groups of rows and the
  // chunks of positions (at least 256 each), as far as the workspace holds their
  // partial sums
  const int64_t groups = (R + kProjRows - 1) / kProjRows;
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>({1024 / groups, (m + 255) / 256,
                                                              std::max<int64_t>(kProjChunks, m / R)}));
  const int64_t len = round_up((m + want - 1) / want, 64), nch = (m + len - 1) / len;
  timed(c, VDS_TIMER_PROJ, 4.0 * m * R, [&] {
    by_bonds(nb, [&](auto n) {
      k_pod_project<decltype(n)::value>
          <<<dim3((unsigned)groups, (unsigned)nch), kProjThreads, 0, c->stream>>>(U, m, R, len, q, part);
    });
    k_pod_project_sum<<<(nb * R + 3) / 4, 256, 0, c->stream>>>(part, nb * R, (int)nch, p);
  });
  return hip_check(c, hipGetLastError(), "project");
}

vds_status vds_pod_reconstruct(vds_ctx c, const float *U, int32_t R, const float *p, float *q, void *ws,
                               size_t bytes) {
  if (c == nullptr) return VDS_ERR_ARG;
  if (!U || !q || !p || !ws || R < 1) return set_err(c, VDS_ERR_ARG, "bad arguments");
  if (bytes < vds_pod_map_workspace_bytes(&c->prob, R)) return set_err(c, VDS_ERR_NOMEM, "workspace too small");
  const int64_t m = 3 * c->prob.P;
  const int nb = c->prob.nb;
  timed(c, VDS_TIMER_PROJ, 4.0 * m * R, [&] { launch_pod_reconstruct(U, m, R, nb, p, q, c->stream); });
  return hip_check(c, hipGetLastError(), "reconstruct");
}

}  // extern "C"
