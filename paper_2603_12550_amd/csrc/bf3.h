// Device pieces of the kernels that take FP32 products from three BF16 parts
// (operand layouts: vds_internal.h; the method: pair_kernels.hip).
#pragma once

#include "vds_internal.h"

namespace vds {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The three BF16 parts of an FP64 number, each rounded to nearest (the third
// leaves 2^-27 of it); bit patterns.
struct Bf3 {
  uint16_t h, m, l;
};
__device__ inline uint16_t bf16_bits(double v) {
  return __builtin_bit_cast(uint16_t, (__bf16)(float)v);
}
__device__ inline double bf16_value(uint16_t u) { return (double)__uint_as_float((uint32_t)u << 16); }
__device__ inline Bf3 split_bf3(double v) {
  Bf3 s;
  s.h = bf16_bits(v);
  v -= bf16_value(s.h);
  s.m = bf16_bits(v);
  v -= bf16_value(s.m);
  s.l = bf16_bits(v);
  return s;
}
__device__ inline bf16x8 as_bf8(uint4 u) {
  bf16x8 r;
  __builtin_memcpy(&r, &u, sizeof(r));
  return r;
}
// (a, b) = h + m + l, each two BF16 numbers rounded to nearest, exact down to
// the FP32 subnormals (not for |a| or |b| that round up to infinity).
__device__ __forceinline__ void split_pair_bf3(float a, float b, uint32_t (&o)[3]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(o[p]) : "v"(a), "v"(b));
    if (p < 2) {
      a -= __uint_as_float(o[p] << 16);
      b -= __uint_as_float(o[p] & 0xffff0000u);
    }
  }
}

// The upper halves of eight values, a BF16 operand (truncation: what is left of
// a value after two such cuts is again a BF16 number).
__device__ __forceinline__ bf16x8 upper_halves(const floatx4 &a, const floatx4 &b) {
  uint32_t u[4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    u[j] = __builtin_amdgcn_perm(__float_as_uint(a[2 * j + 1]), __float_as_uint(a[2 * j]), 0x07060302u);
    u[2 + j] = __builtin_amdgcn_perm(__float_as_uint(b[2 * j + 1]), __float_as_uint(b[2 * j]), 0x07060302u);
  }
  return as_bf8(uint4{u[0], u[1], u[2], u[3]});
}

// Row operand of the 16-row block rb from its column operand (layout at
// bf3_index): the slots of a component swap within a dword, the norm's dwords
// change places (see there).
template <int D>
__device__ __forceinline__ void bf3_row_operand(const uint4 *__restrict__ K3, int64_t rb, int lane,
                                                bf16x8 (&q)[bf3_slices(D)]) {
  constexpr int NQ = bf3_slices(D);
  constexpr int dA = 3 * D, dB = dA + 1, dC = dA + 2;
  const int g = lane >> 4;
  uint32_t k[NQ][4];
#pragma unroll
  for (int m = 0; m < NQ; ++m) {
    const uint4 u = K3[(rb * NQ + m) * 64 + lane];
    k[m][0] = u.x, k[m][1] = u.y, k[m][2] = u.z, k[m][3] = u.w;
  }
  const uint32_t nA = __shfl(k[dA / 16][dA % 4], (lane & 15) + 16 * (dA % 16 / 4));
#pragma unroll
  for (int m = 0; m < NQ; ++m) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int dd = 16 * m + 4 * g + j;
      const uint32_t v = k[m][j], sw = (v >> 16) | (v << 16);
      o[j] = (dd % 3 != 0 && dd < dA) || dd == dB ? sw : v;
      if (dd == dA) o[j] = 0x3f803f80u;
      if (dd == dC) o[j] = nA;
    }
    q[m] = as_bf8(uint4{o[0], o[1], o[2], o[3]});
  }
}

// Minus the identity as the A operand that picks, for row m of block b of an
// e tile, the slot holding column J = m of that block, k = 8 (m / 4) + 4 b + m % 4:
// mfma(neg[b], upper halves of e, e[b]) is what the cut leaves of block b.
__device__ __forceinline__ void minus_identity(int lane, bf16x8 (&neg)[2]) {
  const int d = (lane & 15) - 4 * (lane >> 4);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 8; ++i) neg[b][i] = (d >= 0 && d < 4 && i == 4 * b + d) ? (__bf16)-1.f : (__bf16)0.f;
}

// One piece of 64 x 16 bytes straight from memory to LDS (asynchronous: the
// wave waits on vmcnt before it meets the barrier that publishes the piece).
__device__ __forceinline__ void piece_to_lds(const uint4 *src, uint4 *dst, int lane) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + lane),
                                   (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

}  // namespace vds
