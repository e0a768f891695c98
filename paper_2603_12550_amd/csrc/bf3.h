// Device pieces of the kernels that take FP32 products from three BF16 parts
// (operand layouts: vds_internal.h; the method: pair_kernels.hip).
#pragma once

#include <type_traits>

#include "vds_internal.h"

namespace vds {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The three BF16 parts of an FP64 number, each rounded to nearest (the third
// leaves 2^-27 of it); bit patterns.  In two FP32 halves: the upper one's cut
// leaves an exact remainder, which takes the lower one in with 2^-33 of the number
// (a conversion from FP64 to BF16 is ten instructions).
struct Bf3 {
  uint16_t h, m, l;
};
__device__ inline float bf16_float(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ inline double bf16_value(uint16_t u) { return (double)bf16_float(u); }
__device__ inline Bf3 split_bf3(double v) {
  Bf3 s;
  float r = (float)v;
  const float lo = (float)(v - (double)r);
  s.h = __builtin_bit_cast(uint16_t, (__bf16)r);
  r = (r - bf16_float(s.h)) + lo;
  s.m = __builtin_bit_cast(uint16_t, (__bf16)r);
  r -= bf16_float(s.m);
  s.l = __builtin_bit_cast(uint16_t, (__bf16)r);
  return s;
}
__device__ inline bf16x8 as_bf8(uint4 u) {
  bf16x8 r;
  __builtin_memcpy(&r, &u, sizeof(r));
  return r;
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

// Lane i of each row of 16 gets lane (i + R) % 16 of its row.
template <int R>
__device__ __forceinline__ float row_rotate(float v) {
  if constexpr (R % 16 == 0) return v;
  else
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + (16 - R % 16), 0xf, 0xf, true));
}

constexpr int kFlush3 = 8;  // 32-column chunks per FP32 accumulation group of the pair sums

// The three parts of every sum (columns p (D + 1) + n of the tiles) added up in
// lane n of each row of 16, into FP64; clears the FP32 sums.
template <int D>
__device__ __forceinline__ void bf3_flush(floatx4 (&acc)[bf3_tiles(D)], int lane, double (&tot)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v = 0.f;
    auto part = [&](auto pc) {
      constexpr int s = decltype(pc)::value * (D + 1);
      float u = row_rotate<s % 16>(acc[s / 16][i]);
      if constexpr (s % 16 + D + 1 > 16) {
        const float u2 = row_rotate<s % 16>(acc[s / 16 + 1][i]);
        u = (lane & 15) < 16 - s % 16 ? u : u2;
      }
      v += u;
    };
    part(std::integral_constant<int, 2>{});
    part(std::integral_constant<int, 1>{});
    part(std::integral_constant<int, 0>{});
    tot[i] += (double)v;
  }
#pragma unroll
  for (int T = 0; T < bf3_tiles(D); ++T) acc[T] = floatx4{0.f, 0.f, 0.f, 0.f};
}

// The sums of one 16-row block over a 32-column chunk from its exponents
// (t in e): e = 2^t cut into three parts, each with V's columns (see
// pair_kernels.hip).  With `self`, block b1 of the chunk holds the rows' self
// pairs, which are left out.
template <int D>
__device__ __forceinline__ void bf3_accumulate(floatx4 (&e)[2], const bf16x8 (&va)[bf3_tiles(D)], const bf16x8 (&neg)[2],
                                               bool self, int b1, int diag_i, floatx4 (&acc)[bf3_tiles(D)]) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      e[b][i] = __builtin_amdgcn_exp2f(e[b][i]);
      e[b][i] = self && b == b1 && diag_i == i ? 0.f : e[b][i];
    }
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const int nt = ((3 - p) * (D + 1) + 15) / 16;
    const bf16x8 ep = upper_halves(e[0], e[1]);
    if (p < 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) e[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(neg[b], ep, e[b], 0, 0, 0);
    }
#pragma unroll
    for (int T = 0; T < nt; ++T) acc[T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ep, va[T], acc[T], 0, 0, 0);
  }
}

// One piece of 64 x 16 bytes straight from memory to LDS (asynchronous: the
// wave waits on vmcnt before it meets the barrier that publishes the piece).
__device__ __forceinline__ void piece_to_lds(const uint4 *src, uint4 *dst, int lane) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + lane),
                                   (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// f(std::integral_constant<int, D>) for the configuration dimension D.
template <class F>
void by_dimension(int D, F &&f) {
  switch (D) {
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    default: f(std::integral_constant<int, 15>{}); break;
  }
}

}  // namespace vds
