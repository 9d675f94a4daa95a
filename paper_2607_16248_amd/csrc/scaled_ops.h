// Packed codes as exact fp16 matrix operands that carry their scales (shared
// by the many-row chunk kernel and the decode kernel of the classes whose
// weights keep their low halves):
//   x^ = z + s code = (z + c0 s) + unit * operand
// operand = (code - c0) / 2 * s (unit 2) with c0 = 1, 8, 128 at 2, 4, 8 bits;
// at one bit s (1 - 2 code), the scale with the code as its sign bit (c0 =
// 1/2, unit -1/2).  Two-bit operands are -1/2, 0, 1/2 or 1 times s, one half;
// the 4- and 8-bit products take two, hi = fl(x) and lo = x - hi.
#pragma once

#include "mfma_common.h"

namespace kvq {
namespace mfma_ops {

// what one bit width's operands look like
template <int B>
struct Code {
  static constexpr int parts = B <= 2 ? 1 : 2;                       // fp16 parts of an operand
  static constexpr float c0 = B == 1 ? 0.5f : B == 2 ? 1.f : B == 4 ? 8.f : 128.f;
  static constexpr float unit = B == 1 ? -0.5f : 2.f;                // code term = unit * operand sum
  static constexpr int reach = B <= 2 ? 0 : B == 4 ? 2 : 6;          // |operand| <= 2^reach * s
};

// (code - c0) / 2 * 2^X of a pair whose codes sit at the bits stated below;
// f holds 2^X (or 2^(X-1)) twice.
__device__ __forceinline__ h2_t half_codes2(uint32_t y, h2_t f) {  // bits 8-9 of each half: 2 + code / 2
  return __builtin_elementwise_fma(u2h((y & 0x03000300u) | 0x40004000u), f, f * (h2_t){(_Float16)-2.5f, (_Float16)-2.5f});
}
// (keys: f is 1/2, and the difference takes it in the same fma; a value's f may
// be too large for that)
template <bool VALUE>
__device__ __forceinline__ h2_t half_codes4(uint32_t y, h2_t f) {  // bits 0-3 of each half: 1024 + code
  if constexpr (!VALUE)
    return __builtin_elementwise_fma(u2h((y & 0x000F000Fu) | 0x64006400u), (h2_t){(_Float16)0.5f, (_Float16)0.5f},
                                     (h2_t){(_Float16)-516.f, (_Float16)-516.f});
  return (u2h((y & 0x000F000Fu) | 0x64006400u) - (h2_t){(_Float16)1032.f, (_Float16)1032.f}) * f;
}
template <bool VALUE>
__device__ __forceinline__ h2_t half_codes8(uint32_t x, int pair, h2_t f) {  // bytes 2 * pair, 2 * pair + 1
  const h2_t h = u2h(__builtin_amdgcn_perm(0x64646464u, x, pair ? 0x04030402u : 0x04010400u));
  if constexpr (!VALUE)
    return __builtin_elementwise_fma(h, (h2_t){(_Float16)0.5f, (_Float16)0.5f}, (h2_t){(_Float16)-576.f, (_Float16)-576.f});
  return (h - (h2_t){(_Float16)1152.f, (_Float16)1152.f}) * f;
}
__device__ __forceinline__ void put_product(h2_t c, uint32_t s, uint32_t& hi, uint32_t& lo) {
  const h2_t h = c * u2h(s);
  hi = h2u(h);
  lo = h2u(__builtin_elementwise_fma(c, u2h(s), -h));
}

// Operand parts of 8 elements.  x: the lane's packed dwords of the operand;
// s: the elements' scales; at: where the codes sit (1 bit: pair t at bits at
// + t, +16; 2-bit keys: pair t at 2t, 2t + 16 of x >> at; 2-bit values:
// element e at 2e of x >> at); f: the operand's power of two (two bits: 2^X,
// else 2^(X-1); one bit: 2^X).
template <int B, bool VALUE>
__device__ __forceinline__ void unpack_scaled(const uint32_t (&x)[2], u4_t s, int at, h2_t f, u4_t& hi, u4_t& lo) {
  if constexpr (B == 1) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      hi[t] = ((x[0] << (15 - at - t)) & 0x80008000u) | (VALUE ? h2u(u2h(s[t]) * f) : s[t]);
  } else if constexpr (B == 2 && !VALUE) {
    const uint32_t y = x[0] >> at;
#pragma unroll
    for (int t = 0; t < 4; ++t) hi[t] = h2u(half_codes2(y << (8 - 2 * t), f) * u2h(s[t]));
  } else if constexpr (B == 2) {
    const uint32_t v = (x[0] >> at) & 0xFFFFu, y = v | (v << 14);  // element pair t at 4t, 4t + 16
#pragma unroll
    for (int t = 0; t < 4; ++t) hi[t] = h2u(half_codes2(t < 2 ? y << (8 - 4 * t) : y >> (4 * t - 8), f) * u2h(s[t]));
  } else if constexpr (B == 4) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      uint32_t h, l;
      put_product(half_codes4<VALUE>(x[0] >> (4 * t), f), s[t], h, l);
      hi[t] = h;
      lo[t] = l;
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      uint32_t h, l;
      put_product(half_codes8<VALUE>(x[t >> 1], t & 1, f), s[t], h, l);
      hi[t] = h;
      lo[t] = l;
    }
  }
}

// The power of two X of a head's value operands, from the bound on its scales
// (fp16 bits): |operand| * 2^X < 2^15, and every factor of the operand a finite
// half (2.5 * 2^X, 2^reach * 2^X).  Small scales are lifted out of the
// subnormal range.
template <int BV>
__device__ __forceinline__ int value_shift(uint32_t vbits) {
  constexpr int kMaxX = (BV == 2 ? 13 : 15) - Code<BV>::reach;
  if (vbits == 0u || vbits >= 0x7C00u) return kMaxX;
  int ex = 0;
  frexpf((float)__builtin_bit_cast(_Float16, (uint16_t)vbits), &ex);
  return min(kMaxX, 15 - ex - Code<BV>::reach);
}
// The factor f of unpack_scaled for that power of two (0 for keys).
template <int B>
__device__ __forceinline__ h2_t operand_factor(int X) {
  const _Float16 f = (_Float16)ldexpf(1.f, B > 2 ? X - 1 : X);
  return (h2_t){f, f};
}

}  // namespace mfma_ops
}  // namespace kvq
