// Quantize-on-append for the packed low-bit KV cache (gfx950).
//
// One launch packs every key group that leaves the fp16 window and copies
// the remaining new tokens into the per-head fp16 ring.  The quantizer is
// asymmetric min-max with an fp16 scale rounded up and an fp16 zero-point
// equal to the group minimum; codes round half to even.  The paper names
// b-bit keys and values (Motivation, "Accuracy Loss under Aggressive KV
// Quantization") and asymmetric key/value formats (Related Work) but leaves
// the rule open; this is the rule the library defines in kvq.h.
//
// What bounds it: a prefill reads 512 B of fp16 per token and kv head and
// writes a fraction of that, so HBM should (16384 tokens of 8 heads: 67 MB,
// 14 us at the rate of a large copy); a single key group (decode) is bound
// by its dependent memory round trips.  One workgroup of four waves takes
// one (sequence, kv head, key group), reads every element once into
// registers and packs there:
//   - keys: a lane holds 8 consecutive channels of a token (16-byte loads,
//     four tokens per wave and load).  These are the 8 elements of one matrix
//     operand, so a row dword is one lane's codes, or the OR of two or four
//     lanes 4 apart (DPP row shifts).  Minima and maxima run packed in fp16,
//     across the lane rows by row swaps, across the waves through 2 KB of LDS.
//   - values: wave w holds the 8 tokens of K-group w of a 32-token block, a
//     lane two channels of each, which again are the 8 elements of one
//     operand.  (min, -max) of a token travel as one packed pair; a butterfly
//     over the 16 lanes leaves lane t with token t's pair, so a wave computes
//     all its scales at once and row broadcasts hand them back.
// Codes need no division: see threshold() and quantize().  Measured, against one thread per channel with
// fp64 quotients and bit-by-bit packing: 16384 tokens at K2V2 43 us (164 in
// two launches), 131072 tokens at K1V1 175 us or 3.4 TB/s (1034), the key
// group of a decode step 9 us (42); the vector instructions take about half
// of the 16384-token launch (670 per wave), its ramp and tail the rest.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "decode_common.h"
#include "kvq_internal.h"
#include "kvq_layout.h"

namespace kvq {
namespace {

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ h2_t u2h(uint32_t v) { return __builtin_bit_cast(h2_t, v); }
__device__ __forceinline__ uint32_t h2u(h2_t v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float lo_f(uint32_t v) { return (float)u2h(v).x; }
__device__ __forceinline__ float hi_f(uint32_t v) { return (float)u2h(v).y; }
// Packed fp16 minimum and maximum as one instruction (the builtins quiet each
// operand first; a NaN is found by probe_nan, whatever these return for it).
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kRowShl4 = 0x104, kRowShl8 = 0x108, kRowRor4 = 0x124, kRowRor8 = 0x128, kRowBcast = 0x150;

// The value of the lane 16 (or 32) away joined with the own one by OP.
template <typename OP>
__device__ __forceinline__ uint32_t join16(uint32_t v, OP op) {
  const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return op((uint32_t)s[0], (uint32_t)s[1]);
}
template <typename OP>
__device__ __forceinline__ uint32_t join32(uint32_t v, OP op) {
  const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return op((uint32_t)s[0], (uint32_t)s[1]);
}

// A packed maximum that turns to +inf where the NaN probe (a sum of 0 * x)
// says that the group holds a NaN or an infinity: no finite scale then.
__device__ __forceinline__ uint32_t spoil(uint32_t mx, uint32_t probe) {
  if (__builtin_isnan((float)u2h(probe).x)) mx = (mx & 0xFFFF0000u) | 0x7C00u;
  if (__builtin_isnan((float)u2h(probe).y)) mx = (mx & 0x0000FFFFu) | 0x7C000000u;
  return mx;
}
// Non-finite halves of x as 0 (in groups that got no finite scale).
__device__ __forceinline__ uint32_t finite_or_zero(uint32_t x) {
  if ((x & 0x7C00u) == 0x7C00u) x &= 0xFFFF0000u;
  if ((x & 0x7C000000u) == 0x7C000000u) x &= 0x0000FFFFu;
  return x;
}
__device__ __forceinline__ bool has_nan(uint32_t probe) {
  return __builtin_isnan((float)u2h(probe).x) || __builtin_isnan((float)u2h(probe).y);
}
__device__ __forceinline__ uint32_t probe_nan(uint32_t x, uint32_t acc) {
  return h2u(__builtin_elementwise_fma(u2h(x), (h2_t){(_Float16)0.f, (_Float16)0.f}, u2h(acc)));
}

__device__ __forceinline__ void raise_range(uint8_t* arena) {
  *reinterpret_cast<volatile uint32_t*>(arena) = 4u;  // KVQ_ERR_RANGE
}

// Scale (low half) and zero-point (high half) of a group: the smallest fp16
// s with s * (2^B - 1) >= max - min.  The range and the products are exact
// in fp64, so the step from a rounded guess ends at the exact answer
// (positive fp16 patterns increase with their value).  A group without a
// finite scale gets the NaN pattern 0x7E00 and raises the range flag.
template <int B>
__device__ __forceinline__ uint32_t scale_zero(uint8_t* arena, float mn, float mx) {
  if (mn == 0.f) mn = 0.f;  // +0 zero-point
  const uint32_t zb = __builtin_bit_cast(uint16_t, (_Float16)mn);
  constexpr double n = (double)((1 << B) - 1);
  const double range = (double)mx - (double)mn;
  if (!(range <= 65504.0 * n)) {
    raise_range(arena);
    return 0x7E00u | (zb << 16);
  }
  uint32_t b = 0u;
  if (range > 0.0) {
    // the guess is a neighbour of the quotient: one step at most is missing
    b = min((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)((float)range * (float)(1.0 / n))), 0x7BFFu);
    const uint32_t below = b > 0u ? b - 1u : 0u;
    if ((double)__builtin_bit_cast(_Float16, (uint16_t)b) * n < range) b += 1u;
    else if ((double)__builtin_bit_cast(_Float16, (uint16_t)below) * n >= range) b = below;
  }
  return b | (zb << 16);
}

// One- and two-bit codes compare the fp16 input with the code's thresholds:
// code > k iff x > T_k, T_k the largest fp16 below the boundary z + (k + 1/2) s
// (an x on the boundary rounds to the even code: it stays at k for even k and
// moves up for odd k).  The boundary is exact in fp64, and the sign of the
// fp16 difference T_k - x is exact, two elements at a time.  Groups of one
// value, or without a finite scale, get T_k = +inf: code 0.
constexpr uint32_t kInf16 = 0x7C00u;
template <int K>
__device__ __forceinline__ uint32_t threshold(uint32_t sz) {
  const uint32_t sb = sz & 0xFFFFu;
  if (sb == 0u || sb == 0x7E00u) return kInf16;
  const double b = (double)lo_f(sz) * (K + 0.5) + (double)hi_f(sz);
  const _Float16 t = (_Float16)(float)b;  // a neighbour of b: above it, one step down
  uint32_t u = __builtin_bit_cast(uint16_t, t);
  const bool above = (K & 1) ? (double)t >= b : (double)t > b;
  if (above) u = (u & 0x7FFFu) == 0u ? 0x8001u : (u & 0x8000u) ? u + 1u : u - 1u;
  return u;
}
template <int B>
struct Thresholds {  // both halves of t[k] hold T_k (values), or two channels' T_k (keys)
  uint32_t t[B == 1 ? 1 : 3];
};
// Bits 15 and 31 of p[i] are code bit i of the two elements of x.
template <int B>
__device__ __forceinline__ void code_bits(uint32_t x, const Thresholds<B>& T, uint32_t (&p)[B]) {
  if constexpr (B == 1) {
    p[0] = h2u(u2h(T.t[0]) - u2h(x));
  } else {
    const uint32_t u0 = h2u(u2h(T.t[0]) - u2h(x)), u1 = h2u(u2h(T.t[1]) - u2h(x)), u2 = h2u(u2h(T.t[2]) - u2h(x));
    p[0] = u0 ^ u1 ^ u2;
    p[1] = u1;
  }
}
// Code bits moved to bit `at` (+ the code bit) of each half of acc.
template <int B>
__device__ __forceinline__ void add_codes(uint32_t x, const Thresholds<B>& T, int at, uint32_t& acc) {
  uint32_t p[B];
  code_bits<B>(x, T, p);
#pragma unroll
  for (int i = 0; i < B; ++i) acc |= (p[i] >> (15 - at - i)) & (0x00010001u << (at + i));
}

// fp32 scale, its reciprocal (an estimate) and zero-point of a group.  A
// group without a finite scale gets s = inf: every code 0.
struct Grid {
  float s, rs, z;
};
__device__ __forceinline__ Grid grid_of(uint32_t sz) {
  const bool bad = (sz & 0xFFFFu) == 0x7E00u;
  Grid g;
  g.s = bad ? __builtin_inff() : lo_f(sz);
  g.rs = (sz & 0xFFFFu) != 0u && !bad ? __builtin_amdgcn_rcpf(g.s) : 0.f;
  g.z = bad ? 0.f : hi_f(sz);
  return g;
}

// code = round-half-even((x - z) / s), exactly, without a division.  With
// f = floor of the estimated quotient, the code is f or f + 1 (an estimate
// off by an ulp next to an integer moves f, not the result): r, the sign of
// x - z - (f + 1/2) s, decides.  d = fl(x - z) and (f + 1/2) s (at most 20
// bits) enter one fma, whose sign is exact for d; the rest d_lo = (x - z) - d
// is below half an ulp of d while any nonzero r is at least an ulp of d (the
// product is a multiple of 2^-19 d), so d_lo matters only when r = 0, as does
// the tie to the even code.
template <int B>
__device__ __forceinline__ uint32_t quantize(float x, const Grid& g) {
  const float d = x - g.z;
  const float f = __builtin_floorf(d * g.rs);
  const float r = fmaf(-(f + 0.5f), g.s, d);
  bool up = r > 0.f;
  const uint32_t fi = (uint32_t)f;
  if (__builtin_amdgcn_ballot_w64(r == 0.f)) {
    const float zp = d - x, xp = d - zp, dlo = (x - xp) + (-g.z - zp);  // exact rest of x - z
    if (r == 0.f) up = dlo > 0.f || (dlo == 0.f && (fi & 1u));
  }
  return fi + (up ? 1u : 0u);
}

// 8 halves of a row at p: one 16-byte load, or halves (inputs that are not
// 16-byte aligned).
template <bool AL>
__device__ __forceinline__ u4_t load8(const uint16_t* p) {
  if constexpr (AL) return *reinterpret_cast<const u4_t*>(p);
  u4_t v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = (uint32_t)p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
  return v;
}
template <bool AL>
__device__ __forceinline__ uint32_t load2(const uint16_t* p) {
  if constexpr (AL) return *reinterpret_cast<const uint32_t*>(p);
  return (uint32_t)p[0] | ((uint32_t)p[1] << 16);
}

// Row of token p: in the ring (appended by an earlier call) or in the input.
struct Rows {
  const uint16_t* in;    // input row of token L_old of this head
  const uint16_t* ring;
  size_t stride;         // halves from one input token to the next
  int L_old, W;
  bool fresh;            // none of the group's tokens sits in the ring (uniform)
  __device__ __forceinline__ const uint16_t* at(int p) const {
    if (!fresh && p < L_old) return ring + (size_t)(p % W) * kHeadDim;
    return in + (size_t)(p - L_old) * stride;
  }
};

// The lane's part of its key row dwords (kvq_layout.h: key_bit)
// into the row at o: operand block kb, lane group g4.
template <int B>
__device__ __forceinline__ void store_key_words(const uint32_t (&w)[2], int kb, int g4, uint32_t* o) {
  if constexpr (B == 1) {  // dword g4: the four blocks kb, lanes 4 apart
    uint32_t v = w[0] << (4 * kb);
    v |= dpp<kRowShl4>(v);
    v |= dpp<kRowShl8>(v);
    if (kb == 0) o[g4] = v;
  } else if constexpr (B == 2) {  // dword 2*g4 + (kb >> 1): two blocks
    uint32_t v = w[0] << (8 * (kb & 1));
    v |= dpp<kRowShl4>(v);
    if ((kb & 1) == 0) o[2 * g4 + (kb >> 1)] = v;
  } else if constexpr (B == 4) {
    o[4 * g4 + kb] = w[0];
  } else {
    *reinterpret_cast<uint2*>(o + 8 * g4 + 2 * kb) = make_uint2(w[0], w[1]);
  }
}

// Keys of one group, second half: codes of the lane's 8 channels of the
// tokens t = 16*i + 4*wv + row.  par: per channel,
// the thresholds [k][128] (fp16) at one and two bits, (scale, zero) else.
template <int B, int GK>
__device__ __forceinline__ void key_codes(const u4_t (&x)[GK / 16], const uint32_t* par, uint8_t* dst,
                                          int lane, int wv) {
  const int cc = lane & 15, row = lane >> 4, kb = cc >> 2, g4 = cc & 3;
  if constexpr (B <= 2) {
    constexpr int NT = B == 1 ? 1 : 3;
    u4_t tk[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) tk[k] = *reinterpret_cast<const u4_t*>(par + 64 * k + 4 * cc);
#pragma unroll
    for (int i = 0; i < GK / 16; ++i) {
      uint8_t* rowp = dst + (size_t)(16 * i + 4 * wv + row) * 16 * B;
      uint32_t acc = 0u;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        Thresholds<B> T;
#pragma unroll
        for (int k = 0; k < NT; ++k) T.t[k] = tk[k][m];
        add_codes<B>(x[i][m], T, B * m, acc);  // pair m at bits B*m and 16 + B*m
      }
      const uint32_t w[2] = {acc, 0u};
      store_key_words<B>(w, kb, g4, reinterpret_cast<uint32_t*>(rowp));
    }
  } else {
    Grid g[8];
    const u4_t a = *reinterpret_cast<const u4_t*>(par + 8 * cc), b = *reinterpret_cast<const u4_t*>(par + 8 * cc + 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = grid_of(e < 4 ? a[e] : b[e - 4]);
#pragma unroll
    for (int i = 0; i < GK / 16; ++i) {
      uint32_t c[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) c[e] = quantize<B>(e & 1 ? hi_f(x[i][e >> 1]) : lo_f(x[i][e >> 1]), g[e]);
      uint8_t* rowp = dst + (size_t)(16 * i + 4 * wv + row) * 16 * B;
      uint32_t w[2] = {0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (B == 8) w[e >> 2] |= c[e] << (8 * (e & 3));
        else w[0] |= c[e] << (B * (e >> 1) + 16 * (e & 1));
      }
      store_key_words<B>(w, kb, g4, reinterpret_cast<uint32_t*>(rowp));
    }
  }
}

// (min, -max) of the two halves of x in one packed pair: minima alone join
// two such pairs.
__device__ __forceinline__ uint32_t min_negmax(uint32_t x) {
  const uint32_t l2 = __builtin_amdgcn_perm(0u, x, 0x01000100u) ^ 0x80000000u;
  const uint32_t h2 = __builtin_amdgcn_perm(0u, x, 0x03020302u) ^ 0x80000000u;
  return pk_min(l2, h2);
}

// f(std::integral_constant<int, t>) for the 8 tokens of a lane.
template <typename F>
__device__ __forceinline__ void for_tokens(F f) {
  f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{});
  f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{});
  f(std::integral_constant<int, 4>{}); f(std::integral_constant<int, 5>{});
  f(std::integral_constant<int, 6>{}); f(std::integral_constant<int, 7>{});
}

// Values of one 32-token block: wave wv = K-group, lane =
// channels 2*lane, 2*lane + 1, x[t] = token value_token(wv, t).  FINE: groups
// of 8 or 16 channels.  Returns the
// wave's largest scale (fp16 bits).
template <int B, bool FINE>
__device__ __forceinline__ uint32_t value_block(uint8_t* arena, uint32_t (&x)[8], int gv, uint8_t* vcb,
                                                       uint8_t* vmb, int lane, int wv) {
  uint32_t m[8], nan = 0u;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    m[t] = min_negmax(x[t]);
    nan = probe_nan(x[t], nan);
  }
  if (__builtin_amdgcn_ballot_w64(has_nan(nan))) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (finite_or_zero(x[t]) != x[t]) {
        m[t] = 0xFC007C00u;  // range +inf
        x[t] = finite_or_zero(x[t]);
      }
  }
  // butterfly over four lanes: o[j] = token 4j + (lane & 3) of their 8 channels
  const bool b0 = lane & 1, b1 = lane & 2;
  uint32_t n[4], o[2];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    n[j] = pk_min(b0 ? m[2 * j + 1] : m[2 * j], dpp<dec::kQuadXor1>(b0 ? m[2 * j] : m[2 * j + 1]));
#pragma unroll
  for (int j = 0; j < 2; ++j)
    o[j] = pk_min(b1 ? n[2 * j + 1] : n[2 * j], dpp<dec::kQuadXor2>(b1 ? n[2 * j] : n[2 * j + 1]));
  // the rest of the group's lanes; a lane then takes token (lane & 7), groups
  // of 8 channels both of its tokens
  const int lpg = gv / 2, ng = kHeadDim / gv;  // lanes per group
  uint32_t sz, sz2 = 0u;
  uint16_t* meta = reinterpret_cast<uint16_t*>(vmb);  // scales [g][pos], then zeros (value_meta_s / value_meta_z)
  auto put_meta = [&](int g, int t, uint32_t v) {
    meta[g * 32 + 8 * wv + t] = (uint16_t)v;
    meta[(ng + g) * 32 + 8 * wv + t] = (uint16_t)(v >> 16);
  };
  if constexpr (!FINE) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      o[j] = pk_min(o[j], dpp<kRowRor4>(o[j]));
      o[j] = pk_min(o[j], dpp<kRowRor8>(o[j]));
    }
    uint32_t v = (lane & 4) ? o[1] : o[0];
    if (gv >= 64) v = join16(v, pk_min);
    if (gv >= 128) v = join32(v, pk_min);
    sz = scale_zero<B>(arena, lo_f(v), -hi_f(v));
    if ((lane & 15) < 8 && (lane & (lpg - 1)) < 16) put_meta(lane / lpg, lane & 7, sz);
  } else if (gv == 16) {
#pragma unroll
    for (int j = 0; j < 2; ++j) o[j] = pk_min(o[j], (uint32_t)__shfl_xor((int)o[j], 4));
    const uint32_t v = (lane & 4) ? o[1] : o[0];
    sz = scale_zero<B>(arena, lo_f(v), -hi_f(v));
    put_meta(lane / lpg, lane & 7, sz);
  } else {
    sz = scale_zero<B>(arena, lo_f(o[0]), -hi_f(o[0]));
    sz2 = scale_zero<B>(arena, lo_f(o[1]), -hi_f(o[1]));
    put_meta(lane / lpg, lane & 3, sz);
    put_meta(lane / lpg, 4 + (lane & 3), sz2);
  }
  // a value that its group's lanes hold for token t, in every lane (v2: tokens
  // 4-7 of groups of 8 channels)
  auto of_token = [&](auto tc, uint32_t v, uint32_t v2) -> uint32_t {
    constexpr int t = decltype(tc)::value;
    if constexpr (!FINE) return dpp<kRowBcast + t>(v);
    if (gv == 16) return (uint32_t)__shfl((int)v, (lane & ~7) + t);
    return (uint32_t)__shfl((int)(t < 4 ? v : v2), (lane & ~3) + (t & 3));
  };
  // codes of the two channels, element t of their operand words w0, w1
  uint32_t w0[2] = {0u, 0u}, w1[2] = {0u, 0u};
  if constexpr (B <= 2) {
    constexpr int NT = B == 1 ? 1 : 3;
    uint32_t own[3], own2[3] = {0u, 0u, 0u};
    own[0] = threshold<0>(sz) * 0x10001u;
    if constexpr (B == 2) {
      own[1] = threshold<1>(sz) * 0x10001u;
      own[2] = threshold<2>(sz) * 0x10001u;
    }
    if (FINE && gv == 8) {
      own2[0] = threshold<0>(sz2) * 0x10001u;
      if constexpr (B == 2) {
        own2[1] = threshold<1>(sz2) * 0x10001u;
        own2[2] = threshold<2>(sz2) * 0x10001u;
      }
    }
    uint32_t acc = 0u;  // low half: the even channel, high half: the odd one
    for_tokens([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      Thresholds<B> T;
#pragma unroll
      for (int k = 0; k < NT; ++k) T.t[k] = of_token(tc, own[k], own2[k]);
      add_codes<B>(x[t], T, B == 1 ? (t >> 1) + 4 * (t & 1) : 2 * t, acc);
    });
    if constexpr (B == 1) {  // pairs apart: elements 2i at bit i, 2i + 1 at bit 16 + i
      w0[0] = (acc & 0xFu) | ((acc & 0xF0u) << 12);
      w1[0] = ((acc >> 16) & 0xFu) | ((acc >> 4) & 0xF0000u);
    } else {
      w0[0] = acc & 0xFFFFu;
      w1[0] = acc >> 16;
    }
  } else {
    for_tokens([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      const Grid g = grid_of(of_token(tc, sz, sz2));
      constexpr int sh = B == 4 ? 4 * (t >> 1) + 16 * (t & 1) : 8 * (t & 3);
      w0[B == 8 ? t >> 2 : 0] |= quantize<B>(lo_f(x[t]), g) << sh;
      w1[B == 8 ? t >> 2 : 0] |= quantize<B>(hi_f(x[t]), g) << sh;
    });
  }
  const int mb = lane >> 3, c16 = 2 * (lane & 7);
  uint32_t* o32 = reinterpret_cast<uint32_t*>(vcb);
  auto bit_or = [](uint32_t p, uint32_t q) { return p | q; };
  if constexpr (B <= 2) {
    // operands that share a dword sit in lanes 8 (and 16) apart; of the
    // lanes that then hold the same word, one stores the even channel and
    // one the odd
    w0[0] <<= B == 1 ? 4 * (mb & 3) : 16 * (mb & 1);
    w1[0] <<= B == 1 ? 4 * (mb & 3) : 16 * (mb & 1);
    w0[0] |= dpp<kRowRor8>(w0[0]);
    w1[0] |= dpp<kRowRor8>(w1[0]);
    uint32_t w = (mb & 1) ? w1[0] : w0[0];
    const int L = c16 + (mb & 1) + 16 * wv;
    if constexpr (B == 1) {
      w = join16(w, bit_or);
      if ((lane & 16) == 0) o32[L * 2 + (mb >> 2)] = w;
    } else {
      o32[L * 4 + (mb >> 1)] = w;
    }
  } else if constexpr (B == 4) {
    o32[(c16 + 16 * wv) * 8 + mb] = w0[0];
    o32[(c16 + 1 + 16 * wv) * 8 + mb] = w1[0];
  } else {
    *reinterpret_cast<uint2*>(o32 + (c16 + 16 * wv) * 16 + 2 * mb) = make_uint2(w0[0], w0[1]);
    *reinterpret_cast<uint2*>(o32 + (c16 + 1 + 16 * wv) * 16 + 2 * mb) = make_uint2(w1[0], w1[1]);
  }
  const uint32_t s = sz & 0xFFFFu, s2 = sz2 & 0xFFFFu;
  return max(s == 0x7E00u ? 0u : s, s2 == 0x7E00u ? 0u : s2);
}

template <bool FINE>
__device__ __forceinline__ uint32_t quantize_values(const AppendArgs& a, int bv, uint32_t (&vx)[8], uint8_t* vcb,
                                                    uint8_t* vmb, int lane, int wv) {
  switch (bv) {
    case 1: return value_block<1, FINE>(a.arena, vx, a.gv, vcb, vmb, lane, wv);
    case 2: return value_block<2, FINE>(a.arena, vx, a.gv, vcb, vmb, lane, wv);
    case 4: return value_block<4, FINE>(a.arena, vx, a.gv, vcb, vmb, lane, wv);
    default: return value_block<8, FINE>(a.arena, vx, a.gv, vcb, vmb, lane, wv);
  }
}

template <int GK, bool AL>
__device__ __forceinline__ void quantize_group(const AppendArgs& a, const AppendSeq& S, int h, int gi, int bk, int bv,
                                               uint32_t* minmax, uint32_t* par) {
  uint8_t* blk = a.arena + S.head0 + (uint64_t)h * a.head_stride;  // the fp16 ring's region
  const int p0 = S.Lq_old + gi * GK;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cc = lane & 15, row = lane >> 4;
  const size_t in0 = ((size_t)S.seq * a.n_max * a.hkv + h) * kHeadDim;
  const Rows rk{a.K + in0, reinterpret_cast<const uint16_t*>(blk + region(a.tk)), (size_t)a.hkv * kHeadDim, S.L_old, a.W, p0 >= S.L_old};
  const Rows rv{a.V + in0, reinterpret_cast<const uint16_t*>(blk + region(a.tv)), (size_t)a.hkv * kHeadDim, S.L_old, a.W, p0 >= S.L_old};

  u4_t kx[GK / 16];
#pragma unroll
  for (int i = 0; i < GK / 16; ++i) kx[i] = load8<AL>(rk.at(p0 + 16 * i + 4 * wv + row) + 8 * cc);
  uint32_t vx[8];
  auto load_v = [&](int b) {
#pragma unroll
    for (int t = 0; t < 8; ++t) vx[t] = load2<AL>(rv.at(p0 + 32 * b + value_token(wv, t)) + 2 * lane);
  };
  load_v(0);
  uint32_t* bound = reinterpret_cast<uint32_t*>(blk + region(a.vb));
  const uint32_t seen = __hip_atomic_load(bound, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // the packed segment (head region or page) of the group, and the group's
  // first token in it
  int t0;
  uint8_t* seg = a.arena + packed_seg(a.pm, S.head0, a.head_stride, S.seq, h, p0, t0);

  // minima and maxima of the lane's channel pairs over its tokens, then over
  // the lane rows; the waves' results meet in LDS
  {
    u4_t mn = kx[0], mx = kx[0], nan = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < GK / 16; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i > 0) {
          mn[k] = pk_min(mn[k], kx[i][k]);
          mx[k] = pk_max(mx[k], kx[i][k]);
        }
        nan[k] = probe_nan(kx[i][k], nan[k]);
      }
    if (__builtin_amdgcn_ballot_w64(has_nan(nan[0]) || has_nan(nan[1]) || has_nan(nan[2]) || has_nan(nan[3]))) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        mx[k] = spoil(mx[k], nan[k]);
#pragma unroll
        for (int i = 0; i < GK / 16; ++i) kx[i][k] = finite_or_zero(kx[i][k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      mn[k] = join32(join16(mn[k], pk_min), pk_min);
      mx[k] = join32(join16(mx[k], pk_max), pk_max);
    }
    if (row == 0) {
      *reinterpret_cast<u4_t*>(minmax + wv * 128 + 4 * cc) = mn;
      *reinterpret_cast<u4_t*>(minmax + wv * 128 + 64 + 4 * cc) = mx;
    }
  }
  __syncthreads();
  if (threadIdx.x < kHeadDim) {
    const int c = threadIdx.x;
    const uint16_t* mm = reinterpret_cast<const uint16_t*>(minmax);
    float mn = __builtin_inff(), mx = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      mn = fminf(mn, (float)__builtin_bit_cast(_Float16, mm[w * 256 + c]));
      mx = fmaxf(mx, (float)__builtin_bit_cast(_Float16, mm[w * 256 + 128 + c]));
    }
    uint16_t* t16 = reinterpret_cast<uint16_t*>(par);
    uint32_t v;
    switch (bk) {
      case 1:
        v = scale_zero<1>(a.arena, mn, mx);
        t16[c] = (uint16_t)threshold<0>(v);
        break;
      case 2:
        v = scale_zero<2>(a.arena, mn, mx);
        t16[c] = (uint16_t)threshold<0>(v);
        t16[128 + c] = (uint16_t)threshold<1>(v);
        t16[256 + c] = (uint16_t)threshold<2>(v);
        break;
      case 4: par[c] = v = scale_zero<4>(a.arena, mn, mx); break;
      default: par[c] = v = scale_zero<8>(a.arena, mn, mx); break;
    }
    uint16_t* km = reinterpret_cast<uint16_t*>(seg + region(a.km)) + (size_t)(t0 / GK) * 2 * kHeadDim;
    km[c] = (uint16_t)v;
    km[kHeadDim + c] = (uint16_t)(v >> 16);
  }

  // values: they need no other wave, and overlap the keys' scales
  const int ng = kHeadDim / a.gv;
  uint32_t most = 0u;
  for (int b = 0; b < GK / 32; ++b) {
    if (b > 0) load_v(b);
    uint8_t* vcb = seg + region(a.vc) + (size_t)(t0 + 32 * b) * 16 * bv;
    uint8_t* vmb = seg + region(a.vm) + (size_t)(t0 + 32 * b) * 4 * ng;
    const uint32_t s = a.gv >= 32 ? quantize_values<false>(a, bv, vx, vcb, vmb, lane, wv)
                   : quantize_values<true>(a, bv, vx, vcb, vmb, lane, wv);
    most = max(most, s);
  }
  // the largest value scale raises the head's bound (decode sizes its weight
  // shift by it); the bound only grows, so a wave below a value seen earlier
  // has nothing to add
  if (__builtin_amdgcn_ballot_w64(most > seen)) {
    for (int d = 32; d > 0; d >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, d));
    if (lane == 0) atomicMax(bound, most);
  }

  __syncthreads();
  uint8_t* kdst = seg + region(a.kc) + (size_t)t0 * 16 * bk;
  switch (bk) {
    case 1: key_codes<1, GK>(kx, par, kdst, lane, wv); break;
    case 2: key_codes<2, GK>(kx, par, kdst, lane, wv); break;
    case 4: key_codes<4, GK>(kx, par, kdst, lane, wv); break;
    default: key_codes<8, GK>(kx, par, kdst, lane, wv); break;
  }
}

// Copy part `part` (kCopyTokens tokens) of the new tokens that stay fp16 into
// the ring of head h.
template <bool AL>
__device__ __forceinline__ void copy_ring(const AppendArgs& a, const AppendSeq& S, int h, int part) {
  uint8_t* blk = a.arena + S.head0 + (uint64_t)h * a.head_stride;
  const int first = max(S.Lq_new, S.L_old) + part * kCopyTokens, end = min(S.L_new, first + kCopyTokens);
  const size_t in0 = ((size_t)S.seq * a.n_max * a.hkv + h) * kHeadDim;
  constexpr int kPer = kCopyTokens * (kHeadDim / 8) / kAppendThreads;  // 16-byte pieces per thread and tensor
  u4_t x[2][kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = i * kAppendThreads + threadIdx.x, p = first + (idx >> 4);
    if (p < end) {
      const size_t src = in0 + (size_t)(p - S.L_old) * a.hkv * kHeadDim + (idx & 15) * 8;
      x[0][i] = load8<AL>(a.K + src);
      x[1][i] = load8<AL>(a.V + src);
    }
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = i * kAppendThreads + threadIdx.x, p = first + (idx >> 4);
    if (p < end) {
      const size_t dst = ((size_t)(p % a.W) * kHeadDim + (idx & 15) * 8) * 2;
      *reinterpret_cast<u4_t*>(blk + region(a.tk) + dst) = x[0][i];
      *reinterpret_cast<u4_t*>(blk + region(a.tv) + dst) = x[1][i];
    }
  }
}

template <int GK, bool AL>
__global__ __launch_bounds__(kAppendThreads) void append_kernel(AppendArgs a, int bk, int bv) {
  __shared__ __attribute__((aligned(16))) uint32_t minmax[4 * 128], par[192];
  const int wg = blockIdx.x;
  int si = 0;
  for (int i = 1; i < a.nseq; ++i) si = (a.seq[i].wg_begin <= wg) ? i : si;
  const AppendSeq& S = a.seq[si];
  // kv heads fastest: neighbouring workgroups read neighbouring 256-byte rows
  const int local = wg - S.wg_begin, part = local / a.hkv, h = local - part * a.hkv;
  const int nquant = a.quantize ? S.n_quant : 0;
  if (part < nquant) {
    quantize_group<GK, AL>(a, S, h, part, bk, bv, minmax, par);
  } else {
    copy_ring<AL>(a, S, h, part - nquant);
  }
}

__global__ __launch_bounds__(256) void table_set_kernel(TableSet t) {
  for (int i = threadIdx.x; i < t.n; i += blockDim.x) t.table[t.idx[i]] = t.val[i];
}

__global__ __launch_bounds__(256) void word_reset_kernel(WordReset r) {
  for (int i = threadIdx.x; i < r.n; i += blockDim.x) *reinterpret_cast<uint32_t*>(r.arena + r.off[i]) = 0u;
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

}  // namespace

int launch_append(const AppendArgs& a, int bk, int bv, void* stream) {
  if (a.total_wg <= 0) return 0;
  // 16-byte input loads where both inputs allow them
  const bool al = (reinterpret_cast<uintptr_t>(a.K) | reinterpret_cast<uintptr_t>(a.V)) % 16 == 0;
  const dim3 grid(a.total_wg), block(kAppendThreads);
  hipStream_t s = (hipStream_t)stream;
  switch (a.gk) {
    case 32:
      if (al) hipLaunchKernelGGL((append_kernel<32, true>), grid, block, 0, s, a, bk, bv);
      else hipLaunchKernelGGL((append_kernel<32, false>), grid, block, 0, s, a, bk, bv);
      break;
    case 64:
      if (al) hipLaunchKernelGGL((append_kernel<64, true>), grid, block, 0, s, a, bk, bv);
      else hipLaunchKernelGGL((append_kernel<64, false>), grid, block, 0, s, a, bk, bv);
      break;
    case 128:
      if (al) hipLaunchKernelGGL((append_kernel<128, true>), grid, block, 0, s, a, bk, bv);
      else hipLaunchKernelGGL((append_kernel<128, false>), grid, block, 0, s, a, bk, bv);
      break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_table_set(const TableSet& t, void* stream) {
  if (t.n <= 0) return 0;
  hipLaunchKernelGGL(table_set_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, t);
  return (int)hipGetLastError();
}

int launch_word_reset(const WordReset& r, void* stream) {
  if (r.n <= 0) return 0;
  hipLaunchKernelGGL(word_reset_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, r);
  return (int)hipGetLastError();
}

int launch_fill_zero(void* dst, size_t words, void* stream) {
  if (words == 0) return 0;
  const unsigned blocks = (unsigned)((words + 255) / 256 < 1024 ? (words + 255) / 256 : 1024);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream,
                     (uint32_t*)dst, words);
  return (int)hipGetLastError();
}

}  // namespace kvq
