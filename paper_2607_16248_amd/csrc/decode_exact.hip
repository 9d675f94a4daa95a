// Decode and chunk attention on the matrix cores for the caches whose weights
// keep fp32 precision (gfx950): 1- or 2-bit keys with 4- or 8-bit values (or
// the reverse), value groups of 8 or 16 channels, and heads past 4 GiB.
//
// Every factor of both products is exact or carried to 22 bits: q as the fp16
// it is, keys and values as codes times scales in one or two halves
// (scaled_ops.h), weights p as hi + lo halves.  The products are transposed,
//   S^T = K' Q^T   (16 tokens x 16 rows; a lane holds 8 of its row's weights)
//   O^T = V'^T P^T (the same lanes' weights are the B operand),
// so a wave needs no LDS between them; zero-points enter as products of their
// own: K' Q^T with the group's z (and s) in every row gives sum_c q z in
// every lane, and z + c0 s of the value groups, in hi + lo halves, times P^T
// the value terms (z and s apart are opposite and leave their rounding where
// the values average out: 1e-6 over 512 tokens of equal weight, 2e-7 so).
//
// What bounds it: the vector unit, by the unpacking: 2 to 6 instructions per
// operand dword, 64 or more dwords per 32-token block, against 40 to 60
// products.  Each wave takes blocks of its own (key groups j0 + wave + 4n of
// the split), the next block's loads in flight but for the widest classes
// (kAhead); two waves per SIMD, spills of 10 registers in K8V8 with groups of 8
// or 16 and of one or two in K1V8, K2V8 and K8V1 with wider ones.
// The vector kernel it replaces multiplied each code by each row's query (64 *
// rows multiply-adds per token half) from LDS.  Measured, 8 kv heads, split
// kernel alone: 32768 tokens, four heads each, K4V2 16.9 us (vector 29.8),
// K8V1 17.9 (30.5), K2V2 with groups of 16 channels 16.8 (29.3); four sequences
// of that length with five heads K4V2 47 (122), with eight heads and groups of
// 16 K1V4 47 (187); error against 64 bits 2e-7 to 9e-7 (3e-7 to 1e-6).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "decode_common.h"
#include "kvq_internal.h"
#include "kvq_layout.h"
#include "mfma_common.h"
#include "scaled_ops.h"
#include "tail_mfma.h"

namespace kvq {
namespace {

using namespace dec;
using namespace mfma_ops;

constexpr float kTop = 14.f;        // weights stay below 2^14 ...
constexpr float kHeadroom = 6.f;    // ... a new reference puts the largest at 2^8
constexpr float kNoScore = -1e30f;  // below any score
constexpr int kPartRows = 8;        // rows of one pass of the cross-wave reduction

// What a wave reads of one 32-token block a block ahead.  FINE: value groups
// of 8 or 16 channels, a scale row per operand; else one per 32 channels.
template <int BK, int BV>
struct ExactBlock {
  uint32_t kx[2][BK], vx[2 * BV];
  u4_t ks[4], kz[4];
  uint32_t cs, cz;  // the lane's two of the key group's 128 scales and zeros
};
// Its value meta; with FINE groups loaded at the block's start instead of a
// block ahead (32 registers more).
template <bool FINE>
struct ValueMeta {
  u4_t s[FINE ? 8 : 4], zz, zs;
};

template <int BK, int BV, bool FINE>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_exact_kernel(DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) Reduce<kPartRows> red;
  __shared__ float zsh[kWaves][16][17];  // value zero-point terms: [group][row]
  const Work wk = find_work<true>(a);
  const DecodeSeq& S = a.seq[wk.si];
  const uint8_t* ring = a.arena + S.head0 + (uint64_t)wk.h * a.head_stride;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, blk = lane >> 4;
  const int rows = a.qpr * a.gqh;  // of the group; a tile holds 16
  const int inv = (65536 + a.gqh - 1) / a.gqh;
  const size_t rec_rows = (size_t)a.hq * a.nqry;

  // the waves' results of rows r0 .. r0 + 7, merged into records
  auto write_rows = [&](int r0) {
    for (int idx = threadIdx.x; idx < kPartRows * kHeadDim; idx += blockDim.x) {
      const int r = idx / kHeadDim, c = idx % kHeadDim, g = r0 + r;
      const int x = (g * inv) >> 16, j = wk.rg * a.qpr + x;
      if (g >= rows || j >= a.nqry) continue;
      float M = -__builtin_inff();
#pragma unroll
      for (int w = 0; w < kWaves; ++w) M = fmaxf(M, red.m[w][r]);
      float val = 0.f, l = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = red.m[w][r] == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(red.m[w][r] - M);
        val = fmaf(f, red.acc[w][idx], val);
        l = fmaf(f, red.l[w][r], l);
      }
      float* rec = a.ws + ((size_t)(S.ws_base + wk.sp) * rec_rows + (size_t)j * a.hq + wk.h * a.gqh + g - x * a.gqh) * kRecFloats;
      rec[4 + c] = val;
      if (c == 0) { rec[0] = M; rec[1] = l; }
    }
  };

  if (wk.sp >= S.nq) {  // fp16 tail tokens
    TailState<1> st;
    tail_split<1, 16, true>(a, S, wk.h, wk.rg, ring, st, lane, wv);
    for (int r0 = 0; r0 < rows; r0 += kPartRows) {
      __syncthreads();
      stage_tail<kPartRows, 1>(st, 0, r0, red, lane, wv);
      __syncthreads();
      write_rows(r0);
    }
    return;
  }

  // row `col` of the group: its query operand and limit (rows past whole
  // queries, and queries past the last, repeat the last query)
  const int seen0 = S.L - a.nqry + 1;
  u4_t q[4];
  int lim;
  {
    typedef u4_t u4_any __attribute__((aligned(4)));
    const int x = (col * inv) >> 16, j = min(wk.rg * a.qpr + (x < a.qpr ? x : kSpareRow), a.nqry - 1);
    lim = seen0 + j;
    const uint16_t* qr = a.q + (((size_t)S.seq * a.nqry + j) * a.hq + wk.h * a.gqh + (col - x * a.gqh)) * kHeadDim + 8 * blk;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      q[kb] = *reinterpret_cast<const u4_any*>(qr + 32 * kb);
      if constexpr (BK == 1) q[kb] ^= 0x80008000u;  // -q: the code term's factor is negative
    }
  }
  const int first_limit = seen0 + min(wk.rg * a.qpr, a.nqry - 1);

  const int ng = kHeadDim / a.gv, gsh = __builtin_ctz(a.gk), bsh = gsh - 5;
  const int t0 = wk.sp * a.split_tokens, t1 = min(S.Lq, t0 + a.split_tokens);
  const int wslot = (wv + 2 * ((int)blockIdx.x >> 8)) & (kWaves - 1);
  const int j0 = (t0 >> gsh) + wslot, jend = t1 >> gsh;
  const int ngroups = j0 < jend ? (jend - j0 + kWaves - 1) / kWaves : 0;
  const int nblocks = ngroups << bsh;
  auto token_of = [&](int i) { return ((j0 + kWaves * (i >> bsh)) << gsh) + ((i & ((1 << bsh) - 1)) << 5); };

  int vgl[FINE ? 8 : 4];  // byte offset of each scale row's 8 tokens
#pragma unroll
  for (int n = 0; n < (FINE ? 8 : 4); ++n) vgl[n] = ((FINE ? 16 * n + col : 32 * n) / a.gv) * 64 + 16 * blk;
  const int zrow = col < ng ? col : 0;
  auto load = [&](auto lift_c, int i, ExactBlock<BK, BV>& o) {
    int t;
    const uint8_t* seg = a.arena + packed_seg(a.pm, S.head0, a.head_stride, S.seq, wk.h, token_of(i), t);
    const uint8_t* kr = seg + region(a.kc) + (size_t)t * 16 * BK + col * 16 * BK + blk * 4 * BK;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      if constexpr (BK == 1) {
        o.kx[mb][0] = *reinterpret_cast<const uint32_t*>(kr + mb * 256);
      } else if constexpr (BK == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(kr + mb * 512);
        o.kx[mb][0] = v.x;
        o.kx[mb][1] = v.y;
      } else {
#pragma unroll
        for (int w = 0; w < BK / 4; ++w) {
          const u4_t v = *reinterpret_cast<const u4_t*>(kr + mb * 256 * BK + 16 * w);
#pragma unroll
          for (int n = 0; n < 4; ++n) o.kx[mb][4 * w + n] = v[n];
        }
      }
    }
    const uint8_t* km = seg + region(a.km) + (size_t)(t >> gsh) * 512 + 16 * blk;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      o.ks[kb] = *reinterpret_cast<const u4_t*>(km + 64 * kb);
      o.kz[kb] = *reinterpret_cast<const u4_t*>(km + 256 + 64 * kb);
    }
    const uint32_t* kmw = reinterpret_cast<const uint32_t*>(seg + region(a.km) + (size_t)(t >> gsh) * 512);
    if constexpr (decltype(lift_c)::value) {
      o.cs = kmw[lane];
      o.cz = kmw[64 + lane];
    }
    const uint8_t* vr = seg + region(a.vc) + (size_t)(t >> 5) * 512 * BV + lane * 8 * BV;
    if constexpr (BV == 1) {
      const uint2 v = *reinterpret_cast<const uint2*>(vr);
      o.vx[0] = v.x;
      o.vx[1] = v.y;
    } else {
#pragma unroll
      for (int w = 0; w < BV / 2; ++w) {
        const u4_t v = *reinterpret_cast<const u4_t*>(vr + 16 * w);
#pragma unroll
        for (int n = 0; n < 4; ++n) o.vx[4 * w + n] = v[n];
      }
    }
  };
  auto load_meta = [&](int i, ValueMeta<FINE>& o) {
    int t;
    const uint8_t* seg = a.arena + packed_seg(a.pm, S.head0, a.head_stride, S.seq, wk.h, token_of(i), t);
    const uint8_t* vm = seg + region(a.vm) + (size_t)(t >> 5) * 128 * ng;
#pragma unroll
    for (int n = 0; n < (FINE ? 8 : 4); ++n) o.s[n] = *reinterpret_cast<const u4_t*>(vm + vgl[n]);
    o.zs = *reinterpret_cast<const u4_t*>(vm + zrow * 64 + 16 * blk);
    o.zz = *reinterpret_cast<const u4_t*>(vm + (ng + zrow) * 64 + 16 * blk);
  };

  const int X = value_shift<BV>(*reinterpret_cast<const uint32_t*>(ring + region(a.vb)) & 0xFFFFu);
  const h2_t vfac = operand_factor<BV>(X), kfac = operand_factor<BK>(0);
  // raw = alpha sum q z + beta sum q s + sum q K', score = ksc raw (q as held)
  constexpr float kAlpha = BK == 1 ? -2.f : 0.5f, kBeta = BK == 1 ? -1.f : Code<BK>::c0 * 0.5f;
  const float ksc = (BK == 1 ? 0.5f : 2.f) * a.qscale;

  // Small key numbers lose bits: halves below 2^-14 in the products, scales below
  // 2^-13 already in their half and in the lo parts, about 2^-25 of the query for
  // each.  Under queries of 8 or more they enter lifted by 2^12, in products of
  // their own next to larger ones (under smaller queries they move a weight by
  // less than 3e-7): keys of 2^-18 under queries of 2^14 are off by 5e-4 without
  // it and 1e-6 with it.  The test and the lift's registers cost a loop with a
  // block in flight 2 to 17%, so such queries take a loop of their own without
  // one (2 to 8% slower).  Classes whose loop with a block in flight spills go
  // without for every query: 32768 tokens, groups of 16 channels, K8V8 23 us
  // (32), K4V8 23 (27).
  constexpr bool kAhead = BK + BV < 10 || BK == 2;
  constexpr uint32_t kTinyScale = 0x0800u;  // 2^-13
  auto any_half = [](uint32_t w, uint32_t from, uint32_t to) -> bool {  // of the wave's, in [from, to)
    return __builtin_amdgcn_ballot_w64((w & 0xFFFFu) - from < to - from || (w >> 16) - from < to - from) != 0;
  };

  float m = kNoScore, most = kNoScore, l = 0.f, zterm = 0.f;  // the row's reference, the lane's maximum
  f4_t acc[8], zal = {0.f, 0.f, 0.f, 0.f}, zar = {0.f, 0.f, 0.f, 0.f};  // value zero-point terms: lifted, as they are
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] = (f4_t){0.f, 0.f, 0.f, 0.f};

  auto process = [&](auto lift_c, const ExactBlock<BK, BV>& cur, ValueMeta<FINE>& vm, int i) {
    if constexpr (FINE) load_meta(i, vm);
    constexpr bool LIFT = decltype(lift_c)::value;
    const bool first = (i & ((1 << bsh) - 1)) == 0;  // of its key group
    // raw scores of the scales ks (the group's, or a part of them; the rest 0)
    auto raw_scores = [&](const u4_t (&ks)[4], f4_t (&d)[2]) {
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        d[mb] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          uint32_t x[2];
          x[0] = cur.kx[mb][BK == 1 ? 0 : BK == 2 ? kb >> 1 : BK == 4 ? kb : 2 * kb];
          x[1] = BK == 8 ? cur.kx[mb][2 * kb + 1 < BK ? 2 * kb + 1 : 0] : 0u;
          u4_t hi, lo;
          unpack_scaled<BK, false>(x, ks[kb], BK == 1 ? 4 * kb : 8 * (kb & 1), kfac, hi, lo);
          d[mb] = mfma(__builtin_bit_cast(h8_t, hi), __builtin_bit_cast(h8_t, q[kb]), d[mb]);
          if constexpr (Code<BK>::parts == 2)
            d[mb] = mfma(__builtin_bit_cast(h8_t, lo), __builtin_bit_cast(h8_t, q[kb]), d[mb]);
        }
      }
    };
    auto q_sum = [&](const u4_t (&x)[4]) {  // sum over the channels of q x, the same in every lane of the row
      f4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) t = mfma(__builtin_bit_cast(h8_t, x[kb]), __builtin_bit_cast(h8_t, q[kb]), t);
      return t[0];
    };
    const int tok = token_of(i), left = lim - tok - 4 * blk;  // token 16mb + 4blk + r is visible below it
    const bool masked = tok + 32 > first_limit;
    float s[8];
    if (LIFT && (any_half(cur.cs, 1u, kTinyScale) || any_half(cur.cz & 0x7FFF7FFFu, 1u, 0x0400u))) {
      // the small numbers lifted, apart from the others
      u4_t part[4], rest[4];
      if (first) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            uint32_t x, y;
            split_subnormal(cur.kz[kb][n], x, y);
            part[kb][n] = x;
            rest[kb][n] = y;
          }
        zterm = kAlpha * ksc * fmaf(1.f / kLift, q_sum(rest), q_sum(part));
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] = 0.f;
      f4_t d[2];
      auto add = [&](float f) {
        raw_scores(part, d);
        if (first) zterm = fmaf(kBeta * f, q_sum(part), zterm);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = fmaf(d[e >> 2][e & 3], f, s[e]);
      };
      auto keep = [&](bool small) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const uint32_t w = cur.ks[kb][n];
            const uint32_t lo = ((w & 0xFFFFu) < kTinyScale) == small ? 0xFFFFu : 0u, hi = ((w >> 16) < kTinyScale) == small ? 0xFFFF0000u : 0u;
            part[kb][n] = w & (lo | hi);
          }
      };
      if (any_half(cur.cs, kTinyScale, 0x7FFFu)) {
        keep(false);
        add(ksc);
      }
      if (any_half(cur.cs, 1u, kTinyScale)) {
        keep(true);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) part[kb] = __builtin_bit_cast(u4_t, lifted(part[kb], false));
        add(ksc * (1.f / kLift));
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] += zterm;
    } else {
      if (first) zterm = fmaf(kAlpha, q_sum(cur.kz), kBeta * q_sum(cur.ks)) * ksc;
      f4_t d[2];
      raw_scores(cur.ks, d);
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] = fmaf(d[e >> 2][e & 3], ksc, zterm);
    }
    if (masked) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] = 16 * (e >> 2) + (e & 3) < left ? s[e] : kNoScore;
    }
    float top = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
    most = fmaxf(most, top);
    if (__builtin_amdgcn_ballot_w64(top - m > kTop)) {
      // the row's maximum over its four lanes; rows above the limit move
      // their reference
      top = fmaxf(top, __shfl_xor(top, 16));
      top = fmaxf(top, __shfl_xor(top, 32));
      const float mn = top - m > kTop ? top + (kHeadroom - kTop) : m;
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] *= alpha;
      zal *= alpha;
      zar *= alpha;
    }
    u4_t hw, lw;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float p0 = __builtin_amdgcn_exp2f(s[2 * t] - m), p1 = __builtin_amdgcn_exp2f(s[2 * t + 1] - m);
      if (masked) {
        p0 = 16 * (t >> 1) + ((2 * t) & 3) < left ? p0 : 0.f;
        p1 = 16 * (t >> 1) + ((2 * t + 1) & 3) < left ? p1 : 0.f;
      }
      l += p0 + p1;
      const h2_t hi = {(_Float16)p0, (_Float16)p1};
      hw[t] = h2u(hi);
      lw[t] = h2u((h2_t){(_Float16)(p0 - (float)hi.x), (_Float16)(p1 - (float)hi.y)});
    }
    const h8_t ph = __builtin_bit_cast(h8_t, hw), pl = __builtin_bit_cast(h8_t, lw);
    // z + c0 s of the value groups, in hi + lo halves (22 bits): lifted below 8,
    // as it is in an accumulator of its own from there on
    auto add_mid = [&](const float (&x)[8], f4_t& sum) {
      u4_t hi, lo;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const h2_t h = {(_Float16)x[2 * t], (_Float16)x[2 * t + 1]};
        hi[t] = h2u(h);
        lo[t] = h2u((h2_t){(_Float16)(x[2 * t] - (float)h.x), (_Float16)(x[2 * t + 1] - (float)h.y)});
      }
      sum = mfma(__builtin_bit_cast(h8_t, hi), ph, sum);
      sum = mfma(__builtin_bit_cast(h8_t, hi), pl, sum);
      sum = mfma(__builtin_bit_cast(h8_t, lo), ph, sum);
    };
    float mid[8], mtop = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const h2_t z = u2h(vm.zz[t]) * (h2_t){(_Float16)kLift, (_Float16)kLift}, sc = u2h(vm.zs[t]);
      mid[2 * t] = fmaf((float)sc.x, Code<BV>::c0 * kLift, (float)z.x);
      mid[2 * t + 1] = fmaf((float)sc.y, Code<BV>::c0 * kLift, (float)z.y);
      mtop = fmaxf(mtop, fmaxf(fabsf(mid[2 * t]), fabsf(mid[2 * t + 1])));
    }
    if (__builtin_amdgcn_ballot_w64(!(mtop < 8.f * kLift)) == 0) {
      add_mid(mid, zal);
    } else {
      float big[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const h2_t z = u2h(vm.zz[e >> 1]), sc = u2h(vm.zs[e >> 1]);
        const float x = fmaf((float)(e & 1 ? sc.y : sc.x), Code<BV>::c0, (float)(e & 1 ? z.y : z.x));
        const bool is_big = fabsf(x) >= 8.f;
        big[e] = is_big ? x : 0.f;
        mid[e] = is_big ? 0.f : x * kLift;
      }
      add_mid(mid, zal);
      add_mid(big, zar);
    }
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      uint32_t x[2];
      x[0] = cur.vx[BV == 1 ? mb >> 2 : BV == 2 ? mb >> 1 : BV == 4 ? mb : 2 * mb];
      x[1] = BV == 8 ? cur.vx[2 * mb + 1 < 2 * BV ? 2 * mb + 1 : 0] : 0u;
      u4_t hi, lo;
      unpack_scaled<BV, true>(x, vm.s[FINE ? mb : mb >> 1], BV == 1 ? 4 * (mb & 3) : 16 * (mb & 1), vfac, hi, lo);
      acc[mb] = mfma(__builtin_bit_cast(h8_t, hi), ph, acc[mb]);
      acc[mb] = mfma(__builtin_bit_cast(h8_t, hi), pl, acc[mb]);
      if constexpr (Code<BV>::parts == 2) {
        acc[mb] = mfma(__builtin_bit_cast(h8_t, lo), ph, acc[mb]);
        acc[mb] = mfma(__builtin_bit_cast(h8_t, lo), pl, acc[mb]);
      }
    }
  };

  auto run = [&](auto lift_c) {
    const int last = nblocks - 1;
    ExactBlock<BK, BV> b0, b1;
    ValueMeta<FINE> m0, m1;
    auto fetch = [&](int i, ExactBlock<BK, BV>& o, ValueMeta<FINE>& vm) {
      load(lift_c, i, o);
      if constexpr (!FINE) load_meta(i, vm);
    };
    if constexpr (decltype(lift_c)::value || !kAhead) {
      for (int i = 0; i < nblocks; ++i) {
        fetch(i, b0, m0);
        process(lift_c, b0, m0, i);
      }
      return;
    }
    fetch(0, b0, m0);
    int i = 0;
    for (; i + 2 <= nblocks; i += 2) {
      fetch(min(i + 1, last), b1, m1);
      process(lift_c, b0, m0, i);
      fetch(min(i + 2, last), b0, m0);
      process(lift_c, b1, m1, i + 1);
    }
    if (i < nblocks) process(lift_c, b0, m0, i);
  };
  if (nblocks > 0) {
    uint32_t qtop = 0u;  // the tile's largest |q| (the lanes hold all of it)
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int n = 0; n < 4; ++n) qtop = max(qtop, max(q[kb][n] & 0x7FFFu, (q[kb][n] >> 16) & 0x7FFFu));
    if (__builtin_amdgcn_ballot_w64(qtop >= 0x4800u) != 0) run(std::true_type{});  // 8.0
    else run(std::false_type{});
  }

  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  most = fmaxf(most, __shfl_xor(most, 16));
  most = fmaxf(most, __shfl_xor(most, 32));
  const float to_max = __builtin_amdgcn_exp2f(m - most);  // records are relative to the maximum
  // zero-point terms of group 4blk + r, row col, to the lanes of its channels
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    zsh[wv][4 * blk + r][col] = fmaf(zal[r], 1.f / kLift, zar[r]);
  }
  wave_lds_sync();
  const float unit = Code<BV>::unit * ldexpf(1.f, -X);
  const int gvsh = __builtin_ctz(a.gv);
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int g = (FINE ? 16 * t + 4 * blk + r : 16 * t) >> gvsh;
      acc[t][r] = fmaf(acc[t][r], unit, zsh[wv][g][col]) * to_max;
    }
  TailState<1> st;
  st.m[0] = l > 0.f ? most : -__builtin_inff();
  st.l[0] = l * to_max;
#pragma unroll
  for (int t = 0; t < 8; ++t) st.acc[0][t] = acc[t];
  for (int r0 = 0; r0 < rows; r0 += kPartRows) {
    __syncthreads();
    stage_tail<kPartRows, 1>(st, 0, r0, red, lane, wv);
    __syncthreads();
    write_rows(r0);
  }
}

template <int BK, int BV>
int launch_fine(const DecodeArgs& a, void* stream) {
  if (a.gv < 32)
    hipLaunchKernelGGL((decode_exact_kernel<BK, BV, true>), dim3(a.total_wg), dim3(64 * kWaves), 0, (hipStream_t)stream, a);
  else
    hipLaunchKernelGGL((decode_exact_kernel<BK, BV, false>), dim3(a.total_wg), dim3(64 * kWaves), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace

// This source is compiled once per key width (KVQ_BK, set by the build).
template <>
int launch_exact_class<KVQ_BK>(const DecodeArgs& a, int bv, void* stream) {
  switch (bv) {
    case 1: return launch_fine<KVQ_BK, 1>(a, stream);
    case 2: return launch_fine<KVQ_BK, 2>(a, stream);
    case 4: return launch_fine<KVQ_BK, 4>(a, stream);
    case 8: return launch_fine<KVQ_BK, 8>(a, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace kvq
