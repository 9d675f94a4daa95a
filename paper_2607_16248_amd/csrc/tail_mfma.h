// The fp16-tail split on the matrix cores: the tokens [Lq, L) of one
// (sequence, kv head), at most a window and a key group of them, read from
// the fp16 ring (or, in a fused append, the call's own new tokens from its
// inputs) and attended by up to 16 * NT (query, head) rows of a workgroup.
//
// Both products are transposed: S^T = K Q^T leaves a row's 8 weights of a
// 32-token block in the lanes that are the B operand of O^T = V^T P^T.  The
// keys' rows are operands as they lie in memory; an operand of V^T gathers 8
// tokens of one channel, 16 channels (32 bytes) per row.  q, k and v are exact
// fp16 operands; p = 2^(score - maximum) enters as hi + lo halves (22 bits),
// times 2^14 so that both stay normal numbers (a reference 14 below the maximum
// would round the difference to 2^-21 instead).  Records hold the maximum.
//
// What bounds it: latency.  A wave's first block is four dependent steps
// (arguments, the rows, two products, the reduction), and four waves share
// the blocks.  The vector version kept the query in LDS and issued 64 * rows
// fused multiply-adds per token half after as many LDS reads: with a tail of
// 128-160 tokens a decode launch over 2000 tokens took 14.8 us and takes 8.1,
// five chunk queries of 32 rows over 32768 tokens took 50 and take 27.
#pragma once

#include "decode_common.h"
#include "kvq_layout.h"
#include "mfma_common.h"

namespace kvq {
namespace dec {

using mfma_ops::f4_t;
using mfma_ops::h2_t;
using mfma_ops::h8_t;
using mfma_ops::u4_t;

constexpr float kTailUnit = 16384.f;  // weights times 2^14 inside tail_split

// row 16u + col of the tile in lane (col, block): maximum, its weights' sum
// over the lane's tokens, accumulators of channels 16t + 4 * block + r
template <int NT>
struct TailState {
  float m[NT], l[NT];
  f4_t acc[NT][8];
};

// Rows g0 .. g0 + 16 * NT - 1 of the workgroup's group of ROWS rows (those past
// it repeat its first row and are dropped by the caller).
template <int NT, int ROWS, bool CHUNK, int AHEAD = 4>
__device__ __forceinline__ void tail_split(const DecodeArgs& a, const DecodeSeq& S, int h, int rg, const uint8_t* ring,
                                           TailState<NT>& st, int lane, int wv) {
  typedef u4_t u4_any __attribute__((aligned(4)));
  const int col = lane & 15, blk = lane >> 4;
  const int seen0 = S.L - a.nqry + 1;
  u4_t q[NT][4];
  int lim[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    int g = 16 * u + col;
    size_t at;
    if constexpr (CHUNK) {
      // query x of the group and head of row g; rows past whole queries and
      // queries past the last repeat the last query
      const int x = (g * ((65536 + a.gqh - 1) / a.gqh)) >> 16;  // g / gqh (g < 32)
      const int j = min(rg * a.qpr + (x < a.qpr ? x : kSpareRow), a.nqry - 1);
      lim[u] = seen0 + j;
      at = ((size_t)S.seq * a.nqry + j) * a.hq + h * a.gqh + (g - x * a.gqh);
    } else {
      g = g < ROWS ? g : 0;
      lim[u] = S.L;
      at = (size_t)S.seq * a.hq + (size_t)h * ROWS + g;
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      q[u][kb] = *reinterpret_cast<const u4_any*>(a.q + at * kHeadDim + 32 * kb + 8 * blk);
    st.m[u] = -__builtin_inff();
    st.l[u] = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) st.acc[u][t] = (f4_t){0.f, 0.f, 0.f, 0.f};
  }

  // Fused append: this workgroup stores the call's new tokens, which all stay
  // fp16, into the ring; it attends over them from the inputs, so the stores
  // are not waited for.
  const int n_new = a.K_new != nullptr ? S.L - S.L_old : 0;
  const size_t new0 = ((size_t)S.seq * a.n_max * a.hkv + h) * kHeadDim, new_stride = (size_t)a.hkv * kHeadDim;
  if (n_new > 0) {
    uint32_t* rk = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(ring) + region(a.tk));
    uint32_t* rv = reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(ring) + region(a.tv));
    constexpr int kRow = kHeadDim / 2;  // dwords per token row
    for (int idx = threadIdx.x; idx < n_new * kRow; idx += blockDim.x) {
      const int t = idx / kRow, c = idx % kRow;
      const size_t dst = (size_t)((S.L_old + t) % a.W) * kRow + c;
      rk[dst] = reinterpret_cast<const uint32_t*>(a.K_new + new0 + t * new_stride)[c];
      rv[dst] = reinterpret_cast<const uint32_t*>(a.V_new + new0 + t * new_stride)[c];
    }
  }
  const int ntail = S.L - S.Lq, slot0 = S.Lq % a.W;
  // the row of tail token i (past the last: the last), in the ring or the inputs
  auto row_at = [&](int i, const uint16_t* in, uint64_t at) -> const uint16_t* {
    i = min(i, ntail - 1);
    int slot = slot0 + i;
    slot = slot >= a.W ? slot - a.W : slot;
    const uint16_t* r = reinterpret_cast<const uint16_t*>(ring + at + (uint64_t)(uint32_t)slot * (kHeadDim * 2));
    if (n_new > 0 && i >= ntail - n_new) r = in + new0 + (size_t)(i - (ntail - n_new)) * new_stride;
    return r;
  };

  bool raw[8] = {};  // per tile of 16 channels: its values enter lifted while they are small
  for (int b = wv; 32 * b < ntail; b += kWaves) {
    // scores: tokens 32b + 16mb + 4blk + r of row 16u + col
    f4_t d[NT][2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const uint16_t* kr = row_at(32 * b + 16 * mb + col, a.K_new, region(a.tk)) + 8 * blk;
      u4_t k[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) k[kb] = *reinterpret_cast<const u4_any*>(kr + 32 * kb);
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        d[u][mb] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
          d[u][mb] = mfma_ops::mfma(__builtin_bit_cast(h8_t, k[kb]), __builtin_bit_cast(h8_t, q[u][kb]), d[u][mb]);
      }
    }
    const uint16_t* vr[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) vr[e] = row_at(32 * b + value_token(blk, e), a.V_new, region(a.tv)) + col;
    h8_t ph[NT], pl[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int left = min(lim[u] - S.Lq, ntail) - 32 * b - 4 * blk;  // token 16mb + 4blk + r is visible below it
      float s[8], top = -__builtin_inff();
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        s[e] = 16 * (e >> 2) + (e & 3) < left ? d[u][e >> 2][e & 3] * a.qscale : -__builtin_inff();
        top = fmaxf(top, s[e]);
      }
      top = fmaxf(top, __shfl_xor(top, 16));
      top = fmaxf(top, __shfl_xor(top, 32));
      // a row with no visible token yet keeps m = -inf
      const float mn = fmaxf(st.m[u], top);
      const bool none = mn == -__builtin_inff();
      const float alpha = none ? 1.f : __builtin_amdgcn_exp2f(st.m[u] - mn);
      st.m[u] = mn;
      st.l[u] *= alpha;
#pragma unroll
      for (int t = 0; t < 8; ++t) st.acc[u][t] *= alpha;
      u4_t hw, lw;
      float sum[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float p0 = none ? 0.f : __builtin_amdgcn_exp2f(s[2 * t] - mn);
        const float p1 = none ? 0.f : __builtin_amdgcn_exp2f(s[2 * t + 1] - mn);
        const h2_t hi = {(_Float16)(p0 * kTailUnit), (_Float16)(p1 * kTailUnit)};
        hw[t] = mfma_ops::h2u(hi);
        lw[t] = mfma_ops::h2u((h2_t){(_Float16)fmaf(p0, kTailUnit, -(float)hi.x), (_Float16)fmaf(p1, kTailUnit, -(float)hi.y)});
        sum[t] = mfma_ops::add_halves(lw[t], mfma_ops::add_halves(hw[t], 0.f));
      }
      st.l[u] += (sum[0] + sum[1]) + (sum[2] + sum[3]);
      ph[u] = __builtin_bit_cast(h8_t, hw);
      pl[u] = __builtin_bit_cast(h8_t, lw);
    }
    // AHEAD tiles are under way while one is in work (the branches below keep
    // loads from moving up by themselves: a tail of 142 tokens 9.8 us, 10.4 without).
    // The kernels of four waves per SIMD have no registers for it.
    u4_t ahead[8];
    auto gather = [&](int t) {
      typedef uint16_t us2_t __attribute__((ext_vector_type(2)));
#pragma unroll
      for (int e = 0; e < 4; ++e)
        ahead[t][e] = __builtin_bit_cast(uint32_t, (us2_t){vr[2 * e][16 * t], vr[2 * e + 1][16 * t]});
    };
#pragma unroll
    for (int t = 0; t < AHEAD; ++t) gather(t);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      if (t + AHEAD < 8) gather(t + AHEAD);
      const u4_t w = ahead[t];
      if (!raw[t] && mfma_ops::needs_raw(w)) {
        raw[t] = true;
#pragma unroll
        for (int u = 0; u < NT; ++u) st.acc[u][t] *= 1.f / mfma_ops::kLift;
      }
      f4_t x[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u) x[u] = st.acc[u][t];
      if (raw[t]) {  // (rows that see no large value keep the bits of their small ones)
        mfma_ops::add_raw<NT>(w, ph, pl, x);
      } else {
        const h8_t v8 = mfma_ops::lifted(w, false);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          x[u] = mfma_ops::mfma(v8, ph[u], x[u]);
          x[u] = mfma_ops::mfma(v8, pl[u], x[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < NT; ++u) st.acc[u][t] = x[u];
    }
  }
#pragma unroll
  for (int u = 0; u < NT; ++u) {
#pragma unroll
    for (int t = 0; t < 8; ++t) st.acc[u][t] *= raw[t] ? 1.f / kTailUnit : 1.f / kTailUnit / mfma_ops::kLift;
    st.l[u] *= 1.f / kTailUnit;
    st.l[u] += __shfl_xor(st.l[u], 16);
    st.l[u] += __shfl_xor(st.l[u], 32);
  }
}

// Rows r0 .. r0 + N - 1 (one tile u holds them) into the staging area of wave wv.
template <int N, int NT>
__device__ __forceinline__ void stage_tail(const TailState<NT>& st, int u, int r0, Reduce<N>& r, int lane, int wv) {
  const int row = (lane & 15) - (r0 & 15), blk = lane >> 4;
  if (row < 0 || row >= N) return;
#pragma unroll
  for (int t = 0; t < 8; ++t)
    *reinterpret_cast<f4_t*>(&r.acc[wv][row * kHeadDim + 16 * t + 4 * blk]) = st.acc[u][t];
  if (blk == 0) {
    r.m[wv][row] = st.m[u];
    r.l[wv][row] = st.l[u];
  }
}

}  // namespace dec
}  // namespace kvq
