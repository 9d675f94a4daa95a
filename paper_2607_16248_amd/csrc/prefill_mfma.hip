// Matrix-core attention of many chunk queries over the packed cache (gfx950):
// chunked prefill, where one kv head has hundreds of (query, head) rows.
//
// The decode and the 16/32-row chunk kernels keep the codes as they are and
// fold the scales into the rows (Q' = q s, P' = p s), which costs vector
// instructions per row and block.  With many rows the scales go to the codes
// instead, once per block and workgroup: every wave of a 256-row workgroup
// unpacks a share of the block's operands into LDS, and eight waves of 32
// rows each read them.  The operands stay exact:
//   keys    K' = (code - c0) / 2 * s,  score = sum_c q (z + c0 s) + 2 sum_c q K'
//   values  V' = (code - c0) / 2 * s 2^X,  O = sum_t p (z + c0 s) + 2^(1-X) sum_t p V'
// with c0 = 1 at two bits (multiples -1/2, 0, 1/2, 1 of s), c0 = 8 and 128 at
// four and eight bits, whose products take two fp16 parts, hi = fl(x) and
// lo = x - hi.  One bit has K' = s (1 - 2 code), the scale with the code as
// its sign bit: score = sum_c q (z + s/2) - 1/2 sum_c q K'.  q enters as the
// fp16 it is, p as hi + lo halves (weights up to 2^14); only the packed values'
// product at four and eight bits takes the hi half alone.
//
// Both products are transposed, so that the first one's output is the second
// one's operand without a lane exchange:
//   S^T = K' Q^T: lane (row n, block b) holds tokens 4b + r and 16 + 4b + r
//         of its row, 8 weights that are the B operand of
//   O^T = V'^T P^T (the A operand's 8 tokens per lane are stored in that
//         order, kvq_layout.h), with the row's softmax state in the lane.
// A further product of P^T with [z; s; 1; z'] gives the zero-point terms and the
// sum of the weights: s lifted like the operands, and the zero-points that are
// subnormal lifted into rows z' of their own, since products of subnormal
// halves lose bits (mfma_common.h).  Per 32 tokens and 16 rows: 8 + 16 + 2 MFMAs at one and
// two bits.  Key zero-point terms come from a table per wave, 16 key groups
// at a time.
//
// Blocks run over the packed tokens and then over the fp16 tail, whose raw
// keys and values are operands already.  A workgroup takes a range of blocks
// (a split); a call with one split writes its output directly.
//
// What bounds it: a wave's block is 52 MFMAs (one and two bits; 832 cycles)
// and about 145 vector instructions, of which the exponentials and the hi and
// lo packing are 80 and its share of the unpacking 45; two waves per SIMD
// (242 registers) take 1.33 us for their blocks of 32 tokens (1.16 without the
// values' products with the low halves), so latencies still show.  A barrier
// every second block instead of every block, with four operand buffers, gave
// 3%; the value operands read before the packing 1%.  Measured, 512 queries of
// 32 heads on 8 kv heads, K2V2: over 65536 tokens 745 us, 735 TFLOP/s (32-row
// groups 1980 us), over 8192 tokens 114 us (304), over 512 tokens 28 us; K4V4
// over 8192 tokens 137 us (320).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "decode_common.h"
#include "kvq_internal.h"
#include "kvq_layout.h"
#include "mfma_common.h"
#include "scaled_ops.h"

namespace kvq {
namespace {

using namespace dec;
using namespace mfma_ops;

constexpr int kNW = kPrefillWaves;
constexpr int kTile = 16;           // rows of one tile (the N dimension); a wave has two
constexpr int kSlots = 4;            // operand buffers (blocks in flight between two barriers)
constexpr int kZGroups = 16;        // key groups per zero-point table
constexpr int kSubRow = 12;         // first row z' of the operand [z; s; 1; z']
constexpr int kZRow = 132;          // dwords per staged key group: s[128], z[128] (+ 4: rows start in distinct banks)
constexpr float kTop = 14.f;        // weights stay below 2^14 ...
constexpr float kHeadroom = 6.f;    // ... a new reference puts the largest at 2^8
constexpr float kNoScore = -1e30f;  // below any score

// q and out need no more than their element's alignment
typedef u4_t u4_any __attribute__((aligned(4)));
typedef f4_t f4_any __attribute__((aligned(4)));

template <int BK, int BV>
struct PrefillSmem {
  static constexpr int kOps = 8 * Code<BK>::parts + 8 * Code<BV>::parts + 1;  // K', V', [z; s; 1; z']
  u4_t op[kSlots][kOps][64];
  uint32_t zs[kZGroups * kZRow];
  float dz[kNW][kZGroups][32];
  uint32_t raw[kNW];  // fp16 tail: whether the value tile's operand is as it is (else lifted)
};

// What a wave holds of a block between its loads and the unpacking: its key
// or value operand (packed dwords and scales; tail: the raw halves in s) and
// a dword of the rows [z; s] of the values.
struct Staged {
  uint32_t x[2], zz;
  u4_t s;
};

template <int BK, int BV, bool PAGED>
__global__ __launch_bounds__(64 * kNW) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_mfma_kernel(DecodeArgs a) {
  constexpr int PK = Code<BK>::parts, PV = Code<BV>::parts, kZOp = 8 * PK + 8 * PV;
  __shared__ __attribute__((aligned(16))) PrefillSmem<BK, BV> sm;
  const int wg = blockIdx.x;
  int si = 0;
  for (int i = 1; i < a.nseq; ++i) si = (a.seq[i].wg_begin <= wg) ? i : si;
  const DecodeSeq& S = a.seq[si];
  // (kv head, split) fastest: the row workgroups of a unit, which read the
  // same tokens, are hkv * nsplit ids apart (one XCD when that divides by 8)
  const int local = wg - S.wg_begin, units = a.hkv * S.nsplit, rw = local / units, unit = local - rw * units;
  const int sp = unit / a.hkv, h = unit - sp * a.hkv;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, blk = lane >> 4;
  const int ng = kHeadDim / a.gv, gsh = __builtin_ctz(a.gk);

  // blocks of 32 tokens: packed ones, then the fp16 tail's
  const int rg = rw * kNW + wv, rg_last = min(rw * kNW + kNW, a.nrg) - 1;
  const bool active = rg < a.nrg;
  const int seen0 = S.L - a.nqry + 1;  // tokens query 0 sees
  const int wg_limit = seen0 + min(rg_last * a.qpr + a.qpr - 1, a.nqry - 1);
  const int nb_packed = S.Lq / 32;
  const int b0 = sp * S.nq, b1 = min(min(b0 + S.nq, (S.L + 31) / 32), (wg_limit + 31) / 32);
  const int wave_first = active ? seen0 + min(rg * a.qpr, a.nqry - 1) : 0;
  const int wave_limit = active ? seen0 + min(rg * a.qpr + a.qpr - 1, a.nqry - 1) : 0;

  const uint8_t* ring = a.arena + S.head0 + (uint64_t)h * a.head_stride;
  const uint32_t vbits = *reinterpret_cast<const uint32_t*>(ring + region(a.vb)) & 0xFFFFu;

  // row g of a row group: query x of the group (one past the last for the
  // rows beyond whole queries) and query head, without a lane-wise read of
  // the launch arguments
  const int inv = (65536 + a.gqh - 1) / a.gqh;
  auto row_of = [&](int g, int& x, int& head) {
    x = (g * inv) >> 16;  // g / gqh (g < 32)
    head = h * a.gqh + g - x * a.gqh;
    x = x < a.qpr ? x : kSpareRow;
  };
  // rows 16u + col of the wave's row group: query operand, limit
  u4_t q[2][4];
  int lim[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    int x, head;
    row_of(kTile * u + col, x, head);
    const int j = min(rg * a.qpr + x, a.nqry - 1);
    lim[u] = seen0 + j;
    const uint16_t* qr = a.q + ((size_t)((size_t)S.seq * a.nqry + j) * a.hq + head) * kHeadDim + 8 * blk;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      q[u][kb] = *reinterpret_cast<const u4_any*>(qr + 32 * kb);
      if constexpr (BK == 1) q[u][kb] ^= 0x80008000u;  // -q: the code term's factor is negative
    }
  }

  const int X = value_shift<BV>(vbits);
  const h2_t vfac = operand_factor<BV>(X), kfac = operand_factor<BK>(0);
  const float unit_packed = Code<BV>::unit * ldexpf(1.f, -X);
  const _Float16 sf = (_Float16)ldexpf(1.f, min(X + Code<BV>::reach, 13));  // scales lifted like the operands
  const h2_t sfac = {sf, sf};

  // this wave's operands: keys, 16-token tile kmb and channel block kkb;
  // values, channels 16 wv .. (value group vg)
  const int kmb = wv & 1, kkb = wv >> 1, vg = wv * 16 / a.gv;
  const int fresh_vm = ng * 64;  // zeros of a value block follow its scales
  const uint32_t lo_k = (16 * kmb + col) * 16 * BK + blk * 4 * BK + 4 * (BK == 8 ? 2 * kkb : BK == 4 ? kkb : BK == 2 ? kkb >> 1 : 0);
  const uint32_t lo_ks = (32 * kkb + 8 * blk) * 2;
  const uint32_t lo_v = lane * 8 * BV + 4 * (BV == 8 ? 2 * wv : BV == 4 ? wv : BV == 2 ? wv >> 1 : wv >> 2);
  const uint32_t lo_vs = (vg * 32 + 8 * blk) * 2;
  // rows 0-3 (zeros) and 4-7 (scales) of the operand [z; s; 1; z']: 16 threads a row
  const int zrow = threadIdx.x >> 4, zpos = threadIdx.x & 15;
  const bool has_zz = zrow < 8 && (zrow & 3) < ng;
  const uint32_t lo_zz = (zrow < 4 ? fresh_vm : 0) + (zrow & 3) * 64 + zpos * 4;
  const __amdgpu_buffer_rsrc_t ring_rs = head_rsrc(ring, PAGED ? 0 : a.head_stride);
  auto seg_of = [&](int b, int& tin) -> __amdgpu_buffer_rsrc_t {
    tin = 32 * b;
    if constexpr (!PAGED) return ring_rs;
    const int pg = tin >> a.pm.page_shift;
    tin &= a.pm.page_tokens - 1;
    return head_rsrc(a.arena + a.pm.pool0 + (uint64_t)a.pm.table[(size_t)S.seq * a.pm.max_pages + pg] * a.pm.page_bytes +
                         (uint64_t)h * a.pm.page_head_bytes,
                     a.pm.page_head_bytes);
  };
  auto load_key = [&](int b, Staged& o) {
    int tin;
    const __amdgpu_buffer_rsrc_t r = seg_of(b, tin);
    const uint32_t kc = region(a.kc) + (uint32_t)tin * 16 * BK;
    if constexpr (BK == 8) {
      const uint2 v = ld64(r, lo_k, kc);
      o.x[0] = v.x;
      o.x[1] = v.y;
    } else {
      o.x[0] = ld32(r, lo_k, kc);
    }
    o.s = ld128(r, lo_ks, region(a.km) + (uint32_t)(tin >> gsh) * 512);
  };
  auto load_value = [&](int b, Staged& o) {
    int tin;
    const __amdgpu_buffer_rsrc_t r = seg_of(b, tin);
    const uint32_t vc = region(a.vc) + (uint32_t)(tin / 32) * 512 * BV, vm = region(a.vm) + (uint32_t)(tin / 32) * 128 * ng;
    if constexpr (BV == 8) {
      const uint2 v = ld64(r, lo_v, vc);
      o.x[0] = v.x;
      o.x[1] = v.y;
    } else {
      o.x[0] = ld32(r, lo_v, vc);
    }
    o.s = ld128(r, lo_vs, vm);
    if (wv < 2) o.zz = ld32(r, has_zz ? lo_zz : lo_vs, vm);
  };
  auto put_key = [&](int b, u4_t hi, u4_t lo) {
    u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
    op[(kmb * 4 + kkb) * PK][lane] = hi;
    if constexpr (PK == 2) op[(kmb * 4 + kkb) * PK + 1][lane] = lo;
  };
  auto put_value = [&](int b, u4_t hi, u4_t lo) {
    u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
    op[8 * PK + wv * PV][lane] = hi;
    if constexpr (PV == 2) op[8 * PK + wv * PV + 1][lane] = lo;
  };
  auto put_zz = [&](int b, uint32_t zz) {
    if (wv < 2 && has_zz) {
      u4_t* op = &sm.op[b & (kSlots - 1)][kZOp][16 * (zpos >> 2)];
      if (zrow < 4) {
        uint32_t normal, sub;
        split_subnormal(zz, normal, sub);
        reinterpret_cast<uint32_t*>(&op[zrow])[zpos & 3] = normal;
        reinterpret_cast<uint32_t*>(&op[kSubRow + zrow])[zpos & 3] = sub;
      } else {
        reinterpret_cast<uint32_t*>(&op[zrow])[zpos & 3] = h2u(u2h(zz) * sfac);
      }
    }
  };
  auto unpack_key = [&](int b, const Staged& o) {
    u4_t hi, lo;
    unpack_scaled<BK, false>(o.x, o.s, BK == 1 ? 4 * kkb : 8 * (kkb & 1), kfac, hi, lo);
    put_key(b, hi, lo);
  };
  auto unpack_value = [&](int b, const Staged& o) {
    u4_t hi, lo;
    unpack_scaled<BV, true>(o.x, o.s, BV == 1 ? 4 * (wv & 3) : 16 * (wv & 1), vfac, hi, lo);
    put_value(b, hi, lo);
    put_zz(b, o.zz);
  };
  // fp16 tail: the raw halves are the operands (keys negated with q)
  auto load_tail = [&](int b, u4_t& k, u4_t& v) {
    k = v = (u4_t){0u, 0u, 0u, 0u};
    const int t = 32 * b + 16 * kmb + col;
    if (t < S.L)
      k = *reinterpret_cast<const u4_t*>(ring + region(a.tk) + ((size_t)(t % a.W) * kHeadDim + 32 * kkb + 8 * blk) * 2);
    if constexpr (BK == 1) k ^= 0x80008000u;
    const uint16_t* rv = reinterpret_cast<const uint16_t*>(ring + region(a.tv)) + 16 * wv + col;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int tv = 32 * b + (e < 4 ? 4 * blk + e : 12 + 4 * blk + e);
      const uint32_t x = tv < S.L ? rv[(size_t)(tv % a.W) * kHeadDim] : 0u;
      v[e >> 1] |= x << (16 * (e & 1));
    }
  };
  // key zero-point tables: block b starts one when it is the first block of
  // the first of 16 key groups, counted from the split's first
  const int bsh = gsh - 5, j0 = b0 >> bsh;  // 2^bsh blocks per key group
  auto table_start = [&](int b) {
    return (b == b0 || ((b & ((1 << bsh) - 1)) == 0 && ((b >> bsh) - j0) % kZGroups == 0));
  };
  u4_t zreg = {0u, 0u, 0u, 0u};
  auto load_zs = [&](int b) {  // 512 threads: 16 groups of 512 bytes, 16 each
    const int j = min((b >> bsh) + (int)(threadIdx.x >> 5), (S.Lq >> gsh) - 1);
    const int t = j << gsh, pg = PAGED ? t >> a.pm.page_shift : 0, tin = PAGED ? t & (a.pm.page_tokens - 1) : t;
    const uint8_t* seg = PAGED ? a.arena + a.pm.pool0 +
                                     (uint64_t)a.pm.table[(size_t)S.seq * a.pm.max_pages + pg] * a.pm.page_bytes +
                                     (uint64_t)h * a.pm.page_head_bytes
                               : ring;
    zreg = *reinterpret_cast<const u4_t*>(seg + region(a.km) + (size_t)(tin >> gsh) * 512 + (threadIdx.x & 31) * 16);
  };
  auto store_zs = [&]() {
    *reinterpret_cast<u4_t*>(&sm.zs[(threadIdx.x >> 5) * kZRow + (threadIdx.x & 31) * 4]) = zreg;
  };
  static_assert(64 * kNW == kZGroups * 32, "one 16-byte piece per thread");
  // raw starts at alpha sum q z + beta sum q s (q as held: negated at one bit)
  constexpr float kAlpha = BK == 1 ? -2.f : 0.5f, kBeta = BK == 1 ? -1.f : Code<BK>::c0 * 0.5f;
  auto fill_dz = [&]() {
    f4_t tz[2], ts[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) tz[u] = ts[u] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const h8_t s8 = *reinterpret_cast<const h8_t*>(&sm.zs[col * kZRow + 16 * kb + 4 * blk]);
      const h8_t z8 = *reinterpret_cast<const h8_t*>(&sm.zs[col * kZRow + 64 + 16 * kb + 4 * blk]);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        tz[u] = mfma(z8, __builtin_bit_cast(h8_t, q[u][kb]), tz[u]);
        ts[u] = mfma(s8, __builtin_bit_cast(h8_t, q[u][kb]), ts[u]);
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.dz[wv][4 * blk + r][16 * u + col] = fmaf(kAlpha, tz[u][r], kBeta * ts[u][r]);
    wave_lds_sync();
  };

  float m[2] = {kNoScore, kNoScore};
  f4_t acc[2][8], zac[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    zac[u] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[u][t] = (f4_t){0.f, 0.f, 0.f, 0.f};
  }

  // raw scores of block b: S^T tiles of rows 16u + col, tokens 16mb + 4blk + r
  auto scores = [&](int b, f4_t (&d)[2][2]) {
    const u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
#pragma unroll
    for (int u = 0; u < 2; ++u) d[u][0] = d[u][1] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int p = 0; p < PK; ++p) {
          const h8_t k8 = __builtin_bit_cast(h8_t, op[(mb * 4 + kb) * PK + p][lane]);
#pragma unroll
          for (int u = 0; u < 2; ++u) d[u][mb] = mfma(k8, __builtin_bit_cast(h8_t, q[u][kb]), d[u][mb]);
        }
  };
  // Softmax of block b (its raw scores in d): the weights as value-product
  // operands, hi and lo parts.  next() runs between the exponentials, after
  // which d is free, and the packing.
  h8_t ph[2], pl[2];
  auto softmax = [&](auto masked_c, auto packed_c, int b, f4_t (&d)[2][2], auto next) {
    constexpr bool MASKED = decltype(masked_c)::value, PACKED = decltype(packed_c)::value;
    const float ksc = PACKED ? (BK == 1 ? 0.5f : 2.f) * a.qscale : a.qscale;
    float z[2], top[2];
    int left[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      z[u] = PACKED ? sm.dz[wv][((b >> bsh) - j0) % kZGroups][16 * u + col] * ksc : 0.f;
      left[u] = lim[u] - 32 * b - 4 * blk;  // token 16 mb + 4 blk + r is visible below it
      if constexpr (MASKED) {
#pragma unroll
        for (int e = 0; e < 8; ++e) d[u][e >> 2][e & 3] = 16 * (e >> 2) + (e & 3) < left[u] ? d[u][e >> 2][e & 3] : kNoScore;
      }
      const f4_t x = d[u][0], y = d[u][1];
      top[u] = fmaf(fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3]))), ksc, z[u]);
    }
    if (__builtin_amdgcn_ballot_w64(top[0] - m[0] > kTop || top[1] - m[1] > kTop)) {
      // the rows' maxima over their four lanes; rows above the limit move
      // their reference
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t v = __builtin_bit_cast(uint32_t, top[u]);
        const auto s32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        float t = fmaxf(__builtin_bit_cast(float, (uint32_t)s32[0]), __builtin_bit_cast(float, (uint32_t)s32[1]));
        const uint32_t w = __builtin_bit_cast(uint32_t, t);
        const auto s16 = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        t = fmaxf(__builtin_bit_cast(float, (uint32_t)s16[0]), __builtin_bit_cast(float, (uint32_t)s16[1]));
        const float mn = t - m[u] > kTop ? t + (kHeadroom - kTop) : m[u];
        const float alpha = __builtin_amdgcn_exp2f(m[u] - mn);
        m[u] = mn;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[u][i] *= alpha;
        zac[u] *= alpha;
      }
    }
    float p[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float bias = z[u] - m[u];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[u][e] = __builtin_amdgcn_exp2f(fmaf(d[u][e >> 2][e & 3], ksc, bias));
        if constexpr (MASKED) p[u][e] = 16 * (e >> 2) + (e & 3) < left[u] ? p[u][e] : 0.f;
      }
    }
    next();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      u4_t hw, lw;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float f0 = p[u][2 * t], f1 = p[u][2 * t + 1];
        const uint32_t w = h2u((h2_t){(_Float16)f0, (_Float16)f1});
        float g0, g1;  // f - (float)half, one mixed-precision fma each
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[0,0,1]" : "=v"(g0) : "v"(f0), "v"(w));
        asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(g1) : "v"(f1), "v"(w));
        hw[t] = w;
        lw[t] = h2u((h2_t){(_Float16)g0, (_Float16)g1});
      }
      ph[u] = __builtin_bit_cast(h8_t, hw);
      pl[u] = __builtin_bit_cast(h8_t, lw);
    }
  };
  h8_t z8, v8[8];  // the first operands of the value products, read early
  auto fetch = [&](int b) {
    const u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
    __builtin_amdgcn_sched_barrier(0);
    z8 = __builtin_bit_cast(h8_t, op[kZOp][lane]);
#pragma unroll
    for (int t = 0; t < 8; ++t) v8[t] = __builtin_bit_cast(h8_t, op[8 * PK + t][lane]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto values = [&](auto lows_c, int b) {
    const u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      zac[u] = mfma(z8, ph[u], zac[u]);
      zac[u] = mfma(z8, pl[u], zac[u]);
    }
#pragma unroll
    for (int t = 0; t < 8 * PV; ++t) {
      const h8_t v = t < 8 ? v8[t] : __builtin_bit_cast(h8_t, op[8 * PK + t][lane]);
#pragma unroll
      for (int u = 0; u < 2; ++u) acc[u][t / PV] = mfma(v, ph[u], acc[u][t / PV]);
      if (decltype(lows_c)::value && t % PV == 0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u][t / PV] = mfma(v, pl[u], acc[u][t / PV]);
      }
    }
  };

  // fp16 tail: both halves of the weights meet the raw values (the product the
  // other chunk kernels' tails make, tail_mfma.h), which the wave that loads them
  // lifts while they are small.  A tail is a window and a key group long, so its
  // blocks are few.
  auto tail_values = [&](int b, uint32_t& raw) {
    const u4_t(*op)[64] = sm.op[b & (kSlots - 1)];
    const uint32_t now = (uint32_t)__builtin_amdgcn_ballot_w64(lane < kNW && sm.raw[lane & (kNW - 1)] != 0u);
    const h8_t ones = __builtin_bit_cast(h8_t, op[kZOp][lane]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      zac[u] = mfma(ones, ph[u], zac[u]);
      zac[u] = mfma(ones, pl[u], zac[u]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const u4_t w = op[8 * PK + t * PV][lane];
      f4_t x[2] = {acc[0][t], acc[1][t]};
      if ((now >> t) & 1u) {
        if (!((raw >> t) & 1u)) {
#pragma unroll
          for (int u = 0; u < 2; ++u) x[u] *= 1.f / kLift;
        }
        add_raw<2>(w, ph, pl, x);
      } else {
        const h8_t v = __builtin_bit_cast(h8_t, w);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          x[u] = mfma(v, ph[u], x[u]);
          x[u] = mfma(v, pl[u], x[u]);
        }
      }
      acc[0][t] = x[0];
      acc[1][t] = x[1];
    }
    raw = now;
  };

  // the constant part of the operand [z; s; 1; z']
  for (int i = threadIdx.x; i < kSlots * 64; i += 64 * kNW) {
    const uint32_t w = (i & 15) == 8 ? 0x3C003C00u : 0u;
    sm.op[i >> 6][kZOp][i & 63] = (u4_t){w, w, w, w};
  }
  __syncthreads();
  const std::true_type yes{};
  const std::false_type no{};
  const int bp = min(b1, nb_packed);  // packed blocks [b0, bp), then the tail's
  // Pipeline: step b reads the keys of block b + 1 and the values of block b,
  // and writes the keys of b + 3 and the values of b + 2, whose loads went out
  // a step earlier; a barrier before every second step then keeps each
  // buffer's writes two steps away from its reads on both sides.  Past the
  // last block everything repeats it or goes unused.
  auto packed_blocks = [&](auto lows_c) {
    const int last = bp - 1;
    Staged sk, sv;
    {
      Staged k0, k1, v0, v1;
      load_key(b0, k0);
      load_value(b0, v0);
      load_zs(b0);
      load_key(min(b0 + 1, last), k1);
      load_value(min(b0 + 1, last), v1);
      load_key(min(b0 + 2, last), sk);
      load_value(min(b0 + 2, last), sv);
      unpack_key(b0, k0);
      unpack_value(b0, v0);
      store_zs();
      unpack_key(b0 + 1, k1);
      unpack_value(b0 + 1, v1);
    }
    __syncthreads();
    f4_t d[2][2];
    scores(b0, d);
    unpack_key(b0 + 2, sk);
    load_key(min(b0 + 3, last), sk);
    auto begin = [&](int b) {
      if (((b - b0) & 1) == 0) __syncthreads();
      if (table_start(b)) fill_dz();
    };
    auto refill = [&](int b) {
      unpack_key(b + 3, sk);
      unpack_value(b + 2, sv);
      load_key(min(b + 4, last), sk);
      load_value(min(b + 3, last), sv);
      // (a table's staging area is free again: its readers passed a barrier
      // since the block that started it)
      if (b > b0 && table_start(b + 2)) store_zs();
      if (table_start(b + 3)) load_zs(b + 3);
    };
    // three phases with the same barriers: all tokens visible to the wave's
    // rows, some, none (the wave only unpacks for the others)
    const int bv = max(b0, min(bp, wave_first / 32)), bm = max(b0, min(bp, (wave_limit + 31) / 32));
    int b = b0;
    for (; b < bv; ++b) {
      begin(b);
      softmax(no, yes, b, d, [&] { scores(b + 1, d); fetch(b); });
      values(lows_c, b);
      refill(b);
    }
    for (; b < bm; ++b) {
      begin(b);
      softmax(yes, yes, b, d, [&] { scores(b + 1, d); fetch(b); });
      values(lows_c, b);
      refill(b);
    }
    for (; b < bp; ++b) {
      begin(b);
      refill(b);
    }
  };
  // Weights of one half (11 bits) leave a row 1e-4 off.  At one and two bits the
  // smaller row groups are closer where one token leads the softmax (prompts
  // up to some thousand tokens: 5e-5 to 1e-4 against 1.2e-4 to 1.9e-4), so the
  // low halves join (5e-7 to 1e-6; 8192 tokens 120 us, 105 without them).  At
  // four and eight bits the smaller groups are at 1.6e-4 to 2.9e-4 themselves,
  // and the low halves matter only where the scales are subnormal: their
  // rounding leaves codes unused, and the products are lopsided.
  if (b0 < bp) {
    if (PV == 1 || vbits < 0x0400u) packed_blocks(yes);
    else packed_blocks(no);
  }
  float unit_acc = unit_packed;  // factor of the value accumulators
  if (max(b0, nb_packed) < b1) {
    // the tail's values carry no unit but the lift, and its rows [z; s] are zero
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[u][t] *= unit_acc * kLift;
    unit_acc = 1.f;
    uint32_t raw = 0u;  // bit t: the accumulators of tile t are no longer lifted
    bool own_raw = false;  // this wave's value tile met a number of 8 or more
    const u4_t none = {0u, 0u, 0u, 0u};
    u4_t k, v;
    load_tail(max(b0, nb_packed), k, v);
    for (int b = max(b0, nb_packed); b < b1; ++b) {
      __syncthreads();  // every wave is done with the buffer
      put_key(b, k, none);
      own_raw = own_raw || needs_raw(v);
      if (lane == 0) sm.raw[wv] = own_raw ? 1u : 0u;
      put_value(b, __builtin_bit_cast(u4_t, lifted(v, own_raw)), none);
      put_zz(b, 0u);
      if (b + 1 < b1) load_tail(b + 1, k, v);
      __syncthreads();
      if (32 * b < wave_limit) {
        f4_t d[2][2];
        scores(b, d);
        softmax(yes, no, b, d, [] {});
        tail_values(b, raw);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[u][t] *= (raw >> t) & 1u ? 1.f : 1.f / kLift;
  }
  if (!active) return;

  // zero-point terms and the sum of weights to every lane of the row
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float zt[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      zt[r] = fmaf(Code<BV>::c0 / (float)sf, __shfl(zac[u][r], 16 + col),
                   fmaf(1.f / kLift, __shfl(zac[u][r], 48 + col), __shfl(zac[u][r], col)));
    const float l = __shfl(zac[u][0], 32 + col);
    int x, head;
    row_of(kTile * u + col, x, head);
    if (rg * a.qpr + x >= a.nqry) continue;  // a spare row
    const int row = (rg * a.qpr + x) * a.hq + head;
    const size_t rows = (size_t)a.hq * a.nqry;
    float* o;
    float f = unit_acc, fz = 1.f;
    if (a.out != nullptr && S.nsplit == 1) {
      o = a.out + ((size_t)S.seq * rows + row) * kHeadDim;
      f = unit_acc / l;
      fz = 1.f / l;
    } else {
      float* rec = a.ws + ((size_t)(S.ws_base + sp) * rows + row) * kRecFloats;
      if (blk == 0) {
        rec[0] = l > 0.f ? m[u] : -__builtin_inff();
        rec[1] = l;
      }
      o = rec + 4;
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float z = (ng == 4 ? zt[t >> 1] : ng == 2 ? zt[t >> 2] : zt[0]) * fz;
      f4_t v;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fmaf(acc[u][t][r], f, z);
      *reinterpret_cast<f4_any*>(o + 16 * t + 4 * blk) = v;
    }
  }
}

template <int BK, int BV>
int launch_pages(const DecodeArgs& a, void* stream) {
  if (a.pm.table != nullptr)
    hipLaunchKernelGGL((prefill_mfma_kernel<BK, BV, true>), dim3(a.total_wg), dim3(64 * kNW), 0, (hipStream_t)stream, a);
  else
    hipLaunchKernelGGL((prefill_mfma_kernel<BK, BV, false>), dim3(a.total_wg), dim3(64 * kNW), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace

int launch_prefill(const DecodeArgs& a, int bk, int bv, void* stream) {
  if (a.total_wg <= 0) return 0;
  if (bk == 1 && bv == 1) return launch_pages<1, 1>(a, stream);
  if (bk == 1 && bv == 2) return launch_pages<1, 2>(a, stream);
  if (bk == 2 && bv == 1) return launch_pages<2, 1>(a, stream);
  if (bk == 2 && bv == 2) return launch_pages<2, 2>(a, stream);
  if (bk == 4 && bv == 4) return launch_pages<4, 4>(a, stream);
  if (bk == 4 && bv == 8) return launch_pages<4, 8>(a, stream);
  if (bk == 8 && bv == 4) return launch_pages<8, 4>(a, stream);
  if (bk == 8 && bv == 8) return launch_pages<8, 8>(a, stream);
  return (int)hipErrorInvalidValue;
}

}  // namespace kvq
