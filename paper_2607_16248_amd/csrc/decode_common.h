// Pieces shared by the decode kernels: wave reductions over DPP, the mapping of
// workgroups and rows, and the combination of per-wave partial results into
// one split record.
#pragma once

#include <hip/hip_runtime.h>

#include "kvq_internal.h"

namespace kvq {
namespace dec {

constexpr int kWaves = 4;

__device__ __forceinline__ float h2f(uint32_t bits16) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_mov(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                               __builtin_bit_cast(int, v), CTRL,
                                                               ROW_MASK, 0xF, false));
}

// DPP controls: quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror,
// row_mirror, row_bcast:15, row_bcast:31.
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140,
              kBcast15 = 0x142, kBcast31 = 0x143;

__device__ __forceinline__ float readlane63(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_mov<kQuadXor1>(0.f, v);
  v += dpp_mov<kQuadXor2>(0.f, v);
  v += dpp_mov<kHalfMirror>(0.f, v);
  v += dpp_mov<kMirror>(0.f, v);
  v += dpp_mov<kBcast15, 0xA>(0.f, v);
  v += dpp_mov<kBcast31, 0xC>(0.f, v);
  return readlane63(v);
}

__device__ __forceinline__ float wave_max(float v) {
  const float ninf = -__builtin_inff();
  v = fmaxf(v, dpp_mov<kQuadXor1>(ninf, v));
  v = fmaxf(v, dpp_mov<kQuadXor2>(ninf, v));
  v = fmaxf(v, dpp_mov<kHalfMirror>(ninf, v));
  v = fmaxf(v, dpp_mov<kMirror>(ninf, v));
  v = fmaxf(v, dpp_mov<kBcast15, 0xA>(ninf, v));
  v = fmaxf(v, dpp_mov<kBcast31, 0xC>(ninf, v));
  return readlane63(v);
}

// LDS written and read back by the same wave: order the accesses.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Locate this workgroup's (sequence, kv head, row group, split).
struct Work {
  int si, h, rg, sp;
};

// CHUNK = false: single-token decode (one query, one row group of the kv
// head's GQ query heads), where the row arithmetic reduces to h * GQ + g.
template <bool CHUNK>
__device__ __forceinline__ Work find_work(const DecodeArgs& a) {
  const int wg = blockIdx.x;
  int si = 0;
  for (int i = 1; i < a.nseq; ++i) si = (a.seq[i].wg_begin <= wg) ? i : si;
  const int local = wg - a.seq[si].wg_begin;
  const int ns = a.seq[si].nsplit;
  const int hv = local / ns;
  Work w{si, hv, 0, local % ns};
  if (a.nqry == 1) {
    // single-token decode: the packed splits of every kv head first, the
    // fp16-tail workgroups (split nq, a few tokens each) after them
    const int nq = a.seq[si].nq, packed = a.hkv * nq;
    if (local < packed) {
      w.h = local / nq;
      w.sp = local - w.h * nq;
    } else {
      w.h = local - packed;
      w.sp = nq;
    }
  }
  if (CHUNK && a.nrg > 1) {  // chunk queries: kv head and row group
    const int units = a.hkv * ns;  // (kv head, split) pairs
    if (units % 8 == 0) {
      // Row groups of one (kv head, split) unit read the same tokens: give
      // them workgroup ids 8 apart, so that they land on one XCD (ids go
      // round-robin over the 8) and their re-reads hit its L2.
      const int q = local >> 3, u = ((q / a.nrg) << 3) + (local & 7);
      w.rg = q % a.nrg;
      w.h = u / ns;
      w.sp = u % ns;
    } else {
      w.h = hv / a.nrg;
      w.rg = hv - w.h * a.nrg;
    }
  }
  return w;
}

// Chunk queries: when qpr does not divide nqry, the last row group holds
// fewer queries; its rows past the last query repeat the last query (they
// read its q row and see its tokens, so every access stays in bounds) and
// write no record.
__device__ __forceinline__ bool row_padded(const DecodeArgs& a, int rg, int g) {
  return rg * a.qpr + a.row_x[g] >= a.nqry;
}
// the query row g computes: rg * qpr + row_x[g], or the last query
__device__ __forceinline__ int row_query(const DecodeArgs& a, int rg, int g) {
  return min(rg * a.qpr + a.row_x[g], a.nqry - 1);
}
// offset of row g's q row from that of the row group's row 0 (a valid query)
__device__ __forceinline__ int row_q_offset(const DecodeArgs& a, int rg, int g) {
  return a.row_off[g] - (rg * a.qpr + a.row_x[g] - row_query(a, rg, g)) * a.hq;
}

// Row g of the workgroup's row group: its index in q / out
// ([batch][nqry][Hq]), its record row within a split (query * Hq + head),
// and the end of the tokens it sees.
template <int GQ, bool CHUNK>
__device__ __forceinline__ size_t q_index(const DecodeArgs& a, const DecodeSeq& S, int h, int rg, int g) {
  if constexpr (!CHUNK) return (size_t)S.seq * a.hq + (size_t)h * GQ + g;
  return ((size_t)S.seq * a.nqry + rg * a.qpr) * a.hq + h * a.gqh + row_q_offset(a, rg, g);
}

template <int GQ, bool CHUNK>
__device__ __forceinline__ int rec_row(const DecodeArgs& a, int h, int rg, int g) {
  if constexpr (!CHUNK) return h * GQ + g;
  return rg * a.qpr * a.hq + h * a.gqh + a.row_off[g];
}

__device__ __forceinline__ int row_limit(const DecodeArgs& a, const DecodeSeq& S, int rg, int g) {
  return S.L - a.nqry + 1 + row_query(a, rg, g);
}

// The smallest limit of the row group: every token below it is visible to
// every row.
__device__ __forceinline__ int group_limit(const DecodeArgs& a, const DecodeSeq& S, int rg) {
  return S.L - a.nqry + 1 + rg * a.qpr;
}

// Per-wave partial results of GQ query heads, staged for the combine.
template <int GQ>
struct Reduce {
  float m[kWaves][GQ], l[kWaves][GQ];
  float acc[kWaves][GQ * kHeadDim];
};

// After a barrier: merge the waves' partial results and write the record of
// split sp for the GQ query heads of kv head h.
template <int GQ, bool CHUNK>
__device__ __forceinline__ void write_record(const DecodeArgs& a, const DecodeSeq& S, int h, int rg, int sp,
                                             const Reduce<GQ>& r, int g0 = 0) {
  for (int idx = threadIdx.x; idx < GQ * kHeadDim; idx += blockDim.x) {
    const int g = idx / kHeadDim, c = idx % kHeadDim;
    if (CHUNK && row_padded(a, rg, g0 + g)) continue;  // a repeat of the last query
    float M = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, r.m[w][g]);
    float val = 0.f, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      // a wave that saw no visible token of a chunk row has m = -inf, l = 0
      // (in single-token decode some wave of every split has a block, so M
      // is finite and exp2(-inf - M) = 0 already)
      const float f = CHUNK && r.m[w][g] == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(r.m[w][g] - M);
      val = fmaf(f, r.acc[w][idx], val);
      lsum = fmaf(f, r.l[w][g], lsum);
    }
    const size_t rows = CHUNK ? (size_t)a.hq * a.nqry : (size_t)a.hq;
    float* rec = a.ws + ((size_t)(S.ws_base + sp) * rows + rec_row<GQ, CHUNK>(a, h, rg, g0 + g)) * kRecFloats;
    rec[4 + c] = val;
    if (c == 0) { rec[0] = M; rec[1] = lsum; }
  }
}

}  // namespace dec
}  // namespace kvq
