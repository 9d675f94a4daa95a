// DGAP's logit-side runtime step (gfx950): features of the quantized
// logits, the risk detector, the top-K window and, on risky rows, the
// corrector and the sparse merge (Methodology: "DGAP Overview" online
// restoration framework, "Distribution-Risk Detector", "Selective Top-K
// Distribution Corrector"; the feature and MLP readings are stated in
// include/dgap.h).
//
// Two launches per call, both latency-bound at batch 1:
//   scan    one workgroup per (row, 2048-logit chunk): the chunk's max m and
//           its sums of e^(z-m), (m-z) e^(z-m) and e^(2(z-m)), and the largest
//           key of each of its G groups of 2048 / G neighbouring logits (G the
//           largest power of two up to K);
//   finish  one workgroup per row: the log-sum-exp and entropy from the
//           chunk sums, the global top-K, its order by rank counting, the 12
//           features, the detector and, when r > tau, the corrector over the
//           window and the in-place merge.
// Top-K: the K-th largest group maximum bounds the window from below, so only
// groups whose maximum reaches it can hold a window entry.  Neighbouring
// threads give a first bound (each set of them holds some maximum), a
// histogram of 1024 bins over the maxima above it the bin of the K-th, and the
// logits of the K and a few groups from that bin up are read again, filtered
// and ranked by counting.  Where that resolves too little (ties, an outlier
// far above the rest, NaN or +inf among the maxima) a radix selection over the
// keys takes its place.  V = 128256, K = 128, one row: scan 3.7 and finish
// 11.0 us; with a radix selection of every chunk's own top-K in the scan and
// another of the 8064 survivors in the finish 9.1 and 13.8.  Of the finish's
// 25 thousand cycles 6 are the first loads, 5 the selection, 5 the second read
// of the logits, 3 the ranks and 6 the features and the two MLPs, one after
// the other on one compute unit.
//
// Keys: the high 32 bits order the fp32 logits (sign-flipped bit patterns),
// the low 32 bits hold ~index, so that among equal logits the lower index
// is the larger key.  Keys are unique, so "the K largest keys" is exactly
// the window the paper selects with ties broken by index.
#include <hip/hip_runtime.h>

#include "decode_common.h"
#include "kvq_internal.h"

namespace kvq {
namespace {

using dec::dpp_mov;
using dec::kBcast15;
using dec::kBcast31;
using dec::kHalfMirror;
using dec::kMirror;
using dec::kQuadXor1;
using dec::kQuadXor2;
using dec::wave_max;
using dec::wave_sum;

constexpr int kScanThreads = 256;
constexpr int kScanItems = kDgapChunk / kScanThreads;  // logits per thread in a chunk
constexpr int kFinishThreads = 1024;
static_assert(32 * kFinishThreads == kDgapMaxCandidates, "the largest finish kernel holds every candidate");

__device__ __forceinline__ uint32_t order_bits(float f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_order_bits(uint32_t o) {
  return __builtin_bit_cast(float, (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}
__device__ __forceinline__ uint64_t make_key(float v, uint32_t idx) {
  return ((uint64_t)order_bits(v) << 32) | (uint64_t)(~idx);
}
__device__ __forceinline__ float key_value(uint64_t k) { return from_order_bits((uint32_t)(k >> 32)); }
__device__ __forceinline__ uint32_t key_index(uint64_t k) { return ~(uint32_t)k; }

// Inclusive prefix sum over the 64 lanes of a wave: shifts by 1, 2, 4, 8
// within each 16-lane row (lanes without a source add 0), then the row
// totals through row broadcasts 15 and 31.  No LDS round trips.
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROW_MASK, 0xF, false);
}

// Wave-wide maximum / minimum of unsigned 32-bit values (DPP, then lane 63).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, dpp_u32<kQuadXor1>(0u, v));
  v = max(v, dpp_u32<kQuadXor2>(0u, v));
  v = max(v, dpp_u32<kHalfMirror>(0u, v));
  v = max(v, dpp_u32<kMirror>(0u, v));
  v = max(v, dpp_u32<kBcast15, 0xA>(0u, v));
  v = max(v, dpp_u32<kBcast31, 0xC>(0u, v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  v = min(v, dpp_u32<kQuadXor1>(~0u, v));
  v = min(v, dpp_u32<kQuadXor2>(~0u, v));
  v = min(v, dpp_u32<kHalfMirror>(~0u, v));
  v = min(v, dpp_u32<kMirror>(~0u, v));
  v = min(v, dpp_u32<kBcast15, 0xA>(~0u, v));
  v = min(v, dpp_u32<kBcast31, 0xC>(~0u, v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Radix selection: the smallest key T with #{valid keys >= T} == want
// (keys unique and nonzero, at least `want` valid; 0 marks an empty slot).
// The search starts below the bits that the largest and the smallest valid
// key share (a window's candidates agree on their leading bits, which would
// otherwise pile into one histogram bucket), then takes digits of up to 8
// bits; a pass ends the search once the bucket holding the want-th key is
// needed whole.  LDS: hist[256], sel[3], ext[2 * 2 * NT / 64]; every thread
// of the block calls it.
template <int NT, int IPT>
__device__ uint64_t select_threshold(const uint64_t (&key)[IPT], int want, uint32_t* hist, uint32_t* sel,
                                     uint32_t* ext) {
  constexpr int kWavesPerBlock = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // block-wide largest and smallest valid key
  uint64_t kmax = 0, kmin = ~0ull;
#pragma unroll
  for (int j = 0; j < IPT; ++j)
    if (key[j] != 0) {
      kmax = key[j] > kmax ? key[j] : kmax;
      kmin = key[j] < kmin ? key[j] : kmin;
    }
  {
    const uint32_t hmax = wave_max_u32((uint32_t)(kmax >> 32));
    const uint32_t lmax = wave_max_u32((uint32_t)(kmax >> 32) == hmax ? (uint32_t)kmax : 0u);
    const uint32_t hmin = wave_min_u32((uint32_t)(kmin >> 32));
    const uint32_t lmin = wave_min_u32((uint32_t)(kmin >> 32) == hmin ? (uint32_t)kmin : ~0u);
    if (lane == 0) {
      ext[4 * wv] = hmax;
      ext[4 * wv + 1] = lmax;
      ext[4 * wv + 2] = hmin;
      ext[4 * wv + 3] = lmin;
    }
  }
  __syncthreads();
  kmax = 0;
  kmin = ~0ull;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    const uint64_t a = ((uint64_t)ext[4 * w] << 32) | ext[4 * w + 1];
    const uint64_t b = ((uint64_t)ext[4 * w + 2] << 32) | ext[4 * w + 3];
    kmax = a > kmax ? a : kmax;
    kmin = b < kmin ? b : kmin;
  }
  if (kmax == kmin) return kmax;  // a single valid key
  const int top = 63 - __builtin_clzll(kmax ^ kmin);  // highest bit that differs
  int width = min(8, top + 1), shift = top + 1 - width;
  uint64_t prefix = top == 63 ? 0 : kmax >> (top + 1);
  int rem = want;
  for (;;) {
    for (int i = tid; i < 256; i += NT) hist[i] = 0;
    __syncthreads();
    const uint32_t mask = (1u << width) - 1u;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const uint64_t k = key[j];
      if (k != 0 && (shift + width == 64 || (k >> (shift + width)) == prefix))
        atomicAdd(&hist[(uint32_t)(k >> shift) & mask], 1u);
    }
    __syncthreads();
    if (tid < 64) {
      // lane l holds buckets 255 - 4l .. 252 - 4l (descending)
      uint32_t c[4], own = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        c[i] = hist[255 - 4 * tid - i];
        own += c[i];
      }
      uint32_t before = wave_prefix_sum(own) - own;  // keys in the buckets above this lane's
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (before < (uint32_t)rem && before + c[i] >= (uint32_t)rem) {
          sel[0] = 255 - 4 * tid - i;
          sel[1] = before;
          sel[2] = c[i];
        }
        before += c[i];
      }
    }
    __syncthreads();
    const uint32_t digit = sel[0], above = sel[1], inbucket = sel[2];
    prefix = (prefix << width) | digit;
    rem -= (int)above;
    __syncthreads();  // sel and hist are rewritten by the next pass
    if ((int)inbucket == rem || shift == 0) return prefix << shift;
    width = min(8, shift);
    shift -= width;
  }
}

// Logit groups per chunk: the largest power of two up to k (at most 256).
__host__ __device__ inline int chunk_groups(int k) {
  int g = 8;
  while (2 * g <= k && g < kScanThreads) g *= 2;
  return g;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, mask), hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), mask);
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(kScanThreads) void dgap_scan_kernel(DgapArgs a) {
  __shared__ float4 part[kScanThreads / 64];
  __shared__ float wmax[kScanThreads / 64];
  static_assert(kScanThreads == 256, "four waves");
  typedef float f4_t __attribute__((ext_vector_type(4)));
  typedef f4_t f4_any __attribute__((aligned(4)));
  const int row = blockIdx.x / a.nchunk, chunk = blockIdx.x % a.nchunk, tid = threadIdx.x;
  const float* z = a.logits + (size_t)row * a.vocab;
  const int i0 = chunk * kDgapChunk + tid * kScanItems, n = min(kScanItems, a.vocab - i0);  // this thread's logits
  static_assert(kScanItems == 8, "two 16-byte loads per thread");
  float v[kScanItems];
  if (n == kScanItems) {
    const f4_t x = *reinterpret_cast<const f4_any*>(z + i0), y = *reinterpret_cast<const f4_any*>(z + i0 + 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = x[j];
      v[4 + j] = y[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) v[j] = j < n ? z[i0 + j] : -__builtin_inff();
  }
  float m = v[0];
  uint32_t top = order_bits(v[0]);
  int at = 0;  // the first of the largest
#pragma unroll
  for (int j = 1; j < kScanItems; ++j) {
    const uint32_t o = j < n ? order_bits(v[j]) : 0u;
    at = o > top ? j : at;
    top = max(top, o);
    m = fmaxf(m, v[j]);
  }
  // the largest key of each group: one lane, or up to 32 neighbours
  uint64_t key = n > 0 ? ((uint64_t)top << 32) | (uint64_t)(~(uint32_t)(i0 + at)) : 0;
  const int G = chunk_groups(a.k), tpg = kScanThreads / G;
  for (int d = 1; d < tpg; d *= 2) {
    const uint64_t o = shfl_xor_u64(key, d);
    key = o > key ? o : key;
  }
  if (tid % tpg == 0) a.ws_cand[((size_t)row * a.nchunk + chunk) * a.k + tid / tpg] = key;
  m = wave_max(m);
  if ((tid & 63) == 0) wmax[tid >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  float s = 0.f, t = 0.f, u = 0.f;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    if (j < n) {
      const float e = expf(v[j] - m);
      s += e;
      t = fmaf(e, m - v[j], t);  // >= 0 term by term: the entropy needs no cancellation
      u = fmaf(e, e, u);
    }
  }
  s = wave_sum(s);
  t = wave_sum(t);
  u = wave_sum(u);
  if ((tid & 63) == 0) part[tid >> 6] = make_float4(m, s, t, u);
  __syncthreads();
  if (tid < 4) {  // lane 0: m, 1: s, 2: t, 3: u
    const float* p = &part[0].x + tid;
    const float sum = (p[0] + p[4]) + (p[8] + p[12]);
    a.ws_stats[((size_t)row * a.nchunk + chunk) * 4 + tid] = tid == 0 ? m : sum;
  }
}

constexpr int kBins = 1024;
constexpr int kListMax = 2048;   // groups that are binned
constexpr int kRegather = 8;     // logits of the selected groups a finish thread holds at most
constexpr int kRankMax = 1024;   // candidates that rank counting takes
constexpr int kRankPad = 64;     // zeros past them: a thread reads 16 keys, every fourth pair, at a time

// This thread's first slot of `own` in a list that the block fills: one LDS
// atomic per wave (of its own accord the compiler adds lane by lane).
__device__ __forceinline__ uint32_t wave_slots(uint32_t own, uint32_t* count) {
  const uint32_t sum = wave_prefix_sum(own);
  uint32_t base = 0;
  if ((threadIdx.x & 63) == 63 && sum != 0) base = atomicAdd(count, sum);
  return (uint32_t)__builtin_amdgcn_readlane((int)base, 63) + sum - own;
}

// IPT: group maxima per thread (the launch picks the smallest of 8, 16, 32
// that holds them).
template <int IPT>
__global__ __launch_bounds__(kFinishThreads) void dgap_finish_kernel(DgapArgs a) {
  // one row of 64 hidden units (zeros past the last) per input, then the bias and the output weights
  constexpr int kWaves = kFinishThreads / 64, kDet = kDgapFeatures + 2, kCorrIn = kDgapCandInputs + kDgapFeatures;
  static_assert(kDgapMaxHidden == 64, "a weight row per wave");
  __shared__ __attribute__((aligned(16))) float wdet[kDet][64], wcor[kCorrIn + 2][64];
  __shared__ __attribute__((aligned(16))) uint32_t bins[kBins];
  __shared__ __attribute__((aligned(16))) uint32_t ext[4 * kWaves];
  __shared__ uint32_t hist[256], sel[4], cnt[4];
  __shared__ uint2 list[kListMax];  // (order of the maximum, group)
  __shared__ uint16_t groups[kRegather * kFinishThreads / 8];  // selected groups (8 logits at least each)
  __shared__ __attribute__((aligned(16))) uint64_t win[kRankMax + kRankPad], skey[kDgapMaxK];
  __shared__ float stat[8];      // lse, H, sum p^2, r
  __shared__ float phi[kDgapFeatures];
  __shared__ float vsorted[kDgapMaxK];
  __shared__ __attribute__((aligned(16))) float uphi[kDgapMaxHidden];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int K = a.k, G = chunk_groups(K), gshift = __builtin_ctz(G), ngroup = a.nchunk * G;
  float* z = a.logits + (size_t)row * a.vocab;
  const int hd = a.hidden_det, hc = a.hidden_corr;

  // Every global load is issued first so that their latencies overlap: the
  // candidate keys, the MLP weights (three elements per thread of the
  // concatenation det_w1, det_b1, det_w2, corr_w1, corr_b1, corr_w2) and,
  // in wave 0, the statistics of the first 64 chunks.
  uint64_t key[IPT];
  const uint64_t* cand = a.ws_cand + (size_t)row * a.nchunk * K;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const int i = j * kFinishThreads + tid;
    key[j] = i < ngroup ? cand[(size_t)(i >> gshift) * K + (i & (G - 1))] : 0;
  }
  constexpr int kRows = kDet + kCorrIn + 2, kRowsPerWave = (kRows + kWaves - 1) / kWaves;
  float wrow[kRowsPerWave];
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    const int r = wv + i * kWaves, c = r - kDet;  // c: row of the corrector
    const float* src = r < kDgapFeatures       ? a.det_w1 + r * hd
                       : r == kDgapFeatures    ? a.det_b1
                       : r < kDet              ? a.det_w2
                       : c < kCorrIn           ? a.corr_w1 + c * hc
                       : c == kCorrIn          ? a.corr_b1
                                               : a.corr_w2;
    wrow[i] = r < kRows && lane < (r < kDet ? hd : hc) ? src[lane] : 0.f;
  }
  const float* st = a.ws_stats + (size_t)row * a.nchunk * 4;
  float4 st0 = make_float4(-__builtin_inff(), 0.f, 0.f, 0.f);
  if (wv == 0 && lane < a.nchunk) st0 = *reinterpret_cast<const float4*>(st + 4 * lane);
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    const int r = wv + i * kWaves;
    if (r < kDet)
      wdet[r][lane] = wrow[i];
    else if (r < kRows)
      wcor[r - kDet][lane] = wrow[i];
  }

  // log-sum-exp, entropy and concentration from the chunk sums (wave 0)
  if (wv == 0) {
    float M = st0.x;
    for (int c = lane + 64; c < a.nchunk; c += 64) M = fmaxf(M, st[4 * c]);
    M = wave_max(M);
    const bool has0 = lane < a.nchunk;  // (lanes past the last chunk add nothing)
    float S = has0 ? expf(st0.x - M) * st0.y : 0.f;
    for (int c = lane + 64; c < a.nchunk; c += 64) S += expf(st[4 * c] - M) * st[4 * c + 1];
    S = wave_sum(S);
    const float lse = M + logf(S);
    // H = sum_i p_i (lse - z_i) = sum_chunks e^(m-lse) ((lse - m) s + sum_i e_i (m - z_i)),
    // every term non-negative
    const float f0 = has0 ? expf(st0.x - lse) : 0.f;
    float h = has0 ? f0 * fmaf(lse - st0.x, st0.y, st0.z) : 0.f, p2 = f0 * f0 * st0.w;
    for (int c = lane + 64; c < a.nchunk; c += 64) {
      const float f = expf(st[4 * c] - lse);
      h = fmaf(f, fmaf(lse - st[4 * c], st[4 * c + 1], st[4 * c + 2]), h);
      p2 = fmaf(f * f, st[4 * c + 3], p2);
    }
    h = wave_sum(h);
    p2 = wave_sum(p2);
    if (lane == 0) {
      stat[0] = lse;
      stat[1] = h;
      stat[2] = p2;
    }
  }

  // The groups that can hold a window entry.  First a value that at least K maxima reach: 16,
  // 8 or 4 neighbouring threads hold some maximum, and there are 64, 128 or 256 such sets.
  // (Where a set holds none, the smallest maximum.)
  static_assert(kBins == kFinishThreads && kRankMax == kFinishThreads, "one entry per thread to clear");
  static_assert(kFinishThreads / 4 >= kDgapMaxK, "a quad per window entry");
  bins[tid] = 0;
  win[tid] = 0;
  if (tid < kRankPad) win[kRankMax + tid] = 0;
  if (tid < 4) cnt[tid] = 0;
  uint32_t top = 0, bottom = ~0u;
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    const uint32_t o = (uint32_t)(key[j] >> 32);
    top = max(top, o);
    bottom = min(bottom, key[j] != 0 ? o : ~0u);
  }
  uint32_t set = max(top, dpp_u32<kQuadXor1>(0u, top));
  set = max(set, dpp_u32<kQuadXor2>(0u, set));
  if (K <= kFinishThreads / 8) set = max(set, dpp_u32<kHalfMirror>(0u, set));
  if (K <= kFinishThreads / 16) set = max(set, dpp_u32<kMirror>(0u, set));
  set = wave_min_u32(set);
  top = wave_max_u32(top);
  bottom = wave_min_u32(bottom);
  if (lane == 0) *reinterpret_cast<uint4*>(&ext[4 * wv]) = make_uint4(set, top, bottom, 0u);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint4 x = *reinterpret_cast<const uint4*>(&ext[4 * w]);
    set = min(set, x.x);
    top = max(top, x.y);
    bottom = min(bottom, x.z);
  }
  const uint32_t lo_bits = max(set, bottom);
  const int E = kDgapChunk >> gshift, eshift = __builtin_ctz(E);  // logits per group
  const int most = kRegather * kFinishThreads >> eshift;          // groups that can be read again
  // NaN and +inf have no bins, and fewer than K maxima say nothing of the rest
  bool binned = top < order_bits(__builtin_inff()) && bottom >= order_bits(-__builtin_inff());
  const float lo = from_order_bits(lo_bits), scale = (float)kBins / (from_order_bits(top) - lo);
  // monotone; NaN products (an infinite scale or distance) go to bin 0
  auto bin_of = [&](float v) -> int { return (int)fminf(fmaxf((v - lo) * scale, 0.f), (float)(kBins - 1)); };
  int thr = 0, id = tid;  // a group's number is id + 1024 j: computed anew, or the loads' 32 indices stay in registers
  asm volatile("" : "+v"(id));
  if (binned) {
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) own += (uint32_t)(key[j] >> 32) >= lo_bits;  // (-inf is above an empty slot)
    uint32_t slot = wave_slots(own, &cnt[3]);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const uint32_t o = (uint32_t)(key[j] >> 32);
      if (o >= lo_bits && slot < (uint32_t)kListMax) list[slot++] = make_uint2(o, j * kFinishThreads + id);
    }
    __syncthreads();
    const int n = (int)cnt[3];
    binned = n >= K && n <= kListMax;
    if (binned) {
      int bin[kListMax / kFinishThreads];
      uint16_t group[kListMax / kFinishThreads];
#pragma unroll
      for (int i = 0; i < kListMax / kFinishThreads; ++i) {
        bin[i] = -1;
        if (i * kFinishThreads + tid >= n) continue;
        const uint2 x = list[i * kFinishThreads + tid];
        group[i] = (uint16_t)x.y;
        bin[i] = bin_of(from_order_bits(x.x));
        atomicAdd(&bins[bin[i]], 1u);
      }
      __syncthreads();
      if (wv == 0) {  // lane l holds bins kBins - 1 - 16 l and the 15 below it
        static_assert(kBins == 16 * 64, "16 bins per lane");
        uint32_t c[16], own = 0;
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          const uint4 x = *reinterpret_cast<const uint4*>(&bins[kBins - 4 - 16 * lane - i]);
          c[i] = x.w;
          c[i + 1] = x.z;
          c[i + 2] = x.y;
          c[i + 3] = x.x;
          own += (x.x + x.y) + (x.z + x.w);
        }
        uint32_t before = wave_prefix_sum(own) - own;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if (before < (uint32_t)K && before + c[i] >= (uint32_t)K) sel[0] = kBins - 1 - 16 * lane - i;
          before += c[i];
        }
      }
      __syncthreads();
      thr = (int)sel[0];
#pragma unroll
      for (int i = 0; i < kListMax / kFinishThreads; ++i)
        if (bin[i] >= thr) {
          const uint32_t slot = atomicAdd(&cnt[0], 1u);
          if (slot < (uint32_t)most) groups[slot] = group[i];
        }
      __syncthreads();
    }
  }
  if (!binned) {  // every group
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) own += key[j] != 0;
    uint32_t slot = wave_slots(own, &cnt[0]);
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (key[j] != 0 && slot < (uint32_t)most) groups[slot++] = (uint16_t)(j * kFinishThreads + id);
    }
    __syncthreads();
  }
  uint64_t floor_key = 0;  // a lower bound on the window's keys, where the bins resolve too little
  if (cnt[0] > (uint32_t)most) {
    floor_key = select_threshold<kFinishThreads, IPT>(key, K, hist, sel, ext);
    if (tid == 0) cnt[0] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (key[j] >= floor_key && key[j] != 0) groups[atomicAdd(&cnt[0], 1u)] = (uint16_t)(j * kFinishThreads + id);  // K of them
    __syncthreads();
  }
  // their logits again: at most kRegather per thread
  const int nsel = (int)cnt[0], nread = nsel << eshift;
  uint64_t again[kRegather];  // as read: value, ~index
#pragma unroll
  for (int j = 0; j < kRegather; ++j) {
    again[j] = 0;
    if (j * kFinishThreads >= nread) continue;
    const int i = j * kFinishThreads + tid;
    const int at = i < nread ? (groups[i >> eshift] << eshift) + (i & (E - 1)) : a.vocab;  // chunk * 2048 + group * E + element
    if (at < a.vocab) again[j] = ((uint64_t)__builtin_bit_cast(uint32_t, z[at]) << 32) | (uint64_t)(~(uint32_t)at);
  }
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < kRegather; ++j) {
    if (j * kFinishThreads >= nread || again[j] == 0) continue;
    const float v = __builtin_bit_cast(float, (uint32_t)(again[j] >> 32));
    const uint64_t k = make_key(v, key_index(again[j]));
    again[j] = (floor_key != 0 ? k >= floor_key : !binned || (v >= lo && bin_of(v) >= thr)) ? k : 0;
    mine += again[j] != 0;
  }
  {
    uint32_t slot = wave_slots(mine, &cnt[1]);
#pragma unroll
    for (int j = 0; j < kRegather; ++j)
      if (again[j] != 0) {
        if (slot < (uint32_t)kRankMax) win[slot] = again[j];
        ++slot;
      }
  }
  __syncthreads();
  int nwin = (int)cnt[1];
  if (nwin > kRankMax) {  // too many for rank counting: exactly the K largest
    const uint64_t T = select_threshold<kFinishThreads, kRegather>(again, K, hist, sel, ext);
    win[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRegather; ++j)
      if (again[j] != 0 && again[j] >= T) {
        const uint32_t slot = atomicAdd(&cnt[2], 1u);
        if (slot < (uint32_t)K) win[slot] = again[j];  // exactly K keys pass
      }
    nwin = K;
    __syncthreads();
  }
  {
    // rank of candidate c = #{larger ones}: four, two or one threads each
    const int pshift = nwin <= kFinishThreads / 4 ? 2 : nwin <= kFinishThreads / 2 ? 1 : 0, parts = 1 << pshift;
    const int c = tid >> pshift, part = tid & (parts - 1);
    const uint64_t mine_key = c < nwin ? win[c] : 0;
    int rank = 0;
    if (c < nwin) {
      for (int j0 = 2 * part; j0 < nwin; j0 += 16 * parts) {
        ulonglong2 o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) o[u] = *reinterpret_cast<const ulonglong2*>(&win[j0 + 2 * u * parts]);
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (o[u].x > mine_key) + (o[u].y > mine_key);
      }
    }
    // the threads of a candidate are neighbouring lanes
    if (pshift >= 1) rank += (int)dpp_u32<kQuadXor1>(0u, (uint32_t)rank);
    if (pshift >= 2) rank += (int)dpp_u32<kQuadXor2>(0u, (uint32_t)rank);
    if (c < nwin && part == 0 && rank < K) {
      skey[rank] = mine_key;
      vsorted[rank] = key_value(mine_key);
    }
  }
  __syncthreads();

  // features (wave 0; four window entries per lane)
  const float lse = stat[0];
  if (wv == 0) {
    float P[4], vv[4];
    float mass = 0.f, top8 = 0.f, vsum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = lane + 64 * i;
      vv[i] = k < K ? vsorted[k] : 0.f;
      P[i] = k < K ? expf(vv[i] - lse) : 0.f;
      mass += P[i];
      vsum += vv[i];
      if (k < 8) top8 += P[i];
    }
    mass = wave_sum(mass);
    top8 = wave_sum(top8);
    const float mean = wave_sum(vsum) / K;
    float var = 0.f, hk = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = lane + 64 * i;
      if (k < K) {
        var = fmaf(vv[i] - mean, vv[i] - mean, var);
        const float q = P[i] / mass;
        if (q > 0.f) hk -= q * logf(q);
      }
    }
    var = wave_sum(var) / K;
    hk = wave_sum(hk);
    if (lane == 0) {
      const float H = stat[1];
      float mg = vsorted[0] - vsorted[1];
      for (int k = 1; k < 7; ++k) mg = fminf(mg, vsorted[k] - vsorted[k + 1]);
      phi[0] = H;
      phi[1] = H / logf((float)a.vocab);
      phi[2] = vsorted[0] - lse;
      phi[3] = mass;
      phi[4] = top8;
      phi[5] = stat[2];
      phi[6] = vsorted[0] - vsorted[1];
      phi[7] = vsorted[1] - vsorted[2];
      phi[8] = (vsorted[0] - vsorted[K - 1]) / (float)(K - 1);
      phi[9] = mg;
      phi[10] = sqrtf(var);
      phi[11] = hk;
    }
  }
  __syncthreads();

  // detector: lane h is hidden unit h (wave 0); the phi part of the corrector's
  // hidden units, the same for every candidate (wave 1)
  if (wv == 0) {
    float acc = wdet[kDgapFeatures][lane];
#pragma unroll
    for (int i = 0; i < kDgapFeatures; ++i) acc = fmaf(phi[i], wdet[i][lane], acc);
    const float y = lane < hd ? fmaxf(acc, 0.f) * wdet[kDgapFeatures + 1][lane] : 0.f;
    const float s = wave_sum(y) + a.det_b2;
    if (lane == 0) stat[3] = 1.f / (1.f + expf(-s));
  } else if (wv == 1) {
    float uh = wcor[kCorrIn][lane];
#pragma unroll
    for (int i = 0; i < kDgapFeatures; ++i) uh = fmaf(phi[i], wcor[kDgapCandInputs + i][lane], uh);
    uphi[lane] = uh;
  }
  __syncthreads();
  const float r = stat[3];
  const bool correct = r > a.tau;
  float* info = a.info ? a.info + (size_t)row * (kDgapInfoHead + 2 * K) : nullptr;

  if (correct) {
    // corrector: four threads (a lane quad) per candidate, 16 hidden units
    // each (those past the last are left out: 0 times an infinite input)
    const int k = tid >> 2, g = tid & 3;
    float part = 0.f, vk = 0.f;
    if (k < K) {
      vk = vsorted[k];
      const float xi[kDgapCandInputs] = {vk - vsorted[0], vk - lse, (float)k / (float)(K - 1),
                                         k > 0 ? vsorted[k - 1] - vk : 0.f, k + 1 < K ? vk - vsorted[k + 1] : 0.f};
#pragma unroll
      for (int u = 0; u < 16; u += 4) {  // the quad reads 64 bytes side by side
        const int h0 = 4 * u + 4 * g;
        float acc[4];
        *reinterpret_cast<float4*>(acc) = *reinterpret_cast<const float4*>(&uphi[h0]);
#pragma unroll
        for (int i = 0; i < kDgapCandInputs; ++i) {
          float w[4];
          *reinterpret_cast<float4*>(w) = *reinterpret_cast<const float4*>(&wcor[i][h0]);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaf(xi[i], w[e], acc[e]);
        }
        float w2[4];
        *reinterpret_cast<float4*>(w2) = *reinterpret_cast<const float4*>(&wcor[kCorrIn + 1][h0]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (h0 + e < hc) part = fmaf(fmaxf(acc[e], 0.f), w2[e], part);
      }
    }
    part += __builtin_bit_cast(float, dpp_u32<kQuadXor1>(0u, __builtin_bit_cast(uint32_t, part)));
    part += __builtin_bit_cast(float, dpp_u32<kQuadXor2>(0u, __builtin_bit_cast(uint32_t, part)));
    if (k < K && g == 0) {
      const float d = part + a.corr_b2;
      const uint32_t idx = key_index(skey[k]);
      if (idx < (uint32_t)a.vocab) z[idx] = vk + d;
      if (info) info[kDgapInfoHead + K + k] = d;
    }
  } else if (info) {
    for (int k = tid; k < K; k += kFinishThreads) info[kDgapInfoHead + K + k] = 0.f;
  }
  if (info) {
    for (int k = tid; k < K; k += kFinishThreads)
      info[kDgapInfoHead + k] = __builtin_bit_cast(float, key_index(skey[k]));
    if (tid < kDgapFeatures) info[4 + tid] = phi[tid];
    if (tid == 0) {
      info[0] = r;
      info[1] = correct ? 1.f : 0.f;
      info[2] = lse;
      info[3] = 0.f;
    }
  }
}

}  // namespace

int launch_dgap(const DgapArgs& a, int batch, void* stream) {
  hipLaunchKernelGGL(dgap_scan_kernel, dim3(batch * a.nchunk), dim3(kScanThreads), 0, (hipStream_t)stream, a);
  int e = (int)hipGetLastError();
  if (e) return e;
  const int ncand = a.nchunk * chunk_groups(a.k);
  if (ncand <= 8 * kFinishThreads)
    hipLaunchKernelGGL(dgap_finish_kernel<8>, dim3(batch), dim3(kFinishThreads), 0, (hipStream_t)stream, a);
  else if (ncand <= 16 * kFinishThreads)
    hipLaunchKernelGGL(dgap_finish_kernel<16>, dim3(batch), dim3(kFinishThreads), 0, (hipStream_t)stream, a);
  else
    hipLaunchKernelGGL(dgap_finish_kernel<32>, dim3(batch), dim3(kFinishThreads), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace kvq
