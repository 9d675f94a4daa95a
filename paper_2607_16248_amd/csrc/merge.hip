// Merge of split records (gfx950): the partial softmax results (max, sum,
// accumulator) of a (sequence, query row)'s splits joined into its output row
// (flash-decoding's second pass; Introduction: the scaled dot-product
// attention the decoder runs at each step).
#include <hip/hip_runtime.h>

#include "decode_common.h"
#include "kvq_internal.h"

namespace kvq {
namespace {

using namespace dec;

// One workgroup per (sequence, query head, 32-channel slice): thread
// (part, c) folds the records of splits part, part + 8, ... into a running
// (max, denominator, channel c numerator), loading U records at a time, U the
// smallest of 4, 5, 8, 9 and 17 for which one memory round trip covers all
// splits (up to 32, 40, 64, 72 or 136: a power of two of packed splits and
// the fp16-tail split fit; loads past the last split would re-read it); the
// eight parts then meet in LDS.  Four slices per head spread a head's records
// over four compute units.
constexpr int kMergeParts = 8;
constexpr int kMergeSlice = 32;
constexpr int kMergeSlices = kHeadDim / kMergeSlice;
constexpr int kMergeThreads = kMergeParts * kMergeSlice;

template <int U>
__device__ __forceinline__ void merge_fold(const float* base, size_t step, int n, int part, int c, float& M,
                                           float& D, float& A) {
  for (int i0 = part; i0 < n; i0 += kMergeParts * U) {
    float mv[U], lv[U], av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + kMergeParts * u;
      const float* r = base + (size_t)min(i, n - 1) * step;
      mv[u] = r[0];
      lv[u] = r[1];
      av[u] = r[4 + c];
    }
    float mx = M;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + kMergeParts * u < n) mx = fmaxf(mx, mv[u]);
    // M = -inf on the first batch: f = 0.  A split that saw no token of a
    // chunk query's row has m = -inf (l = 0, acc = 0); while every record so
    // far is such a split, mx = -inf and nothing is added.
    const bool none = mx == -__builtin_inff();
    const float f = none ? 1.f : __builtin_amdgcn_exp2f(M - mx);
    D *= f;
    A *= f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + kMergeParts * u < n) {
        const float w = none ? 0.f : __builtin_amdgcn_exp2f(mv[u] - mx);
        D = fmaf(w, lv[u], D);
        A = fmaf(w, av[u], A);
      }
    M = mx;
  }
}

__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeArgs a) {
  __shared__ float sm[kMergeParts], sl[kMergeParts], sa[kMergeParts][kMergeSlice];
  const int head = blockIdx.x / kMergeSlices, slice = blockIdx.x % kMergeSlices;
  const int si = head / a.hq, hq = head % a.hq;
  const MergeSeq& S = a.seq[si];
  const int tid = threadIdx.x, cs = tid % kMergeSlice, part = tid / kMergeSlice;
  const int c = slice * kMergeSlice + cs;
  float* o = a.out + ((size_t)S.seq * a.hq + hq) * kHeadDim;
  const int n = S.nsplit;
  if (n == 0) {
    if (tid < kMergeSlice) o[c] = 0.f;
    return;
  }
  const float* base = a.ws + ((size_t)S.ws_base * a.hq + hq) * kRecFloats;
  const size_t step = (size_t)a.hq * kRecFloats;
  float M = -__builtin_inff(), D = 0.f, A = 0.f;
  if (n <= kMergeParts * 4) merge_fold<4>(base, step, n, part, c, M, D, A);
  else if (n <= kMergeParts * 5) merge_fold<5>(base, step, n, part, c, M, D, A);
  else if (n <= kMergeParts * 8) merge_fold<8>(base, step, n, part, c, M, D, A);
  else if (n <= kMergeParts * 9) merge_fold<9>(base, step, n, part, c, M, D, A);
  else merge_fold<17>(base, step, n, part, c, M, D, A);
  if (cs == 0) {
    sm[part] = M;
    sl[part] = D;
  }
  sa[part][cs] = A;
  __syncthreads();
  if (tid < kMergeSlice) {
    float mx = sm[0];
#pragma unroll
    for (int p = 1; p < kMergeParts; ++p) mx = fmaxf(mx, sm[p]);
    float den = 0.f, num = 0.f;
#pragma unroll
    for (int p = 0; p < kMergeParts; ++p) {
      // a part without splits, or without a visible token, has sm = -inf:
      // w = 0 (every row sees at least one token, so mx is finite)
      const float w = __builtin_amdgcn_exp2f(sm[p] - mx);
      den = fmaf(w, sl[p], den);
      num = fmaf(w, sa[p][cs], num);
    }
    o[c] = num / den;
  }
}

// Merges of many rows (chunk queries): one wave per row, two channels per
// lane, eight records in flight.  Bound by the records it reads: 16384 rows of
// four splits (35 MB) take 12.5 us, against 54 with one workgroup per 32
// channels of a row.
constexpr int kMergeRowsFrom = 2048;  // rows of a launch: enough waves for every SIMD
__global__ __launch_bounds__(256) void merge_rows_kernel(MergeArgs a) {
  const int row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int si = row / a.hq, r = row - si * a.hq;
  if (si >= a.nseq) return;
  const MergeSeq& S = a.seq[si];
  const int n = S.nsplit;
  typedef float f2_t __attribute__((ext_vector_type(2)));
  typedef f2_t f2_any __attribute__((aligned(4)));
  f2_any* o = reinterpret_cast<f2_any*>(a.out + ((size_t)S.seq * a.hq + r) * kHeadDim) + lane;
  if (n == 0) {
    *o = (f2_t){0.f, 0.f};
    return;
  }
  const float* base = a.ws + ((size_t)S.ws_base * a.hq + r) * kRecFloats;
  const size_t step = (size_t)a.hq * kRecFloats;
  float M = -__builtin_inff(), D = 0.f;
  f2_t A = {0.f, 0.f};
  constexpr int U = 8;
  for (int i0 = 0; i0 < n; i0 += U) {
    float mv[U], lv[U];
    f2_t av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* rec = base + (size_t)min(i0 + u, n - 1) * step;
      mv[u] = i0 + u < n ? rec[0] : -__builtin_inff();
      lv[u] = rec[1];
      av[u] = reinterpret_cast<const f2_t*>(rec + 4)[lane];
    }
    float mx = M;
#pragma unroll
    for (int u = 0; u < U; ++u) mx = fmaxf(mx, mv[u]);
    // records without a visible token have m = -inf and zeros; while every
    // record so far is such a one nothing is added
    const bool none = mx == -__builtin_inff();
    const float f = none ? 1.f : __builtin_amdgcn_exp2f(M - mx);
    D *= f;
    A *= f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float w = none ? 0.f : __builtin_amdgcn_exp2f(mv[u] - mx);
      D = fmaf(w, lv[u], D);
      A[0] = fmaf(w, av[u][0], A[0]);
      A[1] = fmaf(w, av[u][1], A[1]);
    }
    M = mx;
  }
  *o = (f2_t){A[0] / D, A[1] / D};
}

}  // namespace

int launch_merge(const MergeArgs& a, void* stream) {
  if (a.nseq <= 0) return 0;
  if (a.nseq * a.hq >= kMergeRowsFrom) {
    hipLaunchKernelGGL(merge_rows_kernel, dim3((a.nseq * a.hq + 3) / 4), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
  }
  hipLaunchKernelGGL(merge_kernel, dim3(a.nseq * a.hq * kMergeSlices), dim3(kMergeThreads), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace kvq
