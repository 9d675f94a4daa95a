// Dequantization of a token range of one sequence, for checking (gfx950).
//
// A packed element becomes fma(code, s, z) in fp32: the exact z + code * s
// rounded once.  A tail element is its fp16 value.
#include <hip/hip_runtime.h>

#include "kvq_internal.h"
#include "kvq_layout.h"

namespace kvq {
namespace {

__device__ __forceinline__ float h2f(uint32_t bits16) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

// Code of channel c from a key row / value block.
__device__ __forceinline__ uint32_t key_code(const uint8_t* row, int c, int bits) {
  uint32_t code = 0;
  for (int p = 0; p < bits; ++p) {
    const BitLoc b = key_bit(c, p, bits);
    code |= ((reinterpret_cast<const uint32_t*>(row)[b.word] >> b.bit) & 1u) << p;
  }
  return code;
}

__device__ __forceinline__ uint32_t value_code(const uint8_t* block, int r, int c, int bits) {
  uint32_t code = 0;
  for (int p = 0; p < bits; ++p) {
    const BitLoc b = value_bit(r, c, p, bits);
    code |= ((reinterpret_cast<const uint32_t*>(block)[b.word] >> b.bit) & 1u) << p;
  }
  return code;
}

__global__ __launch_bounds__(128) void dequant_kernel(DequantArgs a) {
  const int ti = blockIdx.x / a.hkv, h = blockIdx.x % a.hkv;
  const int p = a.tok0 + ti, c = threadIdx.x;
  const uint8_t* blk = a.arena + a.head0 + (uint64_t)h * a.head_stride;
  float kv, vv;
  if (p < a.Lq) {
    int q;  // p's position in its packed segment
    const uint8_t* seg = a.arena + packed_seg(a.pm, a.head0, a.head_stride, a.seq, h, p, q);
    const uint16_t* km = reinterpret_cast<const uint16_t*>(seg + region(a.km)) + (size_t)(q / a.gk) * 2 * kHeadDim;
    const uint8_t* krow = seg + region(a.kc) + (size_t)q * 16 * a.bk;
    const uint32_t kcode = key_code(krow, c, a.bk);
    kv = fmaf((float)kcode, h2f(km[c]), h2f(km[kHeadDim + c]));
    const int ng = kHeadDim / a.gv, g = c / a.gv;
    const uint8_t* vblk = seg + region(a.vc) + (size_t)(q / 32) * 512 * a.bv;
    const uint8_t* vmb = seg + region(a.vm) + (size_t)(q / 32) * 128 * ng;
    const int r = q % 32;
    vv = fmaf((float)value_code(vblk, r, c, a.bv),
              h2f(*reinterpret_cast<const uint16_t*>(vmb + value_meta_s(g, r))),
              h2f(*reinterpret_cast<const uint16_t*>(vmb + value_meta_z(g, r, ng))));
  } else {
    const size_t slot = (size_t)(p % a.W) * kHeadDim + c;
    kv = h2f(reinterpret_cast<const uint16_t*>(blk + region(a.tk))[slot]);
    vv = h2f(reinterpret_cast<const uint16_t*>(blk + region(a.tv))[slot]);
  }
  const size_t o = ((size_t)ti * a.hkv + h) * kHeadDim + c;
  a.K_out[o] = kv;
  a.V_out[o] = vv;
}

// Fields of B bits moved apart: field i of the low 4 * B bits to field 2i.
template <int B>
__device__ __forceinline__ uint32_t spread(uint32_t x) {
  if constexpr (B == 1) {
    x = (x | (x << 2)) & 0x33u;
    return (x | (x << 1)) & 0x55u;
  } else if constexpr (B == 2) {
    x = (x | (x << 4)) & 0x0F0Fu;
    return (x | (x << 2)) & 0x3333u;
  } else {
    x = (x | (x << 8)) & 0x00FF00FFu;
    return (x | (x << 4)) & 0x0F0F0F0Fu;
  }
}

// Canonical dword w of a key row from the row's dwords: per 8
// channels (operand block kb, lane group g) the even elements sit below the
// odd ones, 16 bits apart (kvq_layout.h, key_bit).
template <int B>
__device__ __forceinline__ uint32_t canonical_key(const uint32_t* row, int w) {
  if constexpr (B == 8) {  // channels 4w ..: kb = w >> 3, g = (w >> 1) & 3
    return row[8 * ((w >> 1) & 3) + 2 * (w >> 3) + (w & 1)];
  } else {
    uint32_t v = 0u;
#pragma unroll
    for (int n = 0; n < 4 / B; ++n) {  // the dword's sets of 8 channels
      const int set = w * (4 / B) + n, kb = set >> 2, g = set & 3;
      const uint32_t x = B == 1 ? row[g] >> (4 * kb) : B == 2 ? row[2 * g + (kb >> 1)] >> (8 * (kb & 1)) : row[4 * g + kb];
      constexpr uint32_t kMask = (1u << (4 * B)) - 1u;
      v |= (spread<B>(x & kMask) | (spread<B>((x >> 16) & kMask) << B)) << (8 * B * n);
    }
    return v;
  }
}

// Canonical dword w of token r from a value block (in LDS): the token is one
// element of one K-group, its channels sit in the group's lanes (value_bit).
template <int B>
__device__ __forceinline__ uint32_t canonical_value(const uint32_t* blk, int r, int w) {
  const int kg = (r & 15) >> 2, e = (r & 3) + 4 * (r >> 4);
  constexpr uint32_t kMask = (1u << B) - 1u;
  uint32_t v = 0u;
  if constexpr (B == 1) {  // operands 2w and 2w + 1 share a dword
    const int sh = 16 * (e & 1) + 8 * (w & 1) + (e >> 1);
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const uint32_t x = blk[(c + 16 * kg) * 2 + (w >> 1)] >> sh;
      v |= ((x & 1u) << c) | (((x >> 4) & 1u) << (16 + c));
    }
  } else {
    constexpr int kPer = 32 / B;  // channels of the dword, all in operand mb
    const int c0 = w * kPer, mb = c0 >> 4;
    const int word = B == 2 ? mb >> 1 : B == 4 ? mb : 2 * mb + (e >> 2);
    const int sh = B == 2 ? 16 * (mb & 1) + 2 * e : B == 4 ? 4 * (e >> 1) + 16 * (e & 1) : 8 * (e & 3);
#pragma unroll
    for (int c = 0; c < kPer; ++c)
      v |= ((blk[((c0 & 15) + c + 16 * kg) * 2 * B + word] >> sh) & kMask) << (B * c);
  }
  return v;
}

// One workgroup per 32-token block, then one per 32 tail tokens.  Bound by the
// launch at one head's size: 16384 tokens of one head at K2V2 (1.6 MB in, as
// much out) take 4 to 6 us in one launch; a kernel that fetched the codes bit
// by bit took 18, next to copies of the key meta and the tail of 3 us each.
template <int BK, int BV>
__global__ __launch_bounds__(256) void export_kernel(ExportArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t vblk[128 * BV];
  const int b = blockIdx.x, nblocks = a.Lq / 32, tid = threadIdx.x;
  const uint8_t* ring = a.arena + a.head0 + (uint64_t)a.h * a.head_stride;
  if (b >= nblocks) {  // tail tokens: 32 rows of keys and of values, a dword per thread and step
    const int t0 = (b - nblocks) * 32, n = min(32, a.ntail - t0);
    for (int i = tid; i < n * 64; i += 256) {
      const int t = t0 + (i >> 6), d = i & 63;
      const size_t src = (size_t)((a.Lq + t) % a.W) * 64 + d, dst = (size_t)t * 64 + d;
      reinterpret_cast<uint32_t*>(a.tk_out)[dst] = reinterpret_cast<const uint32_t*>(ring + region(a.tk))[src];
      reinterpret_cast<uint32_t*>(a.tv_out)[dst] = reinterpret_cast<const uint32_t*>(ring + region(a.tv))[src];
    }
    return;
  }
  const int ng = kHeadDim / a.gv;
  int t;  // the block's first token in its packed segment
  const uint8_t* seg = a.arena + packed_seg(a.pm, a.head0, a.head_stride, a.seq, a.h, 32 * b, t);
  const uint32_t* kc = reinterpret_cast<const uint32_t*>(seg + region(a.kc) + (size_t)t * 16 * BK);
  const uint32_t* vc = reinterpret_cast<const uint32_t*>(seg + region(a.vc) + (size_t)t * 16 * BV);
  const uint8_t* vm = seg + region(a.vm) + (size_t)t * 4 * ng;
  uint32_t* kc_out = reinterpret_cast<uint32_t*>(a.kc_out + (size_t)b * 512 * BK);
  uint32_t* vc_out = reinterpret_cast<uint32_t*>(a.vc_out + (size_t)b * 512 * BV);
  uint32_t* vm_out = reinterpret_cast<uint32_t*>(a.vm_out) + (size_t)b * 32 * ng;
  if ((32 * b) % a.gk == 0 && tid < 128)  // a key group's scales and zeros: 512 bytes
    reinterpret_cast<uint32_t*>(a.km_out)[(size_t)(32 * b / a.gk) * 128 + tid] =
        reinterpret_cast<const uint32_t*>(seg + region(a.km))[(size_t)(t / a.gk) * 128 + tid];
  for (int i = tid; i < 32 * BV; i += 256) reinterpret_cast<uint4*>(vblk)[i] = reinterpret_cast<const uint4*>(vc)[i];
  for (int i = tid; i < 128 * BK; i += 256) kc_out[i] = canonical_key<BK>(kc + i / (4 * BK) * (4 * BK), i % (4 * BK));
  for (int i = tid; i < 32 * ng; i += 256) {
    const int r = i / ng, g = i % ng;
    const uint32_t s = *reinterpret_cast<const uint16_t*>(vm + value_meta_s(g, r));
    const uint32_t z = *reinterpret_cast<const uint16_t*>(vm + value_meta_z(g, r, ng));
    vm_out[i] = s | (z << 16);
  }
  __syncthreads();
  for (int i = tid; i < 128 * BV; i += 256) vc_out[i] = canonical_value<BV>(vblk, i / (4 * BV), i % (4 * BV));
}

template <int BK>
int launch_export_bv(const ExportArgs& a, void* stream) {
  const dim3 grid(a.Lq / 32 + (a.ntail + 31) / 32), block(256);
  hipStream_t s = (hipStream_t)stream;
  switch (a.bv) {
    case 1: hipLaunchKernelGGL((export_kernel<BK, 1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((export_kernel<BK, 2>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((export_kernel<BK, 4>), grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL((export_kernel<BK, 8>), grid, block, 0, s, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

}  // namespace

int launch_export(const ExportArgs& a, void* stream) {
  if (a.Lq + a.ntail <= 0) return 0;
  switch (a.bk) {
    case 1: return launch_export_bv<1>(a, stream);
    case 2: return launch_export_bv<2>(a, stream);
    case 4: return launch_export_bv<4>(a, stream);
    case 8: return launch_export_bv<8>(a, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

int launch_dequant(const DequantArgs& a, void* stream) {
  if (a.ntok <= 0) return 0;
  hipLaunchKernelGGL(dequant_kernel, dim3(a.ntok * a.hkv), dim3(kHeadDim), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}


// ---------------------------------------------------------------- read probe
//
// Streaming-read ceiling of the device: every thread reads 16-byte words in
// a grid-stride loop and folds them with XOR; one word per workgroup goes to
// `sink` so that the loads stay.  The decode kernels' algorithmic bytes are
// compared with this measured rate as well as with the nominal HBM peak.
namespace {
constexpr int kProbeBlocks = 2048;
__global__ __launch_bounds__(256) void read_probe_kernel(const uint4* __restrict__ src, size_t n, uint32_t* sink) {
  uint32_t acc = 0u;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const uint4 v = src[i];
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  __shared__ uint32_t red[256];
  red[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t x = 0u;
    for (int t = 0; t < 256; ++t) x ^= red[t];
    sink[blockIdx.x] = x;
  }
}
}  // namespace

int read_probe_blocks() { return kProbeBlocks; }

int launch_read_probe(const void* src, size_t bytes, uint32_t* sink, void* stream) {
  if (bytes == 0) return 0;
  hipLaunchKernelGGL(read_probe_kernel, dim3(kProbeBlocks), dim3(256), 0, (hipStream_t)stream,
                     static_cast<const uint4*>(src), bytes / 16, sink);
  return (int)hipGetLastError();
}

}  // namespace kvq
