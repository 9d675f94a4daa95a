// Host stand-ins for the HIP runtime calls and kernel launchers of the
// library (see hip/hip_runtime.h in this directory).  "Device" buffers are host
// buffers, and every launch reads and writes the ranges that its kernel would
// (packed codes and meta, the fp16 ring, input rows, split records, outputs,
// the export image), so that AddressSanitizer checks the offsets the host code
// computes into them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "kvq_internal.h"

int g_launches = 0;
int g_row_plans = 0;  // chunk launches whose row groups were checked

hipError_t hipGetDevice(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
  *value = 256;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipMemcpy(void* dst, const void* src, size_t bytes, hipMemcpyKind) {
  std::memmove(dst, src, bytes);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

// The regions of a head in the order of the layout, none starting before the
// one ahead of it ends: vb is the last, one alignment unit before the head's
// end.  (A page holds the packed regions, the ring's block the others.)
template <class Args>
static void check_regions(const Args& a, const uint32_t* vb_units) {
  const uint64_t kc = kvq::region(a.kc), km = kvq::region(a.km), vc = kvq::region(a.vc), vm = kvq::region(a.vm),
                 tk = kvq::region(a.tk), tv = kvq::region(a.tv),
                 ring = kvq::align_up((uint64_t)a.W * kvq::kHeadDim * 2, kvq::kAlign),
                 vb = vb_units ? kvq::region(*vb_units) : tv + ring,
                 packed_end = a.pm.table != nullptr ? a.pm.page_head_bytes : tk;
  if (kc <= km && km <= vc && vc <= vm && vm <= packed_end && tv - tk == ring && vb - tv == ring &&
      vb + kvq::kAlign == a.head_stride)
    return;
  std::fprintf(stderr, "region check failed: kc %llx km %llx vc %llx vm %llx tk %llx tv %llx vb %llx, stride %llx\n",
               (unsigned long long)kc, (unsigned long long)km, (unsigned long long)vc, (unsigned long long)vm,
               (unsigned long long)tk, (unsigned long long)tv, (unsigned long long)vb,
               (unsigned long long)a.head_stride);
  std::abort();
}

// Ranges a kernel reads or writes (both through intercepted calls).
static void rd(const void* p, size_t n) {
  static std::vector<uint8_t> sink;
  if (sink.size() < n) sink.resize(n);
  if (n) std::memcpy(sink.data(), p, n);
}
static void wr(const void* p, size_t n) {
  if (n) std::memset(const_cast<void*>(p), 0, n);
}
constexpr size_t kTokenBytes = kvq::kHeadDim * 2;

// f(range) for the packed codes and meta of tokens [from, to) of a head.
template <class Args, class F>
static void packed_ranges(const Args& a, uint64_t head0, int seq, int h, int from, int to, int bk, int bv, F f) {
  const size_t ng = kvq::kHeadDim / a.gv, gk = a.gk;
  for (int t = from; t < to; t += a.gk) {
    int in;
    const uint8_t* seg = a.arena + kvq::packed_seg(a.pm, head0, a.head_stride, seq, h, t, in);
    f(seg + kvq::region(a.kc) + (size_t)in * 16 * bk, gk * 16 * bk);
    f(seg + kvq::region(a.km) + in / gk * 512, 512);
    f(seg + kvq::region(a.vc) + (size_t)in * 16 * bv, gk * 16 * bv);
    f(seg + kvq::region(a.vm) + in * 4 * ng, gk * 4 * ng);
  }
}
// f(key range, value range) for the ring slots of tokens [from, to) of a head.
template <class Args, class F>
static void ring_ranges(const Args& a, uint64_t head0, int h, int from, int to, F f) {
  const uint8_t* ring = a.arena + head0 + (uint64_t)h * a.head_stride;
  for (int t = from; t < to; ++t) {
    f(ring + kvq::region(a.tk) + (size_t)(t % a.W) * kTokenBytes, kTokenBytes);
    f(ring + kvq::region(a.tv) + (size_t)(t % a.W) * kTokenBytes, kTokenBytes);
  }
}

namespace kvq {
int launch_append(const AppendArgs& a, int bk, int bv, void*) {
  check_regions(a, &a.vb);
  for (int i = 0; i < a.nseq; ++i) {
    const AppendSeq& S = a.seq[i];
    auto input = [&](int t, int h) {
      const size_t at = (((size_t)S.seq * a.n_max + (t - S.L_old)) * a.hkv + h) * kHeadDim;
      rd(a.K + at, kTokenBytes);
      rd(a.V + at, kTokenBytes);
    };
    const int packed = a.quantize ? S.n_quant * a.gk : 0, copy0 = std::max(S.Lq_new, S.L_old),
              copied = S.n_copy > 0 ? S.L_new - copy0 : 0;
    if (packed != (a.quantize ? S.Lq_new - S.Lq_old : 0) || (copied + kCopyTokens - 1) / kCopyTokens != S.n_copy) {
      std::fprintf(stderr, "append check failed: sequence %d, %d groups, %d copies\n", S.seq, S.n_quant, S.n_copy);
      std::abort();
    }
    for (int h = 0; h < a.hkv; ++h) {
      ring_ranges(a, S.head0, h, S.Lq_old, std::min(S.L_old, S.Lq_old + packed), rd);
      for (int t = std::max(S.L_old, S.Lq_old); t < S.Lq_old + packed; ++t) input(t, h);
      packed_ranges(a, S.head0, S.seq, h, S.Lq_old, S.Lq_old + packed, bk, bv, wr);
      for (int t = copy0; t < copy0 + copied; ++t) input(t, h);
      ring_ranges(a, S.head0, h, copy0, copy0 + copied, wr);
      rd(a.arena + S.head0 + (uint64_t)h * a.head_stride + region(a.vb), 4);
    }
  }
  return ++g_launches, 0;
}
int launch_table_set(const TableSet& t, void*) {
  // the table lives in the arena: write it as the kernel would
  for (int i = 0; i < t.n; ++i) t.table[t.idx[i]] = t.val[i];
  return ++g_launches, 0;
}
int launch_word_reset(const WordReset& r, void*) {
  for (int i = 0; i < r.n; ++i) std::memset(r.arena + r.off[i], 0, 4);
  return ++g_launches, 0;
}
}  // namespace kvq

// The row groups of a chunk launch, checked the way the kernels read them
// (query of row g = min(rg * qpr + row_x[g], nqry - 1), q row offset from the
// group's row 0, no record for spare rows): every q row read lies in the
// sequence's [nqry][Hq] block, every record row in [0, nqry * Hq), and every
// (query, head) of a kv head is written by exactly one row.
static void check_rows(const kvq::DecodeArgs& a, int rows) {
  check_regions(a, &a.vb);
  if (a.nqry <= 1) return;
  auto bad = [&](const char* what, int rg, int g) {
    std::fprintf(stderr, "row check failed (%s): nqry %d qpr %d nrg %d gqh %d rows %d, group %d row %d\n", what,
                 a.nqry, a.qpr, a.nrg, a.gqh, rows, rg, g);
    std::abort();
  };
  if (rows < 1 || rows > 32 || a.qpr < 1 || a.qpr * a.gqh > rows || a.nrg != (a.nqry + a.qpr - 1) / a.qpr)
    bad("shape", -1, -1);
  std::vector<int> hits((size_t)a.nqry * a.gqh, 0);
  for (int h = 0; h < a.hkv; ++h)
    for (int rg = 0; rg < a.nrg; ++rg)
      for (int g = 0; g < rows; ++g) {
        const int j0 = rg * a.qpr + a.row_x[g];
        const int j = std::min(j0, a.nqry - 1);
        const int64_t qrow = (int64_t)rg * a.qpr * a.hq + h * a.gqh + a.row_off[g] - (int64_t)(j0 - j) * a.hq;
        if (qrow < 0 || qrow >= (int64_t)a.nqry * a.hq || qrow / a.hq != j) bad("q row", rg, g);
        const int64_t head = qrow % a.hq - (int64_t)h * a.gqh;
        if (head < 0 || head >= a.gqh) bad("q head", rg, g);
        if (j0 >= a.nqry) continue;  // spare: no record
        const int64_t rec = (int64_t)rg * a.qpr * a.hq + h * a.gqh + a.row_off[g];
        if (rec != qrow) bad("record row", rg, g);
        if (h == 0) ++hits[(size_t)j * a.gqh + head];
      }
  for (int v : hits)
    if (v != 1) bad("coverage", -1, -1);
  ++g_row_plans;
}

// What a decode or chunk launch reads of the cache and writes: the records of
// every split, or the output of a sequence that is not merged.
static void touch_decode(const kvq::DecodeArgs& a, int bk, int bv) {
  const size_t rows = (size_t)a.hq * a.nqry, row = kvq::kHeadDim * 4;
  for (int i = 0; i < a.nseq; ++i) {
    const kvq::DecodeSeq& S = a.seq[i];
    for (int h = 0; h < a.hkv; ++h) {
      packed_ranges(a, S.head0, S.seq, h, 0, S.Lq, bk, bv, rd);
      ring_ranges(a, S.head0, h, S.Lq, S.L_old, rd);
      if (a.K_new == nullptr) continue;
      ring_ranges(a, S.head0, h, S.L_old, S.L, wr);
      for (int t = S.L_old; t < S.L; ++t) {
        const size_t at = (((size_t)S.seq * a.n_max + (t - S.L_old)) * a.hkv + h) * kvq::kHeadDim;
        rd(a.K_new + at, kTokenBytes);
        rd(a.V_new + at, kTokenBytes);
      }
    }
    rd(a.q + (size_t)S.seq * rows * kvq::kHeadDim, rows * kTokenBytes);
    if (a.out != nullptr && S.nsplit == 1)
      wr(a.out + (size_t)S.seq * rows * kvq::kHeadDim, rows * row);
    else
      wr(a.ws + (size_t)S.ws_base * rows * kvq::kRecFloats, S.nsplit * rows * kvq::kRecFloats * 4);
  }
  ++g_launches;
}

namespace kvq {
int launch_decode(const DecodeArgs& a, int bk, int bv, int rows, void*) {
  return check_rows(a, rows), touch_decode(a, bk, bv), 0;
}
int launch_decode_matrix(const DecodeArgs& a, int bk, int bv, int rows, void*) {
  return check_rows(a, rows), touch_decode(a, bk, bv), 0;
}
int launch_chunk_matrix(const DecodeArgs& a, int bk, int bv, int rows, void*) {
  return check_rows(a, rows), touch_decode(a, bk, bv), 0;
}
int launch_export(const ExportArgs& a, void*) {
  check_regions(a, nullptr);
  packed_ranges(a, a.head0, a.seq, a.h, 0, a.Lq, a.bk, a.bv, rd);
  ring_ranges(a, a.head0, a.h, a.Lq, a.Lq + a.ntail, rd);
  wr(a.kc_out, (size_t)a.Lq * 16 * a.bk);
  wr(a.km_out, (size_t)a.Lq / a.gk * 512);
  wr(a.vc_out, (size_t)a.Lq * 16 * a.bv);
  wr(a.vm_out, (size_t)a.Lq * 4 * (kHeadDim / a.gv));
  wr(a.tk_out, a.ntail * kTokenBytes);
  wr(a.tv_out, a.ntail * kTokenBytes);
  return ++g_launches, 0;
}
int launch_merge(const MergeArgs& a, void*) {
  for (int i = 0; i < a.nseq; ++i) {
    const MergeSeq& S = a.seq[i];
    rd(a.ws + (size_t)S.ws_base * a.hq * kRecFloats, (size_t)S.nsplit * a.hq * kRecFloats * 4);
    wr(a.out + (size_t)S.seq * a.hq * kHeadDim, (size_t)a.hq * kHeadDim * 4);
  }
  return ++g_launches, 0;
}
int launch_dgap(const DgapArgs&, int, void*) { return ++g_launches, 0; }
int launch_dequant(const DequantArgs& a, void*) {
  check_regions(a, nullptr);
  for (int h = 0; h < a.hkv; ++h) {
    packed_ranges(a, a.head0, a.seq, h, std::min(a.tok0, a.Lq) / a.gk * a.gk, std::min(a.tok0 + a.ntok, a.Lq), a.bk, a.bv, rd);
    ring_ranges(a, a.head0, h, std::max(a.tok0, a.Lq), a.tok0 + a.ntok, rd);
  }
  wr(a.K_out, (size_t)a.ntok * a.hkv * kHeadDim * 4);
  wr(a.V_out, (size_t)a.ntok * a.hkv * kHeadDim * 4);
  return ++g_launches, 0;
}
int launch_fill_zero(void* dst, size_t words, void*) {
  std::memset(dst, 0, words * 4);
  return ++g_launches, 0;
}
int launch_read_probe(const void*, size_t, uint32_t*, void*) { return ++g_launches, 0; }
int read_probe_blocks() { return 2048; }
int scratch_workspace(void** ptr) {
  static void* buf = nullptr;
  if (!buf) buf = std::calloc(1, kScratchBytes);
  *ptr = buf;
  return 0;
}
}  // namespace kvq
