"""GPU parity of kvq_chunk_attention (the last n_q tokens of every sequence
attend causally) against the fp64 oracle (oracle.chunk_seq) on the same
seeded, byte-identical cache, through the C ABI.

- row-normwise relative error <= 2e-3 for every (sequence, query, head);
- masked tokens inside packed blocks (no fp16 window: the chunk reaches
  into the last key groups), inside the fp16 tail, and n_q = L (the first
  query sees one token: its value row);
- every row-group shape: the chunk kernel with 16 and 32 rows, the decode
  kernel with 4, 5 and 8 rows (one or two queries per group, also of one or
  two heads), the exact kernel's tiles of 16 rows; a last row group with spare rows (n_q not a multiple of its queries: the
  spare rows repeat the last query and write nothing);
- n_q = 1 equals kvq_decode_attention bit for bit; results are bitwise
  reproducible.
- value scales of ~1e-5 (the weight shift from the head's value-scale
  bound), on contiguous and paged caches.
"""
import numpy as np
import pytest

import oracle
from helpers import ATTN_TOL, Case, log, row_rel_err
from workloads import Workload, gen_q_chunk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def W(name, batch, hq, hkv, lens, bk, bv, gk=32, gv=32, R=0, dist="normal", cfg=91):
    if isinstance(lens, int):
        lens = (lens,) * batch
    if isinstance(bk, int):
        bk = (bk,) * batch
    if isinstance(bv, int):
        bv = (bv,) * batch
    return Workload(name, batch, hq, hkv, 128, tuple(lens), tuple(bk), tuple(bv), gk, gv, R,
                    key_dist=dist, cfg_id=cfg)


def _chunk(c, n_q):
    from paper_2607_16248_amd import kvq
    w = c.w
    q = np.stack([gen_q_chunk(w, n_q, 0, s) for s in range(w.batch)])
    qd = torch.from_numpy(q).cuda()
    out = torch.full((w.batch, n_q, w.num_q_heads, w.head_dim), float("nan"), dtype=torch.float32,
                     device="cuda")
    ws = torch.empty(max(kvq.kvq_chunk_workspace_bytes(c.cache.handle, n_q), 256), dtype=torch.uint8,
                     device="cuda")
    kvq.kvq_chunk_attention(c.cache.handle, qd, n_q, out, ws)
    torch.cuda.synchronize()
    return q, out.cpu().numpy()


def _check(c, q, out, heads=None):
    w = c.w
    worst = 0.0
    for s in range(w.batch):
        ref = oracle.chunk_seq(q[s], c.K[s], c.V[s], w.bits_k[s], w.bits_v[s], w.key_group, w.value_group,
                               w.window, heads=heads)
        rows = slice(None) if heads is None else np.concatenate(
            [np.arange(h * w.group_q, (h + 1) * w.group_q) for h in heads])
        err = row_rel_err(out[s][:, rows], ref[:, rows])
        worst = max(worst, float(err.max()))
        assert err.max() <= ATTN_TOL, (s, np.unravel_index(np.argmax(err), err.shape), err.max())
    return worst


CASES = [
    (W("k1v1_gq4_L1000", 1, 32, 8, 1000, 1, 1), 40),                 # masks inside packed blocks; 32-row groups
    (W("k2v2_gq4_L777_odd", 1, 32, 8, 777, 2, 2), 7),                # odd n_q: one 32-row group, a spare query
    (W("k2v2_gq5_R128_t3", 2, 40, 8, (600, 333), 2, 2, R=128, dist="student_t3"), 16),  # masks in the fp16 tail; five heads, 32 rows
    (W("k4v4_gq8_g64", 1, 64, 8, 900, 4, 4, gk=64), 5),
    (W("k8v8_gq4", 1, 32, 8, 700, 8, 8), 12),
    (W("k1v2_gq4_g128", 1, 32, 8, 1500, 1, 2, gk=128), 24),
    (W("k1v1_gq1_matrix", 1, 8, 8, 500, 1, 1), 8),                   # one head per kv head: 8-query groups
    (W("k2v2_gq2_matrix", 1, 16, 8, 300, 2, 2), 2),                  # two heads: one 2-query group (4 rows)
    (W("k2v2_gq2_pad16", 1, 16, 8, 300, 2, 2), 6),                   # two heads: one 16-row group, two spare queries
    (W("k1v1_gq1_rows5", 1, 8, 8, 500, 1, 1), 5),                    # one head: one 5-query group
    (W("k1v1_gq1_rows32", 1, 8, 8, 600, 1, 1), 32),                  # 32 queries of one head per group
    (W("k2v1_gq2_odd", 1, 16, 8, 400, 2, 1), 7),                     # two heads, odd n_q: one 16-row group, a spare query
    (W("k1v1_gq1_g64_matrix", 1, 8, 8, 500, 1, 1, gk=64), 8),       # matrix kernel, 64-token key groups
    (W("k1v4_gq1_g64_vector", 1, 8, 8, 500, 1, 4, gk=64), 8),       # exact kernel, one tile of 8 rows and 8 spare ones
    (W("k2v4_gq2_g64_vector", 1, 16, 8, 300, 2, 4, gk=64), 6),      # exact kernel, one tile of 12 rows and 4 spare ones
    (W("k1v4_gq4_vector", 1, 32, 8, 800, 1, 4), 9),                  # exact kernel, three tiles of 16 rows
    (W("ragged_mixed_g64", 3, 32, 8, (900, 64, 300), (1, 2, 4), (1, 2, 4), gk=64), 33),
    (W("whole_sequence", 1, 32, 8, 48, 1, 1), 48),                   # n_q = L
    # the chunk kernel: 16-row groups (2 queries x 8 heads at 4 bits, 4 x 4 at
    # 1 and 2 bits for up to 4 queries) and 32-row groups (two row halves:
    # 8 x 4 over two ragged sequences with 64-token key groups and 1-bit
    # values, 4 x 8 heads)
    (W("k4v4_gq8_rows16", 1, 64, 8, 900, 4, 4), 6),
    (W("k1v1_gq4_rows16", 1, 32, 8, 700, 1, 1), 4),
    (W("k2v2_gq4_rows16", 1, 32, 8, 650, 2, 2), 3),
    (W("k2v1_gq4_rows32_g64", 2, 32, 8, (1000, 517), 2, 1, gk=64), 8),
    (W("k1v2_gq8_rows32", 1, 64, 8, 700, 1, 2), 4),
    # spare rows in the last row group: 32 rows with three spare queries,
    # 16 rows of one head with three, 8 rows (decode kernel) with one
    (W("k1v1_gq4_pad32", 1, 32, 8, 900, 1, 1), 5),
    (W("k1v1_gq1_pad16", 2, 8, 8, (600, 450), 1, 1), 13),
    (W("k8v8_gq4_pad8", 1, 32, 8, 700, 8, 8), 3),
    # five heads in the chunk kernel: 6 queries in 32 rows (two rows spare),
    # 3 in 16 (one row spare), each with spare queries in the last group
    (W("k1v1_gq5_rows32", 1, 40, 8, 800, 1, 1), 16),
    (W("k4v4_gq5_rows16", 2, 40, 8, (600, 333), 4, 4), 4),
]


@pytest.mark.parametrize("w,n_q", CASES, ids=[f"{w.name}_nq{n}" for w, n in CASES])
def test_chunk_matches_oracle(w, n_q):
    log(f"[chunk] {w.name} n_q={n_q}: append")
    c = Case(w)
    c.append_all()
    c.cache.check()
    q, out = _chunk(c, n_q)
    worst = _check(c, q, out)
    log(f"[chunk] {w.name} n_q={n_q}: max row-relative error {worst:.3e}")
    assert np.isfinite(out).all()


def test_one_query_equals_decode_and_is_reproducible():
    w = W("k1v1_gq4_L3000", 2, 32, 8, (3000, 1234), 1, 1, R=5)
    c = Case(w)
    c.append_all()
    from paper_2607_16248_amd import kvq
    q1 = torch.from_numpy(np.stack(c.q)).cuda()
    out1 = torch.empty((2, 1, 32, 128), dtype=torch.float32, device="cuda")
    ws = torch.empty(kvq.kvq_chunk_workspace_bytes(c.cache.handle, 1), dtype=torch.uint8, device="cuda")
    kvq.kvq_chunk_attention(c.cache.handle, q1.view(2, 1, 32, 128), 1, out1, ws)
    dec = c.decode()
    assert (out1.cpu().numpy()[:, 0].view(np.uint32) == dec.view(np.uint32)).all()
    qa, a = _chunk(c, 17)
    _, b = _chunk(c, 17)
    assert (a.view(np.uint32) == b.view(np.uint32)).all()
    _check(c, qa, a)


@pytest.mark.parametrize("n_q,bits", [(64, 1), (16, 2)])
def test_long_context_chunk_sampled_heads(n_q, bits):
    # 32K tokens of a Llama-3.1-8B layer, a chunk of n_q queries at the end;
    # two kv heads checked against the oracle
    w = W(f"llama8b_L32768_K{bits}V{bits}", 1, 32, 8, 32768, bits, bits, cfg=92)
    heads = [0, 5]
    c = Case(w, heads=heads)
    c.append_all()
    q, out = _chunk(c, n_q)
    worst = _check(c, q, out, heads=heads)
    log(f"[chunk] {w.name} n_q={n_q}: max row-relative error {worst:.3e}")


@pytest.mark.parametrize("bits,paged", [(1, False), (2, True), (8, False)])
def test_chunk_small_value_scales(bits, paged):
    # values of scale ~1e-5: the causal kernels take the same per-head weight
    # shift as single-token decode, sized by the head's bound on the packed
    # value scales (contiguous and paged caches)
    w = W(f"chunk_vscale_k{bits}", 2, 32, 8, (700, 1300), bits, bits, R=0, cfg=97)
    kw = {"page_tokens": 256, "num_pages": 16} if paged else {}
    c = Case(w, **kw)
    c.V = [(v.astype(np.float32) * 1e-5).astype(np.float16) for v in c.V]
    c.append_all()
    q, out = _chunk(c, 16)
    worst = _check(c, q, out)
    log(f"[chunk] value scale 1e-5, K{bits}V{bits}, paged={paged}: max row-relative error {worst:.3e}")
