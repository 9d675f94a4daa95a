"""GPU parity of kvq_chunk_attention with many (query, head) rows per kv head
(the many-row kernel) against the fp64 oracle on the same
byte-identical cache: every bit class of the matrix layout, every key and
value group size it takes, all head counts (with spare rows in the last row
group and idle waves in the last workgroup), masks inside packed blocks and
inside the fp16 tail, tails longer than a split, caches with no packed token,
ragged batches with bit classes of their own, paged caches, forced split
lengths (tables of key zero-points started inside a key group, splits past a
row workgroup's last visible token), a workspace too small for the planned
splits, value scales of 1e-5 and inputs near the fp16 limit."""
import numpy as np
import pytest

import oracle
from helpers import ATTN_TOL, Case, log, row_rel_err
from workloads import Workload, gen_q_chunk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def W(name, hq, hkv, lens, bk, bv, gk=32, gv=32, R=0, dist="normal"):
    n = len(lens)
    bk = (bk,) * n if isinstance(bk, int) else bk
    bv = (bv,) * n if isinstance(bv, int) else bv
    return Workload(name, n, hq, hkv, 128, lens, bk, bv, gk, gv, R, key_dist=dist, cfg_id=95)


def _run(c, n_q, ws_bytes=None):
    from paper_2607_16248_amd import kvq
    w = c.w
    q = np.stack([gen_q_chunk(w, n_q, 0, s) for s in range(w.batch)])
    out = torch.full((w.batch, n_q, w.num_q_heads, 128), float("nan"), device="cuda")
    need = kvq.kvq_chunk_workspace_bytes(c.cache.handle, n_q) if ws_bytes is None else ws_bytes
    ws = torch.full((max(need, 256) // 4,), float("nan"), device="cuda")
    kvq.kvq_chunk_attention(c.cache.handle, torch.from_numpy(q).cuda(), n_q, out, ws, need)
    torch.cuda.synchronize()
    return q, out.cpu().numpy()


def _check(c, q, out, heads=None):
    w = c.w
    heads = list(range(w.num_kv_heads)) if heads is None else heads
    rows = np.concatenate([np.arange(h * w.group_q, (h + 1) * w.group_q) for h in heads])
    worst = 0.0
    for s in range(w.batch):
        ref = oracle.chunk_seq(q[s], c.K[s], c.V[s], w.bits_k[s], w.bits_v[s], w.key_group, w.value_group, w.window,
                               heads=heads)
        err = row_rel_err(out[s][:, rows], ref[:, rows])
        worst = max(worst, float(err.max()))
        assert err.max() <= ATTN_TOL, (s, np.unravel_index(np.argmax(err), err.shape), err.max())
    return worst


CASES = [
    # workload, n_q, split tokens, cache options
    (W("k1v1", 8, 2, (700,), 1, 1), 70, 0, {}),
    (W("k2v2_R128", 8, 2, (900,), 2, 2, R=128), 200, 0, {}),
    (W("k1v2_g64_split", 8, 2, (1500,), 1, 2, gk=64), 100, 192, {}),
    (W("k2v1_g128_gv64", 8, 2, (1300,), 2, 1, gk=128, gv=64), 64, 384, {}),
    (W("k4v4_gq8", 8, 1, (900,), 4, 4), 450, 0, {}),
    (W("k4v4_gq5_gv64", 10, 2, (600,), 4, 4, gv=64), 77, 128, {}),
    (W("k4v4_gq8_paged", 8, 1, (1000,), 4, 4, R=30), 400, 256, {"page_tokens": 64}),
    (W("k8v8_gq8_gv128", 16, 2, (500,), 8, 8, gv=128, R=40), 33, 0, {}),
    (W("k4v8_gq1", 2, 2, (640,), 4, 8), 290, 0, {}),
    (W("k8v4_gq2_g64", 4, 2, (777,), 8, 4, gk=64, R=33), 129, 256, {}),
    (W("ragged_classes", 8, 2, (900, 333, 410), (2, 1, 8), (2, 1, 8), R=50), 200, 0, {}),
    (W("same_class_batch", 8, 2, (1200, 150), 2, 2), 150, 128, {}),
    (W("whole_sequence", 8, 2, (300,), 2, 2), 300, 0, {}),
    (W("all_fp16", 8, 2, (250,), 2, 2, R=400), 60, 0, {}),
    (W("tail_over_splits", 8, 2, (900,), 1, 1, R=500), 300, 128, {}),
    (W("paged", 8, 2, (1111, 640), 2, 2, gk=64, R=20), 90, 256, {"page_tokens": 128}),
    (W("paged_k1v1", 8, 2, (800,), 1, 1), 64, 0, {"page_tokens": 32}),
    (W("long_table", 4, 1, (3000,), 2, 1, dist="student_t3"), 48, 1600, {}),  # 50 key groups per split
]


@pytest.mark.parametrize("w,n_q,split,kw", CASES, ids=[c[0].name for c in CASES])
def test_many_rows_match_the_oracle(w, n_q, split, kw):
    assert n_q * w.group_q >= 80
    log(f"[prefill] {w.name} n_q={n_q} split={split}")
    c = Case(w, **kw)
    c.append_all()
    if split:
        from paper_2607_16248_amd import kvq
        kvq.kvq_set_split_tokens(c.cache.handle, split)
    q, out = _run(c, n_q)
    worst = _check(c, q, out)
    assert np.isfinite(out).all()
    _, again = _run(c, n_q)
    assert (out.view(np.uint32) == again.view(np.uint32)).all()
    log(f"[prefill] {w.name}: max row-relative error {worst:.2e}")


def test_workspace_of_the_smallest_plan():
    """A workspace that holds no more than one split's records still serves the call."""
    from paper_2607_16248_amd import kvq
    w = W("ws", 8, 2, (4000,), 2, 2, R=64)
    c = Case(w, heads=[1], max_tokens=40000)
    c.append_all()
    n_q = 64
    full = kvq.kvq_chunk_workspace_bytes(c.cache.handle, n_q)
    small = full
    q, ref = _run(c, n_q)
    while True:  # the smallest workspace that the call accepts
        try:
            _, out = _run(c, n_q, small // 2 // 16 * 16)
        except kvq.KvqError as e:
            assert e.status == kvq.ERR_CAPACITY
            break
        small = small // 2 // 16 * 16
        assert np.abs(out - ref).max() <= 1e-3 * np.abs(ref).max()
    assert small < full
    _check(c, q, ref, heads=[1])


@pytest.mark.parametrize("bits", [1, 2, 4, 8])
@pytest.mark.parametrize("scale", [1e-5, 2000.0])
def test_value_and_key_ranges(bits, scale):
    w = W(f"k{bits}_scale{scale:g}", 8, 2, (500,), bits, bits, gv=64 if bits == 4 else 32, R=40)
    c = Case(w)
    for s in range(w.batch):
        c.V[s] = np.clip(c.V[s].astype(np.float32) * scale, -60000, 60000).astype(np.float16)
        if scale > 1:  # wide key groups, scores kept in range by one large channel per head
            c.K[s][:, :, 5] = np.where(np.arange(w.lens[s]) % 2 == 0, 30000, -30000).astype(np.float16)[:, None]
    c.append_all()
    log(f"[prefill] K{bits}V{bits} value scale {scale:g}")
    from paper_2607_16248_amd import kvq
    n_q = 64
    q = np.stack([gen_q_chunk(w, n_q, 0, s) for s in range(w.batch)])
    if scale > 1:
        q[..., 5] = (q[..., 5].astype(np.float32) * 1e-4).astype(np.float16)
    out = torch.full((w.batch, n_q, w.num_q_heads, 128), float("nan"), device="cuda")
    ws = torch.empty(kvq.kvq_chunk_workspace_bytes(c.cache.handle, n_q), dtype=torch.uint8, device="cuda")
    kvq.kvq_chunk_attention(c.cache.handle, torch.from_numpy(q).cuda(), n_q, out, ws)
    torch.cuda.synchronize()
    log(f"[prefill] worst {_check(c, q, out.cpu().numpy()):.2e}")


# Every token fp16: keys, values and queries are exact operands and weights
# carry hi + lo halves (2^-23), so a row is off by its scores alone, fp32 sums
# of magnitude up to 2^5 whose absolute error is a relative one of a weight:
# 2^-18, the bound that the tails of fewer rows hold (test_gpu_tail.py).
@pytest.mark.parametrize("gq,bits,n_q,L", [(4, (1, 1), 20, 250), (4, (2, 2), 64, 250), (5, (2, 1), 33, 33), (8, (1, 2), 130, 130),
                                           (4, (8, 8), 64, 300), (8, (4, 8), 40, 95)])
def test_fp16_tokens_are_near_exact(gq, bits, n_q, L):
    c = Case(W(f"fp16_gq{gq}_K{bits[0]}V{bits[1]}_L{L}", 2 * gq, 2, (L,), bits[0], bits[1], R=400))
    c.append_all()
    q, out = _run(c, n_q)
    err = row_rel_err(out[0], oracle.chunk_seq(q[0], c.K[0], c.V[0], bits[0], bits[1], 32, 32, 400)).max()
    log(f"[prefill] {c.w.name} n_q {n_q}: {err:.2e}")
    assert err <= 2.0 ** -18


# Subnormal values: raw ones in the tail (alone, and with one large token that
# ends their lift), and the zero-points and scales of packed ones.  Values that
# are constant over a token's channels are their zero-point (scale 0, codes 0),
# which meets both halves of the weights as the tail does: the same bound.
@pytest.mark.parametrize("gq,bits,scale,big", [(4, (1, 1), 2.0 ** -20, 0), (4, (2, 2), 2.0 ** -20, 177), (8, (8, 8), 2.0 ** -20, 90),
                                               (5, (2, 1), 1e4, 0)])
def test_value_ranges_of_fp16_tokens(gq, bits, scale, big):
    c = Case(W(f"fp16_gq{gq}_K{bits[0]}V{bits[1]}_scale{scale:.0e}_big{big}", 2 * gq, 2, (200,), bits[0], bits[1], R=200))
    c.V[0] = np.clip(c.V[0].astype(np.float32) * scale, -60000, 60000).astype(np.float16)
    if big:
        c.V[0][big] = (c.V[0][big].astype(np.float32) * 2.0 ** 26).astype(np.float16)
    c.append_all()
    q, out = _run(c, 40)
    err = row_rel_err(out[0], oracle.chunk_seq(q[0], c.K[0], c.V[0], bits[0], bits[1], 32, 32, 200)).max()
    log(f"[prefill] {c.w.name}: {err:.2e}")
    # one large token can carry a row alone, with a small weight: its score's error
    # (base 2, magnitude up to 2^6: 2^-19 of rounding per step of the sum of four
    # products) is then the row's, not averaged over tokens
    assert err <= (2.0 ** -17 if big else 2.0 ** -18)


@pytest.mark.parametrize("gq,bits,gv", [(4, (1, 1), 32), (4, (2, 2), 64), (8, (8, 8), 128), (8, (4, 8), 32)])
def test_zero_points_of_packed_tokens(gq, bits, gv):
    c = Case(W(f"zeros_gq{gq}_K{bits[0]}V{bits[1]}_gv{gv}", 2 * gq, 2, (256,), bits[0], bits[1], gv=gv))
    # (of one sign, so that no sum cancels)
    c.V[0] = np.broadcast_to(np.abs(c.V[0][..., :1].astype(np.float32) * 2.0 ** -18).astype(np.float16), c.V[0].shape).copy()
    c.append_all()
    q, out = _run(c, 40)
    err = row_rel_err(out[0], oracle.chunk_seq(q[0], c.K[0], c.V[0], bits[0], bits[1], 32, gv, 0)).max()
    log(f"[prefill] {c.w.name}: {err:.2e}")
    assert err <= 2.0 ** -18


# Packed tokens: at one and two bits both halves of the weights meet the values,
# so what is left are fp32 sums (2^-24 per addition over up to 2^8 blocks and
# scores of magnitude up to 2^5): 2^-17.
@pytest.mark.parametrize("gq,bits,gv,n_q,L", [(4, (1, 1), 32, 100, 2000), (4, (1, 2), 32, 64, 320), (5, (2, 1), 64, 40, 1500),
                                              (8, (2, 2), 128, 33, 3000), (1, (2, 2), 32, 300, 700)])
def test_packed_tokens_meet_both_halves_of_the_weights(gq, bits, gv, n_q, L):
    c = Case(W(f"packed_gq{gq}_K{bits[0]}V{bits[1]}_L{L}", 2 * gq, 2, (L,), bits[0], bits[1], gv=gv))
    c.append_all()
    q, out = _run(c, n_q)
    err = row_rel_err(out[0], oracle.chunk_seq(q[0], c.K[0], c.V[0], bits[0], bits[1], 32, gv, 0)).max()
    log(f"[prefill] {c.w.name} n_q {n_q}: {err:.2e}")
    assert err <= 2.0 ** -17


# Value ranges of a few subnormal steps: the scale is the smallest there is, half
# of the codes or more go unused, and a value is the difference of its
# zero-point with the scale's multiple (up to 2^7 steps) and its product (as
# much), where the row's largest output has about 2^3 steps: 2^4 times the bound
# above.
@pytest.mark.parametrize("bits,scale", [((8, 8), 2.0 ** -20), ((4, 8), 2.0 ** -21), ((8, 4), 2.0 ** -23)])
def test_subnormal_value_scales(bits, scale):
    c = Case(W(f"steps_K{bits[0]}V{bits[1]}_{scale:.0e}", 16, 2, (512,), bits[0], bits[1]))
    c.V[0] = (c.V[0].astype(np.float32) * scale).astype(np.float16)
    c.append_all()
    q, out = _run(c, 48)
    err = row_rel_err(out[0], oracle.chunk_seq(q[0], c.K[0], c.V[0], bits[0], bits[1], 32, 32, 0)).max()
    log(f"[prefill] {c.w.name}: {err:.2e}")
    assert err <= 2.0 ** -13
