"""GPU parity of the decode kernel of the mixed and fine-grouped classes (1- or
2-bit keys with 4- or 8-bit values and the reverse, value groups of 8 or 16
channels) against the fp64 oracle: every such class and value group, key
groups of 32 to 128 tokens (zero-point terms per group), all head counts,
chunk rows that fill a tile of 16 and that leave spare rows and queries,
pages, ragged batches, and value scales and key ranges at both ends of fp16.

Bound: q, keys and values are exact operands and weights carry 22 bits, so a
row is off by the fp32 sums alone: 2^-24 per addition over up to 2^10 blocks
of partial sums and scores of magnitude up to 2^5 (an absolute score error of
2^-19 is a relative weight error of 2^-19): 2^-17 in all."""
import numpy as np
import pytest

import oracle
from helpers import Case, log, row_rel_err
from paper_2607_16248_amd import kvq
from workloads import Workload, gen_q_chunk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 2.0 ** -17


def W(gq, lens, bk, bv, gk=32, gv=32, R=0):
    n = len(lens)
    return Workload(f"exact_gq{gq}_K{bk}V{bv}_gk{gk}_gv{gv}_R{R}", n, 2 * gq, 2, 128, lens, (bk,) * n, (bv,) * n, gk, gv, R,
                    cfg_id=97)


CLASSES = [(1, 4, 32), (1, 8, 128), (2, 4, 64), (2, 8, 32), (4, 1, 32), (4, 2, 64), (8, 1, 32), (8, 2, 128), (1, 1, 16),
           (2, 2, 8), (4, 4, 16), (8, 8, 8), (1, 2, 8), (4, 8, 8), (8, 4, 16), (2, 8, 16)]


@pytest.mark.parametrize("i", range(len(CLASSES)), ids=[f"K{k}V{v}_gv{g}" for k, v, g in CLASSES])
def test_decode(i):
    bk, bv, gv = CLASSES[i]
    w = W((4, 5, 8, 1, 2)[i % 5], (1111, 64 + 32 * i), bk, bv, (32, 64, 128)[i % 3], gv, (0, 37, 128)[i % 3])
    c = Case(w, **({"page_tokens": 128} if i % 4 == 1 else {}))
    c.append_all((700, 411))
    out = c.decode()
    for s in range(2):
        err = row_rel_err(out[s], c.oracle_out(s)).max()
        log(f"[exact] {w.name} seq {s}: {err:.2e}")
        assert err <= TOL, s


@pytest.mark.parametrize("gq,bk,bv,gk,gv,n_q,R", [(4, 4, 2, 32, 32, 4, 0), (4, 2, 8, 64, 32, 5, 20), (5, 1, 4, 32, 16, 7, 0),
                                                  (8, 8, 1, 128, 8, 3, 64), (1, 2, 2, 32, 8, 17, 0), (2, 4, 4, 64, 16, 9, 300)])
def test_chunk_rows(gq, bk, bv, gk, gv, n_q, R):
    w = W(gq, (700,), bk, bv, gk, gv, R)
    c = Case(w)
    c.append_all()
    q = gen_q_chunk(w, n_q)
    out = c.cache.chunk(torch.from_numpy(q[None]).cuda())[0].cpu().numpy()
    err = row_rel_err(out, oracle.chunk_seq(q, c.K[0], c.V[0], bk, bv, gk, gv, R)).max()
    log(f"[exact] {w.name} n_q {n_q}: {err:.2e}")
    assert err <= TOL


@pytest.mark.parametrize("bk,bv,gv", [(1, 8, 32), (8, 1, 32), (2, 2, 16), (4, 2, 8), (1, 4, 16)])
@pytest.mark.parametrize("scale", [2.0 ** -20, 3000.0])
def test_ranges(bk, bv, gv, scale):
    """Value scales down to single subnormal steps and up to the largest; key groups that span +-30000."""
    w = W(4, (600,), bk, bv, 32, gv)
    c = Case(w)
    c.V[0] = np.clip(c.V[0].astype(np.float32) * scale, -60000, 60000).astype(np.float16)
    if scale > 1:
        c.K[0][:, :, 5] = np.where(np.arange(600) % 2 == 0, 30000, -30000).astype(np.float16)[:, None]
        c.q[0][:, 5] = (c.q[0][:, 5].astype(np.float32) * 1e-4).astype(np.float16)
        c.qd = torch.from_numpy(np.stack(c.q)).cuda()
    c.append_all()
    err = row_rel_err(c.decode()[0], c.oracle_out(0)).max()
    log(f"[exact] {w.name} scale {scale:g}: {err:.2e}")
    assert err <= TOL


def _quantized(x, dim, bits):
    """Min-max quantized and dequantized along dim, in float64: the smallest fp16 scale that covers the range."""
    lo, hi = x.amin(dim, keepdim=True), x.amax(dim, keepdim=True)
    want = (hi - lo) / (2 ** bits - 1)
    s = want.half()
    s = torch.where(s.double() < want, (s.view(torch.int16) + 1).view(torch.half), s).double()
    return lo + s * torch.where(s > 0, (x - lo) / s, 0.0).round()


def test_head_past_4gib():
    """8-bit keys and values with room for 2^24 tokens: the value scales and the fp16 ring lie past 4 GiB.  The key
    codes of the tokens from 2^21 on reach the offsets that those would have modulo 2^32."""
    n, room = (1 << 21) + 4096 + 5, 1 << 24
    gen = torch.Generator(device="cuda").manual_seed(11)
    K, V = (torch.randn((1, n, 1, 128), generator=gen, device="cuda", dtype=torch.half) for _ in range(2))
    q = torch.randn((1, 4, 128), generator=gen, device="cuda", dtype=torch.half)
    cache = kvq.KVCache(1, 4, 1, room, [8], [8], key_group=32, value_group=32, fp16_window=0)
    cache.append(K, V, [n])
    kd, vd = cache.dequant(0, 0, n)
    lq = n // 32 * 32
    for t0, t1 in ((0, 4096), (1 << 20, (1 << 20) + 4096), (1 << 21, lq)):
        k = K[0, t0:t1, 0].double().view(-1, 32, 128)
        v = V[0, t0:t1, 0].double().view(-1, 4, 32)
        assert (kd[t0:t1, 0].double() - _quantized(k, 1, 8).view(-1, 128)).abs().max() <= 2.0 ** -21  # |x| < 8 in fp32
        assert (vd[t0:t1, 0].double() - _quantized(v, 2, 8).view(-1, 128)).abs().max() <= 2.0 ** -21
    assert (kd[lq:, 0] == K[0, lq:, 0].float()).all() and (vd[lq:, 0] == V[0, lq:, 0].float()).all()
    out = cache.decode(q)[0].double()
    s = torch.empty((4, n), device="cuda", dtype=torch.double)
    for t in range(0, n, 1 << 18):
        s[:, t:t + (1 << 18)] = q[0].double() @ kd[t:t + (1 << 18), 0].double().t().contiguous()
    p = torch.softmax(s / 128 ** 0.5, 1)
    ref, size = (sum(p[:, t:t + (1 << 18)].contiguous() @ f(vd[t:t + (1 << 18), 0].double()) for t in range(0, n, 1 << 18))
                 for f in (torch.clone, torch.abs))
    # the bound is on the terms' sum of magnitudes: over two million tokens the values themselves average out
    err = ((out - ref).abs().amax(1) / size.amax(1)).max().item()
    log(f"[exact] {n} tokens of a head past 4 GiB: {err:.2e}")
    assert err <= TOL


@pytest.mark.parametrize("gq,bk,bv,gv", [(4, 4, 2, 32), (8, 2, 2, 16), (5, 1, 8, 64), (4, 2, 2, 32), (8, 4, 4, 32), (1, 1, 1, 64)])
def test_records_hold_the_split_maximum(gq, bk, bv, gv):
    """kvq_decode_partials: [0] is the split's largest base-2 score, [1] and [4..] are relative to it, in every split of
    the mixed and fine-grouped classes and in the fp16 tail's split of every class.  A score's error is 2^-24 of the
    sum of its terms' magnitudes per addition (up to 2^7 of them, half the bits random): 2^-20 of it."""
    w, st = W(gq, (1000,), bk, bv, 32, gv, 100), 256
    c = Case(w)
    c.append_all()
    kvq.kvq_set_split_tokens(c.cache.handle, st)
    ws = torch.full((kvq.kvq_workspace_bytes(c.cache.handle) // 4,), float("nan"), device="cuda")
    kvq.kvq_decode_partials(c.cache.handle, c.qd, ws)
    kd, vd = (x.double().cpu().numpy() for x in c.cache.dequant(0, 0, 1000))
    lq, rows = 896, 2 * gq
    splits = [(t, min(t + st, lq)) for t in range(0, lq, st)] + [(lq, 1000)]
    rec = ws.cpu().numpy()[:len(splits) * rows * 132].reshape(len(splits), rows, 132).astype(np.float64)
    exact = (bk <= 2) != (bv <= 2) or gv < 32
    for i, (t0, t1) in enumerate(splits):
        if not exact and i < len(splits) - 1:
            continue
        for r in range(rows):
            k, v, q = kd[t0:t1, r // gq], vd[t0:t1, r // gq], c.q[0][r].astype(np.float64)
            s = k @ q * (np.log2(np.e) / 128 ** 0.5)
            slack = 2.0 ** -20 * (np.abs(k) @ np.abs(q)).max() * (np.log2(np.e) / 128 ** 0.5)
            assert abs(rec[i, r, 0] - s.max()) <= slack, (i, r)
            p = np.exp2(s - s.max())
            assert abs(rec[i, r, 1] - p.sum()) <= (2.0 ** -18 + slack) * p.sum(), (i, r)
            assert np.abs(rec[i, r, 4:] - p @ v).max() <= (2.0 ** -17 + slack) * (p @ np.abs(v)).max(), (i, r)


@pytest.mark.parametrize("gq,bk,bv,gv,gk", [(4, 4, 2, 32, 32), (8, 8, 1, 32, 64), (5, 2, 8, 64, 32), (4, 8, 8, 16, 128), (2, 1, 4, 32, 32),
                                            (1, 2, 2, 8, 32), (4, 8, 4, 8, 32)])
@pytest.mark.parametrize("ks,qs,outlier", [(2.0 ** -8, 2.0 ** 8, 0), (2.0 ** -12, 2.0 ** 12, 0), (2.0 ** -18, 2.0 ** 14, 0),
                                           (2.0 ** -18, 2.0 ** 14, 1), (2.0 ** -18, 7.0, 0)])
def test_small_keys(gq, bk, bv, gv, gk, ks, qs, outlier):
    """Keys down to subnormal fp16 under queries that bring their scores back, alone and with a channel too large to be
    lifted (then the scores' own sums carry its rounding: 2^-24 of 8192 * 0.5 times log2(e) / sqrt(128), twice)."""
    w = W(gq, (700,), bk, bv, gk, gv, 40)
    c = Case(w)
    c.K[0] = (c.K[0].astype(np.float32) * ks).astype(np.float16)
    c.q[0] = np.clip(c.q[0].astype(np.float32) * qs, -60000, 60000).astype(np.float16)
    if outlier:
        c.K[0][:, :, 5] = np.where(np.arange(700) % 2 == 0, 8192, -8192).astype(np.float16)[:, None]
        c.q[0][:, 5] = np.float16(2.0 ** -12)
    c.qd = torch.from_numpy(np.stack(c.q)).cuda()
    c.append_all()
    err = row_rel_err(c.decode()[0], c.oracle_out(0)).max()
    log(f"[exact] {w.name} keys {ks:g} queries {qs:g} outlier {outlier}: {err:.2e}")
    assert err <= TOL


@pytest.mark.parametrize("bk,bv,gv", [(1, 4, 32), (2, 8, 32), (4, 2, 32), (1, 1, 16), (8, 8, 16)])
def test_equal_weights(bk, bv, gv):
    """All scores near zero: values average out to 1/20 of their size, and their zero-points must not leave a rounding
    of their own size.  Values in 22 bits: 2^-22 of up to 2^2 each, averaged over 2^9 tokens, against outputs of 2^-3."""
    c = Case(W(4, (512,), bk, bv, 32, gv))
    c.q[0] = (c.q[0].astype(np.float32) * 2.0 ** -10).astype(np.float16)
    c.qd = torch.from_numpy(np.stack(c.q)).cuda()
    c.append_all()
    err = row_rel_err(c.decode()[0], c.oracle_out(0)).max()
    log(f"[exact] {c.w.name} equal weights: {err:.2e}")
    assert err <= 2.0 ** -20
