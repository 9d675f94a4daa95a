"""GPU parity of the fp16-tail split (decode and chunk queries) against the
fp64 oracle: tails of one token to several blocks per wave, at the edges of
its 32-token blocks, wrapped around the ring, with every head count on the
kernels of both classes, and fused appends that attend over the call's
own tokens (inputs aligned to 4 bytes only) while storing them.  The bound is
tight where every token is fp16: both products are exact but for fp32 sums
and weights of 22 bits, 2^-20 relative with the sums of a few hundred terms."""
import numpy as np
import pytest

import oracle
from helpers import ATTN_TOL, Case, log, row_rel_err
from workloads import Workload, gen_append, gen_q_chunk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def W(L, gq, bk, bv, R, gk=32, gv=32):
    return Workload(f"tail_L{L}_gq{gq}_K{bk}V{bv}_R{R}", 1, 2 * gq, 2, 128, (L,), (bk,), (bv,), gk, gv, R, cfg_id=96)


@pytest.mark.parametrize("gq,bits", [(1, (2, 2)), (2, (1, 1)), (4, (2, 2)), (5, (2, 2)), (8, (4, 4)), (4, (1, 4)), (8, (8, 1))])
@pytest.mark.parametrize("L,R", [(1, 0), (31, 31), (32, 40), (33, 64), (129, 129), (160, 300), (300, 300)])
def test_all_fp16_is_near_exact(gq, bits, L, R):
    c = Case(W(L, gq, bits[0], bits[1], R))
    c.append_all()
    err = row_rel_err(c.decode()[0], c.oracle_out(0)).max()
    log(f"[tail] {c.w.name}: {err:.2e}")
    assert err <= 2.0 ** -20 * 4


@pytest.mark.parametrize("gq,bits,R,n", [(4, (2, 2), 128, 1), (5, (1, 1), 100, 3), (8, (4, 8), 33, 2), (4, (4, 1), 65, 5),
                                         (1, (2, 2), 0, 1)])
def test_fused_append_attends_over_its_tokens(gq, bits, R, n):
    """Steps of n tokens over more than a ring's length: every ring offset, flushes among them."""
    w = W(400, gq, bits[0], bits[1], R)
    c = Case(w, max_tokens=400 + 60 * n)
    c.append_all()
    K, V, q = c.K[0], c.V[0], torch.from_numpy(c.q[0][None]).cuda()
    for step in range(60):
        kn, vn = gen_append(w, 0, 0, step, n)
        K, V = np.concatenate([K, kn]), np.concatenate([V, vn])
        bufs = []
        for x in (kn, vn):  # 4-byte aligned, not 16
            flat = torch.zeros(x.size + 2, dtype=torch.float16, device="cuda")
            flat[2:] = torch.from_numpy(x.reshape(-1)).cuda()
            bufs.append(flat[2:].view((1,) + x.shape))
        out = c.cache.append_decode(bufs[0], bufs[1], q)
        if step % 7 == 0 or step > 55:
            ref = oracle.decode_seq(c.q[0], K, V, w.bits_k[0], w.bits_v[0], w.key_group, w.value_group, w.window)
            err = row_rel_err(out[0].cpu().numpy(), ref).max()
            assert err <= ATTN_TOL, (step, err)
    for h in range(2):
        assert (c.cache.export(0, h) == oracle.build_head(np.ascontiguousarray(K[:, h]), np.ascontiguousarray(V[:, h]),
                                                          w.bits_k[0], w.bits_v[0], w.key_group, w.value_group,
                                                          w.window)).all()


@pytest.mark.parametrize("gq,bits,n_q", [(4, (2, 2), 3), (4, (1, 1), 8), (5, (2, 2), 6), (8, (4, 4), 3), (4, (8, 8), 3),
                                         (2, (2, 2), 7), (1, (4, 4), 16), (4, (1, 8), 4)])
@pytest.mark.parametrize("L,R", [(200, 200), (333, 128), (40, 100)])
def test_chunk_rows(gq, bits, n_q, L, R):
    c = Case(W(L, gq, bits[0], bits[1], R))
    c.append_all()
    q = gen_q_chunk(c.w, n_q)
    out = c.cache.chunk(torch.from_numpy(q[None]).cuda())[0].cpu().numpy()
    ref = oracle.chunk_seq(q, c.K[0], c.V[0], bits[0], bits[1], 32, 32, R)
    err = row_rel_err(out, ref).max()
    log(f"[tail] {c.w.name} n_q {n_q}: {err:.2e}")
    assert err <= (2.0 ** -20 * 4 if L <= R else ATTN_TOL)


@pytest.mark.parametrize("gq,bits", [(4, (1, 1)), (5, (2, 2)), (8, (4, 1))])
@pytest.mark.parametrize("scale,big", [(2.0 ** -20, 0), (2.0 ** -20, 77), (1e4, 0)])
def test_value_ranges(gq, bits, scale, big):
    """Values down to subnormal fp16, alone and with one large token far into the tail, and large ones."""
    c = Case(W(150, gq, bits[0], bits[1], 150))
    c.V[0] = np.clip(c.V[0].astype(np.float32) * scale, -60000, 60000).astype(np.float16)
    if big:
        c.V[0][big] = (c.V[0][big].astype(np.float32) * 2.0 ** 26).astype(np.float16)
    c.append_all()
    err = row_rel_err(c.decode()[0], c.oracle_out(0)).max()
    log(f"[tail] {c.w.name} scale {scale:g} big {big}: {err:.2e}")
    assert err <= 2.0 ** -20 * 4


@pytest.mark.parametrize("gq,bits,n_q", [(1, (2, 2), 40), (4, (1, 1), 16), (8, (8, 8), 8), (2, (4, 1), 30)])
@pytest.mark.parametrize("big", [90, 130, 147])
def test_rows_that_see_only_small_values(gq, bits, n_q, big):
    """Subnormal values and one large token: the queries before it see subnormal ones alone.  A row that the large token
    carries has its score's error (base 2, magnitude up to 2^6) as its own: 2^-17, as with many rows."""
    c = Case(W(150, gq, bits[0], bits[1], 150))
    c.V[0] = (c.V[0].astype(np.float32) * 2.0 ** -20).astype(np.float16)
    c.V[0][big] = (c.V[0][big].astype(np.float32) * 2.0 ** 26).astype(np.float16)
    c.append_all()
    q = gen_q_chunk(c.w, n_q)
    out = c.cache.chunk(torch.from_numpy(q[None]).cuda())[0].cpu().numpy()
    err = row_rel_err(out, oracle.chunk_seq(q, c.K[0], c.V[0], bits[0], bits[1], 32, 32, 150))
    before = max(0, big - (150 - n_q))  # queries that don't see it
    log(f"[tail] {c.w.name} n_q {n_q} big {big}: {err[:before].max() if before else 0:.2e} {err[before:].max():.2e}")
    assert before == 0 or err[:before].max() <= 2.0 ** -18
    assert err[before:].max() <= 2.0 ** -17
