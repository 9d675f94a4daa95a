"""GPU parity of the append kernel's own branches against the CPU oracle's
canonical image (bytes equal): every bit width with key groups of 32, 64 and
128 tokens, value groups that span part of a lane row, one row and several,
inputs that are not 16-byte aligned, appends that pack groups held in the
ring while the new tokens overwrite its other slots (two launches), appends
to an empty ring longer than the ring (one launch), ring copies of more and
of fewer tokens than one copy workgroup takes, ragged batches, and groups
whose differences need more than 24 bits."""
import numpy as np
import pytest

import oracle
from helpers import log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _inputs(shape, seed, spread):
    r = np.random.default_rng(seed)
    x = r.standard_normal(shape).astype(np.float32)
    if spread:  # magnitudes from the smallest fp16 values to the largest in one group
        x *= np.exp2(r.integers(-22, 14, size=shape)).astype(np.float32)
    x = np.clip(x, -32000, 32000).astype(np.float16)
    x[r.random(shape) < 0.01] = np.float16(-0.0)
    return x


CASES = [
    # bits_k, bits_v, gk, gv, window, q heads per kv head, chunk sizes, spread, input offset (halves)
    (1, 1, 32, 32, 0, 4, (300,), False, 0),
    (2, 2, 64, 64, 40, 4, (700, 1, 130, 64), False, 0),       # packs ring tokens, two launches
    (2, 1, 128, 128, 0, 8, (511, 129), True, 0),
    (4, 4, 64, 32, 128, 5, (200, 200, 33), True, 0),
    (8, 8, 128, 64, 7, 4, (640, 5), True, 0),
    (8, 4, 32, 128, 33, 2, (97, 31, 31, 64), False, 0),
    (1, 2, 32, 32, 32, 4, (90, 45, 45), True, 3),              # 2-byte aligned inputs
    (4, 8, 128, 32, 0, 1, (130, 126), True, 1),
    (2, 2, 32, 8, 16, 4, (200, 60), True, 0),                  # value groups of 8 and 16 channels
    (1, 1, 64, 16, 0, 4, (257,), True, 2),
    (4, 1, 128, 16, 90, 4, (400, 100), False, 0),
    (8, 2, 32, 128, 0, 4, (64, 3, 61), True, 0),
    (4, 8, 64, 8, 10, 8, (150,), True, 5),
]


@pytest.mark.parametrize("bk,bv,gk,gv,R,gq,chunks,spread,off", CASES)
def test_packed_bytes(bk, bv, gk, gv, R, gq, chunks, spread, off):
    from paper_2607_16248_amd import KVCache
    hkv, L = 2, sum(chunks)
    K, V = (_inputs((2, L, hkv, 128), 7 * i + bk + 10 * bv + gk, spread) for i in (1, 2))
    cache = KVCache(2, gq * hkv, hkv, L, [bk] * 2, [bv] * 2, key_group=gk, value_group=gv, fp16_window=R)
    pos = [0, 0]
    for i, n in enumerate(chunks):
        new = [n, n if i else max(1, n - 50)]  # ragged from the first call on
        n_max = max(new)
        bufs = []
        for X in (K, V):
            x = np.zeros((2, n_max, hkv, 128), dtype=np.float16)
            for s in range(2):
                x[s, :new[s]] = X[s, pos[s]:pos[s] + new[s]]
            flat = torch.zeros(off + x.size, dtype=torch.float16, device="cuda")
            flat[off:] = torch.from_numpy(x.reshape(-1)).cuda()
            bufs.append(flat[off:].view(x.shape))
        log(f"[append] K{bk}V{bv} gk {gk} gv {gv} R {R}: {new} tokens at {pos}")
        cache.append(bufs[0], bufs[1], new)
        pos = [p + m for p, m in zip(pos, new)]
        torch.cuda.synchronize()
        for s in range(2):
            for h in range(hkv):
                ref = oracle.build_head(np.ascontiguousarray(K[s, :pos[s], h]), np.ascontiguousarray(V[s, :pos[s], h]),
                                        bk, bv, gk, gv, R)
                got = cache.export(s, h)
                bad = np.flatnonzero(got != ref)
                assert bad.size == 0, (s, h, bad.size, bad[:5])
    cache.check()


@pytest.mark.parametrize("gq,value", [(4, np.nan), (4, np.inf), (1, -np.inf), (1, np.nan)])
@pytest.mark.parametrize("tensor", [0, 1])
def test_non_finite_inputs_raise_the_flag(gq, value, tensor):
    from paper_2607_16248_amd import KVCache, kvq
    K, V = (_inputs((1, 96, 2, 128), i, False) for i in (1, 2))
    (K, V)[tensor][0, 41, 1, 77] = value
    cache = KVCache(1, 2 * gq, 2, 96, [2], [2], key_group=32, value_group=32 if gq > 1 else 16, fp16_window=0)
    cache.append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    torch.cuda.synchronize()
    with pytest.raises(kvq.KvqError):
        cache.check()
    # the other head's image is untouched by the bad group
    ref = oracle.build_head(np.ascontiguousarray(K[0, :, 0]), np.ascontiguousarray(V[0, :, 0]), 2, 2, 32,
                            32 if gq > 1 else 16, 0)
    assert (cache.export(0, 0) == ref).all()
