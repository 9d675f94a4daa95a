"""The logit step's window where its selection takes another path: more
groups of equal maxima than can be read again, masked rows (-inf and the
type's lowest value), +inf and NaN logits, an outlier that leaves one
histogram bin for the rest, and fewer groups than window entries.

The window is the K largest in the total order of the fp32 bit patterns
(sign-flipped, so NaN above +inf), equal ones by index: whole numbers, compared
exactly.  tau = 2 keeps every row uncorrected, so the logits stay the same
bits.
"""
import numpy as np
import pytest

from dgap_inputs import gen_weights

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _logits(kind, V, seed):
    rng = np.random.default_rng(seed)
    z = rng.normal(0, 3, V).astype(np.float32)
    at = rng.permutation(V)
    if kind == "equal":
        z[:] = 1.5
    elif kind == "few_values":
        z = np.round(z).astype(np.float32)
    elif kind == "mask_inf":
        z[at[V // 50:]] = -np.inf
    elif kind == "mask_lowest":
        z[at[V // 50:]] = np.finfo(np.float32).min
    elif kind == "mask_most":
        z[at[5:]] = -np.inf
    elif kind == "inf":
        z[at[:3]] = np.inf
    elif kind == "nan":
        z[at[:3]] = np.nan
        z[at[3:6]] = -np.float32(np.nan)
    elif kind == "all_negative_nan":
        z[:] = -np.float32(np.nan)
        z[at[:4]] = 1.0
    elif kind == "outlier":
        z[at[0]] = 1e30
    elif kind == "signed_zeros":
        z = np.where(rng.integers(0, 2, V) == 0, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
    elif kind == "clustered":  # the largest ones side by side
        z[V // 3:V // 3 + min(V // 4, 600)] += 20.0
    return z


def _window(z, k):
    u = z.view(np.uint32)
    order = np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint64)
    key = (order << np.uint64(32)) | (np.uint64(0xFFFFFFFF) - np.arange(z.size, dtype=np.uint64))
    return np.argsort(key)[::-1][:k].astype(np.int32)


KINDS = ["plain", "equal", "few_values", "mask_inf", "mask_lowest", "mask_most", "inf", "nan", "all_negative_nan",
         "outlier", "signed_zeros", "clustered"]
SIZES = [(256, 256), (300, 9), (2048, 16), (2049, 64), (5000, 65), (32000, 128), (128256, 128), (128256, 129),
         (152064, 256), (524288, 128)]


@pytest.mark.parametrize("V,k", SIZES, ids=[f"V{v}_k{k}" for v, k in SIZES])
def test_window_in_every_path(V, k):
    from paper_2607_16248_amd import kvq
    dev = torch.device("cuda:0")
    z = np.stack([_logits(kind, V, 7 * i + k) for i, kind in enumerate(KINDS)])
    w = gen_weights(seed=3, det_bias=0.0)
    t = {n: torch.from_numpy(np.ascontiguousarray(getattr(w, n))).to(dev) for n in ("w1", "b1", "w2", "c1", "cb1", "c2")}
    p = kvq.dgap_params(V, k, 2.0, t["w1"], t["b1"], t["w2"], w.b2, t["c1"], t["cb1"], t["c2"], w.cb2)
    B = len(KINDS)
    logits = torch.from_numpy(z.copy()).to(dev)
    ws = torch.empty(kvq.dgap_workspace_bytes(B, V, k), dtype=torch.uint8, device=dev)
    info = torch.full((B, kvq.dgap_info_floats(k)), float("nan"), dtype=torch.float32, device=dev)
    kvq.dgap_restore(p, logits, B, ws, info=info)
    torch.cuda.synchronize()
    got = info.cpu().numpy()[:, 16:16 + k].view(np.int32)
    for i, kind in enumerate(KINDS):
        assert np.array_equal(got[i], _window(z[i], k)), kind
    assert np.array_equal(logits.cpu().numpy().view(np.uint32), z.view(np.uint32))
