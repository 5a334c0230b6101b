"""A NaN in an earlier token reaches its sequence's logits, and only those.

Attention skips keys by position, never by score: fmaxf drops NaN, so a lane or
wave whose visible keys all have NaN scores must not look like one without
keys.  Lengths and places around the four lanes that share a query, the 64-key
blocks and the four waves of one-query attention."""
import numpy as np
import pytest
import torch

from paper_2608_10139_amd.device import DeviceModel, DevicePrefill
from synth.configs import ModelSpec
from synth.gen import make_model

pytestmark = pytest.mark.gpu

BAD = 7   # the token whose embedding holds one NaN
MODELS = {
    "f32": ModelSpec(n_layers=1, d_model=128, n_heads=4, n_kv_heads=2, d_ff=128, vocab=256, act="gelu", dtype="f32",
                     weight_seed=71, init_std=0.05),
    "hd64": ModelSpec(n_layers=1, d_model=256, n_heads=4, n_kv_heads=4, d_ff=512, vocab=256, act="swiglu",
                      dtype="bf16", weight_seed=72, init_std=0.05),
    "hd128": ModelSpec(n_layers=2, d_model=768, n_heads=6, n_kv_heads=2, d_ff=512, vocab=256, act="swiglu",
                       dtype="bf16", weight_seed=73, init_std=0.05),
}


def run(dm, seqs):
    cu = np.zeros(len(seqs) + 1, dtype=np.int32)
    cu[1:] = np.cumsum([len(s) for s in seqs])
    pf = DevicePrefill(None, labels=(1, 2), max_tokens=int(cu[-1]), dmodel=dm)
    out = pf.run(torch.from_numpy(np.concatenate(seqs)).cuda(), torch.from_numpy(cu).cuda()).cpu().numpy()
    pf.close()
    return out


@pytest.mark.parametrize("name,compute", [("f32", None), ("hd64", "f16"), ("hd64", "bf16"), ("hd128", "f16")])
def test_nan_of_an_earlier_token_reaches_the_logits(name, compute):
    m = make_model(MODELS[name])
    m["emb"][BAD, 5] = np.float32(np.nan) if name == "f32" else 0x7FC0
    dm = DeviceModel(m, compute=compute)
    r = np.random.default_rng(9)
    seqs, bad = [], []
    for n in (1, 2, 3, 4, 5, 6, 9, 17, 63, 64, 65, 66, 67, 130, 200):
        s = r.integers(8, 256, n).astype(np.int32)
        seqs.append(s)
        bad.append(False)
        for p in sorted({0, 1, n // 2, n - 2, n - 1} & set(range(n))):
            t = s.copy()
            t[p] = BAD
            seqs.append(t)
            bad.append(True)
    bad = np.array(bad)
    got = run(dm, seqs)
    for i in np.flatnonzero(bad):
        at = int(np.flatnonzero(seqs[i] == BAD)[0])
        assert np.isnan(got[i]).all(), (len(seqs[i]), at, got[i])
    clean = run(dm, [s for s, b in zip(seqs, bad) if not b])
    assert np.isfinite(clean).all() and np.array_equal(got[~bad], clean)
