"""The fp32 path (32 x 64 projection tiles, attention with four lanes per query)
at the edges of its tiles and key blocks, for head dims 32 and 64, MHA and
GQA, against the fp64 oracle at the fp32 tolerance; a sequence's bits do not
depend on the others in its batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_10139_amd.device import DeviceModel, DevicePrefill
from synth.configs import ModelSpec
from synth.gen import make_model
from tests._parity import TOL_F32, random_gains

pytestmark = pytest.mark.gpu

LABELS = (1, 2, 3, 250, 5, 6, 7, 0)   # the most a head takes


def run(dm, batch):
    cu = np.zeros(len(batch) + 1, dtype=np.int32)
    cu[1:] = np.cumsum([len(s) for s in batch])
    pf = DevicePrefill(None, labels=LABELS, max_tokens=int(cu[-1]), dmodel=dm)
    out = pf.run(torch.from_numpy(np.concatenate(batch)).cuda(), torch.from_numpy(cu).cuda()).cpu().numpy()
    pf.close()
    return out


@pytest.mark.parametrize("d,heads,kv,ff", [(128, 4, 2, 64), (64, 2, 2, 192), (256, 4, 1, 512)])
def test_f32_model(d, heads, kv, ff):
    spec = ModelSpec(n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, d_ff=ff, vocab=256, act="gelu", dtype="f32",
                     weight_seed=61, init_std=0.05)
    m = random_gains(make_model(spec))
    dm = DeviceModel(m)
    r = np.random.default_rng(3)
    seqs = [r.integers(0, 256, n).astype(np.int32)
            for n in (1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200)]
    got = run(dm, seqs)
    assert np.abs(got - oracle.label_logits(m, seqs, LABELS)).max() <= TOL_F32
    for i, s in enumerate(seqs):
        assert np.array_equal(run(dm, [s])[0], got[i]), len(s)
    # so many items (more than four per workgroup) that waves take short sequences by themselves
    n = 4 * 4096 // heads + 1
    many = [r.integers(0, 256, k).astype(np.int32) for k in r.integers(1, 24, n)]
    at = np.sort(r.choice(n, len(seqs), replace=False))
    for i, s in zip(at, seqs):
        many[i] = s
    assert np.array_equal(run(dm, many)[at], got)
