"""The projection GEMM takes 64 x 64, 128 x 128 or 256 x 256 tiles (or 256-row ones
and smaller ones for the last rows) by the number of rows M of a launch, and
small batches share an attention item's query blocks out.  A row's result must not depend on which of them ran
(each output is one accumulator over K in order): the same sequence alone, in
batches at the edges of the tiles and inside a batch large enough for the
256-row tiles gives the same bits, full-vocabulary head included, and agrees
with the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_10139_amd.device import DeviceModel, DevicePrefill
from synth.configs import ModelSpec
from synth.gen import make_model
from tests._parity import TOL_BF16, random_gains

pytestmark = pytest.mark.gpu

MODELS = {
    "hd64": ModelSpec(n_layers=3, d_model=256, n_heads=4, n_kv_heads=4, d_ff=512, vocab=1024, act="swiglu",
                      dtype="bf16", weight_seed=51),
    "hd128": ModelSpec(n_layers=2, d_model=768, n_heads=6, n_kv_heads=2, d_ff=512, vocab=1024, act="swiglu",
                       dtype="bf16", weight_seed=52),
}
LARGE = 40000   # tokens: 256-row tiles for every projection of both models
# one sequence per length; the batches' totals sit at tile edges
TOTALS = (1, 31, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1023, 1024, 1025, 2049, 8300, 18200)
_M = {}


def model(name, compute):
    if (name, compute) not in _M:
        m = random_gains(make_model(MODELS[name]))
        _M[name, compute] = (m, DeviceModel(m, compute=compute))
    return _M[name, compute]


def prefill(dm, seqs, full_vocab):
    cu = np.zeros(len(seqs) + 1, dtype=np.int32)
    cu[1:] = np.cumsum([len(s) for s in seqs])
    pf = DevicePrefill(None, max_tokens=int(cu[-1]), dmodel=dm)
    out = pf.run(torch.from_numpy(np.concatenate(seqs)).cuda(), torch.from_numpy(cu).cuda(), full_vocab=full_vocab)
    torch.cuda.synchronize()
    r = out.cpu().numpy()
    pf.close()
    return r


@pytest.mark.parametrize("name,compute", [("hd64", "f16"), ("hd128", "f16"), ("hd128", "bf16")])
@pytest.mark.parametrize("full_vocab", [False, True])
def test_row_bits_do_not_depend_on_tiles(name, compute, full_vocab):
    m, dm = model(name, compute)
    r = np.random.default_rng(7)

    def seq(n):
        return r.integers(3, 1024, n).astype(np.int32)

    probe = [seq(1), seq(64), seq(100), seq(255), seq(700)]
    # the probes at the head of a batch large enough for 256-row tiles
    filler = [seq(int(n)) for n in r.integers(16, 400, LARGE // 208)]
    print("large batch", flush=True)
    want = prefill(dm, probe + filler, full_vocab)[:len(probe)]
    for total in TOTALS:
        print("total", total, flush=True)
        for i, p in enumerate(probe):
            rest = total - len(p)
            if rest < 0:
                continue
            seqs = [p] + [seq(min(1000, rest - o)) for o in range(0, rest, 1000)]
            got = prefill(dm, seqs, full_vocab)[0]
            assert np.array_equal(got, want[i]), (total, i)
    # many sequences: the last layer's rows and the head at M = sequences
    for n in (63, 64, 65, 129, 300):
        print("sequences", n, flush=True)
        got = prefill(dm, [seq(9) for _ in range(n - len(probe))] + probe, full_vocab)[-len(probe):]
        assert np.array_equal(got, want), n
    if not full_vocab and compute == "f16":
        assert np.abs(want - oracle.label_logits(m, probe, (1, 2))).max() <= TOL_BF16
