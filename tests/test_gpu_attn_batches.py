"""Attention and the label head share their work out by the batch: query blocks of
one sequence to several workgroups where one sequence outweighs the rest, waves
that take last-position items alone where there are many, as many waves per head
row as its width fills.  A row's logits must not depend on which of them ran: rows
at the edges of the query and key blocks (rows without tokens between them, more
than the 64 that are searched at a time) alone, in a batch of 80 and behind 3,000 and 9,000
others (the short ones among 2,200) give the same bits, with and without a shared prefix, and the fp64 oracle's
values.  The norm gains are random, so that a gain read at a wrong place shows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_10139_amd.device import DeviceModel, DeviceQuery
from synth.configs import ModelSpec, Pred, Query
from synth.gen import make_model
from tests._parity import TOL_BF16, random_gains

pytestmark = pytest.mark.gpu

# (head dim, query heads per K/V head)
HEADS = {(64, 1): (256, 4, 4), (64, 2): (512, 8, 4), (64, 4): (512, 8, 2), (128, 1): (256, 2, 2), (128, 2): (512, 4, 2),
         (128, 3): (768, 6, 2)}
EDGES = (0, 1, 2, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 0, 0, 127, 128, 129, 191, 192, 193, 257, 700)


def run(rows, prefix, m, dm, npre):
    lens = np.array([len(s) for s in rows], dtype=np.int64)
    off = np.zeros(len(rows) + 1, dtype=np.int64)
    off[1:] = np.cumsum(lens)
    probe = {"id": np.arange(len(rows), dtype=np.int32), "c": np.zeros(len(rows), np.int32), "offsets": off,
             "tokens": np.concatenate(rows).astype(np.int32)}
    q = Query(preds=(Pred("c", "ge", 0),), labels=(1, 2), decision="binary_gt", agg="count", n_prefix=npre)
    dq = DeviceQuery({"probe": probe, "build": None, "prefix": prefix}, m, q, dmodel=dm)
    dq.run()
    torch.cuda.synchronize()
    r = dq.results()
    dq.close()
    assert r["status"] == 0 and r["n_selected"] == len(rows)
    return r["logits"]


@pytest.mark.parametrize("npre", [0, 13, 64])
@pytest.mark.parametrize("heads", list(HEADS))
def test_row_bits_do_not_depend_on_the_batch(heads, npre):
    print("case:", heads, npre, flush=True)
    d, h, kv = HEADS[heads]
    m = random_gains(make_model(ModelSpec(n_layers=2, d_model=d, n_heads=h, n_kv_heads=kv, d_ff=512, vocab=1024,
                                          act="swiglu", dtype="bf16", weight_seed=81)))
    dm = DeviceModel(m)
    r = np.random.default_rng(82)
    prefix = r.integers(3, 1024, 64).astype(np.int32)
    lens = list(EDGES) + list(r.integers(0, 260, 57))
    rows = [r.integers(3, 1024, n).astype(np.int32) for n in lens]
    print("  batch of 80", flush=True)
    got = run(rows, prefix, m, dm, npre)
    others = [r.integers(3, 1024, n).astype(np.int32) for n in r.integers(0, 60, 9000)]
    for n in (3000, 9000):   # 3,000: query blocks shared out among 3,080 sequences; 9,000: whole sequences
        print("  among others:", n, flush=True)
        assert np.array_equal(run(others[:n] + rows, prefix, m, dm, npre)[n:], got)
    short = [i for i, n in enumerate(lens) if n <= 64]
    print("  short rows among 2,200 others", flush=True)
    assert np.array_equal(run([rows[i] for i in short] + others[:2200], prefix, m, dm, npre)[:len(short)], got[short])
    for n in (1, 33, 65, 129, 700):
        i = lens.index(n)
        print("  alone:", n, flush=True)
        assert np.array_equal(run([rows[i]], prefix, m, dm, npre)[0], got[i])
    sample = [i for i in range(len(EDGES)) if lens[i] + npre > 0]
    want = oracle.label_logits(m, [np.concatenate([prefix[:npre], rows[i]]) for i in sample], (1, 2))
    assert np.abs(got[sample] - want).max() <= TOL_BF16
