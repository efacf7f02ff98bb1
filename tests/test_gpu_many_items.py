"""Levels with more narrow items than the device holds at once, beside medium items: their narrow
items skip the loads of idle lanes and, from 65,536 items on, the tiny ones run on 4 lanes.  The
factors must not depend on it: bit for bit those of the vector path (dense_mfma = 0, whose levels
run in 256-thread blocks), and in a batch, whose level sums the items of all handles, those of
the handles alone.  Which levels the cases have is checked in test_schedule_levels.py."""
import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LARGE = kktgen.small(42000, config_id=198, steps=1)
BATCH = [kktgen.small(6000, config_id=199, steps=2), kktgen.small(200, config_id=145, steps=2),
         kktgen.small(5000, config_id=200, steps=2, flows=1)]


def factors(q, v, **kw):
    sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), **kw).bind()
    sk.refactor(v)
    out = (sk.export_factors()[0], sk.refactor_status())
    sk.close()
    return out


def test_tiny_items_beside_medium_ones():
    print("[gpu] 42,000 buses: tiny items on a level with medium ones", flush=True)
    q = kktgen.make_sequence(LARGE)
    v = torch.from_numpy(q.values(0)).to("cuda")
    a, b = factors(q, v), factors(q, v, dense_mfma=0)
    assert np.isfinite(a[0]).all() and np.array_equal(a[0], b[0]) and a[1] == b[1]


@pytest.mark.parametrize("prec", [K.FP64, K.FP32], ids=["fp64", "fp32"])
def test_batch_levels_of_many_items(prec):
    print(f"[gpu] batch with levels of over 16,384 narrow items, {prec}", flush=True)
    seqs = [kktgen.make_sequence(s) for s in BATCH]
    hs = [K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), factor_precision=prec).bind() for q in seqs]
    v = [torch.from_numpy(q.values(1)).to("cuda") for q in seqs]
    batch = K.KKTBatch(hs)
    for _ in range(2):
        batch.refactor(v)
    for sk, q, vi in zip(hs, seqs, v):
        ref = factors(q, vi, factor_precision=prec)
        assert np.array_equal(sk.export_factors()[0], ref[0]) and sk.refactor_status() == ref[1]
    batch.close()
