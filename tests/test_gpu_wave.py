"""Medium refactorization items on one wavefront against the vector-FMA path, through the C ABI.

With dense_mfma = 0 a level's medium items run in 256-thread blocks and their updates are chains
of fused multiply-adds in column order, starting from zero; the wavefront path runs the same
products on the matrix cores, whose FP64 and FP32 16x16x4 instructions add their four products
one by one in that order, each sum rounded.  Padding adds exact zeros.  The factors are
therefore equal bit for bit (up to the sign of a zero, which == does not tell).
"""
import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # one medium item per level, panels of 4 to 16 columns, single groups
    ("grid200", kktgen.config(0), {}),
    # several groups of a source, ragged row counts, odd panel widths, more than 16 targets
    ("grid1500_flows1", kktgen.small(1500, config_id=161, steps=2, avg_degree=2.7, flows=1), {}),
    # levels of over 16,384 narrow items beside medium ones, and of over 65,536 narrow ones
    ("grid36000", kktgen.small(36000, config_id=162, steps=1), {}),
    # sources and panels on both sides of the row limit
    ("grid600_tau1e-3", kktgen.small(600, config_id=163, steps=2), {"pivot_tau": 1e-3}),
    ("grid2000_fp32", kktgen.small(2000, config_id=164, steps=2), {"factor_precision": K.FP32}),
]


@pytest.mark.parametrize("name,spec,kw", CASES, ids=[c[0] for c in CASES])
def test_wavefront_items_equal_vector_path(name, spec, kw):
    print(f"[gpu] wavefront items {name}", flush=True)
    q = kktgen.make_sequence(spec)
    t = q.steps - 1
    v = torch.from_numpy(q.values(t)).to("cuda")
    lus = []
    for mfma in (1, 0):
        sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), dense_mfma=mfma, **kw).bind()
        for _ in range(2):
            sk.refactor(v)
        rc, pert = sk.refactor_status()
        lus.append((sk.export_factors()[0], rc, pert))
        sk.close()
    assert lus[0][1:] == lus[1][1:]
    assert np.isfinite(lus[0][0]).all()
    assert np.array_equal(lus[0][0], lus[1][0])


def test_wavefront_items_report_nonfinite():
    print("[gpu] wavefront items: a non-finite value", flush=True)
    q = kktgen.make_sequence(kktgen.small(800, config_id=165, steps=2))
    sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0)).bind()
    for bad in (np.inf, np.nan):
        v = q.values(1)
        v[q.nnz // 3] = bad
        sk.refactor(torch.from_numpy(v).to("cuda"))
        with pytest.raises(K.KKTError) as e:
            sk.refactor_status()
        assert e.value.code == K.ERR_NONFINITE
    sk.refactor(torch.from_numpy(q.values(1)).to("cuda"))
    assert sk.refactor_status()[0] in (K.OK, K.WARN_PIVOT_PERTURBED)
    sk.close()
