"""The merged first solves of kkt_batch_refine against the handles refined alone: equal bit for
bit for FP64 and FP32 (whose FGMRES steps follow handle by handle), for a batch of one, with a
handle that solves in place (its right-hand side and solution are one array), and after a handle
was refactored alone; a handle with non-finite factors is reported while the others are solved."""
import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


SPECS = [kktgen.small(180, config_id=181, steps=3), kktgen.small(1700, config_id=182, steps=3),
         kktgen.small(820, config_id=183, steps=3, flows=1)]


def alone(q, v, b, **kw):
    sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), **kw).bind()
    sk.refactor(v)
    x, info = sk.refine(b)
    sk.close()
    return x, info[0]


@pytest.mark.parametrize("kw", [{}, {"factor_precision": K.FP32}, {"dense_mfma": 0}, {"persistent_solve": 0}],
                         ids=["fp64", "fp32", "vector", "levels"])
@pytest.mark.parametrize("count", [1, 3])
def test_merged_refine_equals_alone(kw, count):
    print(f"[gpu] merged refine {kw} {count}", flush=True)
    seqs = [kktgen.make_sequence(s) for s in SPECS[:count]]
    hs = [K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), **kw).bind() for q in seqs]
    batch = K.KKTBatch(hs)
    for t in range(2):
        v = [cuda(q.values(t)) for q in seqs]
        b = [cuda(q.rhs(t)) for q in seqs]
        ref = [alone(q, v[i], b[i], **kw) for i, q in enumerate(seqs)]
        batch.refactor(v)
        for rep in range(2):
            xs, infos = batch.refine(b)
            for i in range(count):
                assert torch.equal(xs[i], ref[i][0]) and infos[i] == ref[i][1], (t, rep, i)
        inplace = [x.clone() for x in b]
        xs, infos = batch.refine(inplace, inplace)
        for i in range(count):
            assert torch.equal(xs[i], ref[i][0]) and infos[i] == ref[i][1], (t, i)
    # one handle refactored alone since: its residual reads its own values
    v2 = cuda(seqs[0].values(2))
    hs[0].refactor(v2)
    xs, infos = batch.refine(b)
    x0, i0 = alone(seqs[0], v2, b[0], **kw)
    assert torch.equal(xs[0], x0) and infos[0] == i0
    for i in range(1, count):
        assert torch.equal(xs[i], ref[i][0]) and infos[i] == ref[i][1]
    batch.close()


def test_merged_refine_reports_a_bad_handle():
    print("[gpu] merged refine: non-finite values in one handle", flush=True)
    seqs = [kktgen.make_sequence(s) for s in SPECS]
    hs = [K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0)).bind() for q in seqs]
    batch = K.KKTBatch(hs)
    v = [cuda(q.values(1)) for q in seqs]
    b = [cuda(q.rhs(1)) for q in seqs]
    ref = [alone(q, v[i], b[i]) for i, q in enumerate(seqs)]
    bad = v[1].clone()
    bad[seqs[1].nnz // 2] = float("nan")
    batch.refactor([v[0], bad, v[2]])
    xs = [torch.full_like(x, 3.0) for x in b]
    with pytest.raises(K.KKTError) as e:
        batch.refine(b, xs)
    assert e.value.code == K.ERR_NONFINITE
    assert torch.equal(xs[0], ref[0][0]) and torch.equal(xs[2], ref[2][0]) and bool((xs[1] == 3.0).all())
    batch.refactor(v)
    xs, infos = batch.refine(b)
    for i in range(3):
        assert torch.equal(xs[i], ref[i][0]) and infos[i] == ref[i][1]
    batch.close()
