"""Solves with an infinite right-hand side entry (as an overflowing scaled one becomes): the level
launches, the persistent launches and the forward substitution inside the refactorization's
launches give the same infinities and NaNs, and the same finite unknowns bit for bit."""
import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("buses,cid", [(200, 195), (2500, 196)])
@pytest.mark.parametrize("fp32", [0, 1])
def test_infinite_right_hand_sides_agree_between_modes(buses, cid, fp32):
    print(f"[gpu] infinite right-hand sides, {buses} buses, fp32 {fp32}", flush=True)
    q = kktgen.make_sequence(kktgen.small(buses, config_id=cid, steps=2))
    kw = {"factor_precision": fp32, "max_iters": 0}
    pers, lev = (K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), persistent_solve=m, **kw).bind() for m in (1, 0))
    Q = pers.export_symbolic()["Q"]
    v = torch.from_numpy(q.values(1)).to("cuda")
    pers.refactor(v)
    lev.refactor(v)
    # an infinity at a column of the first levels, of the middle and of the last, and at two at once
    for at in ([Q[0]], [Q[q.n // 5]], [Q[q.n // 2]], [Q[-1]], [Q[7], Q[q.n // 3]]):
        b = np.zeros(q.n)
        b[at] = np.inf
        bd = torch.from_numpy(b).to("cuda")
        x = {"persistent": pers.solve(bd), "levels": lev.solve(bd)}
        for name, sk in (("step", pers), ("step, levels", lev)):
            x[name], info = sk.refactor_refine(v, bd)
            assert info.status == K.WARN_NOT_CONVERGED
        ref = x["persistent"].cpu().numpy()
        assert not np.isfinite(ref).all()
        for name, y in x.items():
            assert np.array_equal(ref, y.cpu().numpy(), equal_nan=True), (at, name)
    pers.close()
    lev.close()
