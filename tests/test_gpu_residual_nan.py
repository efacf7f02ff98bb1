"""A NaN in the right-hand side of one block of a block-diagonal system of more rows than one pass
of the residual's grid holds (4,096 blocks of 128 rows): the lane that meets the NaN goes on to a
finite row 524,288 further on, and the call must still report that column as not converged, on
every path that computes a residual."""
import numpy as np
import pytest

import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 524_288 + 40_000


def pairs(n):
    """2 x 2 blocks [[4, 1], [1, 3]] on the diagonal."""
    rowptr = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    colind = (np.arange(n, dtype=np.int32) // 2 * 2)[:, None] + np.array([0, 1], np.int32)
    vals = np.tile(np.array([4.0, 1.0, 1.0, 3.0]), n // 2)
    return rowptr, colind.ravel(), vals


def test_nan_of_an_early_block_is_reported():
    print("[gpu] residual: a NaN in an early row of 564,288", flush=True)
    rowptr, colind, vals = pairs(N)
    sk = K.KKTSolver(N, rowptr, colind, vals, gmres_restart=8).bind(max_nrhs=2)
    v = torch.from_numpy(vals).to("cuda")
    b = torch.ones(2, N, dtype=torch.float64, device="cuda")
    sk.refactor(v)
    for row in (0, 5, 39_999, 40_001, N - 1):
        bad = b.clone()
        bad[0, row] = float("nan")
        pair = slice(row // 2 * 2, row // 2 * 2 + 2)
        x, info = sk.refine(bad)                            # columns beside each other
        assert info[0].status == K.WARN_NOT_CONVERGED and info[1].status == K.OK, row
        assert bool(torch.isnan(x[0, pair]).all()) and bool(torch.isfinite(x[1]).all())
        x, info = sk.refine(bad[0].contiguous())            # one column
        assert info[0].status == K.WARN_NOT_CONVERGED, row
        x, info = sk.refactor_refine(v, bad[0].contiguous())
        assert info.status == K.WARN_NOT_CONVERGED, row
    batch = K.KKTBatch([sk])
    bad = b[0].clone()
    bad[3] = float("nan")
    batch.refactor([v])
    _, infos = batch.refine([bad])
    assert infos[0].status == K.WARN_NOT_CONVERGED
    x, infos = batch.refine([b[0].contiguous()])
    assert infos[0].status == K.OK and bool(torch.isfinite(x[0]).all())
    batch.close()
    sk.close()
