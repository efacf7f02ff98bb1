"""The limit of the static scratch binding for triangular patterns, whose item records are a
large part of the workspace: one that fits without the first pair's record in each item passes
the size check although its workspace exceeds the limit, the next size is refused."""
import numpy as np
import pytest

import paper_2302_08656_amd as K


@pytest.mark.parametrize("n,fits", [(1500, True), (1520, False)])
def test_triangular_pattern_at_the_limit(n, fits):
    a = np.triu(np.random.default_rng(3).random((n, n)) < 0.2)
    a[np.arange(n), np.arange(n)] = True
    rows, cols = np.nonzero(a)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    sk = K.KKTSolver(n, rowptr, cols.astype(np.int32), np.where(rows == cols, float(n), 1.0))
    assert K.SCRATCH_BYTES < sk.workspace_bytes(1) < K.SCRATCH_BYTES + (4 << 20)
    # past the size check the call needs a device
    rc = K._lib().kkt_bind_scratch(sk._h, 1, None)
    assert (rc != K.ERR_NOMEM) if fits else (rc == K.ERR_NOMEM)
