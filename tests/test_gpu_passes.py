"""The passes over the matrix around a step at row and column lengths on both sides of their
batches (8, 16 and 24 entries of a row; 32 and 160 slots of a column): the scaled values and
the factor through the solution, the norm of A and the residual's norms through the backward
error, for one recorded step against the same calls one by one and against the oracle.

The single-precision factor without refinement leaves a backward error of about 1e-8, so that
the residual's rounding hardly shows in it: computed in two orders it differs by at most
2 (L + 2) u (L the longest row, u = 2^-53), as an absolute bound on the backward error, and
the norm of A by (L + 2) u relatively."""
import numpy as np
import pytest

import oracle
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 63, 64, 65, 159, 160, 161, 287, 288, 289]


def bordered(n, seed):
    """a diagonal matrix bordered by rows (and columns) with the given numbers of entries"""
    rng = np.random.default_rng(seed)
    a = np.zeros((n, n))
    a[np.arange(n), np.arange(n)] = rng.uniform(1.0, 2.0, n)
    h0 = n - len(LENGTHS)
    for k, m in enumerate(LENGTHS):
        at = rng.choice(h0, m - 1, replace=False)
        a[h0 + k, at] = rng.uniform(-1.0, 1.0, m - 1) / m
        a[at, h0 + k] = rng.uniform(-1.0, 1.0, m - 1) / m
    rows, cols = np.nonzero(a)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    return rowptr, cols.astype(np.int32), a[rows, cols]


@pytest.mark.parametrize("n", [311, 640])
@pytest.mark.parametrize("prec", [K.FP64, K.FP32])
def test_step_equals_separate_calls(n, prec):
    print(f"[gpu] passes n={n} precision={prec}", flush=True)
    rowptr, colind, v = bordered(n, n)
    rng = np.random.default_rng(n + 1)
    b = rng.standard_normal(n)
    sk = K.KKTSolver(n, rowptr, colind, v, factor_precision=prec, max_iters=0).bind()
    vd, bd = torch.from_numpy(v).cuda(), torch.from_numpy(b).cuda()
    sk.refactor(vd)
    x1, info1 = sk.refine(bd)
    longest = int(np.diff(rowptr).max())
    bound = 2 * (longest + 2) * 2.0 ** -53
    for _ in range(3):
        x2, info2 = sk.refactor_refine(vd, bd)
        assert torch.equal(x1.reshape(-1), x2.reshape(-1))
        i1, i2 = (i[0] if isinstance(i, (list, tuple)) else i for i in (info1, info2))
        assert (i1.status, i1.berr, i1.perturbed_pivots) == (i2.status, i2.berr, i2.perturbed_pivots)
    x = x2.reshape(-1).cpu().numpy()
    _, berr = oracle.residual(n, rowptr, colind, v, x, b)
    assert abs(i2.berr - berr) <= bound + berr * bound, (i2.berr, berr, bound)
    # LU of a matrix with little growth: a small multiple of n unit roundoffs of the factor
    assert berr <= 8 * n * (2.0 ** -53 if prec == K.FP64 else 2.0 ** -24)
    if prec == K.FP32:
        assert berr > 1e-10
