"""The static scratch binding at its limit for dense triangular patterns, whose work items take most
room beside the factor: the largest that fit pass the size check, and bound there they give what
a caller's workspace gives, bit for bit, with the workspace reaching into the array's last part."""
import numpy as np
import pytest

import paper_2302_08656_amd as K

# order, factor precision; twenty rows more no longer fit
CASES = [(1030, K.FP64), (1070, K.FP32)]


def triangle(n):
    rows, cols = np.triu_indices(n)
    rowptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int64)
    rng = np.random.default_rng(11)
    vals = np.where(rows == cols, 4.0, rng.uniform(-1.0, 1.0, len(rows)) / n)
    return n, rowptr, cols.astype(np.int32), vals


def solver(n, prec):
    return K.KKTSolver(*triangle(n), factor_precision=prec, gmres_restart=1)


@pytest.mark.parametrize("n,prec", CASES)
def test_size_check(n, prec):
    fits, not_fits = solver(n, prec), solver(n + 20, prec)
    assert fits.workspace_bytes(1) > K.SCRATCH_BYTES + (4 << 20)
    # past the size check the call needs a device
    assert K._lib().kkt_bind_scratch(fits._h, 1, None) in (K.OK, K.ERR_DEVICE)
    assert K._lib().kkt_bind_scratch(not_fits._h, 1, None) == K.ERR_NOMEM


@pytest.mark.gpu
@pytest.mark.parametrize("n,prec", CASES)
def test_scratch_equals_workspace(n, prec):
    torch = pytest.importorskip("torch")
    print(f"[gpu] scratch binding at its limit, triangle of {n}", flush=True)
    v = torch.from_numpy(triangle(n)[3]).to("cuda")
    b = torch.from_numpy(np.random.default_rng(12).standard_normal(n)).to("cuda")
    out = []
    for scratch in (False, True):
        sk = solver(n, prec)
        sk.bind_scratch() if scratch else sk.bind()
        sk.refactor(v)
        x, info = sk.refine(b)
        out.append((*sk.export_factors(), x.cpu().numpy(), info[0]))
        sk.close()
    assert out[0][4] == out[1][4] and out[0][4].status == K.OK
    for a, c in zip(out[0][:4], out[1][:4]):
        assert np.array_equal(a, c)
