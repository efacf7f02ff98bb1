"""Several right-hand sides solved by one launch against the columns solved one by one, through
the C ABI: every column runs the same items with the same arithmetic, so solutions and info are
equal bit for bit, whatever the number of columns (up to and past the most that one launch
takes), the stride, the precision and the restart length (whose basis holds the columns'
buffers; with a short one the columns go one by one)."""
import ctypes as C

import numpy as np
import pytest

import kktgen
import oracle
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


CASES = [
    ("grid200_2", kktgen.config(0), 2, {}),
    ("grid700_7", kktgen.small(700, config_id=171, steps=2), 7, {}),
    ("grid700_19", kktgen.small(700, config_id=171, steps=2), 19, {}),
    ("grid900_fp32_4", kktgen.small(900, config_id=172, steps=2), 4, {"factor_precision": K.FP32}),
    ("grid400_tau1e-3_3", kktgen.small(400, config_id=173, steps=2), 3, {"pivot_tau": 1e-3}),
    ("grid300_restart3_5", kktgen.small(300, config_id=174, steps=2), 5, {"gmres_restart": 3}),
    ("grid300_restart4_5", kktgen.small(300, config_id=174, steps=2), 5, {"gmres_restart": 4}),
    ("grid300_levels_3", kktgen.small(300, config_id=174, steps=2), 3, {"persistent_solve": 0}),
]


@pytest.mark.parametrize("name,spec,nrhs,kw", CASES, ids=[c[0] for c in CASES])
def test_columns_equal_single_columns(name, spec, nrhs, kw):
    print(f"[gpu] columns {name}", flush=True)
    q = kktgen.make_sequence(spec)
    t = q.steps - 1
    v, b = q.values(t), q.rhs(t, nrhs=nrhs)
    b[1] *= 1e3
    sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), **kw).bind(max_nrhs=nrhs)
    sk.refactor(cuda(v))
    bd = cuda(b)
    one = [sk.solve(bd[j].contiguous()) for j in range(nrhs)]
    ref = [sk.refine(bd[j].contiguous()) for j in range(nrhs)]
    many = sk.solve(bd)
    xs, infos = sk.refine(bd)
    for j in range(nrhs):
        assert torch.equal(many[j], one[j]), j
        assert torch.equal(xs[j], ref[j][0]), j
        assert infos[j] == ref[j][1][0], (j, infos[j], ref[j][1][0])
        _, berr = oracle.residual(q.n, q.rowptr, q.colind, v, xs[j].cpu().numpy(), b[j])
        assert infos[j].status == K.OK and berr <= 1e-10, (j, berr)
    # in place: the solutions overwrite the right-hand sides
    xi = bd.clone()
    sk.solve(xi, xi)
    assert torch.equal(xi, many)
    xi = bd.clone()
    _, inf2 = sk.refine(xi, xi)
    assert torch.equal(xi, xs) and inf2 == infos
    # a stride longer than a column
    ld = q.n + 5
    bs, x2 = torch.zeros(nrhs, ld, dtype=torch.float64, device="cuda"), torch.full((nrhs, ld), 7.0,
                                                                                  dtype=torch.float64, device="cuda")
    bs[:, :q.n] = bd
    rc = K._lib().kkt_solve(sk._h, C.c_void_p(bs.data_ptr()), C.c_void_p(x2.data_ptr()), nrhs, ld,
                            K._stream_ptr())
    assert rc == K.OK
    assert torch.equal(x2[:, :q.n], many) and bool((x2[:, q.n:] == 7.0).all())
    sk.close()
