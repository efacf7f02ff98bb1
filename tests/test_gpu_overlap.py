"""Several right-hand sides whose solutions overlap them: every layout gives what one call per
column, one after the other, gives on the same memory (column j's right-hand side may lie where
an earlier solution was written, and is then that solution).  FP32 factors, whose first solves
miss the target, so that the residuals and FGMRES steps of every column count."""
import ctypes as C

import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NRHS = 4
# name: (stride, distance of x from b), in units of n and of entries
LAYOUTS = {"in_place": (1, 0, 0), "over_previous": (1, -1, 0), "over_next": (1, 1, 0), "over_next_but_one": (1, 2, 0),
           "over_previous_strided": (2, -2, 0), "interleaved": (2, 1, 0), "shifted_3": (1, 0, 3),
           "shifted_back_3": (1, 0, -3)}


def call(sk, fn, buf, b, x, nrhs, ld):
    at = [C.c_void_p(buf.data_ptr() + 8 * o) for o in (b, x)]
    if fn == "solve":
        assert K._lib().kkt_solve(sk._h, *at, nrhs, ld, K._stream_ptr()) == K.OK
        return []
    info = (K._Info * nrhs)()
    rc = K._lib().kkt_refine(sk._h, *at, nrhs, ld, info, K._stream_ptr())
    assert rc >= 0
    return [(i.iters, i.status, i.berr, i.perturbed_pivots) for i in info]


# a right-hand side partly under its own solution (shifted) has no residual to refine with
@pytest.mark.parametrize("fn,layout", [("solve", l) for l in LAYOUTS] +
                         [("refine", l) for l in LAYOUTS if not l.startswith("shifted")])
def test_overlapping_columns(fn, layout):
    print(f"[gpu] overlapping columns {fn} {layout}", flush=True)
    q = kktgen.make_sequence(kktgen.small(350, config_id=197, steps=3))
    sk = K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), factor_precision=K.FP32).bind(max_nrhs=NRHS)
    sk.refactor(torch.from_numpy(q.values(0)).to("cuda"))
    stride, cols, off = LAYOUTS[layout]
    ld, b0 = stride * q.n, 3 * q.n
    x0 = b0 + cols * q.n + off
    host = np.zeros(b0 + NRHS * ld + 4 * q.n)
    for j in range(NRHS):
        host[b0 + j * ld:b0 + j * ld + q.n] = q.rhs(0, nrhs=NRHS)[j]
    one, many = (torch.from_numpy(host).to("cuda") for _ in range(2))
    infos = [i for j in range(NRHS) for i in call(sk, fn, one, b0 + j * ld, x0 + j * ld, 1, ld)]
    if fn == "refine":
        assert infos[0][0] > 0 and infos[0][1] == K.OK   # FGMRES steps run
    got = call(sk, fn, many, b0, x0, NRHS, ld)
    assert got == infos
    assert torch.equal(one, many)
    sk.close()


def test_batch_arrays_beside_each_other():
    """One right-hand side for two handles, their solutions end to end in one array."""
    print("[gpu] batch with adjacent arrays", flush=True)
    q = kktgen.make_sequence(kktgen.small(350, config_id=197, steps=3))
    hs = [K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), factor_precision=K.FP32).bind() for _ in range(2)]
    batch = K.KKTBatch(hs)
    v = torch.from_numpy(q.values(0)).to("cuda")
    b = torch.from_numpy(q.rhs(0)).to("cuda")
    batch.refactor([v, v])
    ref, _ = hs[0].refine(b)
    both = torch.empty(2 * q.n, dtype=torch.float64, device="cuda")
    xs, infos = batch.refine([b, b], [both[:q.n], both[q.n:]])
    assert torch.equal(xs[0], ref) and torch.equal(xs[1], ref) and infos[0].iters == infos[1].iters > 0
    batch.close()
