"""A batch with a handle that was retuned and bound to the same address again: the batch's tables
describe the old layout of that workspace, so kkt_batch_refactor returns STATE and
kkt_batch_refine gives what the handles give alone.  A handle bound to the same address again
with its schedule unchanged stays in the batch."""
import ctypes as C

import numpy as np
import pytest

import kktgen
import paper_2302_08656_amd as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OTHER = {"panel_max": 8, "small_rows": 32, "group": 16}


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def bind_at(sk, ws):
    """kkt_bind to the caller's buffer ws (as a caller with one workspace does)."""
    base = ws.data_ptr() + (-ws.data_ptr()) % 256
    need = sk.workspace_bytes(1)
    assert need <= ws.numel() - 256
    rc = K._lib().kkt_bind(sk._h, C.c_void_p(base), need, 1, K._stream_ptr())
    assert rc == K.OK
    sk._ws, sk.device = ws, ws.device


@pytest.mark.parametrize("fp32", [0, 1])
def test_retuned_handle_leaves_the_merged_path(fp32):
    print(f"[gpu] batch with a retuned handle, fp32 {fp32}", flush=True)
    seqs = [kktgen.make_sequence(s) for s in (kktgen.small(700, config_id=191, steps=2),
                                              kktgen.small(300, config_id=192, steps=2))]
    hs = [K.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), factor_precision=fp32) for q in seqs]
    sizes = [sk.workspace_bytes(1) for sk in hs]
    tuned = K.KKTSolver(seqs[0].n, seqs[0].rowptr, seqs[0].colind, seqs[0].values(0), factor_precision=fp32)
    tuned.set_tuning(**OTHER)
    assert tuned.workspace_bytes(1) != sizes[0]   # another layout
    sizes[0] = max(sizes[0], tuned.workspace_bytes(1))
    buf = [torch.empty(s + 512, dtype=torch.uint8, device="cuda") for s in sizes]
    for sk, ws in zip(hs, buf):
        bind_at(sk, ws)
    batch = K.KKTBatch(hs)
    v, b = [cuda(q.values(1)) for q in seqs], [cuda(q.rhs(1)) for q in seqs]
    batch.refactor(v)
    first = batch.refine(b)
    # bound to the same address again, schedule unchanged: the tables hold
    bind_at(hs[0], buf[0])
    batch.refactor(v)
    again = batch.refine(b)
    for i in range(2):
        assert torch.equal(first[0][i], again[0][i]) and first[1][i] == again[1][i]
    # retuned and bound to the same address
    hs[0].set_tuning(**OTHER)
    bind_at(hs[0], buf[0])
    with pytest.raises(K.KKTError) as e:
        batch.refactor(v)
    assert e.value.code == K.ERR_STATE
    for sk, vi in zip(hs, v):
        sk.refactor(vi)
    xs, infos = batch.refine(b)
    tuned.bind()
    tuned.refactor(v[0])
    x0, i0 = tuned.refine(b[0])
    assert torch.equal(xs[0], x0) and infos[0] == i0[0]
    assert torch.equal(xs[1], first[0][1]) and infos[1] == first[1][1]
    batch.close()
