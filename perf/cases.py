"""The solver's work as a user's program has it done: steps of an interior-point sequence
(refactorization, triangular solves, refinement) on grids from 200 to 70,000 buses, solves
with kept factors, mixed precision, threshold pivoting, batches and serving.

A case names a grid (its pattern is fixed by the case), where in the interior-point sequence
the system lies (`progress`, 0 to 1: the diagonal D spreads from 10^+-2 to 10^+-10 on the way)
and the call.  The seed draws the values of the system and the right-hand sides.
"""
import dataclasses
import functools
import math

import numpy as np
import torch

import kktgen
import paper_2302_08656_amd as kkt

STEPS = 51   # systems of one sequence: progress p is system round(50 p)


def listed():
    step = {"call": "step", "degree": 2.5, "gens": 0.25, "schedule": "widening", "flows": 2, "progress": 0.5,
            "nrhs": 1, "fp32": False, "tau": 0.0, "systems": 1}

    def case(name, buses, **kw):
        return dict(step, name=name, buses=buses, **kw)

    return [
        # the smallest workload, 200 buses: latency and launches; a distribution-size study
        case("step_200", 200, degree=2.7, gens=0.20, schedule="fixed"),
        # an ordinary transmission grid, mid-sequence
        case("step_2000", 2_000, progress=0.3),
        # a regional interconnection near convergence (D spread over 10^+-9)
        case("step_10000", 10_000, progress=0.9),
        # the 25,000-bus-shaped grid, early in the sequence
        case("step_25000", 25_000, progress=0.1),
        # the headline 70,000-bus-shaped grid (N = 665,000)
        case("step_70000", 70_000),
        # KLU's pivot rule (tau = 1e-3): off-diagonal pivots, much fill, hundreds of levels
        case("step_pivoted_500", 500, tau=1e-3, progress=0.2),
        # FP32 factors with FP64 refinement: several FGMRES steps, each a pair of solves
        case("step_fp32_10000", 10_000, fp32=True, progress=0.5),
        # refactorization followed by the refinement of four right-hand sides (sensitivities)
        case("refine_4rhs_5000", 5_000, call="refine", nrhs=4, progress=0.6),
        # one more right-hand side with the factors at hand (a corrector step), small grid
        case("solve_1000", 1_000, call="solve", progress=0.4),
        # predictor and corrector right-hand sides with the factors at hand, large grid
        case("solve_2rhs_25000", 25_000, call="solve", nrhs=2, progress=0.7),
        # scenarios: sixteen systems of four patterns refactored together and refined
        case("batch_16", 1_700, call="batch", systems=16),
        # a burst of twelve requests over four patterns through the serving engine
        case("serve_12", 900, call="serve", systems=12, progress=0.4),
    ]


def draw(rng):
    """The same calls on other grids: sizes spread over their logarithm, ragged branch and
    generator counts, any place in the sequence."""
    call = rng.choice(["step", "step", "step", "step", "fp32", "pivoted", "refine", "solve", "batch", "serve"])
    lo, hi = {"step": (200, 60_000), "fp32": (200, 20_000), "pivoted": (150, 700), "refine": (200, 20_000),
              "solve": (200, 40_000), "batch": (400, 2_500), "serve": (300, 2_000)}[call]
    buses = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return {"call": call if call in ("refine", "solve", "batch", "serve") else "step", "buses": buses,
            "degree": round(rng.uniform(2.3, 2.8), 3), "gens": round(rng.uniform(0.15, 0.3), 3),
            "schedule": "widening", "flows": rng.choice([1, 2, 2]), "progress": round(rng.uniform(0.0, 1.0), 2),
            "nrhs": rng.randint(1, 4) if call in ("refine", "solve") else 1, "fp32": call == "fp32",
            "tau": 1e-3 if call == "pivoted" else 0.0,
            "systems": rng.randint(6, 16) if call in ("batch", "serve") else 1}


# ------------------------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=24)
def _grid(buses, degree, gens, schedule, flows, tau, fp32):
    """A grid's sequence and the sizes of its factors."""
    q = kktgen.make_sequence(kktgen.GridSpec(f"grid{buses}", 900, buses, degree, gens, STEPS, schedule, flows))
    sk = kkt.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), pivot_tau=tau, factor_precision=int(fp32))
    sizes = (sk.stats["nnz_lu"], sk.stats["flops_refactor"])
    sk.close()
    return q, sizes


def _grids(case):
    """The grids of a case: one, or for a batch or a server four of different sizes (half to
    one and a half times the named size apart)."""
    scale = (0.6, 1.0, 1.5, 2.2) if case["call"] in ("batch", "serve") else (1.0,)
    return [_grid(int(round(case["buses"] * f)), case["degree"], case["gens"], case["schedule"], case["flows"],
                  case["tau"], case["fp32"]) for f in scale]


def _systems(case):
    """(grid, right-hand sides) of each system of a pass: a batch takes the grids in turn; a
    server's requests lean to the small ones and bring one to four right-hand sides."""
    if case["call"] == "serve":
        order = (0, 1, 0, 2, 0, 1, 3, 0, 1, 2, 0, 3, 1, 0, 2, 0)
        return [(order[k], 1 + (k * 5) % 4 if k % 3 == 0 else 1) for k in range(case["systems"])]
    if case["call"] == "batch":
        return [(k % 4, 1) for k in range(case["systems"])]
    return [(0, case["nrhs"])]


def _host(case, seed):
    """(sequence, values, right-hand sides) of each system, on the host, from the seed."""
    t = int(round(case["progress"] * (STEPS - 1)))
    out = []
    for k, (g, nrhs) in enumerate(_systems(case)):
        q = _grids(case)[g][0]
        # the same grid with perturbations and right-hand sides of another stream
        own = dataclasses.replace(q, spec=dataclasses.replace(q.spec, config_id=1_000 + seed * 64 + k))
        out.append((q, own.values(t), np.ascontiguousarray(own.rhs(t, nrhs=nrhs))))
    return out


def prepare(case, seed):
    host = _host(case, seed)
    dev = torch.device("cuda", torch.cuda.current_device())
    st = {"call": case["call"], "v": [torch.from_numpy(v).to(dev) for _, v, _ in host],
          "b": [torch.from_numpy(b).to(dev) for _, _, b in host]}
    st["x"] = [torch.empty_like(b) for b in st["b"]]
    opts = {"pivot_tau": case["tau"], "factor_precision": int(case["fp32"])}

    def solver(q, nrhs=1):
        return kkt.KKTSolver(q.n, q.rowptr, q.colind, q.values(0), **opts).bind(max_nrhs=nrhs)

    if case["call"] == "serve":
        st["server"] = kkt.KKTServer(max_inflight=4, max_nrhs=4)
        ids = [st["server"].add_pattern(q.n, q.rowptr, q.colind, q.values(0), **opts) for q, _ in _grids(case)]
        st["pattern"] = [ids[g] for g, _ in _systems(case)]
    elif case["call"] == "batch":
        st["solvers"] = [solver(q) for q, _, _ in host]
        st["batch"] = kkt.KKTBatch(st["solvers"])
    else:
        st["solver"] = solver(host[0][0], case["nrhs"])
        if case["call"] == "solve":
            st["solver"].refactor(st["v"][0])
    torch.cuda.synchronize()
    return st


def _numbers(infos):
    return np.array([[i.iters, i.status, i.perturbed_pivots] for i in infos], dtype=np.int64)


def run(st):
    """One pass: the solutions, and the steps, status and replaced pivots that came with them."""
    if st["call"] == "step":
        x, info = st["solver"].refactor_refine(st["v"][0], st["b"][0], st["x"][0])
        return {"x": [x], "info": _numbers([info])}
    if st["call"] == "refine":
        st["solver"].refactor(st["v"][0])
        x, infos = st["solver"].refine(st["b"][0], st["x"][0])
        return {"x": [x], "info": _numbers(infos)}
    if st["call"] == "solve":
        return {"x": [st["solver"].solve(st["b"][0], st["x"][0])]}
    if st["call"] == "batch":
        st["batch"].refactor(st["v"])
        xs, infos = st["batch"].refine(st["b"], st["x"])
        return {"x": xs, "info": _numbers(infos)}
    sv = st["server"]
    tickets = [sv.submit(p, v, b, x) for p, v, b, x in zip(st["pattern"], st["v"], st["b"], st["x"])]
    infos = [i for t in tickets for i in sv.wait(t)[1]]
    return {"x": st["x"], "info": _numbers(infos)}


# ------------------------------------------------------------------------------- bounds

def work(case):
    """What one pass cannot do without.  A refactorization reads A (values and their slots, 12
    bytes an entry) and writes each factor entry once with its 4-byte index; a pair of
    triangular solves reads the factor once, with its indices, and four vectors; a refinement
    reads A once for the residual.  FGMRES steps are not counted: they depend on the values."""
    nbytes = flops = 0.0
    for g, nrhs in _systems(case):
        q, (nlu, ref_flops) = _grids(case)[g]
        fb = 4 if case["fp32"] else 8
        if case["call"] != "solve":
            nbytes += 12 * q.nnz + (fb + 4) * nlu + 16 * q.n + nrhs * (12 * q.nnz + 28 * q.n)
            flops += ref_flops + nrhs * 2 * q.nnz
        nbytes += nrhs * ((fb + 4) * nlu + 48 * q.n)
        flops += nrhs * 2 * nlu
    return {"bytes": nbytes, "flops": flops}


EXACT_CPU, EXACT_GPU = 5_000, 20_000   # orders up to which a dense solve is quick


def exact(case, seed):
    """The solutions by a dense LU in 64 bits, refined with residuals in extended precision
    until they stand still.  None for the large systems, whose dense matrix is too much."""
    host = _host(case, seed)
    if max(q.n for q, _, _ in host) > (EXACT_GPU if len(host) == 1 else EXACT_CPU):
        return None
    xs = []
    for q, v, b in host:
        rows = np.repeat(np.arange(q.n), np.diff(q.rowptr))
        top = np.maximum.reduceat(np.abs(v), q.rowptr[:-1])
        r = np.exp2(-np.floor(np.log2(np.where(top > 0, top, 1.0))))
        side = np.zeros(q.n)
        np.maximum.at(side, q.colind, np.abs(v) * r[rows])
        c = np.exp2(-np.floor(np.log2(np.where(side > 0, side, 1.0))))
        dev = "cpu" if q.n <= EXACT_CPU else "cuda"
        A = torch.zeros(q.n, q.n, dtype=torch.float64, device=dev)
        A[torch.from_numpy(rows).to(dev), torch.from_numpy(q.colind.astype(np.int64)).to(dev)] = \
            torch.from_numpy(v * r[rows] * c[q.colind]).to(dev)
        lu, piv = torch.linalg.lu_factor(A)
        del A
        cols = np.atleast_2d(b)
        x = np.zeros(cols.shape, np.longdouble)
        for _ in range(8):
            Ax = np.stack([np.add.reduceat(v.astype(np.longdouble) * xi[q.colind], q.rowptr[:-1]) for xi in x])
            rhs = ((cols - Ax).astype(np.float64) * r).T
            d = torch.linalg.lu_solve(lu, piv, torch.from_numpy(np.ascontiguousarray(rhs)).to(dev)).cpu().numpy().T
            x = x + d * c
        xs.append(x.astype(np.float64).reshape(b.shape))
    return {"x": xs, "info": None} if case["call"] != "solve" else {"x": xs}
