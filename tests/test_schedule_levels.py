"""The kinds of levels that the GPU tests of the refactorization kernels mean to run, from the
schedule itself (host code, built with g++): medium items on wavefronts and in blocks, and levels
with more narrow items than the launch's variants switch at."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import kktgen

pytest.importorskip("torch")
import test_gpu_many_items as many  # noqa: E402
import test_gpu_wave as wave  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_08656_amd", "csrc")


def constant(name, path):
    return int(re.search(rf"constexpr int \w*{name} = (\d+);", open(os.path.join(CSRC, path)).read()).group(1))


MANY = constant("kManyItems", "kkt_runtime.hip")
TINY_MIN = constant("kTinyMinItems", "kkt_runtime.hip")
WAVE_ROWS = constant("kWaveRows", "kkt_internal.h")


@pytest.fixture(scope="module")
def levels(tmp_path_factory):
    """{wide, medium, narrow, tiny, wave, rows} of each level of a grid's schedule."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("schedule")
    exe = str(tmp / "levels")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "schedule_driver.cpp"),
                    os.path.join(CSRC, "kkt_symbolic.cpp"), os.path.join(CSRC, "kkt_schedule.cpp"), "-o", exe], check=True)

    def run(spec, tau=0.0):
        q = kktgen.make_sequence(spec)
        path = str(tmp / "m.in")
        with open(path, "wb") as f:
            f.write(np.int32(q.n).tobytes() + np.int64(q.nnz).tobytes() + np.float64(tau).tobytes())
            f.write(np.ascontiguousarray(q.rowptr, np.int64).tobytes())
            f.write(np.ascontiguousarray(q.colind, np.int32).tobytes())
            f.write(np.ascontiguousarray(q.values(0), np.float64).tobytes())
        out = subprocess.run([exe, path], capture_output=True, text=True, check=True, timeout=600).stdout
        return [dict(zip(("wide", "medium", "narrow", "tiny", "wave", "rows"), map(int, l.split())))
                for l in out.splitlines()]

    return run


@pytest.mark.parametrize("name,spec,kw", wave.CASES, ids=[c[0] for c in wave.CASES])
def test_wavefront_levels_of_the_wave_cases(levels, name, spec, kw):
    ls = levels(spec, kw.get("pivot_tau", 0.0))
    on_waves = [l for l in ls if l["wave"]]
    assert sum(l["medium"] for l in on_waves) >= 11
    for l in on_waves:
        assert l["wide"] == l["medium"] > 0 and l["rows"] <= WAVE_ROWS
    in_blocks = [l for l in ls if l["medium"] and not l["wave"]]
    for l in in_blocks:
        assert l["rows"] > WAVE_ROWS
    if kw.get("pivot_tau"):
        assert in_blocks and max(l["rows"] for l in on_waves) > 64   # rows past a wavefront's first 64
    if name == "grid36000":
        assert any(l["narrow"] >= MANY for l in on_waves) and any(l["narrow"] < MANY for l in on_waves)
        assert any(l["narrow"] >= TINY_MIN for l in ls if not l["wide"])


def test_tiny_items_beside_medium_ones(levels):
    ls = levels(many.LARGE)
    assert any(l["wave"] and l["narrow"] >= TINY_MIN and l["tiny"] > 0 and l["narrow"] > l["tiny"] for l in ls)


def test_batch_levels_of_many_items(levels):
    hs = [levels(s) for s in many.BATCH]
    found = []
    for l in range(max(map(len, hs))):
        at = [h[l] for h in hs if l < len(h)]
        if all(x["wave"] or not x["wide"] for x in at) and sum(x["narrow"] for x in at) >= MANY:
            found.append(sum(x["medium"] for x in at))
    assert any(found)   # with medium items beside the narrow ones
