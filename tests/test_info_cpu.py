"""kkt_info of a batch's handle after the merged first solve (host code, built with g++): a solve
whose wait timed out is reported as a device error with an infinite backward error, never as
solved, and so is an error of the FGMRES steps that follow."""
import os
import shutil
import subprocess

import pytest

import paper_2302_08656_amd as K

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_info_after_the_first_solve(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "info")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", os.path.join(ROOT, "tests", "info_driver.cpp"), "-o", exe],
                   check=True)
    # abort, ||A||, ||r||, ||x||, ||b||, perturbed, target -> return, status, berr
    cases = [((1, 2.0, 0.0, 0.0, 0.0, 5, 1e-10), (K.ERR_DEVICE, K.ERR_DEVICE, "inf")),
             ((0, 2.0, 1e-12, 1.0, 1.0, 5, 1e-10), (K.OK, K.OK, 1e-12 / 3.0)),
             ((0, 2.0, 1.0, 1.0, 1.0, 0, 1e-10), (K.WARN_NOT_CONVERGED, K.OK, 1.0 / 3.0)),
             ((0, 2.0, 0.0, 0.0, 0.0, 0, 0.0), (K.OK, K.OK, 0.0)),
             ((0, 0.0, 1.0, 1.0, 0.0, 0, 1e-10), (K.WARN_NOT_CONVERGED, K.OK, "inf")),
             ((0, 2.0, "nan", 1.0, 1.0, 0, 1e-10), (K.WARN_NOT_CONVERGED, K.OK, "nan"))]
    text = "".join(" ".join(str(x) for x in c) + "\n" for c, _ in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    for k, (c, (rc, status, berr)) in enumerate(cases):
        got = out[2 * k].split()
        assert [int(got[0]), int(got[1]), int(got[2]), int(got[4])] == [rc, 0, status, c[5]], (c, got)
        assert got[3].lstrip("-") == berr if isinstance(berr, str) else float(got[3]) == berr, (c, got)
        after = out[2 * k + 1].split()
        assert int(after[0]) == K.ERR_DEVICE and after[1] == "inf" and int(after[2]) == (5 if c[0] else 3)
