"""The plans of the near / far split: an error that does not grow with the number
of ions, and blocks per brick within their range."""
import os
import subprocess

import numpy as np
import pytest

from tests.gpu_util import accel_errors, say

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("check", ["mesh_fit_check", "mesh_parts_check"])
def test_every_plan(tmp_path, check):
    exe = str(tmp_path / check)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-o", exe,
                           os.path.join(ROOT, "tests", check + ".cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout


@pytest.mark.gpu
def test_largest_split_within_the_direct_sums_error():
    """2^22 + 77 ions, sampled accelerations against the oracle.  The bound is
    the relative L2 error of the direct FP32 sum at 2^20 ions, 3.0e-7."""
    from oracle import oracle as O
    from paper_2205_06557_amd import binding as B
    from paper_2205_06557_amd import workloads as W
    w = W.single_grain_small()
    w = w.with_(n_ions=(1 << 22) + 77, R=3 * w.lam, H=6 * w.lam)
    with B.System(w) as s:
        o = O.Oracle(w, init=False)
        x, v, q, step = s.get_state()
        lam, cs, wpi = o.derived["lam"], o.derived["cs"], o.derived["wpi"]
        o.set_state(x.T.astype(np.float64) * lam, v.T.astype(np.float64) * cs, q, step)
        s.step(1)
        s.sync()
        a = s.accelerations().T.astype(np.float64)
        idx = np.sort(np.random.default_rng(1).choice(w.n_ions, 300, replace=False))
        l2, p999, top = accel_errors(a[idx], o.accel_subset(idx) / (lam * wpi * wpi))
        say("split, N", w.n_ions, ":", l2, p999, top)
        assert l2 < 3e-7
