"""Every zone belongs to one wave of the signal-speed kernels and the columns of
a few long rows are spread over the waves (csrc/ppmlr_rows.hpp, plain functions
of sizes, on the CPU); the time step of such grids against the oracle."""
import os
import subprocess

import numpy as np
import pytest

import gpu_cases as GC
from paper_1607_02214_amd import inputs as I

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1607_02214_amd", "csrc")


def test_every_zone_once_and_no_long_chain(tmp_path):
    exe = str(tmp_path / "row_split")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "row_split.cpp"),
                           "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and int(r.stdout.split()[0]) > 500, r.stdout + r.stderr


# few rows of many columns, the last one short or whole; 1e-12 as the other
# comparisons of the same 64-bit arithmetic in another order
@pytest.mark.gpu
@pytest.mark.parametrize("n", [(1000, 1, 1), (4033, 2, 1), (300, 3, 2), (129, 7, 5), (2, 1, 1), (1, 300, 3)])
def test_time_step_on_few_long_rows(n):
    import torch
    rng = np.random.default_rng(n[0])
    faces = [np.concatenate([[0.0], np.cumsum(rng.uniform(0.7, 1.3, k))]) for k in n]
    case = GC.Case("smooth", [f / f[-1] for f in faces], I.random_smooth_state(n[::-1], seed=n[0]))
    for at in (0, n[0] // 2, n[0] - 1):         # the zone that decides, at both ends and inside
        U = case.U.copy()
        U[7, -1, 0, at] *= 50.0
        for dtype in (torch.float64, torch.float32):
            u = torch.from_numpy(U).to("cuda", dtype).contiguous()
            want = case.oracle().cfl_dt(u.double().cpu().numpy(), 0.4)
            assert abs(case.context().cfl_dt(u, 0.4) - want) <= 1e-12 * want
