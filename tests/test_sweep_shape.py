"""The shapes chosen for sweeps of whole pencils (csrc/ppmlr_march.hpp, plain
functions of sizes) on the CPU: kernels exist for them, their chunks cover the
pencil, and grids of few pencils are not swept in chunks that only wait for each
other."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1607_02214_amd", "csrc")


def test_chosen_shapes(tmp_path):
    exe = str(tmp_path / "sweep_shape")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC,
                           os.path.join(HERE, "sweep_shape.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
