"""No lane of a sweep workgroup reads or writes LDS outside what its launch
asks for: the shape rules and the slot arithmetic of the kernels
(csrc/ppmlr_march.hpp, plain functions of sizes) enumerated on the CPU, lanes
that only pad a workgroup to whole waves included."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1607_02214_amd", "csrc")


def test_every_lane_stays_inside_the_allocation(tmp_path):
    exe = str(tmp_path / "lds_layout")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "lds_layout.cpp"),
                           "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    marches, tiles = (int(line.split()[0]) for line in r.stdout.splitlines())
    assert marches > 1000 and tiles > 1000
