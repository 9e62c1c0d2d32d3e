"""The shape that the library chooses for a sweep of whole pencils, from the same
plain functions (csrc/ppmlr_march.hpp) compiled for the host.  Test
infrastructure only."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1607_02214_amd", "csrc")


@functools.lru_cache(maxsize=None)
def _lib():
    tmp = tempfile.mkdtemp()
    so = os.path.join(tmp, "sweep_plan.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, os.path.join(HERE, "sweep_plan.cpp"),
                           "-o", so])
    lib = C.CDLL(so)
    os.remove(so)
    os.rmdir(tmp)
    return lib


def plan(n, axis, elem, pencils=0, trace=0, learned=0, wrap=0):
    """(pencils, chunks, zones per chunk, LDS stride)"""
    out = (C.c_int * 4)()
    _lib().sweep_plan((C.c_int * 3)(*n), axis, elem, trace, learned, wrap, pencils, out)
    return tuple(out)
