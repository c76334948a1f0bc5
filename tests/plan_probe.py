"""The launch plan of the 16-bit attention path, from the library's own header compiled for the host."""

import ctypes as C
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
Plan = namedtuple("Plan", "wide nrb groups n_rg nsplit units slots total grid_ok")


@functools.lru_cache(maxsize=None)
def _probe():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan_probe.so")
        subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2502_11101_amd", "csrc"), os.path.join(ROOT, "tests", "plan_probe.cpp"), "-o", so],
                       check=True, timeout=120)
        f = C.CDLL(so).probe_plan
    f.argtypes = [C.c_int] * 5 + [C.c_int64, C.c_size_t, C.POINTER(C.c_int64)]
    f.restype = None
    return f


def plan(hq, hkv, batch, tq, stride, max_kv, given=2 ** 63):
    out = (C.c_int64 * 9)()
    _probe()(hq, hkv, batch, tq, stride, max_kv, given, out)
    return Plan(*out)
