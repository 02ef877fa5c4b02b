"""The library's planners and launch arithmetic, compiled for the host alone (plan_host.cpp with the sources they are in)."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_15667_amd", "csrc")


@functools.lru_cache(maxsize=None)
def lib():
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "plan_host.so")
        cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
               "-I" + os.path.join(ROOT, "include"), "-x", "c++", os.path.join(ROOT, "tests", "plan_host.cpp"),
               os.path.join(CSRC, "split_plan.hip"), os.path.join(CSRC, "tune.cpp"), "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout
        L = ctypes.CDLL(out)
    L.divide.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_uint, ctypes.c_void_p]
    L.divide.restype = None
    L.wino_split_beyond_range.restype = ctypes.c_longlong
    return L
