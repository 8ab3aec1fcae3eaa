"""The library's host code on the stand-in runtime of host_runtime.cpp: a child
process with the stand-in (rt) loaded before librt.so runs the given statements."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
rt = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
rt.host_launches.restype = rt.host_live.restype = ctypes.c_longlong
rt.host_largest.restype = ctypes.c_ulonglong
rt.host_fail_launch.argtypes = [ctypes.c_longlong]
rt.host_limit.argtypes = [ctypes.c_ulonglong]
import numpy as np
from paper_2110_11873_amd import binding as B, workloads as W
def launches(f):
    n = rt.host_launches()
    f()
    return rt.host_launches() - n
def fails(f):
    try:
        f()
    except B.RTError as e:
        return e.code
    raise SystemExit("no error")
"""


def build(folder):
    so = os.path.join(str(folder), "host_runtime.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host_runtime.cpp"), "-o", so], check=True)
    return so


def run(so, statements):
    lib = os.path.join(ROOT, "paper_2110_11873_amd", "librt.so")
    if not os.path.exists(lib):
        pytest.skip("librt.so is not built")
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + statements], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
