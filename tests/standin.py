"""libtlb over a stand-in HIP runtime (standin_hip.cpp), for tests of its host code without a GPU.

``run(body)`` executes ``body`` in a Python process of its own, which has loaded the stand-in before the library:
``hip`` is the stand-in, ``tlb`` the binding, ``kernels()`` the names of the launches recorded so far (cleared on
each call), ``buffers()`` their source and destination.  Returns the process's output.
"""
import os
import subprocess
import sys

TESTS = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(TESTS)

_HEAD = """
import ctypes, sys
sys.path.insert(0, {root!r})
hip = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
hip.standin_name.restype = ctypes.c_char_p
hip.standin_pointer.restype = ctypes.c_void_p
hip.standin_grid.restype = ctypes.c_uint32
hip.standin_cost.argtypes = [ctypes.c_char_p, ctypes.c_double]
import numpy as np
from paper_1511_02155_amd import tlb


def kernels(show=lambda i: hip.standin_name(i).decode().split("tlb::", 1)[1].replace("(anonymous namespace)::", "")):
    out = [show(i) for i in range(hip.standin_count())]
    hip.standin_clear()
    return out


def buffers():
    return kernels(lambda i: (hip.standin_pointer(i, 0), hip.standin_pointer(i, 1)))
"""


def build(folder):
    lib = os.path.join(str(folder), "standin_hip.so")
    if not os.path.exists(lib):
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", lib, os.path.join(TESTS, "standin_hip.cpp")],
                       check=True)
    return lib


def run(folder, body, env=None):
    code = _HEAD.format(root=ROOT, lib=build(folder)) + body
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, **(env or {})))
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
