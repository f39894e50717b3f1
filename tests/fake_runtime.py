"""Runs the library's host code on the fake HIP runtime of tests/fake_hip.cpp, in a child process.

The child loads the fake runtime with global symbols before the library, so every HIP call of the
library comes to it; "device" memory is host memory there and launches run nothing. `check` runs a
body of Python in such a child, after a prelude with the library (mg), the fake runtime (F) and
helpers that make maps, trees and output arrays."""
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
import numpy as np
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
for f in ("fake_live", "fake_held"):
    getattr(F, f).restype = C.c_size_t
for f in ("fake_mallocs", "fake_frees", "fake_dirty", "fake_waits"):
    getattr(F, f).restype = C.c_int64
F.fake_last_block.restype = C.c_void_p
F.fake_limit.argtypes = [C.c_int, C.c_size_t]
F.fake_held.argtypes = [C.c_int, C.c_size_t]
F.fake_device_of.argtypes = [C.c_void_p]
from paper_2609_40297_amd import mg, workloads as W
L = mg.lib()
SENSOR = W.Sensor(n_az=64, n_el=8, fov_h_deg=90.0, fov_v_deg=60.0, range_m=9.0, yaw_bins=16)
MiB = 1 << 20

class Out:                      # an output array the library is given as device memory
    def __init__(self, n, dtype=np.uint32):
        self.a = np.zeros(n, dtype)
    def data_ptr(self):
        return self.a.ctypes.data

def new_map(dims=(40, 36, 20)):
    nx, ny, nz = dims
    return mg.mg_map_create(np.full((nz, ny, nx), W.UNK, np.uint8), 1.0, (0.0, 0.0, 0.0), stream=0)

def new_tree(m, n, sensor=SENSOR, star=False):
    i = np.arange(n)
    pos = np.stack([i % 19 + 0.5, i % 17 + 0.5, i % 13 + 0.5], 1).astype(np.float32)
    par = np.where(i == 0, -1, 0 if star else (i - 1) // 2).astype(np.int32)
    return mg.mg_tree_upload(m, pos, par, sensor, stream=0)

def code(fn, *a, **k):          # the MG_E_* code of a refused call, 0 of an accepted one
    try:
        fn(*a, **k)
    except mg.MGError as e:
        return e.code
    return mg.MG_OK
"""

_lib = None


def _build():
    global _lib
    if _lib is None:
        d = tempfile.mkdtemp(prefix="fake_hip_")
        out = os.path.join(d, "libfakehip.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", out],
                       check=True, timeout=120)
        _lib = out
    return _lib


def check(body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, _build()], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
