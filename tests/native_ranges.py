"""The library's scoring-range arithmetic, compiled for the host from its own
header (tests/native/ranges.cpp), for the tests without a GPU."""
from __future__ import annotations

import ctypes
import functools
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@functools.lru_cache(maxsize=None)
def lib() -> ctypes.CDLL:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    out = os.path.join(ROOT, "_build", "ranges.so")
    os.makedirs(os.path.dirname(out), exist_ok=True)
    tmp = f"{out}.tmp{os.getpid()}"
    r = subprocess.run(
        [hipcc, "-x", "hip", "-O1", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         f"-I{os.path.join(ROOT, 'include')}",
         f"-I{os.path.join(ROOT, 'paper_2607_26475_amd', 'csrc')}",
         os.path.join(HERE, "native", "ranges.cpp"), "-o", tmp],
        capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    os.replace(tmp, out)
    so = ctypes.CDLL(out)
    for name in ("t_groups_of", "t_range_groups"):
        getattr(so, name).restype = ctypes.c_uint32
    so.t_min_range_groups.argtypes = [ctypes.c_int64, ctypes.c_int]
    so.t_added_min_range.argtypes = [ctypes.c_int64]
    so.t_slots_fit.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    for name in ("t_range_of", "t_unit_ranges"):
        a = [ctypes.c_int if name == "t_range_of" else ctypes.c_uint32, ctypes.c_uint32,
             ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
        getattr(so, name).argtypes, getattr(so, name).restype = a, None
    return so


def pair(fn, *args):
    out = (ctypes.c_uint32 * 2)()
    fn(*args, out)
    return int(out[0]), int(out[1])
