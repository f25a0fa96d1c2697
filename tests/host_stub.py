"""Runs a scenario against libfaco_hip.so with the HIP runtime replaced by
hip_host_stub.cpp (no GPU, kernels do not run), in a process of its own, and
returns what the scenario prints as JSON."""
import json
import os
import subprocess
import sys

import pytest

from paper_2203_02228_amd import faco as F

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "hip_host_stub.cpp")

PRELUDE = """
import ctypes, json, sys
import numpy as np
sys.modules["torch"] = None   # its HIP runtime stays out of this process
S = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
for f in ("stub_copies", "stub_news", "stub_events"):
    getattr(S, f).restype = ctypes.c_int64
from paper_2203_02228_amd import faco as F

def launches():
    out = []
    for i in range(S.stub_launch_count()):
        v = (ctypes.c_uint64 * 7)()
        S.stub_launch(i, v)
        out.append(dict(grid=list(v[0:3]), block=list(v[3:6]), lds=int(v[6])))
    return out

def build(n, ants=16, k=16, **kw):
    i = np.arange(n, dtype=np.int32)
    xy = np.stack([i * 31 % 4099, i], axis=1)
    return F.faco_build_instance(xy, n_ants=ants, cl_size=k, bl_size=4, **kw)
"""


def build_stub(folder):
    out = os.path.join(str(folder), "libhip_host_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", STUB, "-o", out], check=True)
    return out


def run(stub, body):
    if not os.path.exists(F.LIB_PATH):
        pytest.skip("HIP library not built")
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(stub=stub) + body], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])
