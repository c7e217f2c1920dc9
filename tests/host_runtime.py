"""libqd's host side on a machine without a GPU: tests run their script in a process of its own, where
hip_host.cpp answers the HIP calls (kernels are recorded, not run)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PRELUDE = """
import ctypes, sys
sys.path[:0] = [{root!r}, {here!r}]
hip = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)     # found before the runtime that libqd is linked with
for f in ("host_held", "host_peak", "host_made", "host_waits"):
    getattr(hip, f).restype = ctypes.c_longlong
hip.host_limit.argtypes = [ctypes.c_int, ctypes.c_longlong]
hip.host_launch.restype = ctypes.c_char_p
DEVICE, PINNED = 0, 1
def launches():
    out = []
    for i in range(hip.host_launches()):
        g, b, l = ctypes.c_uint32(), ctypes.c_uint32(), ctypes.c_uint64()
        n = hip.host_launch(i, ctypes.byref(g), ctypes.byref(b), ctypes.byref(l)).decode()
        out.append((n, g.value, b.value, l.value))
    return out
import numpy as np
import paper_2211_07918_amd as Q
"""


@pytest.fixture(scope="session")
def host_runtime(tmp_path_factory):
    """run(script): its output; the script has hip (the host_* calls), launches(), np and Q."""
    lib = str(tmp_path_factory.mktemp("hip") / "libhip_host.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_host.cpp"), "-o", lib], check=True)

    def run(script):
        src = PRELUDE.format(root=os.path.dirname(HERE), here=HERE, lib=lib) + script
        r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout
    return run
