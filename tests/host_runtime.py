"""Runs a Python snippet in a process of its own where libcgconv.so finds the
stand-ins of tests/fake_hip.cpp in place of the HIP runtime (no GPU): plans
are created and entry points called, kernel launches are only recorded.

The snippet sees ``P`` (the package), ``ptr(i)`` (distinct aligned addresses
that are never read) and ``launches()``: (grid, block, LDS bytes, allowed LDS
bytes) of each kernel launched since the last call.
"""

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_hip_launches.restype = ctypes.c_int64
import paper_2509_24093_amd as P
P.library()

def ptr(i):
    return 0x100000 * (i + 1)

def launches():
    buf = (ctypes.c_int64 * (8 * 64))()
    n = fake.fake_hip_launches(buf, ctypes.c_int64(64))
    rows = [list(buf[8 * i:8 * i + 8]) for i in range(n)]
    return [(tuple(r[:3]), tuple(r[3:6]), r[6], r[7]) for r in rows]
"""


def run(tmp_path, code):
    so = str(tmp_path / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE + code, so], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout
