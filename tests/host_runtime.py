"""Runs libqsv's host runtime without a GPU, on the recorder of hip_stub.cpp.

`record(tmp, script)` runs the script in a process of its own, where libqsv's
HIP calls go to the recorder, with `stub` (the recorder's entry points),
`Context`, `W` (workloads) and `np` in scope, and returns the JSON value that
the script leaves in `result`."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
sys.modules["torch"] = None  # (it would bring the real runtime)
stub = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
for name in ("stub_count", "stub_stale_replays", "stub_pending", "stub_grid"):
    getattr(stub, name).restype = ctypes.c_long
stub.stub_grid.argtypes = [ctypes.c_long]
stub.stub_fail.argtypes = [ctypes.c_char_p, ctypes.c_long]
count = lambda name: stub.stub_count(name.encode())
import numpy as np
import workloads as W
from paper_2604_11599_amd import Context, QsvError, lower
"""


def record(tmp, script):
    so = os.path.join(str(tmp), "libhipstub.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-o", so, os.path.join(ROOT, "tests", "hip_stub.cpp")], check=True)
    code = _PRELUDE.format(root=ROOT, so=so) + script + "\nprint('RESULT ' + json.dumps(result), flush=True)\n"
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    lines = [x for x in r.stdout.splitlines() if x.startswith("RESULT ")]
    assert r.returncode == 0 and lines, r.stdout + r.stderr
    return json.loads(lines[-1][7:])
