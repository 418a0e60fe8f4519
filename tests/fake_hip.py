"""Run a piece of Python on the library with its HIP runtime replaced by
fake_hip.c (no GPU: launches are recorded, not run).  ``run(code)`` executes
``code`` in a process of its own, in which ``lbm`` is the binding, ``np`` is
numpy, ``hip`` this stand-in, and what the code stores in ``out`` comes back.
"""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
sys.modules["torch"] = None  # it brings a HIP runtime of its own
hip = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
import numpy as np
from paper_1608_06345_amd import lbm

class _Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32),
                ("block", ctypes.c_uint32), ("ticks", ctypes.c_int)]
hip.fake_launch.restype = ctypes.POINTER(_Launch)
hip.fake_live_bytes.restype = ctypes.c_size_t

def launches():
    return [hip.fake_launch(i).contents for i in range(hip.fake_launches())]

out = None
"""


def run(code, tmp_path):
    lib = os.path.join(str(tmp_path), "libfakehip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-w",
                           os.path.join(ROOT, "tests", "fake_hip.c"), "-o", lib])
    script = _PRELUDE.format(root=ROOT, lib=lib) + code + "\nprint('OUT ' + json.dumps(out))\n"
    r = subprocess.run([sys.executable, "-c", script], stdout=subprocess.PIPE,
                       stderr=subprocess.PIPE, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return json.loads([l for l in r.stdout.splitlines() if l.startswith("OUT ")][-1][4:])
