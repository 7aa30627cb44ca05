"""Runs libfbp's host code in a child process over a HIP runtime of host memory (fake_hip.cpp).

`run(body)` executes `body` there with `fbp` (the package), `call` (an entry point of the C
ABI with a geometry and as many arguments, NULL stream; returns the status), `launched`
(kernel names and workgroups since the last reset) and `fake` (the runtime's controls), and
returns what it leaves in `result`.
"""
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_CHILD = """
import ctypes, json, re, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_kernel.restype = ctypes.c_char_p
fake.fake_blocks.restype = ctypes.c_longlong
fake.fake_allocated.restype = ctypes.c_size_t
fake.fake_fail_from.argtypes = [ctypes.c_size_t]
sys.path.insert(0, sys.argv[2])
import math
import numpy as np
import paper_2109_02174_amd as fbp
from paper_2109_02174_amd import _binding as B
lib = B.load()
A, C = 1 << 40, 1 << 44                      # device addresses that no launch touches

def call(name, g, *args):
    return getattr(lib, name)(ctypes.byref(g.as_c()), *args, None)

def launched():
    out = []
    for i in range(fake.fake_launches()):
        m = re.search(r"([a-z_0-9]+_kernel(?:_1)?)(I[A-Za-z0-9_]*?E)?E", fake.fake_kernel(i).decode())
        name = re.sub(r"^.*\\d+(?=[a-z])", "", m.group(1))
        values = [int(v) for v in re.findall(r"L[ib](\\d+)E", m.group(0))]
        out.append((name, values, fake.fake_blocks(i)))
    return out

result = None
"""


def run(body):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "libfakehip.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
        script = os.path.join(tmp, "child.py")
        with open(script, "w") as f:
            f.write(_CHILD + body + "\nprint('RESULT ' + json.dumps(result))\n")
        done = subprocess.run([sys.executable, script, so, ROOT], capture_output=True, text=True, timeout=300)
    lines = [l for l in done.stdout.splitlines() if l.startswith("RESULT ")]
    assert done.returncode == 0 and lines, done.stdout + done.stderr
    return json.loads(lines[-1][7:])
