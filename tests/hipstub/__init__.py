"""Runs a script against libsmx.so on the CPU, with hipstub.cpp in the place of the HIP runtime."""

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

PRELUDE = """
import ctypes, sys
import numpy as np
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
import paper_2004_10811_amd as smx
smx._share_torch_hip_runtime = lambda: None
from waterbox import random_block_system, water_config
NEVER = 1 << 30


def launches(prefix=""):
    \"\"\"(kernel, grid) of the launches since the last call.\"\"\"
    rows = [ln.rsplit(" ", 1) for ln in stub.stub_log().decode().splitlines()]
    stub.stub_clear_log()
    return [(k, int(g)) for k, g in rows if k.startswith(prefix)]

"""


def build(folder):
    lib = os.path.join(str(folder), "libhipstub.so")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2004_10811_amd", "csrc"),
                    os.path.join(HERE, "hipstub.cpp"), "-o", lib], check=True, capture_output=True, text=True)
    return lib


def run(lib, script):
    """The script in a process of its own; what it prints."""
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=lib) + script], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
