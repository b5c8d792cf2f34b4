"""Runs the library's host code on the stub HIP runtime of hip_stub.c: kernels do
nothing, allocations and launches can be refused, and what the library asks the
runtime to do is logged.  In a process of its own, since the stub takes the
runtime's place for the whole process."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, os, sys
import numpy as np
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
from paper_2312_07010_amd import ace
L = ace.lib()

def log(clear=True):
    lines = stub.stub_log().decode().splitlines()
    if clear:
        stub.stub_clear()
    return lines

def solver(d, M, bc, dt=1e-3, kappa=0.05):
    N = [m + (-2, 1, 0)[bc] for m in M]
    return ace.Solver(d, N, [0.0] * d, [float(n) for n in N], (kappa / dt) ** 0.5, dt, bc)

def batch(sizes):
    insts = []
    for M, bc in sizes:
        N = [m + (-2, 1, 0)[bc] for m in M]
        insts.append((len(M), N, [0.0] * len(M), [float(n) for n in N], 7.0, 1e-3, bc))
    return ace.Batch(insts)
"""


def run(tmp_path, code):
    """Executes `code` (after the prelude: ace, L, stub, log(), solver(), batch()) and fails on any error."""
    lib = os.path.join(str(tmp_path), "hip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-o", lib, os.path.join(HERE, "hip_stub.c")], check=True)
    src = PRELUDE.format(root=ROOT, lib=lib) + textwrap.dedent(code)
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
