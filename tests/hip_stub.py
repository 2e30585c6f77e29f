"""Runs a piece of Python against librid.so with the HIP runtime replaced by
tests/hip_stub.cpp (no GPU): `L` is the library with its argument types, `stub`
the replacement, and a few helpers make handles and buffers."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
import numpy as np
sys.path.insert(0, {root!r})
import paper_2408_14070_amd as rid
import ridgen
L = rid.lib()
stub = ctypes.CDLL({so!r})
stub.stub_take_log.restype = ctypes.c_char_p
vp = ctypes.c_void_p

def launched():
    return stub.stub_take_log().decode().split()

def ptr(a):
    return a.ctypes.data_as(vp)

def ensemble(n, widths, K, prec):
    w = np.array(widths, np.int32)
    p = ridgen.xavier_ensemble(2 * n, list(widths), K, 1)
    h = vp()
    assert L.rid_ensemble_create(n, K, len(w), ptr(w), prec, ptr(p), ctypes.byref(h)) == 0
    launched()
    return h

def system(spec):
    q = np.ascontiguousarray(spec.quads, np.int32)
    h = vp()
    assert L.rid_system_create(spec.n_atoms, spec.n_cv, ptr(q), None, ctypes.byref(h)) == 0
    return h
"""


def build(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path / "hip_stub.so")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", so], check=True)
    return so


def run(tmp_path, body):
    so = build(tmp_path)
    env = dict(os.environ, LD_PRELOAD=so)
    r = subprocess.run([sys.executable, "-c",
                        PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(body)],
                       capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
