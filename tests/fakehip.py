"""Runs a piece of Python in a child process whose HIP runtime is fake_hip.cpp:
the library's host side on the CPU, every allocation, copy and launch seen."""
from __future__ import annotations

import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C
import importlib.util
import numpy as np
import sys
sys.path.insert(0, {tests!r})
fake = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
fake.fake_name.restype = C.c_char_p
fake.fake_allocated.restype = fake.fake_copied.restype = fake.fake_stream.restype = C.c_int64
fake.fake_fill.argtypes = [C.c_double]
spec = importlib.util.spec_from_file_location("semlib_c", {lib!r})
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
lib = L.load()
from libhost import make_desc

def mesh(N, nel, **kw):
    d, keep = make_desc(L, N, nel, **kw)
    h = C.c_void_p()
    L.check(lib.sem_setup(C.byref(d), None, C.byref(h)), "sem_setup")
    info = L.MeshInfo()
    L.check(lib.sem_info(h, C.byref(info)), "sem_info")
    return h, info

def launches(part=""):
    return [i for i in range(fake.fake_launches()) if part in fake.fake_name(i).decode()]

def opts(**kw):
    o = L.SolveOpts()
    lib.sem_solve_opts_default(C.byref(o))
    for k, v in kw.items():
        setattr(o, k, v)
    return o
"""


def build(out_dir):
    """Compiles the runtime into out_dir and returns its path."""
    from paper_2109_03592_amd import build as B
    so = os.path.join(str(out_dir), "libfakehip.so")
    src = os.path.join(ROOT, "tests", "fake_hip.cpp")
    obj = so + ".o"
    subprocess.run([B.HIPCC, "-std=c++17", "-O1", "-fPIC", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip",
                    "-I", B.CSRC, "-c", src, "-o", obj], check=True)
    subprocess.run(["g++", "-shared", "-o", so, obj], check=True)
    return so


def run(so, code):
    """Runs code (after PRELUDE) in a child; returns what it printed."""
    lib = os.path.join(ROOT, "paper_2109_03592_amd", "_lib.py")
    text = PRELUDE.format(tests=os.path.join(ROOT, "tests"), so=so, lib=lib) + textwrap.dedent(code)
    r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout
