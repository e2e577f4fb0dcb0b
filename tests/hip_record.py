"""Host tests of the library's launches (imported by test modules): a child
process loads a HIP runtime that records launches instead of running them
(hip_record.cpp) in front of the real one, then the library, and runs the given
code.  Device pointers are never followed there, so any number serves as one."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, importlib.util, os, random, sys
sys.path.insert(0, {root!r})
import scenegen as sg
R = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
R.record_calls.restype = C.c_char_p
spec = importlib.util.spec_from_file_location("h4d_lib", os.path.join({root!r}, "paper_2505_13215_amd", "_lib.py"))
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
D = 1 << 40  # a device pointer
ctx = L.Context()

def calls(clear=True):
    got = [c.split() for c in R.record_calls().decode().splitlines()]
    if clear:
        R.record_clear()
    return got

def kernels(got):
    return [c[1] for c in got if c[0] == "launch"]

def cameras(n, W, H, same=False):
    return L.view_array([sg.look_at((0.01 * (0 if same else k), 0.0, -3.0), (0.0, 0.0, 0.0), W, H, t=0.1 + 0.02 * k)
                         for k in range(n)])

def sets(n3, n4):
    return L.G3D(n3, *[D] * 5), L.G4D(n4, *[D] * 7)

def render(n3, n4, views, n_views, cfg, entry="h4dgs_render_infer", scratch=None):
    g3, g4 = sets(n3, n4)
    st, sc = C.c_size_t(), C.c_size_t()
    ctx.check(ctx.L.h4dgs_workspace_size(ctx.h, n3, n4, views, n_views, C.byref(cfg), C.byref(st), C.byref(sc)))
    return getattr(ctx.L, entry)(ctx.h, C.byref(g3), C.byref(g4), views, n_views, C.byref(cfg),
                                 L.ptr_array([D] * n_views), C.c_void_p(D), st, C.c_void_p(D), sc, None)

def error():
    return ctx.L.h4dgs_last_error(ctx.h).decode()
"""


def build(directory: str) -> str:
    stub = os.path.join(directory, "libhip_record.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_record.cpp"), "-o", stub],
                   check=True, capture_output=True, timeout=300)
    return stub


def run(stub: str, code: str) -> str:
    """Output of ``code`` (after PRELUDE) in a process of its own."""
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, stub=stub) + textwrap.dedent(code)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
