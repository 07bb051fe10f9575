"""libps.so over a HIP runtime that only records (fake_hip.c): the host code's
choices of kernels, launches, graphs and tuned settings, without a GPU.

run(body) executes Python source in a child process (the runtime's symbols are
global there, so no other HIP user may share it) with these names: L (libps.so),
F (the runtime's controls), plan(...), step(...), launches(), check(status).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes as c, sys
F = c.CDLL(sys.argv[1], mode=c.RTLD_GLOBAL)
L = c.CDLL(sys.argv[2])
L.ps_last_error.restype = c.c_char_p
L.ps_plan_workspace_bytes.restype = c.c_size_t
L.ps_rk2_step.argtypes = [c.c_void_p, c.c_void_p, c.c_int, c.c_double, c.c_double, c.c_double, c.c_int]
for f in ("ps_plan_workspace_bytes", "ps_plan_destroy"):
    getattr(L, f).argtypes = [c.c_void_p]
L.ps_plan_set_workspace.argtypes = [c.c_void_p, c.c_void_p, c.c_size_t]
for f in ("ps_plan_set_variant", "ps_plan_set_graphs", "ps_plan_set_timing"):
    getattr(L, f).argtypes = [c.c_void_p] + ([c.c_char_p, c.c_int] if f == "ps_plan_set_variant" else [c.c_int])
L.ps_plan_get_variant.argtypes = L.ps_plan_variant_count.argtypes = [c.c_void_p, c.c_char_p]
for f in ("ps_fft_r2c", "ps_fft_c2r", "ps_nonlinear_ns", "ps_nonlinear_mhd"):
    getattr(L, f).argtypes = [c.c_void_p, c.c_void_p, c.c_void_p]
L.ps_plan_autotune.argtypes = [c.c_void_p, c.c_void_p, c.c_int, c.c_int]
L.ps_plan_autotune_timed.argtypes = [c.c_void_p]
F.fake_cost.argtypes = [c.c_double] * 3
F.fake_fail.argtypes = [c.c_long] * 3
F.fake_fail_launch.argtypes = [c.c_long]
for f in ("fake_launches", "fake_replays", "fake_instantiated"):
    getattr(F, f).restype = c.c_long

class Launch(c.Structure):
    _fields_ = [("func", c.c_void_p), ("blocks", c.c_uint64), ("threads", c.c_uint64), ("stream", c.c_uint64),
                ("captured", c.c_int)]

def launches():
    """(kernel, workgroups, threads of one, stream, captured) since the last reset"""
    p = c.POINTER(Launch)()
    n = F.fake_launches(c.byref(p))
    return [(p[i].func, p[i].blocks, p[i].threads, p[i].stream, p[i].captured) for i in range(n)]

def check(st):
    assert st == 0, (st, L.ps_last_error())

def plan(dims, nf, f64=False, **variants):
    """a cube (int), an nx x ny x nz grid (tuple) or an ensemble of cubes (list)"""
    h = c.c_void_p()
    if isinstance(dims, tuple):
        check(L.ps_plan_create_grid(c.byref(h), *dims, nf, int(f64)))
    else:
        d = dims if isinstance(dims, list) else [dims]
        check(L.ps_plan_create_batch(c.byref(h), len(d), (c.c_int * len(d))(*d), nf, int(f64)))
    # nothing reads or writes the buffers: addresses alone (the plan checks alignment)
    check(L.ps_plan_set_workspace(h, 1 << 40, L.ps_plan_workspace_bytes(h)))
    for k, v in variants.items():
        check(L.ps_plan_set_variant(h, k.encode(), v))
    return h

STATE = 1 << 44

def step(h, nf, n=1, dt=1e-3, state=STATE):
    return L.ps_rk2_step(h, state, int(nf == 6), 1e-3, 1e-3, dt, n)
'''


def library(folder):
    """The fake runtime, compiled into `folder`."""
    out = os.path.join(str(folder), "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-o", out, os.path.join(HERE, "fake_hip.c")],
                   check=True)
    return out


def run(fake, body):
    lib = os.path.join(ROOT, "paper_1003_4322_amd", "libps.so")
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake, lib], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
