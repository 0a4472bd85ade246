"""Runs librkl's host code against fake_hip.c, a stand-in for the HIP runtime
that records launches and runs none, in a child process (the library binds
its runtime once per process).

``run(tmp_path, code)`` executes ``code`` there with these names:

  hip          the stand-in's knobs and counters (ctypes; ``put`` sets a knob,
               ``get`` reads one)
  rkl          paper_1702_05487_amd.rkl, loaded on the stand-in
  T, b, out    addresses to pass as device fields (never dereferenced)
  desc(n, ...) a grid descriptor (periodic, T^2.5, MC unless told otherwise)
  launches()   (kernel, workgroups, threads, LDS bytes) since ``hip.fake_reset()``,
               the kernel as its name with template arguments
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r'''
import ctypes, subprocess, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1702_05487_amd import rkl
lib = rkl.load()
hip.fake_name.restype = ctypes.c_char_p

def put(name, v):
    (ctypes.c_double if isinstance(v, float) else ctypes.c_int).in_dll(hip, "fake_" + name).value = v

def get(name):
    return ctypes.c_int.in_dll(hip, "fake_" + name).value

T, b, out = (ctypes.c_void_p(x) for x in (1 << 40, 2 << 40, 3 << 40))

def desc(n, ndim=3, lim=1, sat=0, law=2.5, edges=(0, 0, 0)):
    return rkl.grid_desc(n, (0.03, 0.04, 0.05), ndim=ndim, limiter=lim, saturation=sat, phi=0.3, kappa_exp=law,
                         boundary=edges)

def launches():
    r, shape = [], (ctypes.c_uint * 3)()
    names = [hip.fake_name(i).decode() for i in range(hip.fake_count())]
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True).stdout.split("\n")
    for i, name in enumerate(plain[:len(names)]):
        hip.fake_shape(i, shape)
        name = name.split("(")[0].replace("void ", "").replace("rkl::", "")
        r.append((name, shape[0], shape[1], shape[2]))
    return r
'''


def run(tmp_path, code, timeout=60):
    so = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-w", os.path.join(HERE, "fake_hip.c"), "-o", so])
    r = subprocess.run([sys.executable, "-c", PRELUDE + code, so, ROOT], capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
