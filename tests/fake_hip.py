"""The library's host code on the CPU: ``run`` starts a process in which
libwl.so's calls of the HIP runtime go to fake_hip.cpp (kernels do not run),
and executes a piece of Python there with these names:

  wl        the package
  fake      fake_hip.cpp's own functions (fake.fake_limit, ...)
  calls()   the recorded calls since the last clear(), a list of strings
  pinned(n) a float64 array of n values in pinned memory
  np        numpy
"""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "fake_hip.cpp")
OUT = os.path.join(ROOT, "tests", "_build", "libfake_hip.so")

PREAMBLE = """
import ctypes, os, sys
fake = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)  # ahead of the real runtime
sys.modules["torch"] = None
sys.path.insert(0, %r)
import numpy as np
import paper_1407_7486_amd as wl
fake.fake_log.restype = ctypes.c_char_p
fake.fake_used.restype = ctypes.c_size_t
fake.fake_limit.argtypes = [ctypes.c_size_t]
clear = fake.fake_reset
def calls():
    return fake.fake_log().decode().splitlines()
def pinned(n):
    p = ctypes.c_void_p()
    assert fake.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(8 * n), 0) == 0
    return np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_double)), (n,))
"""


def build():
    if not os.path.exists(OUT) or os.path.getmtime(OUT) < os.path.getmtime(SRC):
        os.makedirs(os.path.dirname(OUT), exist_ok=True)
        tmp = OUT + ".tmp%d" % os.getpid()
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w",
                        "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", SRC, "-o", tmp],
                       check=True)
        os.replace(tmp, OUT)
    return OUT


def run(code):
    """Runs `code`; returns what it printed.  Fails with its error output."""
    res = subprocess.run([sys.executable, "-c", PREAMBLE % (build(), ROOT) + code],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr[-2000:]
    return res.stdout
