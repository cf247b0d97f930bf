"""Runs the library's host code on the CPU, over tests/fake_hip.cpp in place
of the HIP runtime: `start()` in a process that has not loaded the library."""
import ctypes
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

OUT_OF_MEMORY, CAPTURE_UNSUPPORTED, UNKNOWN = 2, 900, 999  # hipError_t


def build(folder):
    """The stand-in runtime as a shared library in `folder`; None without a compiler."""
    gxx = shutil.which("g++")
    if gxx is None:
        return None
    so = os.path.join(folder, "libfakehip.so")
    subprocess.run([gxx, "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


def start():
    """The loaded stand-in (named by argv[1]); the package then binds to it."""
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    fake.fake_log.restype = ctypes.c_char_p
    fake.fake_fail.argtypes = [ctypes.c_char_p, ctypes.c_int, ctypes.c_int]
    fake.fake_limit.argtypes = [ctypes.c_int, ctypes.c_size_t]
    fake.fake_used.restype = ctypes.c_size_t
    fake.fake_pending.argtypes = [ctypes.c_void_p]
    fake.fake_fast.argtypes = [ctypes.c_char_p]
    sys.path.insert(0, ROOT)
    return fake


def run(so, code, env=None, timeout=120):
    """`code` in a fresh process after `fake = start()`; its output."""
    head = f"import sys; sys.path.insert(0, {HERE!r})\nimport fake_gpu\nfake = fake_gpu.start()\n"
    head += "import numpy as np\nimport paper_0707_2437_amd as lbm\n"
    r = subprocess.run([sys.executable, "-c", head + code, so], capture_output=True, text=True, timeout=timeout,
                       env=dict(os.environ, **(env or {})))
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
