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


PASSES = """
import json, re
def passes(log):
    out = []
    for line in log.decode().splitlines():
        m = re.match(r"launch lbm::(\\w+)<(.*)>", line)
        if not m or m[1] == "init_kernel":
            continue
        name, arg = m[1], m[2].split(", ")
        if name == "cascade_kernel":
            out.append("cascade%d" % (4 * int(arg[3])))
        elif name in ("batch_cascade_kernel", "batch_persistent_cascade_kernel"):
            out.append("pool_cascade%d" % (4 * int(arg[3])))
        else:
            out.append({"block_kernel": "block", "step2_vstack_kernel": "pair", "step_vstack_kernel": "step", "step_kernel": "step",
                        "xbc_kernel": "xbc", "ghost_kernel": "ghosts", "batch_step2_kernel": "pool_pair",
                        "batch_persistent2_kernel": "pool_pair"}.get(name, name))
    return out
"""

_ROUTES = PASSES + """
res = []
for case in json.loads(sys.stdin.read()):
    c = dict({"tile": None, "model": None, "field": False, "inlet": None}, **case)
    with lbm.Lattice(c["nx"], c["ny"], 0.7, 0.3, c["dtype"]) as L:
        if c["model"] is not None: L.set_model(c["model"])
        if c["field"]: assert L._L.lbm_set_c2_field_device(L._h, 4096) == 0  # no kernel reads it
        if c["inlet"]: L.set_x_boundaries(lbm.XBC_INLET_OUTLET, *c["inlet"])
        if c["tile"] == "own": L.set_tile(*L.get_tile())
        elif c["tile"]: L.set_tile(*c["tile"])
        L.init_device(None, None, None)
        fake.fake_log()
        for n in c["calls"]: L.step(n)
        res.append(passes(fake.fake_log()))
print(json.dumps(res))
"""


def routes(so, cases, env=None):
    """The kernels that lbm_step launches for each case: a dict with nx, ny, dtype,
    calls and optionally tile ("own": the one it reports), model, field, inlet."""
    import json
    head = f"import sys; sys.path.insert(0, {HERE!r})\nimport fake_gpu\nfake = fake_gpu.start()\nimport paper_0707_2437_amd as lbm\n"
    r = subprocess.run([sys.executable, "-c", head + _ROUTES, so], input=json.dumps(cases), capture_output=True, text=True,
                       timeout=120, env=dict(os.environ, **(env or {})))
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout)
