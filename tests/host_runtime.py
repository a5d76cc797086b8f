"""Runs a piece of test code in a process whose HIP runtime is host_runtime.cpp: the library's
host side without a GPU (plans, uploads, the choice of kernels and their grids, errors).

The code finds M (the package), W (workloads), np, a stand-in for torch that Solver accepts,
and `host` with the runtime's controls.  Kernels are recorded, not run, except the copy of
loaded blocks into their pool slots."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = '''
import ctypes, sys, types
sys.path.insert(0, {root!r})
import numpy as np
host = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)   # before the library that needs a HIP runtime
host.host_launch.restype = ctypes.c_char_p
host.host_scatter_faults.restype = host.host_null_topologies.restype = ctypes.c_long


class _Array:
    def __init__(self, n, dtype=None, device=None):
        self.a = np.zeros(n, dtype or np.float64)

    def data_ptr(self):
        return self.a.ctypes.data


class _Context:
    cuda_stream = 0

    def __init__(self, *a):
        pass

    def __enter__(self):
        return self

    def __exit__(self, *a):
        return False

    def synchronize(self):
        pass


torch = types.ModuleType("torch")
torch.float64, torch.float32, torch.zeros, torch.device = np.float64, np.float32, _Array, lambda d: d
torch.cuda = types.SimpleNamespace(is_available=lambda: True, device=_Context, Stream=_Context,
                                   synchronize=lambda *a: None, current_stream=_Context)
sys.modules["torch"] = torch
import paper_1902_00088_amd as M
import workloads as W


def launches():
    """(name, workgroups, threads) of the kernels launched since the last call"""
    out = []
    g, t = ctypes.c_ulonglong(), ctypes.c_ulonglong()
    for i in range(host.host_launches()):
        name = host.host_launch(i, ctypes.byref(g), ctypes.byref(t)).decode()
        out.append((name, g.value, t.value))
    host.host_clear()
    return out


def morton(co):
    """order of same-level blocks along the space-filling curve"""
    key = np.zeros(len(co), np.int64)
    for b in range(20):
        for a in range(co.shape[1]):
            key |= ((co[:, a].astype(np.int64) >> b) & 1) << (b * co.shape[1] + a)
    return np.argsort(key)


def pool_free_solver(cfg, levels, coords):
    """a solver whose kernels are recorded only: no memory behind its pools and loads"""
    host.host_run_copies(0)
    torch.zeros = lambda n, dtype=None, device=None: _Array(1)
    s = M.Solver(cfg)
    s.init_forest(levels, coords)
    s.set_graph(0)
    s._chk(M.lib().mrb_load_blocks(s.h, 8, 1))
    launches()
    return s


def solver(cfg, levels, coords):
    s = M.Solver(cfg)
    s.init_forest(levels, coords)
    s.load_blocks(np.zeros((len(levels), cfg.nf, cfg.npts)))
    s.set_graph(0)
    launches()
    return s
'''


def run(tmp_path, code):
    import paper_1902_00088_amd as M
    if not os.path.exists(M.LIB_PATH):
        M.build()
    so = os.path.join(str(tmp_path), "libamdhip64.so.7")
    vers = os.path.join(str(tmp_path), "versions")
    with open(vers, "w") as f:
        f.write("hip_4.2 { global: *; };\n"
                "hip_4.3 { global: hipStreamBeginCapture; hipStreamEndCapture; hipGraph*; } hip_4.2;\n")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROOT, "paper_1902_00088_amd", "csrc"), "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "host_runtime.cpp"), "-o", so,
                           "-Wl,-soname,libamdhip64.so.7", f"-Wl,--version-script={vers}"])
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + code], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
