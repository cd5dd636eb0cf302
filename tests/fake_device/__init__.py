"""The library's host code on a device that is not there (fake_hip.cpp), in a process of its own without torch: which kernels
a call enqueues, what it allocates, and what it does when host memory runs out."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

PRELUDE = """
import ctypes, re, sys
sys.modules["torch"] = None                     # its own copy of the runtime would come in with it
import numpy as np
import paper_2402_02447_amd as B
import workloads as W
from paper_2402_02447_amd import lbs
B.load_library()
fake = ctypes.CDLL("libamdhip64.so.7")
fake.fake_launch_name.restype = fake.fake_kernel_name.restype = ctypes.c_char_p
fake.fake_launch_arg.restype = ctypes.c_void_p
fake.fake_device_allocations.restype = fake.fake_device_frees.restype = ctypes.c_ulonglong

def kernels():
    '''Names (without namespaces and template arguments) and grids of the launches since the last look.'''
    out = []
    for i in range(fake.fake_num_launches()):
        mangled = fake.fake_launch_name(i).decode()
        out.append((re.search(r"k_[a-z_]+", mangled).group().rstrip("_"), fake.fake_launch_grid(i)))
    fake.fake_forget_launches()
    return out
"""


def build(tmp_path) -> str:
    out = os.path.join(str(tmp_path), "libamdhip64.so.7")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wall",
                    os.path.join(HERE, "fake_hip.cpp"), "-Wl,-soname,libamdhip64.so.7", "-o", out], check=True)
    return os.path.dirname(out)


def run(libdir: str, script: str, timeout: float = 120.0) -> str:
    """Runs `script` behind PRELUDE; returns what it printed."""
    env = dict(os.environ, LD_LIBRARY_PATH=libdir, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PRELUDE + script], cwd=ROOT, env=env, capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, f"status {r.returncode}\n{r.stdout[-3000:]}\n{r.stderr[-3000:]}"
    return r.stdout
