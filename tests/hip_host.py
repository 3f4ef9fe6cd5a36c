"""Run a snippet against the library with its HIP calls served by host memory
(tests/hip_host.cpp): in a process of its own, `b` the binding and `h` the
counters and switches of the host calls."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
import ctypes, sys
sys.path.insert(0, sys.argv[1])
lib = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
class Host:
    def __getattr__(self, name): return ctypes.c_long.in_dll(lib, "host_" + name).value
    def __setattr__(self, name, v): ctypes.c_long.in_dll(lib, "host_" + name).value = v
h = Host()
import numpy as np
from paper_cs_0312006_amd import binding as b
"""


def run(tmp_path, snippet):
    so = str(tmp_path / "hip_host.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "hip_host.cpp"),
                    "-o", so, "-lpthread"], check=True)
    r = subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(snippet), ROOT, so], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
