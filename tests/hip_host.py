"""Run a snippet against the library with its HIP calls served by host memory
(tests/hip_host.cpp): in a process of its own, `b` the binding and `h` the
counters and switches of the host calls."""
import os
import subprocess
import sys
import tempfile
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


_built = []


def _library():
    """Built once a process, in a folder that goes with it."""
    if not _built:
        folder = tempfile.TemporaryDirectory()
        so = os.path.join(folder.name, "hip_host.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "hip_host.cpp"),
                        "-o", so, "-lpthread"], check=True)
        _built.append((folder, so))
    return _built[0][1]


def run(snippet):
    r = subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(snippet), ROOT, _library()], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
