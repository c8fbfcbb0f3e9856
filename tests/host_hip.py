"""The library over the host-memory HIP runtime of host_hip.cpp.  run(code)
runs Python code in a process of its own, where `fw` is the binding, `np`
numpy, launches(clear=True) the launches since they were last cleared, `hip`
the runtime."""
from __future__ import annotations

import os
import subprocess
import sys
import textwrap
from pathlib import Path

import pytest

HERE = Path(__file__).resolve().parent

PRELUDE = """
import ctypes, sys
hip = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, {root!r})
sys.modules["torch"] = None  # the library must not find another HIP runtime first
import numpy as np
from paper_2404_08364_amd import flowwalk as fw


class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 96), ("grid", ctypes.c_uint), ("block", ctypes.c_uint),
                ("lds", ctypes.c_ulonglong), ("stream", ctypes.c_void_p)]


hip.host_hip_launches.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
hip.host_hip_launches.restype = ctypes.c_size_t
hip.host_hip_fail_at.argtypes = [ctypes.c_long]


def launches(clear=True):
    a = (Launch * 4096)()
    n = hip.host_hip_launches(a, 4096, int(clear))
    return [l for l in a[:n] if b"reset" not in l.name]


def ring(n=1000, hub=0, **kw):
    '''n vertices in a ring, vertex 0 joined to `hub` more entries (parallel edges to 1).'''
    off = np.arange(n + 1, dtype=np.uint64) + hub
    off[0] = 0
    adj = np.concatenate([np.ones(hub + 1), (np.arange(1, n) + 1) % n]).astype(np.uint32)
    w = np.full(adj.size, 3, np.uint32)
    lab = np.zeros(adj.size, np.uint8)
    return fw.Graph.upload(off, adj, kw.get("weights", w), kw.get("labels", lab))
"""


@pytest.fixture(scope="session")
def host_hip(tmp_path_factory):
    lib = tmp_path_factory.mktemp("host_hip") / "libhost_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wno-unused-result",
                    str(HERE / "host_hip.cpp"), "-o", str(lib)], check=True)

    def run(code: str) -> str:
        text = PRELUDE.format(lib=str(lib), root=str(HERE.parent)) + textwrap.dedent(code)
        p = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True,
                           timeout=120, env=dict(os.environ))
        assert p.returncode == 0, p.stdout + p.stderr
        return p.stdout
    return run
