"""Runs the library's host code on fake_hip.c: which kernels a call launches,
with what grid and LDS, and what it returns when one of the launches fails.

Used from a process of its own (see run): the fake runtime takes the place of
HIP for as long as the process lives."""
import ctypes
import json
import os
import re
import subprocess
import sys
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def run(module: str, call: str):
    """The JSON value of `module.call` evaluated in a process of its own."""
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "fake_hip.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")], check=True)
        code = ("import sys, json; sys.path[:0] = [%r, %r]\nimport fake_hip; fake_hip.load(%r)\nimport %s\n"
                "print('RESULT ' + json.dumps(%s.%s))" % (ROOT, HERE, so, module, module, call))
        out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stderr[-2000:]
        return json.loads(out.stdout.split("RESULT ", 1)[1])


class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 96), ("grid", ctypes.c_uint32), ("block", ctypes.c_uint32),
                ("lds", ctypes.c_uint64)]


fake = None
_keep = []  # memory the library was given


def load(so: str) -> None:
    global fake
    fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
    fake.fake_launch.restype = ctypes.POINTER(Launch)


def memory(n: int):
    """n bytes of "device" memory, 256-byte aligned."""
    a = np.zeros(n + 256, dtype=np.uint8)
    _keep.append(a)
    return ctypes.c_void_p((a.ctypes.data + 255) // 256 * 256)


def launches() -> list:
    """The launches since the last reset: (kernel, grid, block, LDS bytes)."""
    out = []
    for i in range(fake.fake_launches()):
        f = fake.fake_launch(i).contents
        name = re.search(r"(k_[a-z_]+)", f.name.decode())
        out.append([name.group(1) if name else f.name.decode(), f.grid, f.block, f.lds])
    return out


def world(name="c2", flags=0, **kw):
    import paper_2209_12842_amd as R
    from paper_2209_12842_amd import workloads as W
    w = W.make_world(name, **kw)
    obs = np.ascontiguousarray(w["obstacles"], dtype=np.float32)
    _keep.append(obs)
    p = R.make_params(w["params"], len(obs), flags)
    return p, obs.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), (ctypes.c_float * 4)(*w["x0"])


def handle(p, obs):
    import paper_2209_12842_amd as R
    L = R.lib()
    n = L.mppi_workspace_bytes(ctypes.byref(p))
    h = ctypes.c_void_p()
    R.check(L.mppi_create(ctypes.byref(p), obs, memory(n), n, None, ctypes.byref(h)))
    return h


def batch(ps, obstacles):
    import paper_2209_12842_amd as R
    L = R.lib()
    n = len(ps)
    P = (R.Params * n)(*ps)
    nb = L.mppi_batch_workspace_bytes(n, P)
    V = (ctypes.c_void_p * n)(*[memory(8 * p.T) for p in ps])
    O = (ctypes.POINTER(ctypes.c_float) * n)(*obstacles)
    b = ctypes.c_void_p()
    R.check(L.mppi_batch_create(n, P, O, V, memory(nb), nb, None, ctypes.byref(b)))
    return b
