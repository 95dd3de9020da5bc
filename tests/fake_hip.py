"""Runs a piece of Python against libsqn.so with tests/fake_hip.c in place of
the HIP runtime's calls: the host code's choices (launches, allocations,
refusals) on a machine without a GPU."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r"""
import ctypes, json, sys
sys.path.insert(0, ROOT)
# global and first: libsqn.so's calls bind to these, not to the runtime's
fake = ctypes.CDLL(FAKE, mode=ctypes.RTLD_GLOBAL)
from paper_2204_02585_amd import binding as B
lib = B.lib
fake.fake_limit.argtypes = [ctypes.c_size_t]
fake.fake_used.restype = ctypes.c_size_t
fake.fake_log.restype = ctypes.c_char_p
fake.fake_cost.argtypes = [ctypes.c_char_p, ctypes.c_double]
fake.fake_copied.restype = ctypes.c_size_t
fake.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
fake.hipFree.argtypes = [ctypes.c_void_p]
SIZE = {0: 4, 1: 2, B.SQN_F32: 4, B.SQN_F16: 2}

def alloc(n):
    p = ctypes.c_void_p()
    assert fake.hipMalloc(ctypes.byref(p), max(n, 1)) == 0
    return p.value

def desc(n_p, D, n_theta=16, n_phi=16, sigma="f16", uvw="f16", beta="f16"):
    d = B.CacheDesc()
    t = {"f16": B.SQN_F16, "f32": B.SQN_F32}
    d.n_p, d.D, d.n_theta, d.n_phi = n_p, D, n_theta, n_phi
    d.sigma_dtype, d.uvw_dtype, d.beta_dtype = t[sigma], t[uvw], t[beta]
    for r in range(3):
        d.bbox_min[r], d.bbox_max[r] = -1.0, 1.0
    d.t_eps = 1e-4
    return d

def arrays(d, channels=1):
    # three sigma planes, three uvw planes, beta
    tex = d.n_p * d.n_p
    vp = ctypes.c_void_p
    s = (vp * 3)(*[alloc(tex * channels * SIZE[d.sigma_dtype]) for _ in range(3)])
    u = (vp * 3)(*[alloc(tex * 3 * d.D * SIZE[d.uvw_dtype]) for _ in range(3)])
    return s, u, alloc(d.n_theta * d.n_phi * d.D * SIZE[d.beta_dtype])

def free(a):
    for p in list(a[0]) + list(a[1]) + [a[2]]:
        assert fake.hipFree(p) == 0

def launches():
    out = fake.fake_log().decode().splitlines()
    fake.fake_reset()
    return out

def intrinsics(w, h):
    return B._intrinsics(dict(fx=100.0, fy=100.0, cx=w / 2, cy=h / 2, width=w, height=h))
"""


def run(code, data=None, timeout=100):
    """The JSON that `code` prints last, run behind PRELUDE with `data` (plain
    values) as DATA."""
    build = os.path.join(HERE, "..", "paper_2204_02585_amd", "_build")
    os.makedirs(build, exist_ok=True)
    lib = os.path.abspath(os.path.join(build, f"fake_hip_{os.getpid()}.so"))
    try:
        subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "fake_hip.c")],
                       check=True)
        script = f"ROOT, FAKE, DATA = {ROOT!r}, {lib!r}, {data!r}\n" + PRELUDE + code
        p = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True, timeout=timeout)
        assert p.returncode == 0, p.stderr[-3000:]
        return json.loads(p.stdout.splitlines()[-1])
    finally:
        if os.path.exists(lib):
            os.remove(lib)
