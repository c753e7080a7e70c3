"""Host code of the library's entry points without a GPU: the library runs in
a process of its own over a stand-in for the HIP runtime (host_hip.cpp) that
records kernel launches by name and runs none."""

import os
import subprocess
import sys

import pytest

A = pytest.importorskip("paper_2601_01388_amd")

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
import numpy as np
import paper_2601_01388_amd as A
H = ctypes.CDLL({so!r})
for f in ("host_hip_live_bytes", "host_hip_log"):
    getattr(H, f).restype = ctypes.c_size_t
for f in ("host_hip_memory_queries", "host_hip_mallocs", "host_hip_launches", "host_hip_new_left"):
    getattr(H, f).restype = ctypes.c_longlong
H.host_hip_free_memory.argtypes = [ctypes.c_size_t, ctypes.c_int]
for f in ("host_hip_fail_malloc", "host_hip_fail_launch", "host_hip_fail_new"):
    getattr(H, f).argtypes = [ctypes.c_longlong]
H.host_hip_time.argtypes = [ctypes.c_char_p, ctypes.c_float]
GiB = 1 << 30
_buf = ctypes.create_string_buffer(1 << 22)

def launches(part=""):
    n = H.host_hip_log(_buf, len(_buf))
    return [x for x in _buf.raw[:n].decode().split() if part in x]

def graph(ctx, n, d=2):
    global keep
    off = np.arange(n + 1, dtype=np.uint64) * d
    nbr = np.zeros(n * d, dtype=np.uint32)
    keep = off, nbr
    return A.agis_load_csr(ctx, off.ctypes.data, nbr.ctypes.data, n, n * d, 0)

TRI = A.make_pattern(3, [6, 5, 3, 0, 0, 0, 0, 0])
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    if not os.path.exists(A.LIB_PATH):
        from paper_2601_01388_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("host_hip") / "libhost_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "host_hip.cpp"), "-o", so],
                   check=True)
    return so


def run(so, script):
    code = PRELUDE.format(root=ROOT, so=so) + script
    env = dict(os.environ, LD_PRELOAD=so)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-3000:])
    return r.stdout


KERNELS = """
def kernels(ctx, g, t):
    launches()
    A.agis_estimate(ctx, g, t, TRI, 5000, 1, A.make_params(mode="uniform"))
    fixed = launches("k_sample")
    A.agis_estimate(ctx, g, t, TRI, 5000, 1, A.make_params(mode="uniform", eps=0.01, check_every=4096))
    eps = launches("k_sample")
    assert len(fixed) == 1 and len(eps) == 1, (fixed, eps)
    return fixed[0].split("k_sample")[1][:9], eps[0].split("k_sample")[1][:10]

ctx = A.agis_create(0, 0)
g = graph(ctx, 1000)
t = A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)
new = kernels(ctx, g, t)
assert new == ("ILi0ELi8E", "_epsILi6EL"), new
"""


def test_a_new_contexts_launch_shape_can_be_given_back(stand_in):
    run(stand_in, KERNELS + """
A.agis_set_launch(ctx, True, 0, 0, 1, 0)
assert kernels(ctx, g, t) == ("ILi0ELi7E", "_epsILi7EL")
A.agis_set_launch(ctx, True, 0, 0, 0, 0)
assert kernels(ctx, g, t) == ("ILi0ELi6E", "_epsILi6EL")
A.agis_set_launch(ctx)
assert kernels(ctx, g, t) == new
A.agis_set_launch(ctx, True, 0, 0, 1, 0)
A.agis_set_launch(ctx, True, 0, 0, -1, 0)
assert kernels(ctx, g, t) == new
for bad in (-2, 3):
    try:
        A.agis_set_launch(ctx, True, 0, 0, bad, 0)
    except A.AgisError as e:
        assert e.code == A.AGIS_E_INVALID_ARG
    else:
        raise AssertionError(bad)
""")


@pytest.mark.parametrize("times,fixed,eps,variant,default,best", [
    # the default is the fastest, or within the 2% of the fastest
    ((3.0, 2.9, 2.0), "ILi0ELi8E", "_epsILi6EL", 2, 2.0, 2.0),
    ((1.99, 2.9, 2.0), "ILi0ELi8E", "_epsILi6EL", 2, 2.0, 2.0),
    ((3.0, 1.0, 2.0), "ILi0ELi7E", "_epsILi7EL", 1, 2.0, 1.0),
    ((1.0, 3.0, 2.0), "ILi0ELi6E", "_epsILi6EL", 0, 2.0, 1.0),
])
def test_autotune_starts_from_the_default_and_keeps_it_for_runs_to_epsilon(stand_in, times, fixed, eps, variant,
                                                                           default, best):
    run(stand_in, KERNELS + f"""
for name, ms in zip((b"k_sampleILi0ELi6E", b"k_sampleILi0ELi7E", b"k_sampleILi0ELi8E"), {times}):
    H.host_hip_time(name, ms)
tun = A.agis_autotune(ctx, g, t, [TRI], 1000, A.make_params(mode="uniform"))
assert tun.variant == {variant}, tun.variant
assert abs(tun.default_seconds * 1e3 - {default}) < 1e-5 and abs(tun.seconds * 1e3 - {best}) < 1e-5
assert kernels(ctx, g, t) == ({fixed!r}, {eps!r}), kernels(ctx, g, t)
""")
