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
import ctypes, sys, time
sys.path.insert(0, {root!r})
import numpy as np
import paper_2601_01388_amd as A
H = ctypes.CDLL({so!r})
for f in ("host_hip_live_bytes", "host_hip_log"):
    getattr(H, f).restype = ctypes.c_size_t
for f in ("host_hip_memory_queries", "host_hip_mallocs", "host_hip_launches", "host_hip_unwaited", "host_hip_new_left"):
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


@pytest.mark.parametrize("slots,kernel", [(96 << 20, "ILi0ELi8E"), ((96 << 20) + 2, "ILi0ELi7E")])
def test_large_graphs_sample_at_seven_waves(stand_in, slots, kernel):
    # (the neighbours are not read: no kernel runs)
    run(stand_in, KERNELS + f"""
off = np.array([0, {slots}, {slots}, {slots}], dtype=np.uint64)
big = A.agis_load_csr(ctx, off.ctypes.data, off.ctypes.data, 3, {slots}, 0)
tb = A.agis_build_proposal_tables(ctx, big, 1, A.LC_MIN_DEFAULT, False)
assert kernels(ctx, big, tb) == ({kernel!r}, "_epsILi6EL"), kernels(ctx, big, tb)
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


POOL = """
MiB = 1 << 20

def held():
    return H.host_hip_live_bytes() - base

ctx = A.agis_create(0, 0)
base = H.host_hip_live_bytes()
H.host_hip_free_memory(200 * GiB, 0)

def tables(n, free_at_end):
    g = graph(ctx, n)
    t = A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)
    H.host_hip_free_memory(free_at_end, 0)
    A.agis_tables_destroy(t)
    A.agis_graph_destroy(g)
"""


def test_kept_buffers_go_back_on_request(stand_in):
    run(stand_in, POOL + """
tables(8 << 20, 200 * GiB)   # 128 + 3 x 64 MiB
kept = held()
assert kept >= 320 * MiB, kept
before = H.host_hip_mallocs()
tables(8 << 20, 200 * GiB)   # from the kept buffers
assert held() == kept and H.host_hip_mallocs() == before
A.agis_release_scratch(ctx)
assert held() == 0, held()
tables(8 << 20, 200 * GiB)
A.agis_destroy(ctx)
assert H.host_hip_live_bytes() == 0
""")


@pytest.mark.parametrize("n,count", [(8 << 20, 1), (300_000, 40)])
def test_no_more_than_64_mib_is_kept_where_memory_is_short(stand_in, n, count):
    run(stand_in, POOL + f"""
gs = [graph(ctx, {n}) for _ in range({count})]
ts = [A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False) for g in gs]
assert held() > 300 * MiB
H.host_hip_free_memory(100 * GiB, 0)
for t in ts:
    A.agis_tables_destroy(t)
assert held() <= 64 * MiB, held()
""")


def test_kept_buffers_go_back_at_a_call_that_finds_memory_short(stand_in):
    run(stand_in, POOL + """
small = graph(ctx, 1000)
t = A.agis_build_proposal_tables(ctx, small, 1, A.LC_MIN_DEFAULT, False)
feats = np.zeros((1000, 4), dtype=np.float32)
w = np.ones(4801, dtype=np.float32)
row = np.zeros(4, dtype=np.uint32), np.zeros(4, dtype=np.uint8), np.zeros(4, dtype=np.float32), np.ones(4, dtype=np.float32)
ptr = [x.ctypes.data for x in row]
grad = np.zeros(4801, dtype=np.float32)
sums, counts, base_ = np.zeros((3, 1000)), np.zeros((3, 1000), dtype=np.uint32), held()
out = [np.zeros(3000, dtype=d) for d in (np.uint32, np.uint8, np.float32, np.float32)]
calls = {
    "tables": lambda: A.agis_tables_destroy(A.agis_build_proposal_tables(ctx, small, 1, A.LC_MIN_DEFAULT, False)),
    "orient": lambda: A.agis_graph_destroy(A.agis_orient(ctx, small)),
    "features": lambda: A.agis_features(ctx, t, feats.ctypes.data),
    "targets": lambda: A.agis_learn_targets(ctx, small, t, TRI, 10, 1, A.make_params(), sums.ctypes.data, counts.ctypes.data),
    "rows": lambda: A.agis_learn_rows(ctx, sums.ctypes.data, counts.ctypes.data, 3, 1000, 7, 2, *[o.ctypes.data for o in out]),
    "grad": lambda: A.agis_mlp_grad(ctx, w.ctypes.data, feats.ctypes.data, *ptr, 4, 4.0, grad.ctypes.data, 0),
    "train": lambda: A.agis_mlp_train(ctx, w.ctypes.data, feats.ctypes.data, *ptr, 4, 1, 4, 1e-3, 1),
    "estimate": lambda: A.agis_estimate(ctx, small, t, TRI, 100, 1, A.make_params(mode="uniform")),
}
for name, call in calls.items():
    H.host_hip_free_memory(200 * GiB, 0)
    call()   # (what the call itself leaves with the context)
    A.agis_release_scratch(ctx)
    call()
    after = held()
    tables(8 << 20, 200 * GiB)
    assert held() >= after + 300 * MiB, name
    H.host_hip_free_memory(100 * GiB, 0)
    time.sleep(0.005)   # (asked once a millisecond at most)
    call()
    assert held() <= after + 64 * MiB, (name, held(), after)
""")


def test_free_memory_is_asked_of_the_contexts_device(stand_in):
    run(stand_in, POOL + """
g = graph(ctx, 8 << 20)
t = A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)
H.host_hip_current_device(3)
asked = H.host_hip_memory_queries()
A.agis_tables_destroy(t)
assert H.host_hip_memory_queries() > asked and H.host_hip_queried_device() == 0
d = ctypes.c_int(-1)
H.hipGetDevice(ctypes.byref(d))
assert d.value == 3
""")


def test_training_rows_wait_for_their_stream_where_a_launch_fails(stand_in):
    run(stand_in, POOL + """
sums, counts = np.ones((3, 1000)), np.full((3, 1000), 5, dtype=np.uint32)
out = [np.zeros(3000, dtype=d) for d in (np.uint32, np.uint8, np.float32, np.float32)]
bp = np.zeros((3, 1000), dtype=np.int32)
failed = 0
for n in range(1, 5):
    H.host_hip_fail_launch(n)
    try:
        A.agis_learn_rows(ctx, sums.ctypes.data, counts.ctypes.data, 3, 1000, 7, 2, *[o.ctypes.data for o in out],
                          bp.ctypes.data)
    except A.AgisError as e:
        assert e.code == A.AGIS_E_HIP
        failed += 1
    assert H.host_hip_unwaited() == 0, n
assert failed == 4
""")


CALLS = POOL + """
n0 = 300_000
g = graph(ctx, n0)
t = A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)
feats = np.zeros((n0, 4), dtype=np.float32)
w = np.ones(4801, dtype=np.float32)
R = 300_000
row = np.zeros(R, dtype=np.uint32), np.zeros(R, dtype=np.uint8), np.zeros(R, dtype=np.float32), np.ones(R, dtype=np.float32)
ptr = [x.ctypes.data for x in row]
grad = np.zeros(4801, dtype=np.float32)
sums, counts = np.zeros((3, n0)), np.zeros((3, n0), dtype=np.uint32)
out = [np.zeros(3 * n0, dtype=d) for d in (np.uint32, np.uint8, np.float32, np.float32)]
lt = np.zeros(n0, dtype=np.int32)
idx, rec = np.arange(100, dtype=np.uint64), np.zeros(100 * A.RECORD_BYTES, dtype=np.uint8)
mt, q1 = np.zeros(400, dtype=np.uint64), np.zeros(n0, dtype=np.uint32)
H5 = A.make_pattern(5, [0b11010, 0b10101, 0b1010, 0b101, 0b11, 0, 0, 0])
PR = dict(mode="always", rowtab="on")
LE = dict(mode="learned", learned={i: lt.ctypes.data for i in range(5)}, rowtab="on")
calls = {
    "tables": lambda: A.agis_tables_destroy(A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)),
    "orient": lambda: A.agis_graph_destroy(A.agis_orient(ctx, g)),
    "features": lambda: A.agis_features(ctx, t, feats.ctypes.data),
    "targets": lambda: A.agis_learn_targets(ctx, g, t, TRI, 10, 1, A.make_params(), sums.ctypes.data, counts.ctypes.data),
    "rows": lambda: A.agis_learn_rows(ctx, sums.ctypes.data, counts.ctypes.data, 3, n0, 7, 2, *[o.ctypes.data for o in out]),
    "grad": lambda: A.agis_mlp_grad(ctx, w.ctypes.data, feats.ctypes.data, *ptr, R, 4.0, grad.ctypes.data, 0),
    "train": lambda: A.agis_mlp_train(ctx, w.ctypes.data, feats.ctypes.data, *ptr, R, 3, 100000, 1e-3, 1),
    "estimate": lambda: A.agis_estimate(ctx, g, t, H5, 100000, 1, A.make_params(**PR)),
    "blocked": lambda: A.agis_estimate(ctx, g, t, H5, 100000, 1, A.make_params(step1="blocks", **PR)),
    "learned": lambda: A.agis_estimate(ctx, g, t, H5, 100000, 1, A.make_params(**LE)),
    "eps": lambda: A.agis_estimate(ctx, g, t, H5, 100000, 1, A.make_params(eps=0.01, check_every=4096, **PR)),
    "batch": lambda: A.agis_estimate_batch(ctx, g, t, [H5, TRI], [1000, 1000], 1, A.make_params(**PR)),
    "dump": lambda: A.agis_dump_samples(ctx, g, t, H5, 1, A.make_params(**PR), idx.ctypes.data, 100, rec.ctypes.data),
    "meter": lambda: A.agis_meter_samples(ctx, g, t, H5, 1, A.make_params(**PR), idx.ctypes.data, 100, mt.ctypes.data),
    "step1": lambda: A.agis_step1_weights(ctx, g, t, H5, A.make_params(**PR), q1.ctypes.data),
    "load": lambda: A.agis_graph_destroy(graph(ctx, 1000)),
    "autotune": lambda: A.agis_autotune(ctx, g, t, [TRI, H5], 100, A.make_params(**PR)),
    "patterns": lambda: A.agis_connected_patterns(5),
    "compile": lambda: A.agis_compile_pattern(H5),
    "concentrations": lambda: A.agis_concentrations([TRI, A.make_pattern(3, [6, 1, 1, 0, 0, 0, 0, 0])], [5.0, 9.0]),
    "create": lambda: A.agis_destroy(A.agis_create(0, 0)),
}
"""


def test_a_failed_host_allocation_is_a_code_and_no_exception(stand_in):
    run(stand_in, CALLS + """
for name, call in calls.items():
    failed, n = 0, 0
    while True:
        A.agis_tables_destroy(t)   # (nothing cached)
        t = A.agis_build_proposal_tables(ctx, g, 1, A.LC_MIN_DEFAULT, False)
        H.host_hip_fail_new(n)
        try:
            call()
            code = 0
        except A.AgisError as e:
            code = e.code
        through = H.host_hip_new_left() >= 0
        H.host_hip_fail_new(-1)
        assert code in (0, A.AGIS_E_OOM, A.AGIS_E_NOT_CONVERGED), (name, n, code)
        failed += code == A.AGIS_E_OOM
        if through:
            break
        n += 1
    call()   # the context still serves
    print(name, n, failed, flush=True)
""")
