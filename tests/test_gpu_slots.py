"""GPU: the kernels that give a wave runs of consecutive CSR slots
(orientation, validation, vertex tables), at the edges of words and runs and
across rows without slots."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")


@pytest.fixture(scope="module")
def sess():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    yield s
    s.close()


def _spread(n, m, seed, lo=0, hi=None):
    """m edges among the vertices [lo, hi) of n, the others without any."""
    rng = np.random.Generator(np.random.PCG64(seed))
    hi = n if hi is None else hi
    return synth.csr_from_edges(n, rng.integers(lo, hi, m), rng.integers(lo, hi, m))


def _ends(n):
    """A triangle at either end of n vertices."""
    return synth.csr_from_edges(n, [0, 1, 2, n - 1, n - 2, n - 3], [1, 2, 0, n - 2, n - 3, n - 1])


GRAPHS = {
    "edge": lambda: synth.csr_from_edges(2, [0], [1]),
    "star32": lambda: synth.star_graph(32),       # 64 slots
    "star33": lambda: synth.star_graph(33),
    "star512": lambda: synth.star_graph(512),     # 1,024 slots
    "star513": lambda: synth.star_graph(513),
    "star3000": lambda: synth.star_graph(3000),   # one row over three runs
    "ends": lambda: _ends(5000),                  # thousands of rows without slots
    "middle": lambda: _spread(9000, 3000, 1, 4000, 4300),
    "sparse": lambda: _spread(40_000, 9000, 2),
    "K65": lambda: synth.complete_graph(65),
    "skewed": lambda: synth.chung_lu(n=3000, m=20_000, seed=3),
}


def _oriented(g):
    d = g.degrees()
    src = np.repeat(np.arange(g.n), d)
    dst = g.nbr.astype(np.int64)
    keep = (d[dst] > d[src]) | ((d[dst] == d[src]) & (dst > src))
    off = np.zeros(g.n + 1, dtype=np.uint64)
    np.cumsum(np.bincount(src[keep], minlength=g.n), out=off[1:])
    return off, g.nbr[keep]


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_orientation_and_tables(sess, name):
    g = GRAPHS[name]()
    G = sess.graph(g.off, g.nbr)
    D = sess.orient(G)
    off, nbr = D.csr()
    roff, rnbr = _oriented(g)
    assert np.array_equal(off, roff) and np.array_equal(nbr, rnbr)
    for exact in (False, True):
        T = sess.tables(G, cv_seed=3, exact_cv=exact)
        got, ref = T.export(), oracle.Tables(g, cv_seed=3, exact_cv=exact)
        for f in ("deg", "s2", "hits", "trials", "la", "lc"):
            assert np.array_equal(got[f].astype(np.int64), getattr(ref, f).astype(np.int64)), (name, exact, f)
        T.close()
    D.close()
    G.close()


@pytest.mark.parametrize("name", ["edge", "star33", "star513", "middle", "K65", "skewed"])
def test_validation_finds_each_fault(sess, name):
    """One slot made wrong, at the first, a middle and the last edge: every
    kind of fault is refused, in whichever direction of the edge it lies."""
    g = GRAPHS[name]()
    src = np.repeat(np.arange(g.n), g.degrees())
    for e in {0, g.nnz // 2, g.nnz - 1}:
        v = int(src[e])
        row = g.row(v).astype(np.int64)
        bad = {"range": g.n, "loop": v}
        free = np.setdiff1d(np.arange(g.n), np.append(row, v))
        lo = int(g.nbr[e - 1]) if e > int(g.off[v]) else -1
        hi = int(g.nbr[e + 1]) if e + 1 < int(g.off[v + 1]) else g.n
        between = free[(free > lo) & (free < hi)]
        if between.size:
            bad["asymmetric"] = int(between[0])  # the row stays ascending
        if e + 1 < int(g.off[v + 1]):
            bad["duplicate"] = int(g.nbr[e + 1])
        for kind, x in bad.items():
            nbr = g.nbr.copy()
            nbr[e] = x
            with pytest.raises(A.AgisError) as err:
                sess.graph(g.off, nbr)
            assert err.value.code == A.AGIS_E_INVALID_CSR, (name, kind, e)
    sess.graph(g.off, g.nbr).close()
