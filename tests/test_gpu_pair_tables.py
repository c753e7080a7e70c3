"""GPU: the pair-hub tables at the edges of their panels and eighths, and
the core-pair lists, through the samples that read them."""

import numpy as np
import pytest

import oracle
import synth
from oracle.pattern import compile_pattern

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


def _hub_graph(hubs, leaves, seed):
    """`hubs` vertices of degree >= 64, each with a random share of `leaves`
    low-degree vertices and of the other hubs, ids mixed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = hubs + leaves
    per = np.maximum(70, (90 * (1.0 - rng.random(hubs)) ** -0.5).astype(np.int64))
    per = np.minimum(per, n // 2)
    u = np.repeat(np.arange(hubs), per)
    v = rng.integers(0, n, u.size)
    perm = rng.permutation(n)
    return synth.csr_from_edges(n, perm[u], perm[v])


# hubs around one word (32), the first full panel (2,048) and its remainder
@pytest.mark.parametrize("hubs", [3, 33, 64, 129, 2047, 2049, 2300])
def test_pair_tables_against_oracle(sess, hubs):
    g = _hub_graph(hubs, 6 * hubs + 200, seed=hubs)
    G = sess.graph(g.off, g.nbr)
    T = sess.tables(G, cv_seed=1)
    OT = oracle.Tables(g, cv_seed=1)
    idx = np.arange(1500, dtype=np.uint64)
    for name in ("4-cycle", "5-cycle", "house", "4-clique"):
        p = synth.named_pattern(name)
        for mode in ("switch", "uniform"):
            smp = oracle.Sampler(g, OT, compile_pattern(p.k, p.edges, mode=mode), seed=5)
            got, ref = sess.dump(G, T, p, 5, idx, mode=mode, rowtab="on"), smp.records(idx)
            for f in ("v", "num", "den", "x", "steps", "fail_step"):
                assert np.array_equal(got[f], ref[f]), (hubs, name, mode, f)
            st, _, _ = smp.run(0, 4000)
            r = sess.estimate(G, T, p, 4000, 5, mode=mode, rowtab="on")
            assert abs(r.estimate - st.mean) <= 1e-9 * abs(st.mean), (hubs, name, mode)
    T.close()
    G.close()


def test_recycled_buffers_and_handles_that_outlive_their_context():
    """Tables built from buffers of destroyed ones hold nothing of them, the
    kept memory goes back on request, and tables destroyed after their
    context give their memory back."""
    import torch
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    big, small = _hub_graph(2100, 9000, seed=1), _hub_graph(2050, 8800, seed=2)
    idx = np.arange(500, dtype=np.uint64)
    p = synth.named_pattern("house")
    for g in (big, small, big):
        G = s.graph(g.off, g.nbr)
        T = s.tables(G, cv_seed=1)
        smp = oracle.Sampler(g, oracle.Tables(g, cv_seed=1), compile_pattern(p.k, p.edges, mode="switch"), seed=5)
        got, ref = s.dump(G, T, p, 5, idx, mode="switch", rowtab="on"), smp.records(idx)
        for f in ("v", "num", "den", "x", "steps", "fail_step"):
            assert np.array_equal(got[f], ref[f]), f
        T.close()
        G.close()
    kept = torch.cuda.mem_get_info()[0]
    s.release_scratch()
    assert torch.cuda.mem_get_info()[0] > kept
    G = s.graph(big.off, big.nbr)
    T = s.tables(G, cv_seed=1)
    s.close()
    held = torch.cuda.mem_get_info()[0]
    T.close()
    G.close()
    assert torch.cuda.mem_get_info()[0] > held
