"""GPU: tables of graphs with few hubs of very long rows: their samples against
the oracle (rows past 524,280 neighbours are counted with more bit planes),
and their time, which one workgroup's walk of such a row must not set."""

import time

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


def _hubs(shares, leaves, seed):
    """One hub per share, joined to the other hubs and to that share of the
    leaves; ids mixed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    h = len(shares)
    u, v = [], []
    for i, share in enumerate(shares):
        w = h + rng.choice(leaves, int(share * leaves), replace=False)
        u += [np.full(w.size, i), np.full(h - 1 - i, i)]
        v += [w, np.arange(i + 1, h)]
    perm = rng.permutation(h + leaves)
    return synth.csr_from_edges(h + leaves, perm[np.concatenate(u)], perm[np.concatenate(v)])


@pytest.mark.parametrize("shares,leaves", [((1.0, 0.9), 600_000), ((1.0, 0.7, 0.02), 700_000), ((0.5, 0.4, 0.3), 200_000)])
def test_samples_over_long_rows_against_oracle(sess, shares, leaves):
    g = _hubs(shares, leaves, seed=len(shares))
    G = sess.graph(g.off, g.nbr)
    T = sess.tables(G, cv_seed=1)
    OT = oracle.Tables(g, cv_seed=1)
    idx = np.arange(150, dtype=np.uint64)
    for name in ("4-cycle", "diamond"):
        p = synth.named_pattern(name)
        for mode in ("switch", "uniform"):
            smp = oracle.Sampler(g, OT, compile_pattern(p.k, p.edges, mode=mode), seed=5)
            got, ref = sess.dump(G, T, p, 5, idx, mode=mode, rowtab="on"), smp.records(idx)
            for f in ("v", "num", "den", "x", "steps", "fail_step"):
                assert np.array_equal(got[f], ref[f]), (shares, name, mode, f)
    T.close()
    G.close()


def test_tables_of_one_hub_take_no_multiple_of_a_ring(sess):
    # the ring has as many slots; 3.8 times as long, 16 with the hub's row
    # walked by four workgroups
    def tables_ms(g):
        import torch
        G = sess.graph(g.off, g.nbr)
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sess.tables(G, cv_seed=1).close()
            best = min(best, (time.perf_counter() - t0) * 1e3)
        G.close()
        return best

    star, ring = tables_ms(synth.star_graph(1 << 20)), tables_ms(synth.ring_graph(1 << 20))
    print(f"[gpu-test] star {star:.3f} ms, ring {ring:.3f}", flush=True)
    assert star <= 8 * ring
