"""GPU: runs to epsilon whose later workgroups never join (short samples), all
join (long ones) or join for some of a batch's patterns, and launches of
fewer workgroups than one rank: the stop points and estimates are those of
the round-by-round run."""

import math

import pytest

import synth

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")

RUNS = {
    "short": (["3-star"], "always", 0.01),
    "long": (["5-clique"], "always", 0.01),
    "mixed": (["triangle", "house", "5-clique", "4-path"], "switch", 0.01),
}


@pytest.fixture(scope="module")
def state():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    g = synth.rmat(16, 16, seed=2)
    G = s.graph(g.off, g.nbr)
    T = s.tables(G, cv_seed=1)
    yield s, G, T
    s.close()


@pytest.mark.parametrize("blocks_per_cu", [0, 1, 3])
@pytest.mark.parametrize("case", sorted(RUNS))
def test_run_to_eps_equals_rounds(state, case, blocks_per_cu):
    s, G, T = state
    names, mode, eps = RUNS[case]
    pats = [synth.named_pattern(n) for n in names]
    kw = dict(mode=mode, eps=eps, delta=0.05, check_every=4096, min_samples=4096)
    s.set_launch(True, blocks_per_cu, 0, 0, 0)
    for budgets in ([200_000] * len(pats), [1000] * len(pats)):
        dev = s.estimate_batch(G, T, pats, budgets, 5, **kw)
        host = s.estimate_batch(G, T, pats, budgets, 5, host_rounds=True, **kw)
        for a, b in zip(dev, host):
            assert (a.n, a.n_nonzero, a.converged) == (b.n, b.n_nonzero, b.converged)
            assert math.isclose(a.estimate, b.estimate, rel_tol=1e-12)
            assert math.isclose(a.variance, b.variance, rel_tol=1e-12)
