"""GPU: a batch of patterns of unequal cost in one launch: the launch takes
less time in the sampler than its patterns one after the other (the slot
counters run through the patterns side by side), with the same results."""

import pytest

import synth

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")


@pytest.fixture(scope="module")
def state():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    g = synth.rmat(12, 16, seed=2)
    G = s.graph(g.off, g.nbr)
    T = s.tables(G, cv_seed=1)
    yield s, G, T
    s.close()


# the launches alone leave the chip idle at their ends and take 0.59 and 0.95
# ms together, the batch 0.35 and 0.71 (0.76 and 1.56 where the waves of a
# cheap pattern all went on with one counter of a dear one)
@pytest.mark.parametrize("samples", [20_000, 50_000])
def test_batch_takes_less_than_its_patterns_alone(state, samples):
    s, G, T = state
    pats = [synth.named_pattern(n) for n in ("house", "4-clique", "5-cycle", "triangle")]

    def kernel_seconds(ps):
        runs = [s.estimate_batch(G, T, ps, [samples] * len(ps), 4, mode="switch") for _ in range(6)]
        return min(sum(r.sample_kernel_seconds for r in run) for run in runs), runs[0]

    together, batch = kernel_seconds(pats)
    alone = 0.0
    for i, p in enumerate(pats):
        sec, _ = kernel_seconds([p])
        alone += sec
        one = s.estimate(G, T, p, samples, 4, mode="switch", pattern_id=i)
        assert (one.estimate, one.variance, one.n) == (batch[i].estimate, batch[i].variance, batch[i].n)
    print(f"[gpu-test] {samples} samples: together {together * 1e3:.3f} ms, alone {alone * 1e3:.3f}", flush=True)
    assert together < alone
