"""GPU: the sampler's slot queue at its edges (fewer slots than parts, than
waves, one more or less than what is dealt without the counters, uneven
parts): every slot is run exactly once, whatever the launch shape."""

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
    g = synth.chung_lu(n=2000, m=12_000, seed=5)
    G = s.graph(g.off, g.nbr)
    yield s, G, s.tables(G, cv_seed=1)
    s.close()


# (triangle: a wave a sample; 3-star under switching: a lane a sample)
@pytest.mark.parametrize("name", ["triangle", "3-star"])
@pytest.mark.parametrize("samples", [1, 3, 31, 33, 127, 4095, 4097, 8191, 8192, 8193, 65_537, 300_001])
def test_every_slot_once(state, name, samples):
    s, G, T = state
    p = synth.named_pattern(name)

    def run(seed, blocks_per_cu, grab):
        s.set_launch(True, blocks_per_cu, grab, 2, 0)
        r = s.estimate(G, T, p, samples, seed, mode="switch")
        return r.n, r.n_nonzero, r.estimate, r.variance

    want = run(1, 0, 0)
    for shape in ((0, 1), (1, 3), (1, 100)):
        other = run(2, *shape)  # leaves other weights in the buffers
        assert samples < 100 or other != want
        assert run(1, *shape) == want
