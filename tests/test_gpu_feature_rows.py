"""GPU: the learned proposal's features at the edges of the kernels that take
a vertex (a lane, a wave with 1 to 16 registers, a workgroup whose rows stay
in registers or are read again)."""

import numpy as np
import pytest

import oracle
import synth
from oracle import mlp

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")

DEGREES = [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 4095, 4096, 4097,
           9000]


def _graph():
    """Hub i has DEGREES[i] neighbours, drawn from 10,000 vertices that have
    a few hundred edges among the first of them (so that h-indices differ)."""
    rng = np.random.Generator(np.random.PCG64(3))
    n, base = 10_000, 10_000
    u, v = [], []
    for i, d in enumerate(DEGREES):
        picks = rng.choice(n, size=d, replace=False)
        u += [base + i] * d
        v += picks.tolist()
    a = rng.integers(0, 300, 20_000)
    b = rng.integers(0, n, 20_000)
    return synth.csr_from_edges(n + len(DEGREES), np.r_[u, a], np.r_[v, b])


def test_features_at_row_edges():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    g = _graph()
    assert set(DEGREES) <= set(g.degrees()[10_000:].tolist())
    T = s.tables(s.graph(g.off, g.nbr), cv_seed=1)
    got = s.features(T).cpu().numpy().astype(np.float64)
    ref = mlp.features(g, oracle.Tables(g, cv_seed=1))
    # float32 values of log2(1 + x) <= 64: half a unit in the last place is
    # 2^-19 at most, and the oracle's log2 rounds once in 64 bits
    np.testing.assert_allclose(got, ref, rtol=2.0 ** -23, atol=2.0 ** -40)
    s.close()
