"""GPU: training targets and rows at the edges of their chunks, against the
rows taken one vertex after another in 64 bits."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

A = pytest.importorskip("paper_2601_01388_amd")

ZERO = np.iinfo(np.int32).min


@pytest.fixture(scope="module")
def sess():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_01388_amd.session import Session
    s = Session(0)
    yield s
    s.close()


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("n", [1, 63, 257, 2047, 2048, 2049, 70_001])
def test_rows(sess, n, residual):
    import torch
    rng = np.random.Generator(np.random.PCG64(n))
    k, mask, least = 5, 0b10111, 2
    c = rng.integers(0, 5, (k, n)).astype(np.int32)
    c[1] = 0          # a step without rows
    c[2] = 7          # every vertex kept
    s = np.where(c > 0, rng.exponential(50.0, (k, n)), 0.0)
    s[4] = 0.0        # kappa falls back to 1
    b = rng.integers(-5 << 16, 9 << 16, (k, n)).astype(np.int32)
    b[0, ::3] = ZERO
    vtx, cls, tgt, wt = [], [], [], []
    for i in range(k):
        if not mask >> i & 1:
            continue
        keep = (c[i] >= least) & ~((b[i] == ZERO) & residual)
        v = np.flatnonzero(keep)
        sv, cv = s[i, v], c[i, v].astype(np.float64)
        if residual:
            B = np.exp2(b[i, v] / 65536.0)
            kappa = sv.sum() / (cv * B).sum() if sv.sum() > 0 else 1.0
            t = np.log2((sv / (kappa * B) + 1.0) / (cv + 1.0))
        else:
            t = np.log2(1.0 + sv / cv)
        vtx.append(v)
        cls.append(np.full(len(v), min(i, 3)))
        tgt.append(t)
        wt.append(cv)
    d = sess.device
    rows = sess.learn_rows(torch.from_numpy(s).to(d), torch.from_numpy(c).to(d), mask, least,
                           base=torch.from_numpy(b).to(d) if residual else None)
    assert rows["rows"] == sum(map(len, vtx))
    assert np.array_equal(rows["vtx"].cpu().numpy(), np.concatenate(vtx))
    assert np.array_equal(rows["cls"].cpu().numpy(), np.concatenate(cls))
    assert np.array_equal(rows["weight"].cpu().numpy(), np.concatenate(wt))
    # one rounding to float32 (2^-24 of the value); near zero the logarithm's
    # argument, off by a few 2^-53 and kappa's sum of n terms, counts absolutely
    np.testing.assert_allclose(rows["target"].cpu().numpy(), np.concatenate(tgt), rtol=2.0 ** -23, atol=1e-10)
