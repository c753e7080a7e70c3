"""GPU: the gradient of the network where a parameter or an input is not
finite: the entries that are not numbers are those of the FP64 reference,
also where the weight belongs to a position class that no row has."""

import numpy as np
import pytest

from oracle import mlp

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


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("where", ["unused class", "used class", "feature weight", "feature"])
def test_gradient_of_values_that_are_not_finite(sess, where, value):
    import torch
    from paper_2601_01388_amd.session import mlp_init
    rng = np.random.Generator(np.random.PCG64(11))
    n, rows = 50, 130
    feats = (1 + rng.random((n, 4)) * 8).astype(np.float32)
    host = {"vtx": rng.integers(0, n, rows).astype(np.int32), "cls": np.zeros(rows, dtype=np.uint8),
            "target": rng.normal(0, 1, rows).astype(np.float32), "weight": np.ones(rows, dtype=np.float32)}
    params = mlp_init(5, 0.1)
    if where == "feature":
        feats[host["vtx"][7], 1] = value
    else:
        params[5 * 8 + {"unused class": 6, "used class": 4, "feature weight": 1}[where]] = value
    dev = {k: torch.from_numpy(v).cuda() for k, v in host.items()}
    dev["rows"] = rows
    g, loss = sess.mlp_grad(torch.from_numpy(params).cuda(), torch.from_numpy(feats).cuda(), dev)
    with np.errstate(all="ignore"):
        x = mlp.inputs(feats, host["vtx"], host["cls"])
        rg = mlp.grad(params.astype(np.float64), x, host["target"], host["weight"], float(rows))
        rloss = mlp.loss(params.astype(np.float64), x, host["target"], host["weight"], float(rows))
    assert np.array_equal(np.isnan(g.cpu().numpy()), np.isnan(rg))
    assert np.isnan(loss) == np.isnan(rloss)
