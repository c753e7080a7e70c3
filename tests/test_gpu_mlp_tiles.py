"""GPU: the gradient of the network against FP64 at the edges of its tiles
(64 rows) and of the workgroups' shares of them, and training on one
minibatch and on several."""

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


def _set(rows, seed):
    import torch
    from paper_2601_01388_amd.session import mlp_init
    rng = np.random.Generator(np.random.PCG64(seed))
    n = 500
    feats = (rng.random((n, 4)) * 8).astype(np.float32)
    host = {"vtx": rng.integers(0, n, rows).astype(np.int32), "cls": rng.integers(0, 6, rows).astype(np.uint8),
            "target": rng.normal(0, 1, rows).astype(np.float32),
            "weight": (1 + rng.integers(0, 50, rows)).astype(np.float32)}
    params = mlp_init(seed, 0.1)
    dev = {k: torch.from_numpy(v).cuda() for k, v in host.items()}
    dev["rows"] = rows
    return feats, host, params, dev


# FP32 sums of up to 40,000 rows against FP64: each gradient entry is a sum of
# rounded products, so its error is a few units of 2^-24 of the sum of their
# absolute values, which is at most some hundred times the largest entry here
REL = 1e-4


@pytest.mark.parametrize("rows", [1, 2, 63, 64, 65, 127, 4096, 4097, 512 * 64 - 1, 512 * 64, 512 * 64 + 1, 40_000])
def test_gradient_at_tile_edges(sess, rows):
    import torch
    feats, host, params, dev = _set(rows, rows)
    d_feats, d_params = torch.from_numpy(feats).cuda(), torch.from_numpy(params).cuda()
    g, loss = sess.mlp_grad(d_params, d_feats, dev)
    x = mlp.inputs(feats, host["vtx"], host["cls"])
    ws = float(host["weight"].astype(np.float64).sum())
    rloss = mlp.loss(params.astype(np.float64), x, host["target"], host["weight"], ws)
    rg = mlp.grad(params.astype(np.float64), x, host["target"], host["weight"], ws)
    scale = np.abs(rg).max()
    assert np.abs(g.cpu().numpy() - rg).max() <= REL * scale
    assert loss == pytest.approx(rloss, rel=REL)
    g2, _ = sess.mlp_grad(d_params, d_feats, dev)
    assert torch.equal(g, g2)


def test_training_on_one_and_several_minibatches(sess):
    import torch
    rows = 3000
    feats, host, params, dev = _set(rows, 9)
    d_feats = torch.from_numpy(feats).cuda()
    for batch in (rows, 5000, 1000, 999):
        out = []
        for _ in range(2):
            p = torch.from_numpy(params).cuda()
            losses = sess.mlp_train(p, d_feats, dev, epochs=6, batch=batch, lr=3e-3, seed=4)
            out.append((p, np.asarray(losses)))
        assert torch.equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
        assert out[0][1][-1] < out[0][1][0]
        # the first epoch's first loss is the loss at the initial parameters
        if batch >= rows:
            _, loss = sess.mlp_grad(torch.from_numpy(params).cuda(), d_feats, dev)
            assert out[0][1][0] == pytest.approx(loss, rel=1e-6)
