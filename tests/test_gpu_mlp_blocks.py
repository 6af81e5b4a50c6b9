"""The network's passes at the sizes where the choice of block changes (32, 64
and 128 rows and columns) and at the blocks' edges, against the oracle that
rounds to BF16 at the same points; a training step against the same kernels'
gradients."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [([16, 16], 16), ([80, 528, 272], 48), ([64, 48, 16, 96], 272),
                                        ([512, 1024, 1024], 1024), ([32, 2064, 2048], 2048)])
def test_blocks_match_oracle(dims, batch):
    import torch
    from paper_2203_05027_amd import learn
    rng = np.random.default_rng(sum(dims) + batch)
    net = learn.MLP(dims, max_batch=batch, seed=1)
    w, b = net.params()
    b = (0.1 * rng.standard_normal(b.size)).astype(np.float32)
    net.set_params(w, b)
    ws, bs = net.split(w.astype(np.float64), b.astype(np.float64))
    x = rng.standard_normal((batch, dims[0])).astype(np.float32)
    t = rng.standard_normal((batch, dims[-1])).astype(np.float32)
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    y, (yo, _) = net.forward(xd).cpu().numpy(), M.forward(ws, bs, x, bf16=True)
    # FP32 sums of up to 2064 terms; an activation within their rounding of a
    # BF16 boundary can move by 2^-8 of itself
    assert np.linalg.norm(y - yo) <= 1e-3 * np.linalg.norm(yo)
    gw, gb, loss = net.gradients(xd, td)
    lo, gws, gbs = M.loss_and_grads(ws, bs, x, t, bf16=True)
    assert loss == pytest.approx(lo, rel=1e-4)
    gwl, gbl = net.split(gw, gb)
    for l in range(len(dims) - 1):
        assert np.linalg.norm(gwl[l] - gws[l]) <= 2e-3 * np.linalg.norm(gws[l]), l
        assert np.linalg.norm(gbl[l] - gbs[l]) <= 2e-3 * np.linalg.norm(gbs[l]), l
    # the step's gradients are these, and its loss this one
    assert net.train_step(xd, td, lr=1e-2) == loss
    w1, b1 = net.params()
    pw, _, _ = M.adam_step(w.astype(np.float64), gw.astype(np.float64), 0, 0, 1, lr=1e-2)
    pb, _, _ = M.adam_step(b.astype(np.float64), gb.astype(np.float64), 0, 0, 1, lr=1e-2)
    np.testing.assert_allclose(w1, pw, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(b1, pb, rtol=1e-5, atol=1e-6)
