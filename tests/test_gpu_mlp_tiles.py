"""The cost model's matrix-core kernels at the edges of their tiles (32
samples a wave, four waves a work-group, one work-group a tile up to 256
tiles), against the FP64 network reference."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 256 * 32, 256 * 32 + 1,
                               256 * 4 * 32 + 31])
def test_forward_and_gradient_at_tile_edges(n):
    import torch
    import paper_2510_14147_amd as fnn
    from oracle import mlp
    rng = np.random.default_rng(n)
    th = (mlp.init(n) + 0.1 * rng.standard_normal(mlp.N_PARAMS)).astype(np.float32)
    x = rng.standard_normal((n, 16)).astype(np.float32)
    t = rng.standard_normal((n, 2)).astype(np.float32)
    dth, dx, dt = (torch.from_numpy(v).cuda() for v in (th, x, t))
    ref, (_, z1, h1, z2, h2) = mlp.forward(th, x)
    y = fnn.fnn_mlp_forward(dth, dx).cpu().numpy()
    # each layer sums at most 64 products: 66 roundings against the sum of
    # the products' magnitudes, three layers, and the activations' own (4)
    p = mlp.unpack(np.abs(th.astype(np.float64)))
    m1 = np.abs(x) @ p["W1"].T + p["b1"]
    m2 = m1 @ p["W2"].T + p["b2"]
    m3 = m2 @ p["W3"].T + p["b3"]
    assert np.all(np.abs(y - ref) <= 3 * 70 * U * m3)
    loss, g = fnn.fnn_mlp_loss_grad(dth, dx, dt)
    gref = mlp.backward(th, x, t)
    assert abs(loss - mlp.loss(th, x, t)) <= 1e-6 * loss
    # a mean over n samples of such products: the same roundings, and one per
    # addition along a chain (at most the samples of one wave, 256 rows, 4 waves)
    k = 3 * 70 + min(n, 32 * (n // (32 * 1024) + 1)) + 256
    assert np.abs(g.cpu().numpy() - gref).max() <= k * U * 4 * np.abs(gref).max() + 1e-7
    # a fixed order of summation: the same bits again
    l2, g2 = fnn.fnn_mlp_loss_grad(dth, dx, dt)
    assert l2 == loss and torch.equal(g, g2)
    # batches through an index: one epoch over one batch, then the same with
    # the smallest ragged batches, keep the loss
    q = dth.clone()
    ls = fnn.fnn_mlp_train(q, dx, dt, epochs=1, batch=n, lr=1e-3, seed=3)
    assert abs(ls[0] - loss) <= 1e-5 * loss
