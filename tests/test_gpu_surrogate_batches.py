"""Gradients and training at the edges of the batch tiles (16 rows of a
workgroup, 32 rows of a matrix-instruction chunk): batches of one row, just
below, at and just above the tiles, and the largest.  Bars as in the other
surrogate tests: 2e-2 norm-wise per parameter block against the FP64 reference
(BF16 products, FP32 accumulation), loss histories within 3e-2."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


def _weights(k, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(k):
        w = np.zeros(mlp.n_params())
        for W, b in mlp.unpack(w):
            W[:] = rng.uniform(-1, 1, W.shape) * np.sqrt(3.0 / W.shape[1])
            b[:] = rng.normal(0, 0.1, b.shape)
        out.append(w.astype(np.float32).astype(np.float64))
    return out


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 4096])
def test_gradients_at_batch_edges(n):
    from paper_1906_04722_amd import surrogate
    ws = _weights(2, seed=n)
    m = surrogate.Surrogate(members=2)
    for z, w in enumerate(ws):
        m.set_params(z, w)
    rng = np.random.default_rng(n + 1)
    X, T = rng.normal(size=(n, 80)), rng.normal(size=(n, 17))
    g, loss = m.grad(X, T)
    again, _ = m.grad(X, T)
    assert np.array_equal(g, again)
    for z, w in enumerate(ws):
        Y, cache = mlp.forward(w, X)
        ref = mlp.backward(w, cache, Y, T)
        assert abs(loss[z] - mlp.mse(Y, T)) <= 2e-2 * mlp.mse(Y, T)
        o = 0
        for l in range(4):
            nin, nout = mlp.LAYERS[l], mlp.LAYERS[l + 1]
            for size in (nout * nin, nout):
                a, b = g[z, o:o + size].astype(np.float64), ref[o:o + size]
                assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b), (z, l, size)
                o += size
        assert np.array_equal(m.get_params(z), w.astype(np.float32))  # unchanged


def test_training_with_a_ragged_last_batch_follows_the_reference():
    """70 samples in batches of 33, 33 and 4; predictions use the trained
    weights (their packed copies are refreshed by the update)."""
    from paper_1906_04722_amd import surrogate
    rng = np.random.default_rng(12)
    n, epochs, batch = 70, 3, 33
    X = rng.normal(size=(n, 80)) + 0.5
    T = np.tanh(X[:, :17] + X[:, 20:37]) * 2.0
    ws = _weights(2, seed=31)
    order = np.stack([np.stack([rng.permutation(n) for _ in range(2)]) for _ in range(epochs)])
    m = surrogate.Surrogate(members=2)
    for z, w in enumerate(ws):
        m.set_params(z, w)
    hist = m.train(X, T, epochs=epochs, batch=batch, lr=1e-3, order=order)
    ref_w = [w.copy() for w in ws]
    xs, ts, ref_hist = mlp.train(ref_w, X, T, order, batch, 1e-3, epochs)
    print("gpu", hist, "ref", ref_hist)
    assert np.allclose(hist, ref_hist, rtol=3e-2)
    mean, _ = m.predict(X)
    # the same weights in a fresh handle give the same answers
    q = surrogate.Surrogate(members=2)
    for z in range(2):
        q.set_params(z, m.get_params(z))
    q.set_stats(*m.get_stats())
    assert np.array_equal(q.predict(X)[0], mean)
    rmean, _ = mlp.predict(ref_w, xs, ts, X)
    assert np.linalg.norm(mean - rmean) <= 3e-2 * np.linalg.norm(rmean)
