"""The fused network kernels at the edges of their 16-row tiles, of the number
of gradient shares and of the host staging, against the FP64 reference."""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2205_06557_amd import binding
    return binding


def _net(B, seed):
    net = B.Mlp(seed)
    net.set_normalization(-np.ones(5), np.ones(5), np.zeros(16), np.ones(16))
    p = (np.random.default_rng(seed).normal(size=M.N_PARAMS) * 0.15).astype(np.float32)
    net.set_params(p)
    return net, p.astype(np.float64)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 8191, 16384, 16385])
def test_predict_rows(B, n):
    net, p = _net(B, 21)
    X = np.random.default_rng(n).uniform(-1.01, 1.01, size=(n, 5)).astype(np.float32)
    Y, inside = net.predict(X)
    Yr, _ = M.forward(p, X.astype(np.float64))
    assert np.linalg.norm(Y - Yr) < 2e-6 * np.linalg.norm(Yr)
    assert np.array_equal(inside, (np.abs(X) <= 1).all(axis=1))


# one row, around one tile, around 32 tiles (one per gradient share), the largest
@pytest.mark.parametrize("n", [1, 16, 17, 511, 512, 513, 4096])
def test_gradient_rows(B, n):
    net, p = _net(B, 22)
    rng = np.random.default_rng(n)
    X = rng.uniform(-1, 1, size=(n, 5)).astype(np.float32)
    T = rng.normal(size=(n, 16)).astype(np.float32)
    L, g = net.loss_grad(X, T)
    Lr, gr = M.loss_grad(p, X.astype(np.float64), T.astype(np.float64))
    assert L == pytest.approx(Lr, rel=1e-5)
    k = 0
    for (i, o) in M.SIZES:
        for m in (i * o, o):
            assert np.linalg.norm(g[k:k + m] - gr[k:k + m]) < 1e-4 * np.linalg.norm(gr[k:k + m])
            k += m
