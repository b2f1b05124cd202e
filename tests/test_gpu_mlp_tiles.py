"""The network's training, gradient and prediction kernels at the edges of
their row tiles (16, 32 and 128 rows) and of minibatches, against the FP64
oracle."""
import numpy as np
import pytest

from oracle import mlp
from paper_2306_14011_amd import inputs

pytestmark = pytest.mark.gpu


def problem(n, n_in, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, n_in)).astype(np.float32).astype(np.float64)
    y = (0.3 * np.sin(X[:, 0]) + 0.2 * X[:, 3] * X[:, n_in - 1]).astype(np.float32).astype(np.float64)
    return X, y


@pytest.mark.parametrize("n_in", [14, 16])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 96, 127, 128, 129, 200, 256, 257, 1000])
def test_gradient_and_prediction_at_row_counts(n, n_in):
    from paper_2306_14011_amd.autotune import Network
    X, y = problem(n, n_in, n)
    N = Network(n, n_in=n_in)
    theta = N.params.cpu().numpy().astype(np.float64)
    L, g = N.loss_grad(X, y, 1e-2)
    Lr, gr = mlp.loss_grad(theta, X, y, 1e-2)
    # FP32 sums of up to 1000 rows and 64 neurons: some 1e-6 of their size
    assert abs(L - Lr) <= 1e-5 * abs(Lr)
    assert np.abs(g - gr).max() <= 1e-5 * np.abs(gr).max()
    out = N.predict(X)
    ref = mlp.predict(theta, X)
    assert np.abs(out - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("n,batch", [(1, 200), (5, 1), (40, 33), (129, 128), (150, 149), (130, 400), (300, 257)])
def test_minibatches_track_oracle(n, batch):
    from paper_2306_14011_amd.autotune import Network
    X, y = problem(n, 14, n + batch)
    order = inputs.epoch_orders(n, 2, 1)
    N = Network(7)
    theta = N.params.cpu().numpy().astype(np.float64)
    losses = N.train(X, y, order=order, max_epochs=2, batch=batch)
    ref, lref, ne, _, _, _ = mlp.train(theta, X, y, order, max_epochs=2, batch=batch)
    assert len(losses) == ne == 2
    assert np.allclose(losses, lref, rtol=1e-4, atol=0)
    # Adam moves every weight by up to lr a step whatever its gradient: a weight
    # whose gradient is FP32 noise may go the other way
    steps = 2 * -(-n // batch)
    d = np.abs(N.params.cpu().numpy() - ref)
    assert d.max() <= 2 * 9e-4 * steps
    assert np.linalg.norm(d) <= 1e-3 * np.linalg.norm(ref - theta)
    assert int(N.t.item()) == steps


def test_no_epochs_leave_the_network():
    from paper_2306_14011_amd.autotune import Network
    X, y = problem(20, 14, 0)
    N = Network(1)
    before = N.params.clone()
    losses = N.train(X, y, order=np.zeros((1, 20), dtype=np.int32), max_epochs=0)
    assert len(losses) == 0 and bool((N.params == before).all()) and int(N.t.item()) == 0
