"""Training shared by several workgroups, at the minibatch sizes where their
number changes: against the FP64 oracle, repeatable bit for bit, from any
scratch (misaligned, with old contents), on two streams at once, and replayed
from a graph."""
import numpy as np
import pytest

from oracle import mlp
from paper_2306_14011_amd import fv, inputs

pytestmark = pytest.mark.gpu

BATCHES = [64, 65, 128, 129, 193, 321, 448, 449, 600]


def problem(n, n_in, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, n_in)).astype(np.float32)
    return X, (0.3 * np.sin(X[:, 0]) + 0.2 * X[:, 3] * X[:, n_in - 1]).astype(np.float32)


class Run:
    """Device buffers of one fv_mlp_train call."""

    def __init__(self, n, n_in, batch, epochs, shift=0, fill=0):
        import torch
        from paper_2306_14011_amd.autotune import Network
        self.X, self.y = problem(n, n_in, n + batch)
        self.order = inputs.epoch_orders(n, epochs, 1)
        self.net = Network(7, n_in=n_in)
        self.first = self.net.params.cpu().numpy().astype(np.float64)
        self.dev = [torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in (self.X, self.y, self.order.astype(np.int32))]
        self.hp = fv.fv_mlp_hparams(9e-4, 0.95, 0.90, 1e-9, 1e-4, 1e-6, batch, epochs, 10, 0)
        self.bytes = fv.fv_mlp_workspace(min(batch, n))
        self.ws = torch.full((self.bytes + 64,), fill, dtype=torch.uint8, device="cuda")
        self.shift, self.n = shift, n
        self.loss = torch.zeros(epochs, device="cuda")
        self.ne = torch.zeros(1, dtype=torch.int32, device="cuda")

    def launch(self, stream):
        N = self.net
        fv.fv_mlp_train(N.params.data_ptr(), N.n_in, N.m.data_ptr(), N.v.data_ptr(), N.t.data_ptr(),
                        self.dev[0].data_ptr(), self.dev[1].data_ptr(), self.n, self.dev[2].data_ptr(), self.hp,
                        self.loss.data_ptr(), self.ne.data_ptr(), self.ws.data_ptr() + self.shift, self.bytes,
                        stream.cuda_stream)

    def state(self):
        N = self.net
        return [a.cpu().numpy() for a in (N.params, N.m, N.v, N.t, self.loss, self.ne)]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("n_in", [14, 16])
@pytest.mark.parametrize("batch", BATCHES)
def test_shared_minibatches(batch, n_in):
    import torch
    n, epochs = 2 * batch + 3, 2   # the last minibatch has 3 rows: fewer than workgroups
    s = torch.cuda.current_stream()
    a, b = Run(n, n_in, batch, epochs), Run(n, n_in, batch, epochs, shift=4, fill=0xff)
    a.launch(s)
    b.launch(s)
    torch.cuda.synchronize()
    assert same(a.state(), b.state())
    ref, lref, ne, _, _, _ = mlp.train(a.first, a.X.astype(np.float64), a.y.astype(np.float64), a.order,
                                       max_epochs=epochs, batch=batch)
    assert int(a.ne.item()) == ne == epochs and int(a.net.t.item()) == 3 * epochs
    assert np.allclose(a.loss.cpu().numpy(), lref, rtol=1e-4, atol=0)
    # Adam moves every weight by up to lr a step whatever its gradient: a weight
    # whose gradient is FP32 noise may go the other way
    d = np.abs(a.net.params.cpu().numpy() - ref)
    assert d.max() <= 2 * 9e-4 * 3 * epochs
    assert np.linalg.norm(d) <= 1e-3 * np.linalg.norm(ref - a.first)


def test_two_streams_at_once():
    import torch
    alone = [Run(900, 14, b, 3) for b in (200, 500)]
    for r in alone:
        r.launch(torch.cuda.current_stream())
    torch.cuda.synchronize()
    runs = [Run(900, 14, b, 3) for b in (200, 500)]
    torch.cuda.synchronize()
    for r in runs:
        r.launch(torch.cuda.Stream())
    torch.cuda.synchronize()
    for r, a in zip(runs, alone):
        assert same(r.state(), a.state())


def test_replayed_from_a_graph():
    import torch
    g, e = Run(500, 14, 200, 2), Run(500, 14, 200, 2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.launch(torch.cuda.current_stream())
    for _ in range(3):
        graph.replay()
        e.launch(torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert same(g.state(), e.state())
