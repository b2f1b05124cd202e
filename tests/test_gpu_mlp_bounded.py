"""Waits of the training kernel's workgroups for each other, forced to end early
from the host: where they do not meet, one computes every share with the
bits of the shared run; where a later wait is given up, the call says so and
leaves the network as it was."""
import numpy as np
import pytest

from paper_2306_14011_amd import fv
from test_gpu_mlp_workgroups import Run, same

pytestmark = pytest.mark.gpu


def launch(r, roll_polls, wait_polls):
    import torch
    N = r.net
    fv.fv_mlp_train_bounded(N.params.data_ptr(), N.n_in, N.m.data_ptr(), N.v.data_ptr(), N.t.data_ptr(),
                            r.dev[0].data_ptr(), r.dev[1].data_ptr(), r.n, r.dev[2].data_ptr(), r.hp,
                            r.loss.data_ptr(), r.ne.data_ptr(), r.ws.data_ptr() + r.shift, r.bytes, roll_polls,
                            wait_polls, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()


# 64 rows: one workgroup, which waits for nothing; 65, 200, 449: two, four and
# eight; 1100: shares of more than a chunk
@pytest.mark.parametrize("n_in", [14, 16])
@pytest.mark.parametrize("batch", [64, 65, 200, 449, 1100])
def test_shares_computed_by_one_alone(batch, n_in):
    import torch
    n = 2 * batch + 3   # the last minibatch has 3 rows: shares of none
    a, b = Run(n, n_in, batch, 2), Run(n, n_in, batch, 2, shift=4, fill=0xff)
    a.launch(torch.cuda.current_stream())
    torch.cuda.synchronize()
    launch(b, 0, 1 << 20)
    assert int(b.ne.item()) == 2 and same(a.state(), b.state())


@pytest.mark.parametrize("batch", [64, 65, 200, 600])
def test_lost_wait_is_reported(batch):
    r = Run(2 * batch, 14, batch, 2)
    before = r.state()
    launch(r, 1 << 20, 0)
    if batch == 64:  # nothing to lose
        assert int(r.ne.item()) == 2 and int(r.net.t.item()) == 4
        return
    assert int(r.ne.item()) == -1
    assert same(r.state()[:4], before[:4])  # params, moments, step counter
    # and the same buffers train afterwards
    launch(r, 1 << 20, 1 << 20)
    e = Run(2 * batch, 14, batch, 2)
    launch(e, 1 << 20, 1 << 20)
    assert int(r.ne.item()) == 2 and same(r.state(), e.state())


def test_network_raises_when_a_wait_is_lost(monkeypatch):
    from paper_2306_14011_amd.autotune import Network
    full = fv.fv_mlp_train_bounded
    monkeypatch.setattr(fv, "fv_mlp_train", lambda *a: full(*a[:-1], 1 << 20, 0, a[-1]))
    rng = np.random.default_rng(0)
    X, y = rng.standard_normal((300, 14)).astype(np.float32), rng.standard_normal(300).astype(np.float32)
    net = Network(0)
    before = net.params.clone()
    with pytest.raises(RuntimeError, match="lost each other"):
        net.train(X, y, max_epochs=1)
    assert (net.params == before).all()
