"""Training minibatches of more rows than a workgroup holds at once (chunks of
128): shares of more than a chunk, of which some ranks have one chunk less than
others, and whole minibatches on the one workgroup that a stream restricted to
some of the compute units gets. Against the FP64 oracle."""
import ctypes

import numpy as np
import pytest

from oracle import mlp
from test_gpu_mlp_workgroups import Run, same

pytestmark = pytest.mark.gpu


def check(r, batch, epochs):
    steps = -(-r.n // batch) * epochs
    ref, lref, ne, _, _, _ = mlp.train(r.first, r.X.astype(np.float64), r.y.astype(np.float64), r.order,
                                       max_epochs=epochs, batch=batch)
    assert int(r.ne.item()) == ne == epochs and int(r.net.t.item()) == steps
    assert np.allclose(r.loss.cpu().numpy(), lref, rtol=1e-4, atol=0)
    # as for the smaller minibatches: Adam moves every weight by up to lr a step
    d = np.abs(r.net.params.cpu().numpy() - ref)
    assert d.max() <= 2 * 9e-4 * steps
    assert np.linalg.norm(d) <= 1e-3 * np.linalg.norm(ref - r.first)


# eight shares of 128 or 129, 137 or 138, 256 or 257, and 384 or 385 rows
@pytest.mark.parametrize("n_in", [14, 16])
@pytest.mark.parametrize("batch", [1025, 1100, 2050, 3075])
def test_shares_of_several_chunks(batch, n_in):
    import torch
    epochs = 2
    r = Run(2 * batch + 5, n_in, batch, epochs)
    r.launch(torch.cuda.current_stream())
    torch.cuda.synchronize()
    check(r, batch, epochs)


class MaskedStream:
    """A stream that may use half of the compute units."""

    def __init__(self):
        # the HIP runtime that the process has loaded
        path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
        self.hip = ctypes.CDLL(path)
        mask = (ctypes.c_uint32 * 8)(*[0x0000ffff] * 8)
        self.ptr = ctypes.c_void_p()
        assert self.hip.hipExtStreamCreateWithCUMask(ctypes.byref(self.ptr), ctypes.c_uint32(8), mask) == 0
        self.cuda_stream = self.ptr.value

    def synchronize(self):
        assert self.hip.hipStreamSynchronize(self.ptr) == 0

    def close(self):
        assert self.hip.hipStreamDestroy(self.ptr) == 0


@pytest.mark.parametrize("batch", [64, 129, 200, 300])
def test_restricted_stream(batch):
    import torch
    epochs = 2
    r, again = Run(2 * batch + 5, 14, batch, epochs), Run(2 * batch + 5, 14, batch, epochs, shift=4, fill=0xff)
    torch.cuda.synchronize()
    s = MaskedStream()
    try:
        r.launch(s)
        again.launch(s)
        s.synchronize()
    finally:
        s.close()
    check(r, batch, epochs)
    assert same(r.state(), again.state())
    # one workgroup writes nothing to the scratch
    assert int(again.ws.min().item()) == 0xff
