"""The range of densities that the flux takes: every operation of a step is
homogeneous in the conserved state, so a state times a power of two gives the
result times that power, bit for bit, up to densities whose products come near
the ends of double precision."""
import numpy as np
import pytest

from paper_2306_14011_amd import fv, inputs
from tests.test_gpu_whole_step import spec_of

pytestmark = pytest.mark.gpu


def run(g, U, path, table):
    import torch
    s = fv.Solver(g)
    s.set_path(path)
    if table:
        s.set_fused_launch([28, 28, 28], [0, 0, 0])
    s.set_state(U)
    dts = torch.zeros(2, dtype=torch.float64, device="cuda")
    s.step(2, dt_out=dts)
    flags = s.status()[1]
    out = s.get_state(), dts.cpu().numpy(), flags
    s.close()
    return out


@pytest.mark.parametrize("power", [-506, -300, 300, 506])
@pytest.mark.parametrize("kind, path", [("periodic", "split"), ("periodic", "one launch"), ("periodic", "stages"),
                                        ("channel", "stages"), ("3d", "stages"), ("3d", "split")])
def test_state_times_a_power_of_two(kind, path, power):
    if kind == "3d":
        g = inputs.grid3d(24, 11, 9)
        rng = np.random.default_rng(5)
        sh = g.shape[1:]
        U = inputs.primitive_to_conserved(g, 1 + 0.2 * rng.random(sh), tuple(0.3 * rng.random(sh) for _ in range(3)),
                                          1 + 0.2 * rng.random(sh))
    else:
        g, U = spec_of(kind, 61, 50)
    code = fv.FV_PATH_SPLIT if path == "split" else fv.FV_PATH_FUSED
    table = path == "stages" and kind != "3d"
    ref, dts, flags = run(g, U, code, table)
    assert flags == 0
    f = 2.0 ** power
    if kind == "channel":
        g.bc_state = np.asarray(g.bc_state) * f
    got, dtp, flags = run(g, U * f, code, table)
    assert flags == 0
    assert np.array_equal(dtp, dts) and np.array_equal(got, ref * f)
