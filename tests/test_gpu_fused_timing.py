"""Launches that the event timing counts on the fused path."""
import pytest

from paper_2306_14011_amd import fv, inputs

pytestmark = pytest.mark.gpu

FUSED = fv.TIMERS.index("fused")


@pytest.mark.parametrize("steps", [1, 2, 3, 8])
@pytest.mark.parametrize("stages", [False, True])
def test_every_launch_of_the_steps_is_counted(steps, stages):
    g, U = inputs.vortex_case(64, seed=0)
    s = fv.Solver(g)
    s.set_path(fv.FV_PATH_FUSED)
    if stages:
        s.set_fused_launch([28, 28, 28], [0, 0, 0])
    s.set_state(U)
    s.set_timing(True)
    s.step(steps)
    ms, count = s.get_timing()
    s.close()
    # three stage launches a step; or one a step and, after an odd number of
    # steps, the copy of the state from the workspace
    want = 3 * steps if stages else steps + steps % 2
    assert count[FUSED] == want and sum(count) == want
    assert ms[FUSED] > 0.0
