"""Batches of many small grids: the same bits as the grids advanced alone, and no
work in a stage that one workgroup does for all grids."""
import numpy as np
import pytest

from paper_2306_14011_amd import fv
from tests.test_gpu_whole_step import spec_of

pytestmark = pytest.mark.gpu

# one to sixteen wave-speed slots a grid, one to several work items
SHAPES = [(8, 8), (16, 61), (32, 32), (33, 32), (61, 40), (64, 33), (90, 70), (130, 100)]


def fill(B, states):
    import torch
    for g, U in enumerate(states):
        B.view(g).copy_(torch.as_tensor(np.ascontiguousarray(U)).view(B.view(g).shape))


@pytest.mark.parametrize("kind", ["periodic", "channel", "viscous"])
def test_many_grids_as_alone(kind):
    kinds = [spec_of(kind, *n) for n in SHAPES]
    alone = []
    for g, U in kinds:
        s = fv.Solver(g)
        s.set_path(fv.FV_PATH_FUSED, 16)
        s.set_state(U)
        s.step(5)
        alone.append(s.get_state().reshape(4, -1))
        s.close()
    n = 1203
    B = fv.Batch([kinds[q % len(kinds)][0] for q in range(n)])
    fill(B, [kinds[q % len(kinds)][1] for q in range(n)])
    for steps in (1, 3, 1):
        B.step(steps)
    assert B.status()[1] == 0
    for q in range(n):
        assert np.array_equal(B.view(q).cpu().numpy().reshape(4, -1), alone[q % len(kinds)]), q
    B.close()


# more than one round of resident waves: middling grids (advanced in groups by
# calls of four steps or more) and large ones (by every call)
@pytest.mark.parametrize("shapes, n", [([(192, 191), (190, 215)], 111), ([(251, 260), (300, 310)], 61)],
                         ids=["middling", "large"])
@pytest.mark.parametrize("kind", ["periodic", "viscous"])
def test_groups_of_grids_as_alone(kind, shapes, n):
    kinds = [spec_of(kind, *s) for s in shapes]
    alone = []
    for g, U in kinds:
        s = fv.Solver(g)
        s.set_path(fv.FV_PATH_FUSED, 16)
        s.set_state(U)
        s.step(8)
        alone.append(s.get_state().reshape(4, -1))
        s.close()
    for calls in ((8,), (1, 5, 2)):
        B = fv.Batch([kinds[q % 2][0] for q in range(n)])
        fill(B, [kinds[q % 2][1] for q in range(n)])
        for steps in calls:
            B.step(steps)
        assert B.status()[1] == 0
        for q in range(n):
            assert np.array_equal(B.view(q).cpu().numpy().reshape(4, -1), alone[q % 2]), (calls, q)
        B.close()


@pytest.mark.parametrize("n", [1, 700, 4096])
def test_second_stage_takes_no_longer_than_the_others(n):
    g, U = spec_of("periodic", 8, 8)
    B = fv.Batch([g] * n)
    fill(B, [U] * n)
    B.set_timing(9)
    B.step(9)
    assert B.status()[1] == 0
    clk = B.clocks()  # (steps, grids, stages, 2)
    span = np.median(clk[..., 1].max(axis=1) - clk[..., 0].min(axis=1), axis=0)
    assert span[1] <= 2 * max(span[0], span[2]), span
    B.close()
