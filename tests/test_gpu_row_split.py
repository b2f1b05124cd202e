"""The library's own split of the rows of a 2D grid (heights that are not
multiples of four, ragged last items) against explicit heights, bit for bit,
and against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2306_14011_amd import inputs
from tests.test_gpu_whole_step import spec_of

pytestmark = pytest.mark.gpu

# above the one-launch step's sizes; the split takes 2, 3, 5, 10, 14 and 19 rows
SIZES = [(400, 361), (70, 2501), (768, 771), (1024, 1023), (1500, 1103), (3328, 1025)]


def run(g, U0, table):
    import torch
    from paper_2306_14011_amd import fv
    s = fv.Solver(g)
    s.set_path(fv.FV_PATH_FUSED)
    if table:
        s.set_fused_launch(*table)
    s.set_state(U0)
    dts = torch.zeros(2, dtype=torch.float64, device="cuda")
    s.step(2, dt_out=dts)
    _, flags = s.status()
    out = s.get_state(), dts.cpu().numpy(), s.get_fused_launch()
    s.close()
    assert flags == 0
    return out


@pytest.mark.parametrize("kind", ["periodic", "channel", "viscous", "curved"])
@pytest.mark.parametrize("n", SIZES, ids=["x".join(map(str, n)) for n in SIZES])
def test_own_split_of_the_rows(n, kind):
    g, U = spec_of(kind, *n)
    own, dts, (seg, waves) = run(g, U, None)
    assert all(s % 4 == 0 for s in seg) and list(waves) == [0, 0, 0]
    for table in (([28, 36, 32], [0, 0, 0]), (seg, [777, 1000, 1 << 20])):
        got, d, _ = run(g, U, table)
        assert np.array_equal(own, got) and np.array_equal(dts, d), table
    if n[0] * n[1] < 400000:
        ref, rdt, _ = oracle.run(g, U, 2)
        assert np.allclose(dts, rdt, rtol=1e-13, atol=0)
        for v in range(4):
            assert np.abs(own[v] - ref[v]).max() <= 1e-11 * np.abs(ref[v]).max(), v


@pytest.mark.parametrize("kind", ["periodic", "viscous"])
@pytest.mark.parametrize("sizes", [[(64, 31), (61, 130)], [(200, 150), (333, 77), (128, 256), (90, 301)],
                                   [(700, 500), (400, 640), (1000, 333)],
                                   # more than one round of resident waves: advanced in groups
                                   [(1000, 900), (64, 31), (1000, 901), (600, 1500), (1000, 900), (1020, 910)]],
                         ids=["2", "4", "3", "groups"])
def test_own_split_of_a_batch(sizes, kind):
    from paper_2306_14011_amd import fv
    specs, states = zip(*[spec_of(kind, *n) for n in sizes])
    import torch
    outs = []
    for segs in (None, "timed", [4 * (3 + q) for q in range(len(sizes))], [28] * len(sizes)):
        B = fv.Batch(specs)
        if segs == "timed":
            B.set_timing(5)
            segs = None
        if segs:
            B.set_schedule(segs)
        reported, _, nitems = B.info()
        assert all(s % 4 == 0 for s in reported) and (segs is None or reported == segs)
        if segs:
            assert nitems == sum(-(-n[0] // 60) * -(-n[1] // s) for n, s in zip(sizes, segs))
        for q, U in enumerate(states):
            B.view(q).copy_(torch.as_tensor(np.ascontiguousarray(U)).view(B.view(q).shape))
        B.step(3)
        B.step(2)
        outs.append([B.view(q).cpu().numpy() for q in range(len(sizes))] + [B.dt()])
        B.close()
    for other in outs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(outs[0], other))
