"""The one-launch step of small 2D grids against the stage kernels it stands in
for (bit for bit: the same arithmetic per face and cell), at sizes around its
tiles' edges, for every kind of grid it takes; a non-default stage table
selects the stage kernels."""
import numpy as np
import pytest

import oracle
from paper_2306_14011_amd import inputs

pytestmark = pytest.mark.gpu

P, O, W, F = 0, 1, 2, 3
SIZES = [(1, 57), (2, 3), (7, 9), (8, 8), (12, 13), (16, 15), (17, 33), (63, 31), (97, 130), (129, 128), (200, 193),
         (300, 300)]


def spec_of(kind, nx, ny):
    """A grid and a smooth state of a kind of case."""
    g = inputs.grid2d(nx, ny, hi=(1.0, 1.0))
    rng = np.random.default_rng(nx * 1000 + ny)
    x, y, _ = g.centres()
    a = rng.uniform(0.05, 0.15, 4)
    s = np.sin(2 * np.pi * (x + 0.3)) * np.cos(2 * np.pi * (y - 0.2))
    c = np.cos(2 * np.pi * x + 0.7) * np.sin(4 * np.pi * y)
    u0 = 0.0 if kind in ("box", "viscous") else 2.6
    U = inputs.primitive_to_conserved(g, 1.0 + a[0] * s, (u0 + a[1] * c, a[2] * s), 1.0 + a[3] * c)
    if kind == "periodic":
        pass
    elif kind == "open":
        g.bc = ((O, O), (O, O), (P, P))
    elif kind in ("box", "viscous"):
        g.bc = ((W, W), (W, W), (P, P))
    elif kind in ("channel", "curved"):
        g.bc = ((F, O), (W, W if kind == "channel" else O), (P, P))
        q = np.zeros((3, 2, 4))
        q[0, 0] = [1.0, 2.6, 0.0, 2.5 + 0.5 * 2.6 ** 2]
        g.bc_state = q
    elif kind == "inflow_y":
        g.bc = ((P, P), (F, O), (P, P))
        q = np.zeros((3, 2, 4))
        q[1, 0] = [1.0, 0.1, 2.6, 2.5 + 0.5 * (2.6 ** 2 + 0.01)]
        g.bc_state = q
        U = U[[0, 2, 1, 3]].copy()
    if kind == "viscous":
        g.mu = 1e-3
    if kind == "curved":
        g.nodes = inputs.wavy_nodes(nx, ny, hi=(1.0, 1.0), amp=0.03)
    return g, U


def run(g, U0, steps, stages, dt_in=None, source=None):
    import torch
    from paper_2306_14011_amd import fv
    s = fv.Solver(g)
    s.set_path(fv.FV_PATH_FUSED)
    if stages:
        seg, _ = s.get_fused_launch()
        s.set_fused_launch(seg, [1 << 20] * 3)
    s.set_state(U0)
    if source is not None:
        s.set_source(source)
    dts = torch.zeros(sum(steps), dtype=torch.float64, device="cuda")
    at = 0
    for n in steps:
        di = torch.as_tensor(dt_in[at:at + n]).cuda() if dt_in is not None else None
        s.step(n, dt_in=di, dt_out=dts[at:at + n])
        at += n
    rc, flags = s.status()
    out = s.get_state()
    s.close()
    return out, dts.cpu().numpy(), flags


def skip(kind, nx, ny):
    return min(nx, ny) < 2 and kind in ("box", "viscous", "channel", "curved")


@pytest.mark.parametrize("kind", ["periodic", "open", "box", "channel", "inflow_y", "viscous", "curved"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_one_launch_gives_the_bits_of_the_stages(kind, nx, ny):
    if skip(kind, nx, ny):
        pytest.skip("walls need two cells")
    g, U0 = spec_of(kind, nx, ny)
    a = run(g, U0, (1, 2, 3), False)
    b = run(g, U0, (1, 2, 3), True)
    assert a[2] == 0 and b[2] == 0
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[0], b[0])


@pytest.mark.parametrize("limiter,kappa", [(True, -1.0), ("vanleer", -1.0), (False, -1.0), (False, 1.0 / 3.0)])
def test_schemes_source_and_frozen_steps(limiter, kappa):
    g, U0 = spec_of("periodic", 75, 41)
    g.limiter, g.kappa = limiter, kappa
    S = inputs.smooth_source(g, 1)
    for src in (None, S):
        a = run(g, U0, (4,), False, source=src)
        b = run(g, U0, (4,), True, source=src)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        d = 0.9 * a[1]
        c = run(g, U0, (1, 3), False, dt_in=d, source=src)
        e = run(g, U0, (1, 3), True, dt_in=d, source=src)
        assert np.array_equal(c[0], e[0]) and np.array_equal(c[1], d)


def test_matches_oracle_and_flags():
    from paper_2306_14011_amd import fv
    g, U0 = spec_of("channel", 50, 37)
    got, dts, flags = run(g, U0, (5,), False)
    ref, rdts, _ = oracle.run(g, U0, 5)
    assert flags == 0 and np.allclose(dts, rdts, rtol=1e-13, atol=0)
    for v in range(4):
        assert np.abs(got[v] - ref[v]).max() <= 1e-11 * np.abs(ref[v]).max()
    # a non-physical cell in the first state is reported, with the step size given or not
    bad = U0.copy()
    bad[3, 0, 5, 7] = 0.0
    for dt_in in (None, dts):
        assert run(g, bad, (1,), False, dt_in=dt_in)[2] & fv.FV_FLAG_P


def test_replays_of_a_captured_call():
    import torch
    from paper_2306_14011_amd import fv
    for steps in (1, 2, 3, 4):
        g, U0 = spec_of("channel", 70, 45)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            s = fv.Solver(g)
            s.set_path(fv.FV_PATH_FUSED)
            s.set_state(U0)
            s.step(steps)
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                s.step(steps)
        e = fv.Solver(g)
        e.set_path(fv.FV_PATH_FUSED)
        e.set_state(U0)
        e.step(steps)
        for _ in range(4):
            graph.replay()
            torch.cuda.synchronize()
            e.step(steps)
            assert np.array_equal(s.get_state(), e.get_state())
        s.close()
        e.close()
