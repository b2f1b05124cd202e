"""The 3D stage kernels around the edges of their 32 x 7 tiles and segments, for
each face-state rule with and without walls and an inflow face, against the
oracle; segment heights and workgroup counts change no bit; the automatic
segment height."""
import numpy as np
import pytest

import oracle
from paper_2306_14011_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [(31, 6, 3), (32, 7, 4), (33, 8, 5), (64, 15, 9), (5, 40, 2), (96, 3, 13)]
P, O, W, F = 0, 1, 2, 3


def spec_of(kind, n):
    g = inputs.grid3d(*n)
    rng = np.random.default_rng(sum(n))
    x, y, z = g.centres()
    a = rng.uniform(0.02, 0.08, 5)
    s = np.sin(2 * np.pi * (x + 0.3)) * np.cos(2 * np.pi * (y - 0.2)) + np.cos(2 * np.pi * z)
    c = np.cos(2 * np.pi * x + 0.7) * np.sin(4 * np.pi * y) * np.cos(2 * np.pi * (z + 0.1))
    U = inputs.primitive_to_conserved(g, 1.0 + a[0] * s, (a[1] * c, a[2] * s, a[3] * c), 1.0 + a[4] * c)
    if kind == "periodic":
        g.bc = ((P, P), (P, P), (P, P))
    else:
        g.bc = ((W, O), (W, W), (F, W))
        q = np.zeros((3, 2, 5))
        q[2, 0] = (1.0, 0.1, 0.0, 0.4, 2.5 + 0.5 * 0.17)
        g.bc_state = q
    return g, U


# Two steps are six stages of about 300 roundings each on values of order one,
# through slopes and wave speeds that amplify an error by less than 50:
# 6 x 300 x 1.1e-16 x 50 = 1e-11; dt is one such chain without the fluxes.
@pytest.mark.parametrize("limiter", [True, "vanleer", False], ids=["minmod", "vanleer", "unlimited"])
@pytest.mark.parametrize("kind", ["periodic", "walls"])
@pytest.mark.parametrize("n", SIZES, ids=["x".join(map(str, n)) for n in SIZES])
def test_stage_kernels_at_tile_edges(n, kind, limiter):
    import torch
    from paper_2306_14011_amd import fv
    g, U = spec_of(kind, n)
    g.limiter = limiter
    outs = []
    for seg, waves in (([0, 0, 0], [0, 0, 0]), ([4, 8, 16], [4, 0, 9])):
        s = fv.Solver(g)
        s.set_path(fv.FV_PATH_FUSED, 0, 0)
        s.set_fused_launch(seg, waves)
        s.set_state(U)
        dts = torch.zeros(2, dtype=torch.float64, device="cuda")
        s.step(2, dt_out=dts)
        _, flags = s.status()
        assert flags == 0
        outs.append((s.get_state(), dts.cpu().numpy()))
        s.close()
    ref, rdt, _ = oracle.run(g, U, 2, limiter=limiter)
    assert np.allclose(outs[0][1], rdt, rtol=1e-13, atol=0)
    for v in range(5):
        err = np.abs(outs[0][0][v] - ref[v]).max()
        assert err <= 1e-11 * np.abs(ref[v]).max(), (v, err)
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("n", [(8, 8, 8), (97, 61, 45), (130, 120, 110), (256, 256, 256)])
def test_automatic_segment_height(n):
    # the busiest compute unit's items times their planes plus one, 1.4 times
    # as slow for a lone item; the tallest multiple of 4 within 1 % of the least
    import torch
    from paper_2306_14011_amd import fv
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def cost(seg):
        per_cu = -(-(-(-n[0] // 32) * -(-n[1] // 7) * -(-n[2] // seg)) // cus)
        return per_cu * (seg + 1) * (1.4 if per_cu == 1 else 1.0)

    segs = range(4, 257, 4)
    least = min(cost(q) for q in segs)
    s = fv.Solver(inputs.grid3d(*n))
    s.set_path(fv.FV_PATH_FUSED, 0, 0)
    got = s.get_path()[1]
    s.close()
    assert got == max(q for q in segs if cost(q) <= 1.01 * least)
