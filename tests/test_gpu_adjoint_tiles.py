"""The 2D adjoint step at grid sizes around its tiles' edges (16 x 12 cells),
for every boundary kind and limiter rule, against the FP64 oracle's reverse."""
import numpy as np
import pytest

import oracle
from paper_2306_14011_amd import inputs

pytestmark = pytest.mark.gpu

P, O, W, F = 0, 1, 2, 3


def case(bc, nx, ny):
    g = inputs.grid2d(nx, ny, hi=(1.0, 1.0), bc=bc)
    rng = np.random.default_rng(nx * 100 + ny)
    # rough data: no two neighbouring differences tie, so the limiter's
    # selections do not depend on rounding
    rho, p = 1.0 + 0.2 * rng.uniform(-1, 1, (2,) + g.shape[1:])
    u, v = 0.5 * rng.uniform(-1, 1, (2,) + g.shape[1:])
    U = inputs.primitive_to_conserved(g, rho, (u, v), p)
    if F in bc[0] + bc[1]:
        q = np.zeros((3, 2, 4))
        q[...] = [1.1, 0.4, 0.3, 2.9]
        g.bc_state = q
    return g, U, rng.standard_normal(g.shape)


@pytest.mark.parametrize("limiter,kappa", [(True, -1.0), ("vanleer", -1.0), (False, -1.0), (False, 1.0 / 3.0)])
@pytest.mark.parametrize("bc", [((P, P), (P, P)), ((O, O), (W, W)), ((W, W), (O, F)), ((F, O), (P, P))])
@pytest.mark.parametrize("nx,ny", [(3, 2), (15, 11), (16, 12), (17, 13), (18, 25), (33, 14)])
def test_adjoint_step_matches_oracle(nx, ny, bc, limiter, kappa):
    import torch
    from paper_2306_14011_amd import fv
    g, U, lam = case(bc, nx, ny)
    g.limiter, g.kappa = limiter, kappa
    dt = 0.2 * oracle.dt(g, U)[0]
    ref = oracle.rk3_step_vjp(g, U, dt, lam, limiter=limiter, kappa=kappa)
    s = fv.Solver(g)
    s.set_state(U)
    d = torch.full((1,), dt, dtype=torch.float64, device="cuda")
    L = torch.as_tensor(lam).cuda()
    fv.fv_adjoint_step(s.ctx, s.U.data_ptr(), d.data_ptr(), L.data_ptr())
    got = L.cpu().numpy()
    s.close()
    for v in range(4):
        assert np.abs(got[v] - ref[v]).max() <= 1e-10 * np.abs(ref[v]).max(), v
