"""The adjoint and the tangent sweep on grids around the edges of their tiles
(8 and 12 nodes), against the complex-step derivative of the CPU oracle: both
are the derivative of the same discrete map to rounding (1e-9 relative per
parameter, 1e-12 on J, the bars of the other comparisons with it)."""
import pytest

import oracle as O
import paper_2306_07603_amd as M

pytestmark = pytest.mark.gpu

# one tile, one node over and under a tile, tall and wide, and grids with tiles clear of the walls (launched apart
# past 256 tiles of 12 x 12)
GRIDS = [(5, 5, 12), (8, 9, 12), (12, 13, 12), (17, 5, 12), (5, 26, 12), (25, 24, 12), (37, 14, 10), (48, 49, 8),
         (205, 194, 5)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "%dx%d" % g[:2])
def test_gradients_at_tile_edges(grid):
    from oracle import complex_step as CS
    nx, ny, steps = grid
    re, n, th, u = 120.0, 0.8, 55.0, 0.1
    p = O.Params(nx=nx, ny=ny, re=re, n=n, theta_deg=th, u_lid=u, rho0=0.0)
    J_ref, g_ref = CS.kinetic_energy_gradient(p, steps)
    cav, o = M.Cavity(nx, ny, re, n, th, u), M.ifdlbm_default_options(rho0=0.0)
    for name, (J, g) in (("adjoint", M.ifdlbm_adjoint(cav, o, steps, 5)), ("tangent", M.ifdlbm_gradient(cav, o, steps))):
        print(name, nx, ny, J, J_ref, g, g_ref, flush=True)
        assert abs(J - J_ref) <= 1e-12 * J_ref, name
        for q in range(3):
            assert abs(g[q] - g_ref[q]) <= 1e-9 * abs(g_ref[q]), (name, q)
