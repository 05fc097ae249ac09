"""The adjoint and the tangent sweep on grids around the edges of their tiles
(8 and 12 nodes), against the complex-step derivative of the CPU oracle: both
are the derivative of the same discrete map to rounding (1e-9 relative per
parameter, 1e-12 on J, the bars of the other comparisons with it)."""
import numpy as np
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


@pytest.mark.parametrize("precision", ["fp32", "fp32x", "fp32sr", "fp32srf", "fp16dev"])
def test_adjoint_clear_of_the_walls_in_the_storage_modes(precision):
    """The reverse kernel's copy for tiles clear of the walls (past 256 tiles of 12 x 12) reads the stored states: two
    checkpoint segments of the FP64 step linearised about the trajectory of the storage mode, against the oracle's step by
    the complex step from each of that trajectory's states (the bars of the FP64 comparison).  One call per step draws
    the random words that the adjoint draws."""
    import ctypes
    import math

    from oracle import complex_step as CS
    nx, ny, steps, hs = 205, 194, 6, 1e-20
    re, n, th, u = 120.0, 0.8, 55.0, 0.1
    cav, o = M.Cavity(nx, ny, re, n, th, u), M.ifdlbm_default_options(precision=precision, rho0=0.0)
    h = M.ifdlbm_create([cav], o)
    states = [M.ifdlbm_get_state(h, 0)]
    for _ in range(steps):
        M.ifdlbm_step(h, 1)
        states.append(M.ifdlbm_get_state(h, 0))
    h.close()
    L, p, g_ref = CS.lib(), O.Params(nx=nx, ny=ny, re=re, n=n, theta_deg=th, u_lid=u, rho0=0.0), []
    for dx in ({"theta_deg": hs * 180.0 / math.pi}, {"n": hs}, {"u_lid": hs}):
        c = CS._cparams(p, dx)
        F, lam = np.zeros((9, ny, nx), dtype=np.complex128), np.zeros((ny, nx), dtype=np.complex128)
        assert L.orc_init(ctypes.byref(c), F.ctypes.data, lam.ctypes.data) == 0
        for t, (f, l) in enumerate(states):
            F.real, lam.real = f, l
            if t < steps:
                assert L.orc_run(ctypes.byref(c), F.ctypes.data, lam.ctypes.data, 1, None, None) == 0
        J = CS._C()
        L.orc_kinetic_energy_into(ctypes.byref(c), F.ctypes.data, ctypes.byref(J))
        J_ref = J[0]
        g_ref.append(J[1] / hs)
    J, g = M.ifdlbm_adjoint(cav, o, steps, 3)
    print(precision, J, J_ref, g, g_ref, flush=True)
    assert abs(J - J_ref) <= 1e-12 * J_ref
    for q in range(3):
        assert abs(g[q] - g_ref[q]) <= 1e-9 * abs(g_ref[q]), q


def test_tangent_of_a_very_tall_grid():
    """More rows of tiles (of 12 nodes) than the second dimension of a launch holds (65536 workgroups): two steps of the
    tangent sweep against the adjoint, derivatives of one discrete map (the bars of the other comparison of the two)."""
    cav, o = M.Cavity(5, 12 * 65536 + 17, 100.0, 0.8, 60.0), M.ifdlbm_default_options()
    (Jt, gt), (Ja, ga) = M.ifdlbm_gradient(cav, o, 2), M.ifdlbm_adjoint(cav, o, 2, 2)
    print(Jt, gt, Ja, ga, flush=True)
    assert abs(Ja - Jt) <= 1e-11 * abs(Jt)
    for q in range(3):
        assert abs(ga[q] - gt[q]) <= 1e-9 * abs(gt[q]) + 1e-13 * np.abs(gt).max(), q


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32x"])
def test_adjoint_on_packed_rows_by_march_and_tiles(precision):
    """The trajectories of these modes have rows that start anywhere: the march (forced) and the tiles store the same bits
    there, so J and the gradient are equal, on widths one over and under a multiple of 16 and of the strip."""
    for nx, ny in ((17, 23), (31, 18), (57, 40), (113, 19)):
        cav = M.Cavity(nx, ny, 200.0, 0.8, 65.0)
        (Ja, ga), (Jb, gb) = (M.ifdlbm_adjoint(cav, M.ifdlbm_default_options(precision=precision, segment_rows=rows), 14, 5)
                              for rows in (0, 16))
        print(precision, nx, ny, Ja, ga, flush=True)
        assert Ja == Jb and np.array_equal(ga, gb) and np.all(np.isfinite(ga))
