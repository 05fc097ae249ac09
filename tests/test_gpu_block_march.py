"""The FP64 row march of the fused schedule (workgroups of four wavefronts,
four rows at a time) against the tile kernel: the same node arithmetic, so the
states are equal bitwise at every segment length (forced: whole chunks of four
rows and every remainder) and where the march is the automatic choice.  The
sums of E(u) add the same positive FP64 terms in another order: for n terms
that is at most n ulp relative (2.3e-16 each)."""
import numpy as np
import pytest

import paper_2306_07603_amd as M

pytestmark = pytest.mark.gpu

# one strip and several, one column or row past the strip (56) or chunk
GRIDS = [(5, 5), (56, 16), (57, 19), (61, 66), (113, 45)]


def state(cavs, precision, rows, steps, **opt):
    h = M.ifdlbm_create(cavs, M.ifdlbm_default_options(precision=precision, segment_rows=rows, residual_every=steps, **opt))
    M.ifdlbm_step(h, steps)
    out = [M.ifdlbm_get_state(h, c) for c in range(len(cavs))], M.ifdlbm_get_residuals(h)[0]
    h.close()
    return out


def check(a, b, nodes):
    for (fa, la), (fb, lb) in zip(a[0], b[0]):
        assert np.array_equal(fa, fb) and np.array_equal(la, lb)
    assert np.all(np.isfinite(a[1])) and np.all(np.abs(a[1] - b[1]) <= 2.3e-16 * nodes * np.abs(b[1]))


@pytest.mark.parametrize("precision", ["fp64", "fp32x", "fp32sr"])
def test_segment_lengths_equal_tile_bitwise(precision):
    for nx, ny in GRIDS:
        cavs = [M.Cavity(nx, ny, 200.0, 0.8, 65.0)]
        ref = state(cavs, precision, 0, 9)
        for rows in (8, 9, 10, 11, 20, 4096):
            print(precision, nx, ny, rows, flush=True)
            check(state(cavs, precision, rows, 9), ref, nx * ny)


@pytest.mark.parametrize("batched", [1, 0])
def test_automatic_march_of_a_batch(batched):
    """Past the tiles: cavities of several sizes in one launch, and with a launch each."""
    sizes = [(257, 257)] * 9 + [(513, 129), (65, 33), (129, 513)] + [(1025, 1025)]
    cavs = [M.Cavity(nx, ny, 100.0 + 50.0 * c, 0.6 + 0.05 * c, 90.0 - 3.0 * c) for c, (nx, ny) in enumerate(sizes)]
    check(state(cavs, "fp64", 0, 3, batched=batched), state(cavs, "fp64", 24, 3), 1025 * 1025)
