"""The tile kernel of the fused schedule (chosen for small batches) against
its row march (chosen by a forced segment length): the same node arithmetic,
so the states are equal bitwise, in every storage mode and with both forms of
Step (2), on grids around the edges of the tiles and in batches that reach
each tile shape.  The sums of E(u) and of the printed E(P) add the same
positive FP64 terms in another order: for n terms that is at most n ulp
relative (2.3e-16 each)."""
import numpy as np
import pytest

import paper_2306_07603_amd as M

pytestmark = pytest.mark.gpu

PRECISIONS = ["fp64", "fp32", "fp16dev", "fp32x", "fp32sr", "fp32srf"]
# one tile, remainders of one node over the tile sizes, tall and wide, several tiles with and without a wall
GRIDS = [(5, 5), (8, 8), (9, 8), (15, 17), (16, 5), (5, 31), (24, 24), (25, 26), (33, 47), (49, 12), (73, 50)]
# (grid, count): the smallest batches past 512 tiles of shape 0 (8 x 8 nodes) and of shape 1 (24 x 8)
BATCHES = [((65, 65), 8), ((129, 97), 8), ((257, 257), 5)]


def run(cav, precision, rows, steps, **opt):
    o = M.ifdlbm_default_options(precision=precision, segment_rows=rows, residual_every=steps, **opt)
    h = M.ifdlbm_create(cav, o)
    M.ifdlbm_step(h, steps)
    return h


def compare(cav, precision, steps, **opt):
    a, b = run(cav, precision, 0, steps, **opt), run(cav, precision, 16, steps, **opt)
    for c in range(len(cav)):
        (Fa, La), (Fb, Lb) = M.ifdlbm_get_state(a, c), M.ifdlbm_get_state(b, c)
        assert np.array_equal(Fa, Fb) and np.array_equal(La, Lb), c
    n = max(c.n_xi * c.n_eta for c in cav)
    for x, y in ((M.ifdlbm_get_residuals(a)[0], M.ifdlbm_get_residuals(b)[0]),
                 (M.ifdlbm_get_pressure_residuals(a)[0], M.ifdlbm_get_pressure_residuals(b)[0])):
        assert np.all(np.isfinite(x)) and np.all(np.abs(x - y) <= 2.3e-16 * n * np.abs(y))


@pytest.mark.parametrize("implicit", [0, 1])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_tile_equals_march_bitwise(precision, implicit):
    for nx, ny in GRIDS:
        print(precision, implicit, nx, ny, flush=True)
        compare([M.Cavity(nx, ny, 300.0, 0.7, 50.0)], precision, 11, lambda_mode=implicit)


@pytest.mark.parametrize("batched", [1, 0])
@pytest.mark.parametrize("precision", ["fp64", "fp32srf", "fp32"])
def test_tile_shapes_equal_march_bitwise(precision, batched):
    for (nx, ny), count in BATCHES:
        print(precision, batched, nx, ny, count, flush=True)
        compare([M.Cavity(nx, ny, 100.0 + 300.0 * c, 0.6 + 0.1 * c, 90.0 - 5.0 * c) for c in range(count)], precision, 6,
                batched=batched)


# remainders on both axes; tiles of 24 x 8 and of 24 x 24 (shapes 1 and 2): the columns and rows of a tile, and the batch
LARGER = [((131, 99), 4, (24, 8)), ((259, 251), 2, (24, 24))]


@pytest.mark.parametrize("batched", [1, 0])
@pytest.mark.parametrize("implicit", [0, 1])
@pytest.mark.parametrize("precision", PRECISIONS)
def test_larger_tiles_equal_march_in_every_mode(precision, implicit, batched):
    for (nx, ny), count, (cols, rows) in LARGER:
        print(precision, implicit, batched, nx, ny, flush=True)
        cavs = [M.Cavity(nx, ny, 100.0 + 300.0 * c, 0.6 + 0.1 * c, 90.0 - 5.0 * c) for c in range(count)]
        h = M.ifdlbm_create(cavs, M.ifdlbm_default_options(precision=precision))
        assert M.ifdlbm_info(h)["work_items"] == count * -(-nx // cols) * -(-ny // rows)
        h.close()
        compare(cavs, precision, 6, lambda_mode=implicit, batched=batched)
