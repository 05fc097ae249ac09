"""Cavities that stop (here by a non-finite state) take a batch from the row
march to the tiles: those left go on bitwise as in a batch of their own, in
eager steps and in replayed graphs."""
import numpy as np
import pytest

import paper_2306_07603_amd as M

pytestmark = pytest.mark.gpu

# (precision, cavities, cavities left, side): march of all, tiles of those left, which are more items
BATCHES = [("fp64", 40, 10, 129), ("fp32srf", 64, 15, 513)]


@pytest.mark.parametrize("graph", [0, 4])
@pytest.mark.parametrize("batch", BATCHES, ids=lambda b: b[0])
def test_those_left_step_as_if_alone(batch, graph):
    precision, n, left, side = batch
    cavs = [M.Cavity(side, side, 100.0 + 20.0 * c, 0.6 + 0.01 * c, 90.0 - 0.5 * c) for c in range(n)]
    opt = M.ifdlbm_default_options(precision=precision, graph_steps=graph, residual_every=4)
    items, states = [], []
    for k in (n, left):
        h = M.ifdlbm_create(cavs[:k], opt)
        items.append(M.ifdlbm_info(h)["work_items"])
        M.ifdlbm_step(h, 8)
        for c in range(left, k):
            M.ifdlbm_set_state(h, c, np.full((9, side, side), np.nan), np.ones((side, side)))
        M.ifdlbm_step(h, 4)
        M.ifdlbm_get_residuals(h)
        info = M.ifdlbm_info(h)
        print(precision, graph, k, items[-1], info["work_items"], info["n_active"], flush=True)
        assert info["n_active"] == left
        items[-1] = (items[-1], info["work_items"])
        M.ifdlbm_step(h, 11)
        assert np.all(np.isfinite(M.ifdlbm_get_residuals(h)[0][:left]))
        states.append([M.ifdlbm_get_state(h, c) for c in range(left)])
        h.close()
    assert items[0][0] < items[0][1] == items[1][1]
    for (fa, la), (fb, lb) in zip(*states):
        assert np.array_equal(fa, fb) and np.array_equal(la, lb)
