"""Chained launch of small minibatches against the step and accumulation launches, which per-launch timing
selects: the same objects and per-position objectives bit for bit."""

import numpy as np
import pytest

from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,levels,batch,step,epochs", [
    (16, 1, 1, 5, 2),      # one grid, single positions
    (16, 5, 8, 4, 10),     # the largest minibatch of the smallest chained plan; chunks of epochs
    (16, 3, 5, 9, 2),      # a short last minibatch
    (32, 2, 4, 6, 2),      # the largest of its plan
    (32, 5, 3, 11, 2),     # the deepest in-wave hierarchy
    (32, 6, 1, 9, 2),      # V-cycle through LDS: no spare groups
    (64, 3, 1, 16, 2),
    (64, 7, 1, 21, 1),
])
def test_chained_equals_two_launches(m, levels, batch, step, epochs):
    rng = np.random.default_rng(1000 + m + levels)
    c = Case(rng, 2 * m + 21, 2 * m + 8, m, step, noise=0.05)
    # windows in a corner each, and one position measured twice
    c.offs[0] = c.offs[1]
    c.offs[-1] = (c.n_rows - m, c.n_cols - m)
    got = []
    for timing in (False, True):
        g = c.gpu(levels, 0.5)
        g.set_timing(timing)
        g.run_epochs(epochs, batch, seed=5)
        got.append((g.get_object(), g.step_phi(), g.epoch_index))
        g.close()
    assert np.array_equal(got[0][0].view(np.uint32), got[1][0].view(np.uint32))
    assert np.array_equal(got[0][1], got[1][1]) and got[0][2] == got[1][2] == epochs
