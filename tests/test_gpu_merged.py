"""Merged launches (a minibatch's steps with the previous minibatch's update) against the step and accumulation
launches, which per-launch timing selects: the same objects and per-position objectives bit for bit."""

import numpy as np
import pytest

from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,rows,cols,step,levels,batch,epochs", [
    (16, 90, 131, 9, 3, 13, 1),     # an odd number of minibatches, a short last one
    (16, 90, 131, 9, 1, 26, 2),     # an even number
    (16, 240, 250, 9, 5, 256, 10),  # the largest minibatch, several chunks of epochs
    (16, 33, 700, 5, 2, 64, 1),     # windows in a few rows: many overlap
    (32, 128, 128, 12, 2, 8, 3),
    (32, 403, 390, 17, 6, 128, 2),  # V-cycle through LDS
])
def test_merged_equals_two_launches(m, rows, cols, step, levels, batch, epochs):
    rng = np.random.default_rng(1200 + m + batch)
    c = Case(rng, rows, cols, m, step, noise=0.05)
    c.offs[0] = c.offs[1]                        # one position measured twice
    c.offs[-1] = (rows - m, cols - m)            # a window in the corner
    got = []
    for timing in (False, True):
        g = c.gpu(levels, 0.5)
        g.set_timing(timing)
        g.run_epochs(epochs, batch, seed=7)
        g.run_minibatch(np.arange(5, dtype=np.int32))     # the context is left as after two launches
        g.run_epochs(1, max(1, batch // 2), seed=8)
        got.append((g.get_object(), g.step_phi()))
        g.close()
    assert np.array_equal(got[0][0].view(np.uint32), got[1][0].view(np.uint32))
    assert np.array_equal(got[0][1], got[1][1])
