"""Network input map at the edges of its kernels: tile heights, lists longer than the staged chunk,
odd and even map sides, a side of one cell, cells wider than a workgroup, ragged tiles."""

import numpy as np
import pytest

from gpu_cases import Case
from oracle import learned as ol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,m,step,side,tile", [
    (84, 84, 16, 9, 7, 8),        # odd side: unpaired columns only at zero frequency; ragged tiles
    (80, 112, 16, 8, 16, 16),     # cells of 5 x 7 pixels
    (64, 64, 32, 2, 32, 32),      # 289 windows over one tile: two staged chunks
    (48, 576, 8, 7, 2, 8),        # cells of 288 columns
    (300, 300, 64, 40, 1, 16),    # a single cell
    (256, 128, 128, 16, 64, 32),  # the largest side and probe
])
def test_input_map_edges(rows, cols, m, step, side, tile):
    c = Case(np.random.default_rng(rows + m), rows, cols, m, step, noise=0.05)
    g = c.gpu(2, 0.5)
    g.set_tuning(0, tile)
    got = g.input_map(side)
    want = ol.input_map(c.sd32.astype(np.float64), c.Q, c.offs, rows, cols, side)
    # FP64 sums rounded to FP32 once (6e-8 of each value); the phase channel is formed
    # from the rounded maps, so it carries their rounding times its largest gain, 1 / (2 pi / side)
    for ch in range(3):
        assert np.max(np.abs(got[ch] - want[ch])) <= 1.2e-7 * max(np.max(np.abs(want[ch])), 1e-12), ch
    slope = 2 * np.pi / m * max(np.max(np.abs(want[1])) * rows / side, np.max(np.abs(want[2])) * cols / side)
    assert np.max(np.abs(got[3] - want[3])) <= 1.2e-7 * (np.max(np.abs(want[3])) + 2 * side * slope)
    g.close()
