"""Probe step at the edges of its kernels: minibatches that end in a chunk of one slot or fill their chunks,
regions of the probe's hierarchy from 16 pixels to the whole probe, replayed epochs."""

import numpy as np
import pytest

import oracle
from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,levels,batch,alternate,graph", [
    (8, 4, 1, False, False),      # the smallest probe, one slot
    (16, 1, 17, False, True),     # a chunk of one slot, no coarse level, replayed
    (32, 6, 16, True, False),     # whole chunks, the deepest hierarchy (one region)
    (64, 4, 33, False, False),    # 16 regions of 16 pixels
    (128, 5, 18, True, True),     # 64 regions of 16 pixels, the split probe table, replayed
])
def test_probe_step_edges(m, levels, batch, alternate, graph):
    from paper_2504_10118_amd import GRAPH, PROBE_ALTERNATE, UPDATE_PROBE
    rng = np.random.default_rng(800 + m)
    c = Case(rng, m + 40, m + 31, m, 7, noise=0.05)
    q0 = (c.Q32 * (1 + 0.1 * (rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))))).astype(np.complex64)
    orders = [rng.permutation(c.n_pos).astype(np.int32) for _ in range(2)]
    g = c.gpu(levels, 0.5)
    g.set_probe(q0)
    g.set_flags(UPDATE_PROBE | (PROBE_ALTERNATE if alternate else 0) | (GRAPH if graph else 0), 0.2)
    g.run_epochs(2, batch, order=np.stack(orders))
    z, q = g.get_object().astype(np.complex128), g.get_probe().astype(np.complex128)
    g.close()
    zo, qo = oracle.run_epochs_blind(c.z0, q0.astype(np.complex128), c.offs, c.sd, 0.5, levels, orders, batch, 0.2,
                                     alternate=alternate)
    # the repository's per-step bound, over the few dependent steps of these runs
    assert c.rel(z, zo) <= 1e-5
    assert np.linalg.norm(q - qo) <= 1e-5 * np.linalg.norm(qo)
