"""GPU: the work-queue launch against the rounds with full minibatches.

Reconstructions of 512 to 1024 pixels, 64 x 64 and 128 x 128 probes, minibatches of 256, from
the flat start: thousands of workgroups of different plans share the chip, and the waves of a
workgroup drift apart in ways that small scans do not show.  Every run of either form must
give the same objects, bit for bit.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_queue_equals_rounds_full_minibatches():
    import torch

    from paper_2504_10118_amd import PERSISTENT, Magpie, run_epochs_multi
    from synth import batched_workload, make_batched_inputs, poisson_counts_device
    specs = batched_workload()
    specs = [s for s in specs if s.m == 64][:16] + [s for s in specs if s.m == 128][:8]
    ctxs, batches = [], []
    for sp in specs:
        z, q, offs, _ = make_batched_inputs(sp)
        c = Magpie(sp.n, sp.n, sp.m, sp.levels, 0.5, device=0)
        c.set_probe(q.astype(np.complex64))
        c.set_positions(offs)
        d = torch.empty((sp.n_pos, sp.m, sp.m), dtype=torch.float32, device="cuda")
        c.forward_model(z.astype(np.complex64), out=d)
        c.sync()
        counts = poisson_counts_device(d, sp.peak, sp.seed)
        torch.cuda.synchronize()
        c.load_intensities(counts, is_sqrt=False)
        c.sync()
        ctxs.append(c)
        batches.append(sp.batch)
    assert max(batches) == 256

    def run(flags):
        for sp, c in zip(specs, ctxs):
            c.set_flags(flags)
            c.set_object(np.ones((sp.n, sp.n), dtype=np.complex64))
            c.epoch_index = 0
        run_epochs_multi(ctxs, 40, batches, seed=2504)
        return [c.get_object().view(np.uint64) for c in ctxs]

    ref = run(0)
    for name, flags in (("rounds", 0), ("queue", PERSISTENT), ("queue", PERSISTENT)):
        got = run(flags)
        differing = [(sp.m, sp.n, int((a != b).sum())) for sp, a, b in zip(specs, got, ref) if (a != b).any()]
        print(name, "reconstructions", len(specs), "differing", differing, flush=True)
        assert not differing
    for c in ctxs:
        c.close()
