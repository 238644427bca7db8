"""Intensities and objects as callers hand them over: device arrays at any alignment of their type, invalid
values at either end, every plan's order."""

import numpy as np
import pytest

from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [8, 16, 32, 64, 128])
def test_unaligned_and_invalid_inputs(m):
    import torch
    from paper_2504_10118_amd import MagpieError, list_plans
    c = Case(np.random.default_rng(1100 + m), m + 20, m + 27, m, 9, noise=0.05)
    n = c.sd32.size
    g = c.gpu(1, 0.5)
    for rb in list_plans(m):
        g.set_tuning(rb, 0)
        g.load_intensities(c.sd32, is_sqrt=True)
        want = g.objective()
        d = torch.empty(n + 1, device="cuda")[1:].view(c.sd32.shape)       # 4 bytes off
        d.copy_(torch.from_numpy(c.sd32))
        z = torch.empty(c.z0_32.size + 1, dtype=torch.complex64, device="cuda")[1:].view(c.z0_32.shape)   # 8 bytes off
        z.copy_(torch.from_numpy(c.z0_32))
        torch.cuda.synchronize()
        g.load_intensities(d, is_sqrt=True)
        g.set_object(z)
        assert g.objective() == want
        g.set_object(z.to(torch.complex128).cpu().numpy())
        assert g.objective() == want
        for at, bad in ((0, -1.0), (n - 1, np.nan), (n // 2, np.inf)):
            e = c.sd32.copy()
            e.ravel()[at] = bad
            with pytest.raises(MagpieError):
                g.load_intensities(e, is_sqrt=True)
        for at, bad in ((0, np.inf), (c.z0_32.size - 1, 1j * np.nan)):
            e = c.z0_32.copy()
            e.ravel()[at] = bad
            for arg in (e, torch.from_numpy(e).cuda(), torch.from_numpy(e.astype(np.complex128)).cuda()):
                torch.cuda.synchronize()
                with pytest.raises(MagpieError):
                    g.set_object(arg)
        g.set_object(c.z0_32)
    g.close()
