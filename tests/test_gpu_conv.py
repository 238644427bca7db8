"""The network's convolutions at the edges of their tiles (16 x 16, 16 x 8 and 16 x 4 pixels, runs of
tiles per workgroup): outputs are the FP32 FMA chain over (input channel, tap) bit for bit, gradients
agree with FP64, and non-finite gradients come out where they do in plain arithmetic."""

import numpy as np
import pytest

from oracle import learned as ol

pytestmark = pytest.mark.gpu

W = 32


def _problem(seed, cin, side, nb):
    rng = np.random.default_rng(seed)
    p = np.concatenate([np.concatenate([rng.normal(0.0, np.sqrt(2.0 / (9 * ci)), co * ci * 9),
                                        rng.normal(0.0, 0.05, co)]) for co, ci in ol.layer_shapes(cin, W)])
    return p.astype(np.float32), rng.normal(size=(nb, cin, side, side)).astype(np.float32), rng


def _net(cin, side, nb, wdt, p):
    from paper_2504_10118_amd import CNN
    net = CNN(in_ch=cin, side=side, max_batch=nb, weight_dtype=wdt)
    net.set_params(p)
    return net


def _weights(p, cin, bf16):
    q, off = p.astype(np.float32).copy(), 0
    for co, ci in ol.layer_shapes(cin, W):
        n = co * ci * 9
        if bf16:
            q[off:off + n] = ol.bf16_round(q[off:off + n])
        off += n + co
    return q


def _chain(x, w, b, relu):
    """FP32 FMA chain from the bias over input channels, then taps.  The 64-bit significand of the
    extended type holds each product exactly, so rounding its sum to FP32 is the fused result."""
    nb, ci, h, wd = x.shape
    xp = np.pad(x, ((0, 0), (0, 0), (1, 1), (1, 1))).astype(np.longdouble)
    acc = np.broadcast_to(b[None, :, None, None], (nb, len(b), h, wd)).astype(np.float32)
    for c in range(ci):
        for t in range(9):
            v = xp[:, None, c, t // 3:t // 3 + h, t % 3:t % 3 + wd]
            acc = (w[None, :, c, t, None, None].astype(np.longdouble) * v + acc).astype(np.float32)
    return np.maximum(acc, np.float32(0)) if relu else acc


@pytest.mark.parametrize("cin,side,nb,bf16", [(1, 2, 1, False), (3, 8, 2, False), (4, 18, 1, True)])
def test_forward_is_the_fp32_chain(cin, side, nb, bf16):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("needs an extended type of 64 significant bits")
    p, x, _ = _problem(500 + side, cin, side, nb)
    net = _net(cin, side, nb, int(bf16), p)
    y = net.forward(x)
    q, a, off = _weights(p, cin, bf16), x, 0
    for i, (co, ci) in enumerate(ol.layer_shapes(cin, W)):
        if i == 2:
            a = a.repeat(2, 2).repeat(2, 3)
        n = co * ci * 9
        a = _chain(a, q[off:off + n].reshape(co, ci, 9), q[off + n:off + n + co], i < 4)
        off += n + co
    assert np.array_equal(y.view(np.uint32), a.view(np.uint32))
    net.close()


# tiles of 16 x 16 at the larger size: 9 (4 rows per workgroup), 90 (8 rows; 40 of the small layer: 4),
# 180 (16 rows; 80: 8), 630 (workgroups with two tiles)
@pytest.mark.parametrize("nb", [10, 20, 70])
def test_forward_of_a_batch_is_that_of_its_samples(nb):
    p, x, _ = _problem(700, 3, 18, nb)
    net = _net(3, 18, nb, 0, p)
    y = net.forward(x)
    one = np.concatenate([net.forward(x[i:i + 1]) for i in range(nb)])
    net.close()
    assert np.array_equal(y.view(np.uint32), one.view(np.uint32))


# (16 x 16 tiles, 16 x 8 tiles) at the two sizes: one ragged tile; exact; one pixel over; many runs
@pytest.mark.parametrize("cin,side,nb,bf16", [(3, 2, 1, False), (1, 8, 2, True), (4, 18, 3, False), (3, 34, 33, False)])
def test_gradients_at_tile_edges(cin, side, nb, bf16):
    p, x, rng = _problem(600 + side, cin, side, nb)
    dy = rng.normal(size=(nb, 2, 2 * side, 2 * side)).astype(np.float32)
    net = _net(cin, side, nb, int(bf16), p)
    net.forward(x)
    net.backward(dy)
    g = net.get_grads()
    net.close()
    q = _weights(p, cin, bf16).astype(np.float64)
    _, cache = ol.net_forward(q, x.astype(np.float64), cin, W)
    go, _ = ol.net_backward(q, cache, dy.astype(np.float64), cin, W)
    off = 0
    for co, ci in ol.layer_shapes(cin, W):
        for cnt in (co * ci * 9, co):
            # FP32 sums of up to 33 * 68^2 terms in a few hundred parts: 2e-5 as for the other gradient tests
            err = np.linalg.norm(g[off:off + cnt] - go[off:off + cnt]) / np.linalg.norm(go[off:off + cnt])
            assert err <= 2e-5, (co, ci, cnt, err)
            off += cnt


@pytest.mark.parametrize("bf16", [False, True])
def test_infinite_output_gradient(bf16):
    """One infinite value in the second output channel's gradient: the gradients are finite, infinite or
    undefined where products and sums in plain arithmetic are."""
    import torch
    cin, side, nb = 3, 10, 2
    p, x, rng = _problem(700, cin, side, nb)
    dy = rng.normal(size=(nb, 2, 2 * side, 2 * side)).astype(np.float32)
    dy[1, 1, 7, 9] = np.inf
    net = _net(cin, side, nb, int(bf16), p)
    net.forward(x)
    net.backward(dy)
    g = net.get_grads()
    net.close()
    q = _weights(p, cin, bf16).astype(np.float64)
    a, leaves, off = torch.from_numpy(x).double(), [], 0
    for i, (co, ci) in enumerate(ol.layer_shapes(cin, W)):
        if i == 2:
            a = a.repeat_interleave(2, 2).repeat_interleave(2, 3)
        n = co * ci * 9
        w = torch.from_numpy(q[off:off + n].reshape(co, ci * 9)).requires_grad_()
        b = torch.from_numpy(q[off + n:off + n + co]).requires_grad_()
        leaves += [w, b]
        off += n + co
        h = a.shape[-1]
        a = (w @ torch.nn.functional.unfold(a, 3, padding=1) + b[None, :, None]).reshape(nb, co, h, h)
        a = torch.relu(a) if i < 4 else a
    a.backward(torch.from_numpy(dy).double())
    want = np.concatenate([v.grad.numpy().ravel() for v in leaves])
    assert np.array_equal(np.isnan(g), np.isnan(want)) and np.array_equal(np.isinf(g), np.isinf(want))
    fin = np.isfinite(want)
    assert 0 < fin.sum() < want.size and np.array_equal(np.sign(g[np.isinf(want)]), np.sign(want[np.isinf(want)]))
    assert np.linalg.norm(g[fin] - want[fin]) <= 2e-5 * np.linalg.norm(want[fin])


def test_infinite_output_gradient_in_a_batch():
    """630 tiles on workgroups that take two each: an infinite value in the first tile of some leaves the
    second one's products right.  Gradients add over samples, to 2e-5 of their norm as above."""
    cin, side, nb, bad = 1, 18, 70, 3
    p, x, rng = _problem(800, cin, side, nb)
    dy = rng.normal(size=(nb, 2, 2 * side, 2 * side)).astype(np.float32)
    rest = dy.copy()
    rest[bad] = 0
    dy[bad, 1, 7, 9] = np.inf
    net = _net(cin, side, nb, 0, p)

    def grads(xs, ds):
        net.forward(xs)
        net.backward(ds)
        return net.get_grads().astype(np.float64)

    g, g_rest, one = grads(x, dy), grads(x, rest), grads(x[bad:bad + 1], dy[bad:bad + 1])
    net.close()
    fin = np.isfinite(one)
    assert 0 < fin.sum() < one.size
    assert np.array_equal(np.isnan(g), np.isnan(one)) and np.array_equal(np.isinf(g), np.isinf(one))
    want = g_rest[fin] + one[fin]
    assert np.linalg.norm(g[fin] - want) <= 2e-5 * np.linalg.norm(want)


def test_refused_mask_keeps_the_output_gradient():
    """A loss with a refused mask fails and leaves the last valid loss's output gradient in place."""
    from paper_2504_10118_amd import MagpieError
    cin, side, nb = 1, 6, 2
    p, x, rng = _problem(900, cin, side, nb)
    t = np.exp(1j * rng.uniform(-1, 1, (nb, 2 * side, 2 * side))).astype(np.complex64)
    mask = rng.uniform(0.5, 1.0, (2 * side, 2 * side)).astype(np.float32)
    net = _net(cin, side, nb, 0, p)
    net.forward(x)
    net.loss(t, mask, align_phase=True)
    net.backward(nbatch=nb)
    g = net.get_grads()
    for bad in (-1.0, np.nan, np.inf):
        m2 = mask.copy()
        m2[3, 4] = bad
        with pytest.raises(MagpieError, match="finite"):
            net.loss(t, m2, align_phase=False)
    with pytest.raises(MagpieError, match="all zero"):
        net.loss(t, 0 * mask)
    net.backward(nbatch=nb)
    assert np.array_equal(net.get_grads().view(np.uint32), g.view(np.uint32))
    net.close()
