"""Products of the network's gradients, one at a time: with centre-tap weights and an output
gradient that is nonzero at one pixel every gradient entry is a single product of two FP32 values,
and has to be within 2^-23 of it (two roundings).  The mean of n differences from the correctly
rounded products stays below 8 standard deviations of n uniform roundings, 2^-24 8 / sqrt(3 n):
operands with all low bits set show a dropped part of a product at once, as a bias."""

import numpy as np
import pytest

from oracle import learned as ol

pytestmark = pytest.mark.gpu

W = 32


def _values(rng, n, low_ones):
    v = rng.uniform(1.0, 2.0, n).astype(np.float32)
    if low_ones:   # 1.xxxxxxx followed by ones: the largest second and third parts
        v = ((v.view(np.uint32) & np.uint32(0x3FFF0000)) | np.uint32(0xFFFF)).view(np.float32)
    return v


def _check(name, got, a, b):
    got, want, rounded = got.astype(np.float64), a.astype(np.float64) * b.astype(np.float64), a * b
    rel = np.abs((got - want) / want).max()
    bias = ((got - rounded.astype(np.float64)) / want).mean()
    print(name, "n", got.size, "max", rel * 2.0**24, "bias", bias * 2.0**24, "(2^-24)", flush=True)
    assert rel <= 2.0**-23
    assert abs(bias) <= 2.0**-24 * 8 / np.sqrt(3 * got.size)


@pytest.mark.parametrize("low_ones", [False, True])
@pytest.mark.parametrize("cin,bf16", [(1, False), (3, False), (4, False), (4, True)])
def test_gradients_hold_fp32_products(cin, bf16, low_ones):
    from paper_2504_10118_amd import CNN
    rng = np.random.default_rng(900 + cin)
    side, nb, py, px = 10, 2, 9, 14   # output pixel (py, px) of 20 x 20, in the second sample
    shapes = ol.layer_shapes(cin, W)
    bias = [_values(rng, co, low_ones) for co, _ in shapes]
    w = [np.zeros((co, ci, 9), np.float32) for co, ci in shapes]
    for l in (1, 2, 3):
        w[l][:, :, 4] = np.eye(W)
    head = _values(rng, W, low_ones)
    if bf16:
        head = ol.bf16_round(head)
    w[4][0, :, 4] = head
    x = _values(rng, nb * cin * side * side, low_ones).reshape(nb, cin, side, side)
    net = CNN(in_ch=cin, side=side, max_batch=nb, weight_dtype=int(bf16))

    def grads(dy_value):
        net.set_params(np.concatenate([np.concatenate([a.ravel(), b]) for a, b in zip(w, bias)]))
        net.forward(x)
        dy = np.zeros((nb, 2, 2 * side, 2 * side), np.float32)
        dy[1, :, py, px] = dy_value
        net.backward(dy)
        g, out, off = net.get_grads(), [], 0
        for co, ci in shapes:
            out.append((g[off:off + co * ci * 9].reshape(co, ci, 9), g[off + co * ci * 9:off + co * ci * 9 + co]))
            off += co * ci * 9 + co
        return out

    # activations: constant planes, sums of the biases
    a1 = bias[0]
    a2 = bias[1] + a1
    a3 = bias[2] + a2
    a4 = bias[3] + a3
    dy = _values(rng, 2, low_ones)
    g = grads(dy)
    for t in range(9):
        _check("head", g[4][0][:, :, t], dy[:, None], a4[None, :])
    g = grads(np.array([1.0, 0.0], np.float32))   # f = head in every layer
    for l, act in ((3, a3), (2, a2), (1, a1)):
        f = g[l][1]
        assert np.array_equal(f, head)
        for t in range(9):
            _check(f"layer {l}", g[l][0][:, :, t], f[:, None], act[None, :])
    f = g[0][1]
    assert np.array_equal(f, head)
    for t in range(9):
        _check("first", g[0][0][:, :, t], f[:, None], x[1, :, py // 2 + t // 3 - 1, px // 2 + t % 3 - 1][None, :])
    # backward-data: one output channel's gradient through a layer's weights
    w[4][0, 1:, 4] = 0.0
    for l in (3, 2, 1):
        save = w[l]
        w[l] = np.zeros_like(save)
        row = _values(rng, W, low_ones)
        if bf16:
            row = ol.bf16_round(row)
        w[l][0, :, 4] = row
        g = grads(dy[:1] * np.array([1.0, 0.0], np.float32))
        f = g[l][1][0]   # the gradient that enters the layer, at its one channel
        _check(f"data {l}", g[l - 1][1], row, np.full(W, f))
        w[l] = save
    net.close()
