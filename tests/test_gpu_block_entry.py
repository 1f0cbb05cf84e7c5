"""Input gradients of 3x3 / stride-2 convolutions in the kernel for many positions (conv3s2_ring_kernel), against float64 over the very
tensors the library stored: units of part of an image, one image and several, the last one not full, channel tiles of which half
exists, one slice of the reduction and more, with the projection beside it, alone and with the share of another convolution to
add; and the sums of the batch norm below.

Bound, per element: a bf16 rounding, 2^-8, of the result (and of the share that was stored first), and fp32 sums of 9 or 10 cout terms,
each off by at most 2^-24 of the sum of their magnitudes."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_bn_sums import _check_backward, _conv, _tail

pytestmark = pytest.mark.gpu


def _layers(cin, cout, beside):
    s2 = dict(op="conv", src=1, cin=cin, cout=cout, k=3, stride=2, pad=1, bias=False)
    other = dict(s2, k=1, pad=0) if beside == "projection" else s2
    head = [dict(op="conv", src=-1, cin=8, cout=cin, k=1, stride=1, pad=0, bias=True), dict(op="relu", src=0), s2]
    if beside == "none":
        return head + [dict(op="relu", src=2), dict(op="gap", src=3), dict(op="linear", src=4, cin=cout, cout=10, bias=True)]
    return head + [dict(other), dict(op="add", src=2, src2=3), dict(op="relu", src=4), dict(op="gap", src=5),
                   dict(op="linear", src=6, cin=cout, cout=10, bias=True)]


# (units are 512 positions by 64 channels; few of them go to another kernel)
@pytest.mark.parametrize("h,w,cin,cout,beside,off", [
    (32, 32, 64, 128, "projection", [0, 1, 135]),
    (32, 32, 64, 64, "none", [0, 131]),
    (64, 32, 64, 64, "projection", [0, 70]),
    (16, 16, 128, 96, "projection", [0, 2, 263]),
    (16, 16, 64, 64, "twin", [0, 515]),
    (8, 8, 96, 32, "projection", [0, 3, 1029]),
    (8, 8, 160, 64, "none", [0, 701]),
    (16, 64, 64, 64, "projection", [0, 1, 133]),
    (8, 128, 96, 64, "twin", [0, 67]),
    (8, 4, 64, 64, "projection", [0, 4099]),
    (16, 32, 64, 32, "projection", [0, 1, 259]),
    (32, 16, 64, 64, "none", [0, 7, 261]),
])
def test_against_float64(h, w, cin, cout, beside, off):
    import torch
    import paper_2503_17469_amd as omni
    layers = _layers(cin, cout, beside)
    B, K = off[-1], len(off) - 1
    params = synth.he_normal_params(layers, 12, True)
    x, y = synth.make_batch(h * w + cin, B, (h, w, 8), 10, True)
    run = GpuRun(layers, (h, w, 8), "bf16", K, B)
    try:
        assert run.step(params, x, y, off, 0.0)["status"] == 0
        grad = lambda n, a, b, c: omni.net_activation_grad(run.net, run.ws, n, B, "bf16").cpu().float().reshape(B, a, b, c).permute(0, 3, 1, 2)
        X = torch.from_numpy(run.activation(1, B)).reshape(B, h, w, cin).permute(0, 3, 1, 2)
        got = grad(1, h, w, cin).double()
        dY = [grad(i, h // 2, w // 2, cout).double() for i in ([2] if beside == "none" else [2, 3])]
    finally:
        run.close()
    assert all(float(d.abs().max()) > 0 for d in dY)
    sl = synth.param_slices(layers)
    want = torch.zeros_like(got)
    size, slack = torch.zeros_like(got), torch.zeros_like(got)
    for i, d in zip([2, 3], dY):
        k = layers[i]["k"]
        W = torch.from_numpy(params[slice(*sl[i]["w"])].astype(np.float64)).reshape(cout, k, k, cin).permute(0, 3, 1, 2)
        back = lambda a, b: torch.nn.functional.conv_transpose2d(a, b, stride=2, padding=k // 2, output_padding=1)
        share = back(d, W)
        want += share
        size += back(d.abs(), W.abs())
        if beside == "twin" and i == 3:
            slack = 2.0 ** -8 * share.abs()
    want *= (X > 0)
    slack += 2.0 ** -8 * want.abs() + 10 * cout * 2.0 ** -24 * size
    assert float(((got - want).abs() - slack).max()) <= 0


# The most tiles (64 positions by 64 channels) of the kernel for few positions, 320, and one image more; with sums 128
@pytest.mark.parametrize("h,w,cin,cout,beside,B", [(16, 16, 64, 64, "projection", 320), (16, 16, 64, 64, "projection", 321),
                                                   (8, 8, 64, 128, "twin", 1280), (8, 8, 64, 128, "twin", 1281)])
def test_either_side_of_the_rule(h, w, cin, cout, beside, B):
    test_against_float64(h, w, cin, cout, beside, [0, 1, B])


@pytest.mark.parametrize("hw,B", [(16, 128), (16, 129), (32, 32), (32, 33)])
def test_sums_at_either_side_of_the_rule(hw, B):
    test_sums_below_a_block_entry(hw, B)


@pytest.mark.parametrize("hw,B", [(8, 2053), (16, 515), (32, 131)])
def test_sums_below_a_block_entry(hw, B):
    C = 64
    layers = [_conv(-1, C), dict(op="bn", src=0, c=C), dict(op="relu", src=1),
              dict(op="conv", src=2, cin=C, cout=C, k=3, stride=2, pad=1, bias=False), dict(op="bn", src=3, c=C),
              dict(op="conv", src=2, cin=C, cout=C, k=1, stride=2, pad=0, bias=False), dict(op="bn", src=5, c=C),
              dict(op="add", src=4, src2=6), dict(op="relu", src=7)] + _tail(8, C)
    _check_backward(layers, (hw, hw, C), B, [1])
