"""3x3 / stride-1 convolutions and their input gradients whose patches and weights are brought by loads that write LDS
(conv3_wide_bf16.hip), against float64 over the very tensors the library stored: every map width with units that are part of an
image, one image and several, the last unit not full, channel tiles of which half exists, two slices of the reduction, three and
more, the narrow tile in either direction, behind a ReLU (a mask), a batch norm and neither.

Bound, per element: the product of a float64 sum with a bf16 rounding, 2^-8 of it, and fp32 sums of 9 cin terms, each off by at most
2^-24 of the sum of their magnitudes."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun

pytestmark = pytest.mark.gpu


def _layers(cin, cout, before):
    front = [dict(op="conv", src=-1, cin=8, cout=cin, k=3, stride=1, pad=1, bias=True)]
    if before != "none":
        front.append(dict(op="relu", src=0) if before == "relu" else dict(op="bn", src=0, c=cin))
    n = len(front)
    return front + [dict(op="conv", src=n - 1, cin=cin, cout=cout, k=3, stride=1, pad=1, bias=True), dict(op="relu", src=n),
                    dict(op="gap", src=n + 1), dict(op="linear", src=n + 2, cin=cout, cout=10, bias=True)], n


# (units are 256 positions by 64 channels, at least 32 of them)
@pytest.mark.parametrize("h,w,cin,cout,before,off", [
    (8, 8, 64, 64, "relu", [0, 1, 131]),
    (8, 8, 96, 32, "relu", [0, 150]),
    (8, 8, 32, 64, "none", [0, 3, 129]),
    (16, 8, 64, 96, "relu", [0, 70]),
    (32, 8, 64, 64, "none", [0, 1, 40]),
    (8, 16, 128, 64, "relu", [0, 65]),
    (16, 16, 64, 160, "none", [0, 5, 33]),
    (16, 16, 32, 64, "bn", [0, 1, 40]),
    (32, 16, 64, 64, "bn", [0, 2, 20]),
    (32, 32, 64, 64, "relu", [0, 1, 9]),
    (32, 32, 32, 96, "none", [0, 11]),
    (8, 32, 96, 128, "bn", [0, 7, 40]),
])
def test_against_float64(h, w, cin, cout, before, off):
    import torch
    import paper_2503_17469_amd as omni
    layers, i = _layers(cin, cout, before)
    B, K = off[-1], len(off) - 1
    params = synth.he_normal_params(layers, 11, True)
    sl = synth.param_slices(layers)[i]
    rng = np.random.default_rng(h * w + cin)
    params[slice(*sl["b"])] = synth.to_bf16_grid(0.2 * rng.standard_normal(cout).astype(np.float32))
    x, y = synth.make_batch(h * w + cin, B, (h, w, 8), 10, True)
    run = GpuRun(layers, (h, w, 8), "bf16", K, B)
    try:
        assert run.step(params, x, y, off, 0.0)["status"] == 0
        act = lambda n, c: torch.from_numpy(run.activation(n, B)).double().reshape(B, h, w, c).permute(0, 3, 1, 2)
        grad = lambda n, c: omni.net_activation_grad(run.net, run.ws, n, B, "bf16").double().cpu().reshape(B, h, w, c).permute(0, 3, 1, 2)
        X, Y, dY, dX = act(i - 1, cin), act(i + 1, cout), grad(i, cout), grad(i - 1, cin)
    finally:
        run.close()
    W = torch.from_numpy(params[slice(*sl["w"])].astype(np.float64)).reshape(cout, 3, 3, cin).permute(0, 3, 1, 2)
    b = torch.from_numpy(params[slice(*sl["b"])].astype(np.float64))

    def outside(got, want, size, terms):
        return float(((got - want).abs() - 2.0 ** -8 * want.abs() - terms * 2.0 ** -24 * size).max())

    conv = torch.nn.functional.conv2d
    assert outside(Y, conv(X, W, b, padding=1).clamp(min=0), conv(X.abs(), W.abs(), b.abs(), padding=1), 9 * cin + 1) <= 0
    T = W.flip(2, 3).transpose(0, 1)
    keep = (X > 0).double() if before == "relu" else torch.ones_like(X)
    assert outside(dX, conv(dY, T, padding=1) * keep, conv(dY.abs(), T.abs(), padding=1), 9 * cout) <= 0
