"""Weight gradients of 3x3 / stride-1 convolutions through rings in LDS (conv3_wgrad_ring_device.h), against float64 over the very
tensors the library stored: every map width and its smallest heights, channel tiles that are not full, few input channels (the form
in which wavefronts share a block) and many, workers of one image, chunks that end inside images, steps that hold several images
and a last one that is not full.  With a 3x3 layer in front all layers of the call have this form (eight wavefronts to a workgroup),
with a 1x1 layer they share a launch with another (four).

Bound (2-norm, relative): the matrix instruction cuts off, at most 2^-23 of the partial sum per addition; the partial sums of terms of
random sign grow with the root of their number, so m additions in a row are off by at most m / 1.5 2^-23 of the last, on average
half that.  m: a worker's positions, sixteen to an instruction."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun

pytestmark = pytest.mark.gpu


def _layers(stem, cin, cout, h, w):
    return [dict(op="conv", src=-1, cin=8, cout=cin, k=stem, stride=1, pad=stem // 2, bias=True), dict(op="relu", src=0),
            dict(op="conv", src=1, cin=cin, cout=cout, k=3, stride=1, pad=1, bias=True), dict(op="relu", src=2),
            dict(op="gap", src=3), dict(op="linear", src=4, cin=cout, cout=10, bias=True)]


@pytest.mark.parametrize("stem", [1, 3])
@pytest.mark.parametrize("h,w,cin,cout,off", [
    (32, 32, 64, 64, [0, 1, 20]),
    (12, 32, 136, 40, [0, 30, 61]),
    (1, 32, 64, 96, [0, 7, 150]),
    (16, 16, 72, 136, [0, 2, 50]),
    (24, 16, 64, 64, [0, 41]),
    (2, 16, 96, 64, [0, 3, 5, 101]),
    (8, 8, 64, 128, [0, 1, 2, 150]),
    (16, 8, 40, 72, [0, 33, 90]),
    (4, 8, 64, 64, [0, 3, 4, 155]),
    (4, 4, 128, 72, [0, 1, 2, 200]),
    (4, 4, 24, 64, [0, 9, 10]),
    (32, 32, 32, 64, [0, 2, 25]),
    (1, 32, 8, 64, [0, 5, 98]),
    (16, 16, 24, 96, [0, 1, 75]),
    (2, 16, 32, 40, [0, 1, 4, 222]),
    (8, 8, 16, 64, [0, 3, 103]),
    (4, 8, 32, 64, [0, 1, 3, 6, 105]),
])
def test_against_float64(stem, h, w, cin, cout, off):
    import torch
    import paper_2503_17469_amd as omni
    layers = _layers(stem, cin, cout, h, w)
    B, K = off[-1], len(off) - 1
    params = synth.he_normal_params(layers, 11, True)
    x, y = synth.make_batch(h * w + cin, B, (h, w, 8), 10, True)
    run = GpuRun(layers, (h, w, 8), "bf16", K, B)
    try:
        G = run.step(params, x, y, off, 0.0, keep_g=False)["worker_grads"]
        X = torch.from_numpy(run.activation(1, B)).double().reshape(B, h, w, cin)
        dY = omni.net_activation_grad(run.net, run.ws, 2, B, "bf16").double().cpu().reshape(B, h, w, cout)
    finally:
        run.close()
    Xp = torch.nn.functional.pad(X, (0, 0, 1, 1, 1, 1))
    sl = synth.param_slices(layers)[2]
    for k in range(K):
        r = slice(off[k], off[k + 1])
        rows = dY[r].reshape(-1, cout)
        want = torch.stack([rows.T @ Xp[r, u:u + h, v:v + w].reshape(-1, cin) for u in range(3) for v in range(3)], 1)
        m = rows.shape[0] / 16
        for name, ref in (("w", want.reshape(-1)), ("b", rows.sum(0))):
            got = torch.from_numpy(G[k, slice(*sl[name])]).double()
            err = float((got - ref).norm() / ref.norm())
            assert err <= (m / 3 + 2) * 2.0 ** -23, (name, k, err)
