"""Weight gradients of 3x3 / stride-1 convolutions on maps wider than 32 (kernel C of conv_wgrad_bf16.hip), with the float64 reference
and the bound of test_gpu_wgrad_ring.py: 64 wide in units of two rows and of one, 128 wide, one row of either (128 wide and a row of 64:
three staging tasks a thread), several units per image, workers of one image, chunks that end inside images, channel tiles that are
not full, and the layer on the network input, with eight stored channels."""
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_wgrad_ring import test_against_float64 as against_float64

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 64, 64, 64, [0, 1, 40]),
    (2, 64, 72, 40, [0, 1, 30]),
    (8, 64, 64, 136, [0, 3, 11]),
    (32, 64, 136, 64, [0, 1, 4]),
    (1, 128, 64, 64, [0, 1, 2, 35]),
    (2, 128, 40, 72, [0, 1, 20]),
    (5, 128, 64, 64, [0, 2, 9]),
    (32, 128, 64, 96, [0, 1, 3]),
    (3, 64, 64, 64, [0, 1, 14]),
]


@pytest.mark.parametrize("stem", [1, 3])
@pytest.mark.parametrize("h,w,cin,cout,off", SHAPES)
def test_hidden_layer(stem, h, w, cin, cout, off):
    against_float64(stem, h, w, cin, cout, off)


@pytest.mark.parametrize("h,w", [(1, 64), (6, 64), (1, 128), (7, 128)])
def test_layer_on_the_input(h, w):
    import torch
    import paper_2503_17469_amd as omni
    off, cin, cout = [0, 1, 12], 8, 40
    layers = [dict(op="conv", src=-1, cin=cin, cout=cout, k=3, stride=1, pad=1, bias=True), dict(op="relu", src=0),
              dict(op="gap", src=1), dict(op="linear", src=2, cin=cout, cout=10, bias=True)]
    B, K = off[-1], len(off) - 1
    params = synth.he_normal_params(layers, 5, True)
    x, y = synth.make_batch(h * w, B, (h, w, cin), 10, True)
    run = GpuRun(layers, (h, w, cin), "bf16", K, B)
    try:
        G = run.step(params, x, y, off, 0.0, keep_g=False)["worker_grads"]
        dY = omni.net_activation_grad(run.net, run.ws, 0, B, "bf16").double().cpu().reshape(B, h, w, cout)
    finally:
        run.close()
    Xp = torch.nn.functional.pad(torch.from_numpy(x).double().reshape(B, h, w, cin), (0, 0, 1, 1, 1, 1))
    sl = synth.param_slices(layers)[0]
    for k in range(K):
        r = slice(off[k], off[k + 1])
        rows = dY[r].reshape(-1, cout)
        want = torch.stack([rows.T @ Xp[r, u:u + h, v:v + w].reshape(-1, cin) for u in range(3) for v in range(3)], 1).reshape(-1)
        err = float((torch.from_numpy(G[k, slice(*sl["w"])]).double() - want).norm() / want.norm())
        assert err <= (rows.shape[0] / 48 + 2) * 2.0 ** -23, (k, err)
