"""GPU parity of the first layer's forward launch that takes the other layers' weight copies along: input channels stored raw and
padded, one and two blocks of output channels and partly filled ones, units of part of an image, of one and of several with the
last one not full, pooling and none; then a stale zero page and stale copies in the workspace must not matter."""
import numpy as np
import pytest

import synth
from test_gpu_cnn import _check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hw,chans,B,cuts", [
    (32, (3, 32, 32), 9, [0, 1, 9]),          # raw, four units per image
    (16, (3, 40, 64), 67, [0, 30, 67]),       # raw, two blocks of outputs, the second a quarter full; a unit is an image
    (8, (3, 64, 32), 37, [0, 5, 37]),         # a unit is four images, the last one of one
    (8, (1, 8, 32), 22, [0, 22]),             # one channel stored as eight, a block a quarter full
    (16, (5, 32, 32), 19, [0, 4, 19]),
    (16, (8, 24, 64), 11, [0, 3, 11]),        # no padding
])
@pytest.mark.parametrize("pool", [True, False])
def test_first_layer(hw, chans, B, cuts, pool):
    layers = []

    def add(**kw):
        layers.append(dict(kw, src=len(layers) - 1))

    add(op="conv", cin=chans[0], cout=chans[1], k=3, stride=1, pad=1, bias=True)
    add(op="relu")
    if pool:
        add(op="maxpool2")
    add(op="conv", cin=chans[1], cout=chans[2], k=3, stride=1, pad=1, bias=True)
    add(op="relu")
    add(op="gap")
    add(op="linear", cin=chans[2], cout=10, bias=True)
    params = synth.he_normal_params(layers, 6, True)
    x, y = synth.make_batch(17 + hw, B, (hw, hw, chans[0]), 10, True)
    _check_step(layers, (hw, hw, chans[0]), params, x, y, cuts, 0.05, f"first-{hw}px-{chans}-{pool}")


def test_workspace_contents_do_not_matter():
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.cnn3(num_classes=10, hw=32, chans=(3, 32, 64, 64))
    B = 33
    p0 = torch.from_numpy(synth.he_normal_params(layers, 6, True)).cuda()
    x, y = synth.make_batch(3, B, (32, 32, 3), 10, True)
    x = torch.from_numpy(x).cuda().to(torch.bfloat16)
    labels = torch.from_numpy(y).cuda().to(torch.int32)
    net = omni.net_create(layers, (32, 32, 3), "bf16", 1, B)
    size = omni.net_workspace_bytes(net)
    lpw, loss = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    got = []
    for fill in (0, 0xFF, 0x3F):
        ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda")
        p = p0.clone()
        omni.step(net, p, x, labels, [0, B], [B], 0.05, ws, lpw, loss)
        torch.cuda.synchronize()
        got.append((p, loss.clone()))
    for p, l in got[1:]:
        assert torch.equal(p, got[0][0]) and torch.equal(l, got[0][1])
    omni.net_destroy(net)
