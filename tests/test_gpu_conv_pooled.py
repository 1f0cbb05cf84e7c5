"""GPU parity of the wide 3x3 kernel's pooling epilogue and its 32-channel tile: both map widths, one slice of the reduction and
several, full and partly filled channel tiles, units of several images with the last one not full, ReLU and none."""
import numpy as np
import pytest

import synth
from test_gpu_cnn import _check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hw,chans,B,cuts", [
    (32, (3, 32, 64, 64), 150, [0, 1, 67, 150]),       # 16x16: one slice, 64-channel tile; 8x8: two slices
    (32, (3, 64, 24, 32), 140, [0, 139, 140]),         # 16x16: two slices, narrow tile three quarters full; its input gradient generic
    (32, (3, 32, 32, 128), 258, [0, 100, 258]),        # 16x16: one slice, narrow tile, two and one units per workgroup
    (16, (3, 32, 96, 64), 523, [0, 3, 260, 523]),      # 8x8: one slice, second channel tile half empty, last unit three of four images
    (16, (3, 96, 32, 64), 530, [0, 530]),              # 8x8: three slices, narrow tile, last unit two of four images
])
def test_pooled_layers(hw, chans, B, cuts):
    layers = synth.cnn3(num_classes=10, hw=hw, chans=chans)
    rng = np.random.default_rng(hw + B)
    params = synth.he_normal_params(layers, 6, True)
    for sl in synth.param_slices(layers):
        if "b" in sl:
            s, e = sl["b"]
            params[s:e] = synth.to_bf16_grid(rng.standard_normal(e - s).astype(np.float32) * 0.2)
    x, y = synth.make_batch(17 + hw, B, (hw, hw, 3), 10, True)
    _check_step(layers, (hw, hw, 3), params, x, y, cuts, 0.05, f"cnn3-{hw}px-{chans}")


def test_ties_and_infinities():
    """Constant inputs make every window a tie (the first takes the gradient), infinite ones infinite maxima: outputs and codes as
    float comparison gives them, from the stored values."""
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.cnn3(num_classes=10, hw=32, chans=(3, 32, 64, 64))
    B = 160
    rng = np.random.default_rng(2)
    params = synth.he_normal_params(layers, 6, True)
    x = np.repeat(rng.standard_normal((B, 1, 1, 3)), 32, 1).repeat(32, 2).astype(np.float32)
    x = torch.from_numpy(x).cuda().to(torch.bfloat16)
    x[5, 7, 9, 1] = float("inf")
    x[6, 20, 21, 0] = float("-inf")
    p = torch.from_numpy(params).cuda()
    labels = torch.zeros(B, dtype=torch.int32, device="cuda")
    net = omni.net_create(layers, (32, 32, 3), "bf16", 1, B)
    ws = torch.zeros(omni.net_workspace_bytes(net), dtype=torch.uint8, device="cuda")
    lpw, loss = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    omni.step(net, p, x, labels, [0, B], [B], 0.0, ws, lpw, loss, omni.STEP_NO_UPDATE)
    torch.cuda.synchronize()
    convs = [i for i, L in enumerate(layers) if L["op"] == "conv"]
    pools = [i for i, L in enumerate(layers) if L["op"] == "maxpool2"]
    hw = 16
    for conv, pool in list(zip(convs, pools))[1:]:
        a = omni.net_activation(net, ws, pool - 1, B, "bf16").float().reshape(B, hw // 2, 2, hw // 2, 2, -1)
        m = omni.net_activation(net, ws, pool, B, "bf16").float().reshape(B, hw // 2, hw // 2, -1)
        win = a.permute(0, 1, 3, 5, 2, 4).reshape(B, hw // 2, hw // 2, -1, 4)
        # (a ReLU stores no NaN and nothing negative)
        assert not torch.isnan(win).any() and (win >= 0).all()
        assert torch.equal(win.max(-1).values, m)
        # where the gradient went: the first of the maxima, nowhere where the maximum is zero
        g = omni.net_activation_grad(net, ws, pool - 1, B, "bf16").float().reshape(a.shape).permute(0, 1, 3, 5, 2, 4).reshape(win.shape)
        d = omni.net_activation_grad(net, ws, pool, B, "bf16").float().reshape(m.shape)
        first = torch.zeros_like(win).scatter_(-1, (win == m[..., None]).float().argmax(-1, keepdim=True), 1.0)
        keep = (m > 0)[..., None] & (first > 0)
        want = torch.where(keep, d[..., None].expand_as(win), torch.zeros_like(win))
        assert torch.equal(torch.nan_to_num(g, nan=7.0), torch.nan_to_num(want, nan=7.0))
        hw //= 2
    omni.net_destroy(net)
