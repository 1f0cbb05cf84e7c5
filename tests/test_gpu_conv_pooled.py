"""GPU parity of the wide 3x3 kernel's pooling epilogue and its 32-channel tile: both map widths, one slice of the reduction and
several, full and partly filled channel tiles, units of several images with the last one not full, ReLU and none."""
import numpy as np
import pytest

import synth
from test_gpu_cnn import _check_step

pytestmark = pytest.mark.gpu


# Workgroups take units of 256 positions (one 16x16 image, four 8x8 ones) by 64 channels, or 32 where that makes at most 256
# workgroups or the layer has at most 32; layers with few positions (8x8: at most 512 images x channel tiles) go to another kernel.
# One slice is 32 input channels; with one, workgroups take several units once there are more than 512 (32 channels: 768).
@pytest.mark.parametrize("hw,chans,B,cuts", [
    (32, (3, 32, 64, 64), 150, [0, 1, 67, 150]),       # 16x16: one slice, two narrow tiles; 8x8: few positions
    (32, (3, 64, 24, 32), 140, [0, 139, 140]),         # 16x16: two slices, narrow tile three quarters full; its input gradient generic
    (32, (3, 32, 32, 128), 258, [0, 100, 258]),        # 16x16: one slice, one narrow tile; 8x8: the same, four of them
    (32, (3, 32, 24, 64), 770, [0, 1, 400, 770]),      # 16x16: two units per workgroup, narrow tile three quarters full
    (16, (3, 32, 96, 64), 523, [0, 3, 260, 523]),      # 8x8: one slice, second channel tile half empty, last unit three of four images
    (16, (3, 96, 32, 64), 530, [0, 530]),              # 8x8: three slices, narrow tile, last unit two of four images
    (32, (3, 32, 128, 64), 259, [0, 100, 259]),        # 16x16: 64-channel tiles, one slice, two units per workgroup, the last one
    (32, (3, 64, 96, 64), 131, [0, 2, 131]),           # 16x16: 64-channel tiles, two slices, second tile half empty
    (16, (3, 64, 96, 64), 518, [0, 3, 260, 518]),      # 8x8: the same, last unit two of four images
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


@pytest.mark.parametrize("hw,chans,B", [
    (32, (3, 32, 64, 64), 160),      # 16x16 in narrow tiles; 8x8 in the kernel of few positions
    (32, (3, 32, 64, 128), 518),     # 16x16 in 64-channel tiles, one slice; 8x8 in 64-channel tiles, two slices, the last unit two images
    (16, (3, 32, 64, 64), 1018),     # 8x8 in narrow tiles
])
def test_ties_and_infinities(hw, chans, B):
    """Constant inputs make every window a tie (the first takes the gradient), infinite ones infinite maxima: outputs and codes as
    float comparison gives them, from the stored values."""
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.cnn3(num_classes=10, hw=hw, chans=chans)
    rng = np.random.default_rng(2)
    params = synth.he_normal_params(layers, 6, True)
    x = np.repeat(rng.standard_normal((B, 1, 1, 3)), hw, 1).repeat(hw, 2).astype(np.float32)
    x = torch.from_numpy(x).cuda().to(torch.bfloat16)
    for n in (5, B - 1):
        x[n, 7, 9, 1] = float("inf")
        x[n - 1, hw // 2 + 4, hw // 2 + 5, 0] = float("-inf")
    p = torch.from_numpy(params).cuda()
    labels = torch.zeros(B, dtype=torch.int32, device="cuda")
    net = omni.net_create(layers, (hw, hw, 3), "bf16", 1, B)
    ws = torch.zeros(omni.net_workspace_bytes(net), dtype=torch.uint8, device="cuda")
    lpw, loss = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    omni.step(net, p, x, labels, [0, B], [B], 0.0, ws, lpw, loss, omni.STEP_NO_UPDATE)
    torch.cuda.synchronize()
    convs = [i for i, L in enumerate(layers) if L["op"] == "conv"]
    pools = [i for i, L in enumerate(layers) if L["op"] == "maxpool2"]
    hw //= 2
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


def test_several_units_of_several_slices():
    """16x16, 64 input channels, 4100 images: two units per workgroup, two slices each.  What was stored against float64 from the stored
    input, in images at both ends and where one workgroup's units end; a bf16 rounding (2^-8) and fp32 sums of 576 products."""
    import torch
    import paper_2503_17469_amd as omni
    B = 4100
    layers = [dict(op="conv", src=-1, cin=3, cout=64, k=3, stride=1, pad=1, bias=True), dict(op="relu", src=0),
              dict(op="conv", src=1, cin=64, cout=64, k=3, stride=1, pad=1, bias=True), dict(op="relu", src=2),
              dict(op="maxpool2", src=3), dict(op="gap", src=4), dict(op="linear", src=5, cin=64, cout=10, bias=True)]
    params = synth.he_normal_params(layers, 6, True)
    s, e = synth.param_slices(layers)[2]["b"]
    params[s:e] = synth.to_bf16_grid(np.random.default_rng(3).standard_normal(e - s).astype(np.float32) * 0.2)
    x = torch.randn(B, 16, 16, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1)).to(torch.bfloat16)
    net = omni.net_create(layers, (16, 16, 3), "bf16", 1, B)
    ws = torch.zeros(omni.net_workspace_bytes(net), dtype=torch.uint8, device="cuda")
    lpw, loss = torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    omni.step(net, torch.from_numpy(params).cuda(), x, torch.zeros(B, dtype=torch.int32, device="cuda"), [0, B], [B], 0.0, ws, lpw,
              loss, omni.STEP_NO_UPDATE)
    torch.cuda.synchronize()
    src = omni.net_activation(net, ws, 1, B, "bf16").reshape(B, 16, 16, 64)
    out = omni.net_activation(net, ws, 3, B, "bf16").reshape(B, 16, 16, 64)
    pooled = omni.net_activation(net, ws, 4, B, "bf16").reshape(B, 8, 8, 64)
    assert torch.equal(out.float().reshape(B, 8, 2, 8, 2, 64).amax((2, 4)), pooled.float())
    at = [0, 1, 2, 3, 2047, 2048, 2049, 4094, 4095, 4096, 4097, 4098, 4099]
    a, got = src[at].cpu().double().permute(0, 3, 1, 2), out[at].cpu().double().permute(0, 3, 1, 2)
    omni.net_destroy(net)
    w = torch.from_numpy(params[slice(*synth.param_slices(layers)[2]["w"])].astype(np.float64)).reshape(64, 3, 3, 64).permute(0, 3, 1, 2)
    b = torch.from_numpy(params[s:e].astype(np.float64))
    want = torch.nn.functional.conv2d(a, w, b, padding=1)
    size = torch.nn.functional.conv2d(a.abs(), w.abs(), b.abs(), padding=1)
    assert float(((got - want.clamp(min=0)).abs() - 2.0 ** -8 * want.abs() - 576 * 2.0 ** -24 * size).max()) <= 0
