"""Convolutions whose workgroups walk through several units of positions (the next one's loads under way when a unit ends, buffers
changing roles from unit to unit, the last workgroup's share short): the variants without sums of the wide 3x3 kernel (64- and 32-channel
tiles, two slices of the reduction and three), of the block entries' input gradients (one slice, two, three; projection, another share)
and of the gathering kernel (with bias and ReLU), against float64 on some of the images.

Bounds as in test_gpu_conv3_staging.py, test_gpu_block_entry.py and test_gpu_conv_gather.py."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import GpuRun
from test_gpu_block_entry import _layers as entry_layers
from test_gpu_conv3_staging import _layers as wide_layers
from test_gpu_conv_gather import _net as gather_layers

pytestmark = pytest.mark.gpu


class _Step:
    """One step of B images; tensors of the images `at`: first, last, at a worker's edge, and some between."""

    def __init__(self, layers, h, w, off):
        import paper_2503_17469_amd as omni
        B = off[-1]
        self.layers, self.params = layers, synth.he_normal_params(layers, 17, True)
        self.slices = synth.param_slices(layers)
        rng = np.random.default_rng(B + h)
        for L, sl in zip(layers, self.slices):
            if "b" in sl and L["op"] == "conv":
                s, e = sl["b"]
                self.params[s:e] = synth.to_bf16_grid(0.2 * rng.standard_normal(e - s).astype(np.float32))
        x = synth.to_bf16_grid(rng.standard_normal((B, h, w, 8)).astype(np.float32))
        y = rng.integers(0, 10, B).astype(np.int32)
        at = {min(max(i, 0), B - 1) for o in off for i in range(o - 4, o + 4)} | set(range(0, B, B // 24))
        self.at = torch.tensor(sorted(at))
        run = GpuRun(layers, (h, w, 8), "bf16", len(off) - 1, B)
        try:
            assert run.step(self.params, x, y, off, 0.0)["status"] == 0
            shapes = synth.layer_shapes(layers, (h, w, 8))
            self.out, self.grad = {}, {}
            for i, L in enumerate(layers[:-1]):
                if L["op"] not in ("conv", "relu", "bn", "maxpool2"):
                    continue
                for store, get in ((self.out, omni.net_activation), (self.grad, omni.net_activation_grad)):
                    try:
                        t = get(run.net, run.ws, i, B, "bf16").reshape(B, *shapes[i])
                    except omni.OmniError:                     # (not stored)
                        continue
                    store[i] = t[self.at.cuda()].double().cpu().permute(0, 3, 1, 2)
        finally:
            run.close()

    def weight(self, i):
        L = self.layers[i]
        k = L["k"]
        W = torch.from_numpy(self.params[slice(*self.slices[i]["w"])].astype(np.float64)).reshape(L["cout"], k, k, L["cin"])
        return W.permute(0, 3, 1, 2)

    def bias(self, i):
        return torch.from_numpy(self.params[slice(*self.slices[i]["b"])].astype(np.float64))


def _outside(got, want, size, terms, slack=0.0):
    return float(((got - want).abs() - slack - 2.0 ** -8 * want.abs() - terms * 2.0 ** -24 * size).max())


# units of 256 positions x 64 (or 32) channels, two and more to a workgroup from 4096 on
@pytest.mark.parametrize("h,w,cin,cout,before,off", [
    (16, 16, 96, 64, "relu", [0, 5, 4099]),
    (16, 16, 64, 32, "none", [0, 4101]),
    (16, 16, 32, 96, "none", [0, 1, 4101]),
    (8, 8, 64, 64, "relu", [0, 7, 16395]),
    (32, 32, 64, 64, "none", [0, 3, 1027]),
])
def test_wide(h, w, cin, cout, before, off):
    layers, i = wide_layers(cin, cout, before)
    s = _Step(layers, h, w, off)
    conv = torch.nn.functional.conv2d
    X, W, b, T = s.out[i - 1], s.weight(i), s.bias(i), s.weight(i).flip(2, 3).transpose(0, 1)
    assert _outside(s.out[i + 1], conv(X, W, b, padding=1).clamp(min=0), conv(X.abs(), W.abs(), b.abs(), padding=1), 9 * cin + 1) <= 0
    dY, keep = s.grad[i], (X > 0).double() if before == "relu" else torch.ones_like(X)
    assert float(dY.abs().max()) > 0
    assert _outside(s.grad[i - 1], conv(dY, T, padding=1) * keep, conv(dY.abs(), T.abs(), padding=1), 9 * cout) <= 0


# units of 512 positions x 64 channels, two to a workgroup from 2048 on
@pytest.mark.parametrize("h,w,cin,cout,beside,off", [
    (16, 16, 64, 32, "none", [0, 1, 4101]),
    (16, 16, 64, 96, "projection", [0, 4101]),
    (8, 8, 64, 64, "twin", [0, 3, 16397]),
    (32, 32, 64, 64, "none", [0, 2, 1027]),
])
def test_block_entries(h, w, cin, cout, beside, off):
    s = _Step(entry_layers(cin, cout, beside), h, w, off)
    X, got = s.out[1], s.grad[1]
    want, size, slack = torch.zeros_like(got), torch.zeros_like(got), 0.0
    for i in [2] if beside == "none" else [2, 3]:
        back = lambda a, b: torch.nn.functional.conv_transpose2d(a, b, stride=2, padding=s.layers[i]["k"] // 2, output_padding=1)
        d, W = s.grad[i], s.weight(i)
        assert float(d.abs().max()) > 0
        share = back(d, W)
        want += share
        size += back(d.abs(), W.abs())
        if beside == "twin" and i == 3:
            slack = 2.0 ** -8 * share.abs()
    assert _outside(got, want * (X > 0), size, 10 * cout, slack) <= 0


# tiles of 256 positions x 128 channels, two to a workgroup from 2048 on
@pytest.mark.parametrize("h,w,cin,cout,k,stride,off", [
    (16, 16, 32, 256, 3, 2, [0, 5, 4107]),
    (8, 8, 64, 256, 1, 1, [0, 4107]),
    (16, 16, 96, 256, 1, 2, [0, 1, 4107]),
])
def test_gather(h, w, cin, cout, k, stride, off):
    s = _Step(gather_layers(h, w, cin, cout, k, stride, "relu"), h, w, off)
    X, W, b = s.out[1], s.weight(2), s.bias(2)
    conv = lambda *a: torch.nn.functional.conv2d(*a, stride=stride, padding=k // 2)
    assert _outside(s.out[3], conv(X, W, b).clamp(min=0), conv(X.abs(), W.abs(), b.abs()), k * k * cin + 1) <= 0


# (as test_wide; the pooled values are those stored, to the bit)
@pytest.mark.parametrize("h,w,cin,cout,off", [(16, 16, 64, 64, [0, 4099]), (8, 8, 96, 32, [0, 1, 16397])])
def test_wide_with_pooling(h, w, cin, cout, off):
    front = wide_layers(cin, cout, "none")[0][:3]
    s = _Step(front + [dict(op="maxpool2", src=2), dict(op="gap", src=3), dict(op="linear", src=4, cin=cout, cout=10, bias=True)], h, w, off)
    X, W, b = s.out[0], s.weight(1), s.bias(1)
    conv = torch.nn.functional.conv2d
    assert _outside(s.out[2], conv(X, W, b, padding=1).clamp(min=0), conv(X.abs(), W.abs(), b.abs(), padding=1), 9 * cin + 1) <= 0
    assert torch.equal(s.out[3], torch.nn.functional.max_pool2d(s.out[2], 2))
