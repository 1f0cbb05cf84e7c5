"""Forward convolutions at stride 2, and with one tap, whose rows are gathered straight into LDS (conv_gather_bf16.hip), against float64
over the very tensors the library stored: maps of even and odd sides, tiles that end inside an image and with a worker, one step of
the reduction per tap and several, one channel tile and several, several tiles to a workgroup; and the sums of the batch norm behind.

Bound, per element: a bf16 rounding, 2^-8, of the result, and fp32 sums of k k cin terms, each off by at most 2^-24 of the sum of
their magnitudes.  Statistics: that of test_gpu_bn_sums.py."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from oracle import layers as OL

pytestmark = pytest.mark.gpu

# (tiles of 256 positions by 128 channels, at least 256 of them)
CASES = [
    (32, 32, 64, 128, 3, 2, [0, 1, 260]),
    (15, 17, 32, 128, 3, 2, [0, 300, 920]),
    (16, 16, 96, 256, 3, 2, [0, 3, 4, 520]),
    (4, 4, 64, 512, 3, 2, [0, 4100]),
    (2, 2, 64, 128, 3, 2, [0, 7, 65600]),
    (14, 14, 32, 384, 1, 2, [0, 460]),
    (32, 32, 64, 128, 1, 2, [0, 1, 1100]),
    (9, 9, 64, 128, 1, 1, [0, 400, 815]),
]


def _net(h, w, cin, cout, k, s, after):
    c = dict(op="conv", src=1, cin=cin, cout=cout, k=k, stride=s, pad=k // 2, bias=after == "relu")
    return [dict(op="conv", src=-1, cin=8, cout=cin, k=1, stride=1, pad=0, bias=True), dict(op="relu", src=0), c,
            dict(op="relu", src=2) if after == "relu" else dict(op="bn", src=2, c=cout), dict(op="gap", src=3),
            dict(op="linear", src=4, cin=cout, cout=10, bias=True)]


@pytest.mark.parametrize("after", ["relu", "bn"])
@pytest.mark.parametrize("h,w,cin,cout,k,s,off", CASES)
def test_against_float64(h, w, cin, cout, k, s, off, after):
    import torch
    layers = _net(h, w, cin, cout, k, s, after)
    B, K = off[-1], len(off) - 1
    oh, ow = (h - 1) // s + 1, (w - 1) // s + 1
    params = synth.he_normal_params(layers, 13, True)
    rng = np.random.default_rng(h * w + cout)
    sl = synth.param_slices(layers)
    if after == "relu":
        params[slice(*sl[2]["b"])] = synth.to_bf16_grid(0.2 * rng.standard_normal(cout).astype(np.float32))
    else:
        params[slice(*sl[3]["gamma"])] = 1.0
        params[slice(*sl[3]["beta"])] = 0.0
    x = synth.to_bf16_grid(rng.standard_normal((B, h, w, 8)).astype(np.float32))
    y = rng.integers(0, 10, B).astype(np.int32)
    run = GpuRun(layers, (h, w, 8), "bf16", K, B)
    try:
        assert run.step(params, x, y, off, 0.0)["status"] == 0
        X = torch.from_numpy(run.activation(1, B)).reshape(B, h, w, cin).permute(0, 3, 1, 2)
        Y = run.activation(3 if after == "relu" else 2, B).reshape(B, oh * ow, cout)
        Z = run.activation(3, B).reshape(B, oh * ow, cout)
    finally:
        run.close()
    W = torch.from_numpy(params[slice(*sl[2]["w"])].astype(np.float64)).reshape(cout, k, k, cin).permute(0, 3, 1, 2)
    b = torch.from_numpy(params[slice(*sl[2]["b"])].astype(np.float64)) if after == "relu" else None
    # (every worker's first and last images, and some between)
    at = sorted({min(max(i, 0), B - 1) for o in off for i in range(o - 3, o + 3)} | set(range(0, B, max(1, B // 40))))
    xs = X[at].double()
    want = torch.nn.functional.conv2d(xs, W, b, stride=s, padding=k // 2)
    size = torch.nn.functional.conv2d(xs.abs(), W.abs(), None if b is None else b.abs(), stride=s, padding=k // 2)
    if after == "relu":
        want = want.clamp(min=0)
    got = torch.from_numpy(Y[at]).double().reshape(len(at), oh, ow, cout).permute(0, 3, 1, 2)
    assert float(((got - want).abs() - 2.0 ** -8 * want.abs() - (k * k * cin + 1) * 2.0 ** -24 * size).max()) <= 0
    if after == "bn":
        for i in range(K):
            v = Y[off[i]:off[i + 1]].reshape(-1, cout).astype(np.float64)
            mean, inv = v.mean(0), 1.0 / np.sqrt(v.var(0) + 1e-5)
            xhat = (v - mean) * inv
            slack = 2.0 ** -23 * (np.abs(mean) * inv + 8 * np.abs(xhat))
            z = Z[off[i]:off[i + 1]].reshape(-1, cout)
            assert ((z >= OL.round_bf16(xhat - slack)) & (z <= OL.round_bf16(xhat + slack))).all()
