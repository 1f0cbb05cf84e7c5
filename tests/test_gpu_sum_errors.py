"""Errors of the fp32 sums of fully connected layers against float64, over the values the library stored.

A chain of m fp32 additions of independent terms has a relative error of about 0.28 u sqrt(m), u = 2^-24: every rounding is
0.4 u of the partial sum (root mean square), which grows with the root of the terms added.  Sums of sums add up in squares.
The kernels form a piece of a reduction by itself and add the pieces, so that both chains are short; the tests state the
lengths of both and allow 1.3 times the model.  One chain over a whole reduction fails all cases but one of the classifier's."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _limit(*chains):
    return 1.3 * 0.28 * U * np.sqrt(sum(chains)) + 0.3 * U      # (0.3 u: the result's own rounding)


def _run(dims, off, dtype):
    """[(x, dy, gw per worker, z, dx, mask)] per layer, float64"""
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.mlp(dims)
    B, K = off[-1], len(off) - 1
    rng = np.random.default_rng(sum(dims) + B)
    params = synth.he_normal_params(layers, 7, dtype == "bf16")
    x = rng.standard_normal((B, dims[0])).astype(np.float32)
    if dtype == "bf16":
        x = synth.to_bf16_grid(x)
    y = rng.integers(0, dims[-1], B).astype(np.int32)
    run = GpuRun(layers, (1, 1, dims[0]), dtype, K, B)
    out = []
    try:
        got = run.step(params, x, y, off, 0.0, keep_g=False)
        for i, L in enumerate(layers):
            if L["op"] != "linear":
                continue
            last = i == len(layers) - 1
            stored = "f32" if last else dtype
            s, e = synth.param_slices(layers)[i]["w"]
            bs, be = synth.param_slices(layers)[i]["b"]
            xin = x if L["src"] < 0 else run.activation(L["src"], B)
            grad = lambda layer, dt: omni.net_activation_grad(run.net, run.ws, layer, B, dt).double().cpu()
            out.append(dict(
                x=torch.from_numpy(np.ascontiguousarray(xin)).double(),
                w=torch.from_numpy(params[s:e].reshape(L["cout"], L["cin"])).double(),
                b=torch.from_numpy(params[bs:be]).double(),
                z=omni.net_activation(run.net, run.ws, i, B, stored).double().cpu(),
                dy=grad(i, stored),
                dx=grad(L["src"], dtype) if L["src"] >= 0 else None,
                gw=[torch.from_numpy(got["worker_grads"][k, s:e].reshape(L["cout"], L["cin"])).double() for k in range(K)],
                last=last))
    finally:
        run.close()
    return out


def _rel(pairs):
    num = sum(float(((a - e) ** 2).sum()) for a, e in pairs)
    den = sum(float((e ** 2).sum()) for a, e in pairs)
    return (num / den) ** 0.5


def _wgrad_error(L, off):
    return _rel([(L["gw"][k], L["dy"][off[k]:off[k + 1]].T @ L["x"][off[k]:off[k + 1]]) for k in range(len(off) - 1)])


@pytest.mark.parametrize("dims,off,dtype,layer,chains", [
    # tiled: slabs of 32 rows
    ([1024, 1024, 1024, 100], [0, 2000], "f32", 0, (32, 63)),
    ([3072, 1024, 1024, 10], [0, 1024, 2048, 4096], "f32", 0, (32, 64)),
    # small, a wavefront per tile (chunks of 16 rows), and four (the rows dealt to them)
    ([997, 501, 243, 37], [0, 333], "f32", 0, (16, 21)),
    ([257, 61, 7], [0, 900], "f32", 0, (16, 15, 4)),
    # bf16: four slabs of 64 rows, sixteen rows to an instruction
    ([512, 512, 512, 10], [0, 1000, 3000], "bf16", 0, (16, 8)),
    ([512, 512, 512, 10], [0, 1000, 3000], "bf16", 1, (16, 8)),
    # classifier: a row in 64 or 16 per thread, their sums in four chains
    ([3072, 1024, 1024, 10], [0, 256], "f32", 2, (4, 16, 4)),
])
def test_weight_gradients(dims, off, dtype, layer, chains):
    err = _wgrad_error(_run(dims, off, dtype)[layer], off)
    assert err <= _limit(*chains), (err / U, _limit(*chains) / U)


@pytest.mark.parametrize("dims,off,layer,chains", [
    ([3072, 1024, 1024, 10], [0, 1024, 2048, 4096], 0, (32, 96)),     # tiled
    ([784, 256, 10], [0, 1000], 0, (64, 4, 4)),                       # small: two chunks of 32, four wavefronts
    ([997, 501, 243, 37], [0, 333], 0, (64, 4, 4)),
    ([3072, 1024, 1024, 10], [0, 480], 2, (16, 2, 4, 8)),             # classifier: half lines of 16, eight wavefronts
    ([1024, 1024, 1024, 100], [0, 2000], 2, (16, 2, 8, 4)),
])
def test_forward(dims, off, layer, chains):
    L = _run(dims, off, "f32")[layer]
    z = L["x"] @ L["w"].T + L["b"]
    err = _rel([(L["z"], z if L["last"] else z.clamp(min=0))])
    assert err <= _limit(*chains), (err / U, _limit(*chains) / U)


@pytest.mark.parametrize("dims,off,layer,chains", [
    ([1024, 1024, 1024, 100], [0, 2000], 1, (32, 32)),                # tiled
    ([1030, 1022, 600, 5], [0, 300, 1000], 1, (32, 19)),
    ([997, 501, 243, 37], [0, 333], 2, (16, 3)),                      # classifier: sixteen classes
])
def test_input_gradients(dims, off, layer, chains):
    L = _run(dims, off, "f32")[layer]
    dx = (L["dy"] @ L["w"]) * (L["x"] > 0)
    err = _rel([(L["dx"], dx)])
    assert err <= _limit(*chains), (err / U, _limit(*chains) / U)
