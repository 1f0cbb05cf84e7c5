"""A worker's rows have no part in another worker's gradient, loss or statistics: with one worker's inputs not finite, everybody
else's come out as they do without it, bit for bit.  Also a weight that is infinite stays an infinity in what it feeds."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun

pytestmark = pytest.mark.gpu


def _isolated(layers, shape, dtype, off, bad, value, seed):
    import paper_2503_17469_amd as omni
    K, B = len(off) - 1, off[-1]
    rng = np.random.default_rng(seed)
    params = synth.he_normal_params(layers, seed, dtype == "bf16")
    x = rng.standard_normal((B,) + shape).astype(np.float32)
    if dtype == "bf16":
        x = synth.to_bf16_grid(x)
    y = rng.integers(0, layers[-1]["cout"], B).astype(np.int32)
    run = GpuRun(layers, shape, dtype, K, B)
    try:
        clean = run.step(params, x, y, off, 0.0, flags=omni.STEP_NO_UPDATE, keep_g=False)
        x[off[bad]:off[bad + 1]] = value
        dirty = run.step(params, x, y, off, 0.0, flags=omni.STEP_NO_UPDATE, keep_g=False)
    finally:
        run.close()
    assert clean["status"] == 0 and np.all(np.isfinite(clean["worker_grads"]))
    assert not np.all(np.isfinite(dirty["worker_grads"][bad]))
    for k in range(K):
        if k == bad:
            continue
        assert np.array_equal(dirty["worker_grads"][k], clean["worker_grads"][k]), (k, off)
        assert dirty["loss_per_worker"][k] == clean["loss_per_worker"][k]


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("dims,off,bad", [
    ([784, 256, 10], [0, 8, 32], 1),                 # fewer than sixteen rows: the chunk reaches into the next worker's
    ([784, 256, 10], [0, 8, 32], 0),
    ([33, 17, 65, 9], [0, 1, 15, 16, 90], 1),
    ([257, 61, 7], [0, 300, 301, 900], 1),           # four wavefronts a tile
    ([3, 40, 2], [0, 2, 19], 1),                     # narrow layers
    ([64, 40, 10], [0, 1, 600, 1100], 1),            # rows shared out
    ([1030, 1022, 5], [0, 40, 43, 97], 1),           # tiled
    ([512, 1024, 1024, 10], [0, 40, 43, 300], 2),
])
def test_fp32(dims, off, bad, value):
    _isolated(synth.mlp(dims), (1, 1, dims[0]), "f32", off, bad, value, sum(dims))


@pytest.mark.parametrize("dims,off,bad", [([64, 96, 40, 10], [0, 5, 31, 77], 1), ([3072, 1024, 1024, 10], [0, 40, 43, 400], 1)])
def test_bf16_fully_connected(dims, off, bad):
    _isolated(synth.mlp(dims), (1, 1, dims[0]), "bf16", off, bad, np.inf, sum(dims))


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("hw,chans,off,bad", [
    (32, (3, 32, 64, 128), [0, 3, 4, 11], 1),
    (16, (3, 16, 24, 40), [0, 3, 4, 11], 1),
    (8, (3, 8, 32, 64), [0, 3, 4, 11], 1),
    (32, (3, 32, 64, 128), [0, 60, 131, 200], 1),
])
def test_convolutions(hw, chans, off, bad, value):
    _isolated(synth.cnn3(num_classes=10, hw=hw, chans=chans), (hw, hw, 3), "bf16", off, bad, value, hw)


@pytest.mark.parametrize("off,bad", [([0, 3, 4, 11], 1), ([0, 40, 75, 130], 1)])
def test_residual_network(off, bad):
    _isolated(synth.resnet18(num_classes=10, cin=3), (32, 32, 3), "bf16", off, bad, np.nan, off[-1])


@pytest.mark.parametrize("dtype,dims,at", [("f32", [40, 48, 10], 31), ("f32", [20, 24, 10], 0), ("bf16", [72, 104, 10], 69)])
def test_an_infinite_weight_gives_infinities(dtype, dims, at):
    """Widths off the kernels' chunks: what a chunk holds a second time, or in the place of what lies past a row's end (element
    `at` among it), counts zero in both operands."""
    layers = synth.mlp(dims)
    B = 19
    params = synth.he_normal_params(layers, 4, dtype == "bf16")
    sl = synth.param_slices(layers)[0]["w"]
    w = params[sl[0]:sl[1]].reshape(dims[1], dims[0])
    w[5, :] = 0.0
    w[5, at] = np.inf
    x = np.abs(np.random.default_rng(3).standard_normal((B, dims[0]))).astype(np.float32) + 0.5
    if dtype == "bf16":
        x = synth.to_bf16_grid(x)
    y = np.zeros(B, dtype=np.int32)
    run = GpuRun(layers, (1, 1, dims[0]), dtype, 2, B)
    try:
        run.step(params, x, y, [0, 7, B], 0.0, keep_g=False)
        hidden = run.activation(0, B)
    finally:
        run.close()
    assert np.all(np.isposinf(hidden[:, 5])), hidden[:3, 5]
    assert np.all(np.isfinite(np.delete(hidden, 5, axis=1)))
