"""Weight gradients of fully connected layers with few tiles, a workgroup per tile and worker and the update behind them: at both
sides of the rules, workers of one row, of less than a slab, of exactly one and of several, against float64 on the values the
library stored."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_sum_errors import U, _limit, _run, _wgrad_error

pytestmark = pytest.mark.gpu

OFF4 = [0, 1, 64, 128, 400]
OFF8 = [0, 1, 16, 79, 143, 207, 208, 271, 530]
OFF16 = [0] + [3 + 17 * k for k in range(15)] + [330]


@pytest.mark.parametrize("dims,off,dtype,chains", [
    ([216, 160, 232, 10], OFF4, "bf16", (16, 17)),
    ([216, 160, 232, 10], [0, 100, 130, 400], "bf16", (16, 17)),     # three workers: together
    ([648, 512, 64, 7], OFF4, "bf16", (16, 17)),            # 88 + 8 tiles: the most
    ([648, 512, 72, 7], OFF4, "bf16", (16, 17)),            # 104: together
    ([1024, 640, 8], OFF16, "bf16", (16, 6)),               # 160 tiles and sixteen workers
    ([8, 16, 3], OFF8, "bf16", (16, 17)),
    ([64, 128, 10], OFF8, "f32", (16, 5, 4)),
    ([64, 128, 10], OFF8[:8], "f32", (16, 5, 4)),           # seven workers: together
    ([130, 67, 33, 10], OFF16, "f32", (16, 5, 4)),
])
def test_gradients(dims, off, dtype, chains):
    layers = _run(dims, off, dtype)
    for layer in layers[:-1]:
        err = _wgrad_error(layer, off)
        assert err <= _limit(*chains), (err / U, _limit(*chains) / U)


@pytest.mark.parametrize("dims,off,dtype", [([216, 160, 232, 10], OFF4, "bf16"), ([64, 128, 10], OFF8, "f32")])
@pytest.mark.parametrize("momentum", [False, True])
def test_update_of_all_parameters(dims, off, dtype, momentum):
    """theta' and the velocity from the gradients the step left, in float64: fp32 sums of at most eight terms, 1e-6; and twice
    the same bits on a workspace that holds something else."""
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.mlp(dims)
    rng = np.random.default_rng(3)
    params = synth.he_normal_params(layers, 4, dtype == "bf16")
    x = rng.standard_normal((off[-1], dims[0])).astype(np.float32)
    if dtype == "bf16":
        x = synth.to_bf16_grid(x)
    y = rng.integers(0, dims[-1], off[-1]).astype(np.int32)
    K, B = len(off) - 1, off[-1]
    b = np.diff(off).astype(np.float64)
    run = GpuRun(layers, (1, 1, dims[0]), dtype, K, B)
    try:
        got = []
        for fill in (0, 255):
            p, v = torch.from_numpy(params).cuda(), torch.zeros(params.size, device="cuda")
            if momentum:
                omni.net_set_momentum(run.net, v, 0.9, 5e-4)
            run.ws.fill_(fill)
            xs = torch.from_numpy(x).cuda()
            xs = xs.bfloat16() if dtype == "bf16" else xs
            omni.step(run.net, p, xs, torch.from_numpy(y).cuda(), off, [int(t) for t in b], 0.05, run.ws, run.lpw, run.loss)
            torch.cuda.synchronize()
            got.append((p.cpu().numpy(), v.cpu().numpy(), omni.net_worker_grads(run.net, run.ws, K).cpu().numpy()[:, :params.size]))
        for one, two in zip(*got):
            assert np.array_equal(one, two)
    finally:
        run.close()
    p, v, g = got[0]
    step = (b[:, None] / B * g.astype(np.float64)).sum(0)
    if momentum:
        step += 5e-4 * params.astype(np.float64)
        assert np.abs(v - step).max() <= 1e-6 * np.abs(step).max()
    want = params - 0.05 * step
    assert np.abs(p - want).max() <= 1e-6 * np.abs(want).max()
