"""GPU parity of the bf16 fully connected kernels at the edges of their tiles, and the update applied by the
weight-gradient launch against the update as a launch of its own."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_cnn import _check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,off", [
    ([8, 8, 2], [0, 1, 3]),                        # one piece per row, three rows
    ([56, 72, 40, 9], [0, 30, 31, 77]),            # reductions one piece short of a line and one past it
    ([64, 64, 64, 10], [0, 64, 128]),              # exact tiles and slabs
    ([200, 136, 33 * 8, 17], [0, 15, 16, 81, 145]),   # ragged tiles, slabs ending after 1, 15, 16, 17 rows
    ([520, 1024, 776, 5], [0, 300, 777]),          # enough 64 x 64 tiles for the wide forward kernel
])
def test_shapes(dims, off):
    layers = synth.mlp(dims)
    rng = np.random.default_rng(sum(dims))
    params = synth.he_normal_params(layers, 2, True)
    for sl in synth.param_slices(layers):
        if "b" in sl:
            s, e = sl["b"]
            params[s:e] = synth.to_bf16_grid(rng.standard_normal(e - s).astype(np.float32) * 0.2)
    x, y = synth.make_batch(5 + off[-1], off[-1], (1, 1, dims[0]), dims[-1], True)
    _check_step(layers, (1, 1, dims[0]), params, x, y, off, 0.1, f"bf16-mlp-{dims}")


@pytest.mark.parametrize("momentum", [False, True])
def test_update_inside_the_weight_gradient_launch(momentum):
    import torch
    import paper_2503_17469_amd as omni
    dims, off = [200, 136, 72, 10], [0, 9, 10, 90]
    b = [off[k + 1] - off[k] for k in range(len(off) - 1)]
    layers = synth.mlp(dims)
    params = synth.he_normal_params(layers, 3, True)
    x, y = synth.make_batch(6, off[-1], (1, 1, dims[0]), dims[-1], True)
    out = []
    for own_launch in (False, True):
        run = GpuRun(layers, (1, 1, dims[0]), "bf16", len(b), off[-1])
        try:
            p, ys = torch.from_numpy(params).cuda(), torch.from_numpy(y).cuda()
            xs = torch.from_numpy(x.reshape(off[-1], -1)).cuda().to(torch.bfloat16)
            v = torch.zeros_like(p)
            if momentum:
                omni.net_set_momentum(run.net, v, 0.9, 5e-4)
            if own_launch:
                omni.net_timing_enable(run.net, "update", -1, 8)
            for _ in range(3):
                omni.step(run.net, p, xs, ys, off, b, 0.05, run.ws, run.lpw, run.loss)
            torch.cuda.synchronize()
            if own_launch:
                assert omni.net_timing_read(run.net)[1] == 3
            out.append((p.cpu().numpy(), v.cpu().numpy(), omni.net_worker_grads(run.net, run.ws, len(b)).cpu().numpy()))
        finally:
            run.close()
    for a, c in zip(*out):
        assert np.array_equal(a, c)
