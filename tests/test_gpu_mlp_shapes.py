"""GPU parity of the fp32 products at the edges of their kernels' tiles: reductions shorter than a chunk, widths below a
vector, pieces moved back at a row's end, few and many rows, one wavefront per tile and four, and the update applied by the
weight-gradient launch against the update as a launch of its own."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun, assert_close, param_tensor_slices
from oracle import step as oracle_step

pytestmark = pytest.mark.gpu


def _case(dims, off, seed):
    layers = synth.mlp(dims)
    rng = np.random.default_rng(seed)
    params = synth.he_normal_params(layers, seed + 1, False)
    params += (rng.standard_normal(params.size) * 0.05).astype(np.float32)
    x = rng.standard_normal((off[-1], dims[0])).astype(np.float32)
    labels = rng.integers(0, dims[-1], off[-1]).astype(np.int32)
    return layers, params, x, labels


@pytest.mark.parametrize("dims,off", [
    ([1, 5, 3], [0, 1, 2]),                       # one input column: the narrow weight-gradient kernel
    ([3, 40, 2], [0, 2, 19]),                     # fewer inputs than a vector
    ([31, 33, 1], [0, 7, 40]),                    # a reduction one short of a chunk, one class
    ([33, 17, 65, 9], [0, 1, 15, 16, 90]),        # one past a chunk, columns one past a tile
    ([64, 16, 16, 4], [0, 16, 32, 48]),           # exact tiles
    ([130, 67, 33, 129], [0, 5, 70]),             # more classes than the fused head takes
    ([257, 61, 7], [0, 300, 301, 900]),           # few tiles and many rows: four wavefronts per tile
    ([515, 514, 21], [0, 3, 4, 131]),             # 32 x 32 tiles, rows off the vector
    ([1030, 1022, 5], [0, 40, 97]),               # enough 64 x 64 tiles for the tiled weight gradient, odd widths
])
def test_shapes(dims, off):
    layers, params, x, labels = _case(dims, off, sum(dims) + off[-1])
    ref = oracle_step.sgd_step(layers, params, x.reshape(-1, 1, 1, dims[0]), labels, off, 0.05)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", len(off) - 1, off[-1])
    try:
        # (without keeping the aggregated gradient: the update then runs inside the weight-gradient launch)
        got = run.step(params, x, labels, off, 0.05, keep_g=False)
        assert got["status"] == 0
        assert_close(got["loss_per_worker"], ref.loss_per_worker, 1e-4, "L_k")
        for name, s, e in param_tensor_slices(layers):
            for k in range(len(off) - 1):
                assert_close(got["worker_grads"][k, s:e], ref.worker_grads[k, s:e], 1e-4, f"g_{k} {name}", tol_max=5e-4)
            assert_close(got["params"][s:e], ref.params[s:e], 1e-4, f"theta' {name}")
    finally:
        run.close()


@pytest.mark.parametrize("dims,off", [([61, 35, 6], [0, 9, 30]), ([257, 61, 7], [0, 300, 301, 900]),
                                      ([1030, 1022, 5], [0, 40, 97]),
                                      ([3400, 1021, 10], [0, 600, 1300, 1400])])      # split products, workers' rows in two pieces and in one
@pytest.mark.parametrize("momentum", [False, True])
def test_update_inside_the_weight_gradient_launch(dims, off, momentum):
    """Bit for bit the update as a launch of its own (which a caller that times it gets), several steps on."""
    import torch
    import paper_2503_17469_amd as omni
    layers, params, x, labels = _case(dims, off, 5 + sum(dims))
    b = [off[k + 1] - off[k] for k in range(len(off) - 1)]
    out = []
    for own_launch in (False, True):
        run = GpuRun(layers, (1, 1, dims[0]), "f32", len(b), off[-1])
        try:
            p, xs, ys = torch.from_numpy(params).cuda(), torch.from_numpy(x).cuda(), torch.from_numpy(labels).cuda()
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


@pytest.mark.parametrize("dims,off", [([64, 40, 10], [0, 1, 1100]), ([33, 17, 65, 9], [0, 700, 703, 1500]),
                                      ([6, 16, 3], [0, 1024])])
@pytest.mark.parametrize("momentum", [False, True])
def test_rows_of_a_weight_gradient_shared_out(dims, off, momentum):
    """Few weights and many rows: a worker's rows in several shares (one worker with a single row, one with three), whose
    partial gradients wait in the workspace; also on a workspace that holds something else."""
    layers, params, x, labels = _case(dims, off, 9 + sum(dims))
    ref = oracle_step.sgd_step(layers, params, x.reshape(-1, 1, 1, dims[0]), labels, off, 0.05)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", len(off) - 1, off[-1])
    try:
        import torch
        import paper_2503_17469_amd as omni
        if momentum:
            vel = torch.zeros(params.size, device="cuda")
            omni.net_set_momentum(run.net, vel, 0.9, 0.0)     # the first step's update is the plain one
        got = run.step(params, x, labels, off, 0.05, keep_g=False)
        run.ws.fill_(0xFF)
        again = run.step(params, x, labels, off, 0.05, keep_g=False) if not momentum else got
        assert got["status"] == 0 and np.array_equal(got["params"], again["params"])
        for name, s, e in param_tensor_slices(layers):
            for k in range(len(off) - 1):
                assert_close(got["worker_grads"][k, s:e], ref.worker_grads[k, s:e], 1e-4, f"g_{k} {name}", tol_max=5e-4)
            assert_close(got["params"][s:e], ref.params[s:e], 1e-4, f"theta' {name}")
    finally:
        run.close()


@pytest.mark.parametrize("dims,K,B", [([384, 384, 10], 24, 2100),    # as many shares as the scratch holds, fewer than wanted
                                      ([64, 150, 12], 64, 2048),     # one share per worker and a few more
                                      ([384, 384, 10], 64, 2100)])   # not even one per worker: no shares
def test_rows_shared_out_within_the_scratch(dims, K, B):
    off = [0] + [min(B, 1 + k + (k * (B - K)) // K) for k in range(1, K)] + [B]
    assert all(a < c for a, c in zip(off, off[1:]))
    layers, params, x, labels = _case(dims, off, K + B)
    ref = oracle_step.sgd_step(layers, params, x.reshape(-1, 1, 1, dims[0]), labels, off, 0.05)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", K, B)
    try:
        got = run.step(params, x, labels, off, 0.05, keep_g=False)
        assert got["status"] == 0
        for name, s, e in param_tensor_slices(layers):
            for k in range(K):
                assert_close(got["worker_grads"][k, s:e], ref.worker_grads[k, s:e], 1e-4, f"g_{k} {name}", tol_max=5e-4)
            assert_close(got["params"][s:e], ref.params[s:e], 1e-4, f"theta' {name}")
    finally:
        run.close()
