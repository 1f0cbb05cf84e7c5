"""The update by the launch that adds the chunks of the convolutions' weight gradients: bit for bit the update as a launch of its own
(which a caller that times it gets), with and without momentum, several steps on; workers of one chunk and of many, first layers
with a kernel of their own and without, channel tiles that are not full, parameters that are no convolution's.  The same of networks
that have the update in a launch of its own: a layer whose second stage is another, hidden fully connected layers."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_cnn import _check_step

pytestmark = pytest.mark.gpu


def _net(*ops):
    """Of 16x16x3 inputs.  conv: output channels, size, stride (no bias where a batch norm follows); linear: outputs."""
    layers, shape = [], (16, 16, 3)
    for i, (op, *a) in enumerate(ops):
        L = dict(op=op, src=len(layers) - 1)
        if op == "conv":
            L.update(cin=shape[2], cout=a[0], k=a[1], stride=a[2], pad=a[1] // 2, bias=ops[i + 1][0] != "bn")
        elif op == "bn":
            L.update(c=shape[2])
        elif op == "linear":
            L.update(cin=shape[0] * shape[1] * shape[2], cout=a[0], bias=True)
        layers.append(L)
        shape = synth.layer_shapes(layers, (16, 16, 3))[-1]
    return layers


RELU, BN, POOL, GAP = ("relu",), ("bn",), ("maxpool2",), ("gap",)
NETS = {
    "batch norms, 3x3 only": _net(("conv", 32, 3, 1), BN, RELU, ("conv", 64, 3, 1), BN, RELU, POOL, ("conv", 40, 3, 1), RELU, GAP,
                                  ("linear", 10)),
    "stride 2": _net(("conv", 32, 3, 1), RELU, ("conv", 64, 3, 2), RELU, ("conv", 64, 3, 1), RELU, GAP, ("linear", 10)),
    "1x1": _net(("conv", 32, 3, 1), RELU, ("conv", 64, 1, 1), RELU, ("conv", 64, 3, 1), RELU, GAP, ("linear", 10)),
    "hidden fully connected layers": _net(("conv", 32, 3, 1), RELU, POOL, ("conv", 64, 3, 1), RELU, POOL, ("linear", 256), RELU,
                                          ("linear", 72), RELU, ("linear", 10)),
}


@pytest.mark.parametrize("hw,chans,off", [
    (32, (3, 32, 64, 128), [0, 8, 24, 56, 128]),
    (32, (3, 32, 64, 128), [0, 1, 200, 203]),          # workers of one image
    (32, (3, 64, 24, 40), [0, 5, 70]),                 # two blocks of first-layer channels, tiles part full
    (32, (4, 40, 96, 64), [0, 33]),                    # 37 columns in the first layer, two channel tiles, one worker
    (16, (3, 16, 96, 256), [0, 3, 4, 100]),            # the first layer in the patch kernel
    (16, (3, 32, 64, 64), list(range(0, 130, 2))),     # 64 workers of two images
    (32, (3, 32, 64, 128), list(range(16)) + [300]),   # one of sixteen with most chunks (its wavefront the last; in quarters)
    (32, (3, 32, 64, 128), list(range(17)) + [300]),   # one of seventeen
])
@pytest.mark.parametrize("momentum", [False, True])
def test_update_with_the_second_stage(hw, chans, off, momentum):
    _same_as_own_launch(synth.cnn3(num_classes=10, hw=hw, chans=chans), (hw, hw, chans[0]), off, momentum)


# Workgroups of four wavefronts with more workers than that (1595 workgroups add chunks: more than 512) and of sixteen (145, and 30 for
# the other parameters: all resident at once), with one worker in the last turn and with full turns; eight: above.
@pytest.mark.parametrize("chans,off", [
    ((3, 16, 128, 256), [0, 1, 3, 7, 33, 57, 58, 60, 90, 100]),
    ((3, 16, 128, 256), list(range(32)) + [400]),
    ((3, 16, 128, 256), list(range(33)) + [400]),      # (one worker too many: eight)
    ((3, 32, 32, 64), list(range(0, 20, 2))),
    ((3, 32, 32, 64), list(range(0, 34, 2))),
    ((3, 32, 32, 64), [0, 1] + list(range(3, 35, 2))),
])
@pytest.mark.parametrize("momentum", [False, True])
def test_update_with_few_and_many_wavefronts(chans, off, momentum):
    _same_as_own_launch(synth.cnn3(num_classes=10, hw=16, chans=chans), (16, 16, 3), off, momentum)


@pytest.mark.parametrize("net", list(NETS))
@pytest.mark.parametrize("off", [[0, 1, 150, 203], [0, 2, 4, 6]])
@pytest.mark.parametrize("momentum", [False, True])
def test_update_of_other_networks(net, off, momentum):
    _same_as_own_launch(NETS[net], (16, 16, 3), off, momentum)


def _same_as_own_launch(layers, shape, off, momentum):
    import torch
    import paper_2503_17469_amd as omni
    B, K = off[-1], len(off) - 1
    b = [off[k + 1] - off[k] for k in range(K)]
    params = synth.he_normal_params(layers, 6, True)
    x, y = synth.make_batch(3, B, shape, 10, True)
    out = []
    for own_launch in (False, True):
        run = GpuRun(layers, shape, "bf16", K, B)
        try:
            p = torch.from_numpy(params).cuda()
            xs = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().to(torch.bfloat16)
            ys = torch.from_numpy(np.ascontiguousarray(y, dtype=np.int32)).cuda()
            v = torch.zeros_like(p)
            if momentum:
                omni.net_set_momentum(run.net, v, 0.9, 5e-4)
            if own_launch:
                omni.net_timing_enable(run.net, "update", -1, 8)
            for _ in range(3):
                run.ws.fill_(255)                      # nothing is left over from the step before
                omni.step(run.net, p, xs, ys, off, b, 0.002, run.ws, run.lpw, run.loss)
            torch.cuda.synchronize()
            if own_launch:
                assert omni.net_timing_read(run.net)[1] == 3
            out.append((p.cpu().numpy(), v.cpu().numpy(), omni.net_worker_grads(run.net, run.ws, K).cpu().numpy()[:, :params.size]))
        finally:
            run.close()
    assert not np.array_equal(out[0][0], params)
    for a, c in zip(*out):
        assert np.array_equal(a, c)


@pytest.mark.parametrize("layers,shape", [(synth.cnn3(num_classes=10, hw=32, chans=(3, 32, 64, 128)), (32, 32, 3))]
                         + [(layers, (16, 16, 3)) for layers in NETS.values()], ids=["cnn3"] + list(NETS))
@pytest.mark.parametrize("momentum", [False, True])
def test_update_follows_from_the_gradients(layers, shape, momentum):
    """One step: parameters and velocity against the weighted sum of the very gradients that the launch left, by the update entry."""
    import torch
    import paper_2503_17469_amd as omni
    off = [0, 1, 24, 56, 128]
    B, K = off[-1], len(off) - 1
    b = [off[k + 1] - off[k] for k in range(K)]
    params = synth.he_normal_params(layers, 6, True)
    x, y = synth.make_batch(3, B, shape, 10, True)
    run = GpuRun(layers, shape, "bf16", K, B)
    try:
        p = torch.from_numpy(params).cuda()
        xs = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().to(torch.bfloat16)
        ys = torch.from_numpy(np.ascontiguousarray(y, dtype=np.int32)).cuda()
        v = torch.randn(p.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) * 0.01
        p0, v0 = p.clone(), v.clone()
        if momentum:
            omni.net_set_momentum(run.net, v, 0.9, 5e-4)
        omni.step(run.net, p, xs, ys, off, b, 0.05, run.ws, run.lpw, run.loss)
        G = omni.net_worker_grads(run.net, run.ws, K)
        full = torch.zeros(K, (params.size + 63) // 64 * 64, device="cuda")
        full[:, :params.size] = G[:, :params.size]
        if momentum:
            omni.weighted_sgd_momentum(p0, v0, full, b, 0.05, 0.9, 5e-4, None)
        else:
            omni.weighted_sgd(p0, full, b, 0.05, None)
        torch.cuda.synchronize()
        assert torch.equal(p, p0) and torch.equal(v, v0)
    finally:
        run.close()


@pytest.mark.parametrize("net", ["1x1", "hidden fully connected layers"])
def test_step_of_other_networks(net):
    """the gradients themselves, and the update, against the oracle"""
    layers, off = NETS[net], [0, 20, 61, 150]
    params = synth.he_normal_params(layers, 6, True)
    x, y = synth.make_batch(3, off[-1], (16, 16, 3), 10, True)
    _check_step(layers, (16, 16, 3), params, x, y, off, 0.05, net)
