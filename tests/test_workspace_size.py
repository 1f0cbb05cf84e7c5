"""How much workspace a network asks for: what its tensors and gradient rows take, and scratch of a stated size, so that the
static workspace and memory caps take the networks they are meant for."""
import random

import pytest

import paper_2503_17469_amd as omni
import synth

MIB = 1 << 20
FP32_SCRATCH = 16 * MIB
BF16_SCRATCH = 2 * 2048 * (4 * 16 * 256 + 128) * 4 + 16 * MIB    # two side streams' partial tiles, and the main stream's


def _up(v, a):
    return (v + a - 1) // a * a


def _bytes(layers, shape, dtype, K, B):
    net = omni.net_create(layers, shape, dtype, K, B)
    try:
        return omni.net_workspace_bytes(net), omni.net_grad_stride(net)
    finally:
        omni.net_destroy(net)


def _fp32_need(dims, stride, K, B):
    """gradient rows, the aggregated gradient, loss rows, status word, every layer's output and its gradient"""
    tensors = sum(2 * _up(B * d * 4, 256) for d in dims[1:])
    return (K + 1) * stride * 4 + _up(B * 4, 256) + 256 + tensors


def test_fp32_networks_need_their_tensors_and_bounded_scratch():
    rng = random.Random(5)
    with_scratch = 0
    for _ in range(300):
        dims = [rng.randint(1, 800)] + [rng.randint(1, 700) for _ in range(rng.randint(0, 4))] + [rng.randint(1, 120)]
        K = rng.choice((1, 2, 4, 8, 16, 64))
        B = rng.randint(K, 8192)
        got, stride = _bytes(synth.mlp(dims), (1, 1, dims[0]), "f32", K, B)
        need = _fp32_need(dims, stride, K, B)
        assert need <= got <= need + FP32_SCRATCH + 256, (dims, K, B)
        with_scratch += got > need + 256
        # no scratch where the weight gradients have more tiles than the chip has compute units, or few rows
        tiles = sum((o + 15) // 16 * ((i + 63) // 64) for i, o in zip(dims, dims[1:]))
        if tiles >= 256 or B < 850:
            assert got <= need + 256, (dims, K, B)
    assert with_scratch > 20


@pytest.mark.parametrize("dims,K,B", [([200, 300, 100, 50], 16, 1024), ([200, 300, 100, 50], 8, 2048),
                                      ([64, 128, 10], 64, 4096), ([784, 256, 10], 4, 1024)])
def test_small_networks_fit_the_static_workspace(dims, K, B):
    assert _bytes(synth.mlp(dims), (1, 1, dims[0]), "f32", K, B)[0] <= omni.STATIC_WORKSPACE_BYTES


def test_bf16_scratch():
    layers = synth.cnn3(num_classes=10, hw=32, chans=(3, 32, 64, 128))
    one, two = (_bytes(layers, (32, 32, 3), "bf16", 4, B)[0] for B in (128, 256))
    fixed = 2 * one - two                                   # what does not grow with the batch
    P = synth.param_count(layers)
    assert fixed <= BF16_SCRATCH + 5 * _up(P, 64) * 4 + 4 * _up(P, 64) * 2 + MIB
    assert one <= 316 * MIB
