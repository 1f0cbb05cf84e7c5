"""The sums of the batch norm that ends a residual block's branch, taken along by the kernel that forms the input gradient of the
shortcut's: one or several trips of a workgroup, workers of one image, channels of two groups of 64."""
import pytest

from test_gpu_bn_sums import _check_backward, _conv, _tail

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hw,B,C", [(8, 3, 64), (8, 41, 64), (16, 22, 128), (32, 33, 64), (32, 150, 64), (8, 900, 128)])
def test_backward_sums_of_both_branches(hw, B, C):
    layers = [_conv(-1, C), dict(op="bn", src=0, c=C), dict(op="relu", src=1),
              dict(op="conv", src=2, cin=C, cout=C, k=3, stride=2, pad=1, bias=False), dict(op="bn", src=3, c=C), dict(op="relu", src=4),
              _conv(5, C), dict(op="bn", src=6, c=C),
              dict(op="conv", src=2, cin=C, cout=C, k=1, stride=2, pad=0, bias=False), dict(op="bn", src=8, c=C),
              dict(op="add", src=7, src2=9), dict(op="relu", src=10)] + _tail(11, C)
    _check_backward(layers, (hw, hw, C), B, [7])
