"""GPU parity of the fp32 products on both sides of the line between the kernels that split a product's reduction: as many 32 x 32
tiles as the chip has compute units and one row of tiles more, ragged rows, outputs that end inside a 64-column tile."""
import pytest

from gpu_util import GpuRun, assert_close, param_tensor_slices
from oracle import step as oracle_step
from test_gpu_mlp_shapes import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,off", [
    ([256, 1024, 1024, 10], [0, 100, 256]),       # 8 x 32 tiles: the small kernels
    ([256, 1024, 1024, 10], [0, 100, 257]),       # a ninth row of tiles, one row of it used
    ([288, 1002, 520, 10], [0, 31, 390]),         # widths that end inside a tile; the second layer's input gradient one way, its output the other
    ([264, 1024, 10], [0, 300]),                  # a reduction off the step: the small kernels, more than one round
])
def test_rounds(dims, off):
    layers, params, x, labels = _case(dims, off, sum(dims) + off[-1])
    ref = oracle_step.sgd_step(layers, params, x.reshape(-1, 1, 1, dims[0]), labels, off, 0.05)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", len(off) - 1, off[-1])
    try:
        got = run.step(params, x, labels, off, 0.05, keep_g=False)
        assert got["status"] == 0
        assert_close(got["loss_per_worker"], ref.loss_per_worker, 1e-4, "L_k")
        for name, s, e in param_tensor_slices(layers):
            for k in range(len(off) - 1):
                assert_close(got["worker_grads"][k, s:e], ref.worker_grads[k, s:e], 1e-4, f"g_{k} {name}", tol_max=5e-4)
            assert_close(got["params"][s:e], ref.params[s:e], 1e-4, f"theta' {name}")
    finally:
        run.close()
