"""GPU: omni_step_static (the step on the library's own fixed workspace, for callers that cannot allocate)
against omni_step with a workspace of the caller's, through the C-ABI."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _both(omni, torch, net, ws, params_np, x_np, y_np, off, lr, K_max):
    b = [off[k + 1] - off[k] for k in range(len(off) - 1)]
    B = off[-1]
    out = []
    for static in (False, True):
        params = torch.from_numpy(params_np.copy()).cuda()
        x = torch.from_numpy(np.ascontiguousarray(x_np[:B]).reshape(B, -1)).cuda()
        y = torch.from_numpy(np.ascontiguousarray(y_np[:B])).cuda()
        lpw = torch.full((K_max,), -1.0, device="cuda")
        loss = torch.full((1,), -1.0, device="cuda")
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        if static:
            omni.step_static(net, params, x, y, off, b, lr, lpw, loss)
        else:
            omni.step(net, params, x, y, off, b, lr, ws, lpw, loss)
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() == before
        out.append((params.cpu().numpy(), lpw.cpu().numpy()[:len(b)], float(loss.item())))
    return out


def test_static_workspace_step_matches_the_step_with_a_caller_workspace():
    import torch
    import paper_2503_17469_amd as omni
    from oracle import step as OS
    from gpu_util import assert_close
    # a network of a few layers whose products split their reduction over the wavefronts of a workgroup
    dims = [512, 1024, 128, 10]
    layers = synth.mlp(dims)
    rng = np.random.default_rng(31)
    params = synth.he_normal_params(layers, 5, False)
    params += (rng.standard_normal(params.size) * 0.05).astype(np.float32)
    K_max, B_max = 4, 96
    x = rng.standard_normal((B_max, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], B_max).astype(np.int32)
    net = omni.net_create(layers, (1, 1, dims[0]), "f32", K_max, B_max)
    try:
        need = omni.net_workspace_bytes(net)
        assert need <= omni.STATIC_WORKSPACE_BYTES, need
        ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
        # two calls in a row, the second with a smaller input (fewer rows, fewer workers): the array keeps
        # the first call's contents, and nothing of it may leak into the second
        for off in ([0, 5, 40, 41, 96], [0, 7, 33]):
            print(f"case static step: off={off}", flush=True)
            (p0, l0, t0), (p1, l1, t1) = _both(omni, torch, net, ws, params, x, y, off, 0.05, K_max)
            assert np.array_equal(p0, p1) and np.array_equal(l0, l1) and t0 == t1
            ref = OS.sgd_step(layers, params, x[:off[-1]].reshape(off[-1], 1, 1, -1), y[:off[-1]], off, 0.05)
            assert_close(p1, ref.params, 1e-4, "theta' against the oracle")
            assert_close(l1, ref.loss_per_worker, 1e-4, "L_k against the oracle")
            assert not np.array_equal(p1, params)
    finally:
        omni.net_destroy(net)


def test_static_workspace_step_rejects_what_does_not_fit():
    import torch
    import paper_2503_17469_amd as omni
    w = synth.workload(1)          # 3072-1024-1024-10 at B = 480: tens of MB of gradient rows alone
    net = omni.net_create(w.layers, w.in_shape, "f32", w.K, w.B)
    try:
        assert omni.net_workspace_bytes(net) > omni.STATIC_WORKSPACE_BYTES
        params = torch.from_numpy(w.params).cuda()
        before = params.clone()
        x = torch.from_numpy(w.x.reshape(w.B, -1)).cuda()
        y = torch.from_numpy(w.labels).cuda()
        lpw, loss = torch.zeros(w.K, device="cuda"), torch.zeros(1, device="cuda")
        with pytest.raises(omni.OmniError) as e:
            omni.step_static(net, params, x, y, [0, 32, 96, 224, 480], [32, 64, 128, 256], 0.1, lpw, loss)
        assert e.value.code == -4 and "static" in str(e.value)
        torch.cuda.synchronize()
        assert torch.equal(params, before)
    finally:
        omni.net_destroy(net)


@pytest.mark.parametrize("K,B", [(16, 1024), (8, 2048)])
def test_static_workspace_step_of_a_small_network_with_many_rows(K, B):
    import gc
    import torch
    import paper_2503_17469_amd as omni
    dims = [200, 300, 100, 50]
    layers = synth.mlp(dims)
    rng = np.random.default_rng(B)
    params = synth.he_normal_params(layers, 6, False)
    x = rng.standard_normal((B, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], B).astype(np.int32)
    gc.collect()      # (tensors that an earlier test's exception holds must not be freed between the two readings below)
    net = omni.net_create(layers, (1, 1, dims[0]), "f32", K, B)
    try:
        ws = torch.zeros(omni.net_workspace_bytes(net), dtype=torch.uint8, device="cuda")
        off = [B * k // K for k in range(K + 1)]
        (p0, l0, t0), (p1, l1, t1) = _both(omni, torch, net, ws, params, x, y, off, 0.05, K)
        assert np.array_equal(p0, p1) and np.array_equal(l0, l1) and t0 == t1
        assert not np.array_equal(p1, params)
    finally:
        omni.net_destroy(net)
