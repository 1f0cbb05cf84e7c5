"""Host threads that step networks of their own on streams of their own at the same time (the library releases the interpreter
lock): the same results as one after the other."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_threads_with_networks_of_different_shapes():
    import torch
    import paper_2503_17469_amd as omni
    specs = [
        (synth.cnn3(num_classes=10, hw=32, chans=(3, 32, 64, 128)), (32, 32, 3), "bf16", [0, 5, 40]),
        (synth.cnn3(num_classes=10, hw=16, chans=(3, 64, 96, 64)), (16, 16, 3), "bf16", [0, 33, 70]),
        (synth.resnet18(num_classes=10, cin=3), (32, 32, 3), "bf16", [0, 4, 20]),
        (synth.resnet18(num_classes=10, cin=3), (32, 32, 3), "bf16", [0, 50, 160]),
        (synth.mlp([784, 256, 10]), (1, 1, 784), "f32", [0, 8, 32]),
    ]
    steps, state = 4, []
    for i, (layers, shape, dtype, off) in enumerate(specs):
        params = synth.he_normal_params(layers, 40 + i, dtype == "bf16")
        x, y = synth.make_batch(60 + i, off[-1], shape, 10, dtype == "bf16")
        x = torch.from_numpy(np.ascontiguousarray(x)).cuda()
        state.append(dict(net=omni.net_create(layers, shape, dtype, 2, off[-1]), off=off, start=torch.from_numpy(params).cuda(),
                          x=x.to(torch.bfloat16) if dtype == "bf16" else x, y=torch.from_numpy(y).cuda(),
                          b=[off[1], off[2] - off[1]], lpw=torch.zeros(2, device="cuda"), loss=torch.zeros(1, device="cuda"),
                          out=None, failed=None))
        state[-1]["ws"] = torch.zeros(omni.net_workspace_bytes(state[-1]["net"]), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()

    def train(s):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                p = s["start"].clone()
                for _ in range(steps):
                    omni.step(s["net"], p, s["x"], s["y"], s["off"], s["b"], 0.01, s["ws"], s["lpw"], s["loss"])
                torch.cuda.current_stream().synchronize()
            s["out"] = p.cpu().numpy()
        except Exception as e:      # (re-raised below, in the test's own thread)
            s["failed"] = e

    try:
        threads = [threading.Thread(target=train, args=(s,)) for s in state]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        together = []
        for s in state:
            if s["failed"]:
                raise s["failed"]
            together.append(s["out"])
        for s, got in zip(state, together):
            train(s)
            assert s["failed"] is None and np.array_equal(s["out"], got)
            assert not np.array_equal(got, s["start"].cpu().numpy())
    finally:
        for s in state:
            omni.net_destroy(s["net"])
