"""The work that a program using this library has it do, as cases that can be timed.

A case is a dict of plain values; `prepare` makes what such a program holds before the call, `run` is one
pass through the public entry points as the program calls them (for a training step: controller with the
workers' current throughputs, then the step), `work` is what a pass cannot do without and `tolerance` how
far two correct implementations may be apart.

Kinds:
  mlp, cnn, resnet   one synchronous training step (controller, forward, loss, backward with one gradient
                     per worker, weighted aggregation, SGD or momentum update)
  asp                one round of the asynchronous variant: every worker pushes once and computes its next
                     gradient (forward and backward without an update, one worker's rows at a time)
  update             weighted aggregation and update alone, for a program with a backward pass of its own

Shapes: the five benchmark configurations, the batch of 4 x 32 samples of the paper's experiments, and
generic sizes between them.  Inputs and weights follow the repository's recipe (inputs N(0,1), uniform
labels, He-normal weights, integer throughputs within an 8x spread) but are drawn on the GPU.
"""
import math
import random

import torch

import paper_2503_17469_amd as omni
from synth import nets

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # The smallest step there is: a few hundred kiloflop, so launches and host work are all of it.
        dict(name="mlp tiny", kind="mlp", dtype="f32", inputs=64, hidden="128", classes=10, K=2, B=32, momentum=False),
        # Fully connected net on flattened 3x32x32 images, four workers whose speeds differ by 8x.
        dict(name="mlp 3072", kind="mlp", dtype="f32", inputs=3072, hidden="1024,1024", classes=10, K=4, B=480,
             momentum=False),
        # Widths and batch that fit no tile, with the optimiser of the paper's experiments.
        dict(name="mlp odd momentum", kind="mlp", dtype="f32", inputs=997, hidden="501,243", classes=37, K=7, B=333,
             momentum=True),
        # The same net as "mlp 3072" fed by sixteen workers with large batches: throughput, not latency.
        dict(name="mlp 3072 large batch", kind="mlp", dtype="f32", inputs=3072, hidden="1024,1024", classes=10, K=16,
             B=4096, momentum=False),
        # The same net with bf16 operands and momentum.
        dict(name="mlp 3072 bf16", kind="mlp", dtype="bf16", inputs=3072, hidden="1024,1024", classes=10, K=8, B=1024,
             momentum=True),
        # Asynchronous training of "mlp 3072": forward and backward of one worker's rows, then the push.
        dict(name="asp mlp 3072", kind="asp", dtype="f32", inputs=3072, hidden="1024,1024", classes=10, K=4, B=480),
        # Small convolutional net at the paper's batch of 4 x 32 images.
        dict(name="cnn small batch", kind="cnn", hw=32, channels="32,64,128", classes=10, K=4, B=128, dynamic=False),
        # The same net at the benchmark's batch.
        dict(name="cnn", kind="cnn", hw=32, channels="32,64,128", classes=10, K=8, B=1024, dynamic=False),
        # The workers' speeds drift and the controller re-sizes every batch on every step.
        dict(name="cnn dynamic", kind="cnn", hw=32, channels="32,64,128", classes=10, K=16, B=2048, dynamic=True),
        # ResNet-18-shaped net at the paper's batch of 4 x 32 images ...
        dict(name="resnet18 small batch", kind="resnet", classes=100, K=4, B=128),
        # ... and the largest configuration.
        dict(name="resnet18", kind="resnet", classes=100, K=8, B=2048),
        # Eight workers' gradients of an 11 M parameter model combined and applied.
        dict(name="update momentum 11M", kind="update", P=11220132, K=8, momentum=True, shadow=False),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above: widths, batches and worker counts over their whole range."""
    kind = rng.choices(("mlp", "mlp bf16", "asp", "cnn", "resnet", "update"), (30, 10, 10, 25, 15, 10))[0]
    if kind in ("mlp", "mlp bf16", "asp"):
        bf = kind == "mlp bf16"
        width = lambda lo, hi: (_log(rng, lo, hi) + 7) // 8 * 8 if bf else _log(rng, lo, hi)
        c = dict(kind="asp" if kind == "asp" else "mlp", dtype="bf16" if bf else "f32", inputs=width(32, 3072),
                 hidden=",".join(str(width(32, 1024)) for _ in range(rng.randint(1, 3))), classes=_log(rng, 2, 100))
        if kind == "asp":
            c["K"] = rng.randint(2, 8)
            c["B"] = _log(rng, 64, 2048)
        else:
            c["K"] = _log(rng, 1, 32)
            c["B"] = _log(rng, max(16, 2 * c["K"]), 4096)
            c["momentum"] = bf or rng.random() < 0.5
        return c
    if kind == "cnn":
        K = _log(rng, 1, 16)
        ch = (rng.choice((16, 32, 64)), rng.choice((32, 64, 96, 128)), rng.choice((64, 128, 256)))
        return dict(kind="cnn", hw=rng.choice((16, 32)), channels=",".join(map(str, ch)), classes=_log(rng, 2, 100), K=K,
                    B=_log(rng, max(16, 2 * K), 2048), dynamic=rng.random() < 0.5)
    if kind == "resnet":
        K = _log(rng, 1, 16)
        return dict(kind="resnet", classes=_log(rng, 10, 100), K=K, B=_log(rng, 32, 2048))
    K = _log(rng, 1, 64)
    return dict(kind="update", P=_log(rng, 10_000, min(12_000_000, 100_000_000 // K)), K=K,
                momentum=rng.random() < 0.5, shadow=rng.random() < 0.5)


# ------------------------------------------------------------------ state


def _net_of(case):
    """(layers, input shape, dtype)"""
    kind = case["kind"]
    if kind in ("mlp", "asp"):
        dims = [case["inputs"]] + [int(v) for v in case["hidden"].split(",")] + [case["classes"]]
        return nets.mlp(dims), (1, 1, case["inputs"]), case["dtype"]
    if kind == "cnn":
        ch = tuple(int(v) for v in case["channels"].split(","))
        return nets.cnn3(case["classes"], case["hw"], (3,) + ch), (case["hw"], case["hw"], 3), "bf16"
    return nets.resnet18(case["classes"]), (32, 32, 3), "bf16"


class _Net:
    """Owns a network (and controller) handle for as long as the state lives."""

    def __init__(self, layers, in_shape, dtype, K, B):
        self.ctl = omni.ctl_create(K, B)
        self.net = omni.net_create(layers, in_shape, dtype, K, B)

    def __del__(self):
        omni.net_destroy(self.net)
        omni.ctl_destroy(self.ctl)


def _throughputs(rng, K):
    """Integer throughputs in milli-units, the fastest worker 8x the slowest."""
    T = [rng.randint(1000, 8000) for _ in range(K)]
    if K > 1:
        T[T.index(min(T))] = 1000
        T[T.index(max(T))] = 8000
    return T


def _walk(rng, T, steps):
    """Throughputs that drift within their 8x range, one list per step."""
    out = [T]
    for _ in range(steps - 1):
        out.append([min(8000, max(1000, t + rng.randint(-250, 250))) for t in out[-1]])
    return out


def _he_params(layers, gen):
    """He-normal weights, zero biases, beta 0, gamma 1; the gamma that ends a residual branch (the batch norm
    read by an add, on the branch of the two 3x3 convolutions) starts small, as is usual for such nets in
    earnest: every block then starts near the identity, and gradients are better conditioned."""
    params = torch.zeros(nets.param_count(layers), device="cuda")
    adds = {L["src"] for L in layers if L["op"] == "add"}
    for i, (L, sl) in enumerate(zip(layers, nets.param_slices(layers))):
        if L["op"] == "bn":
            s, e = sl["gamma"]
            params[s:e] = 0.1 if i in adds else 1.0
        elif L["op"] in ("linear", "conv"):
            s, e = sl["w"]
            fan_in = L["cin"] * L.get("k", 1) ** 2
            params[s:e] = torch.randn(e - s, device="cuda", generator=gen) * math.sqrt(2.0 / fan_in)
    return params


def prepare(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    K, kind = case["K"], case["kind"]
    s = dict(kind=kind, K=K)
    if kind == "update":
        P = case["P"]
        stride = (P + 63) // 64 * 64
        s["grads"] = torch.randn(K, stride, device="cuda", generator=gen) * 0.01
        s["params"] = torch.randn(P, device="cuda", generator=gen) * 0.03
        s["velocity"] = torch.randn(P, device="cuda", generator=gen) * 0.02 if case["momentum"] else None
        s["shadow"] = torch.empty(P, dtype=torch.bfloat16, device="cuda") if case["shadow"] else None
        s["b"] = [rng.randint(8, 64) for _ in range(K)]
        return s

    layers, in_shape, dtype = _net_of(case)
    B = case["B"]
    s["B"] = B
    s["owner"] = h = _Net(layers, in_shape, dtype, K, B)
    s["ctl"], s["net"] = h.ctl, h.net
    T = [1000 << i for i in range(4)] if K == 4 else _throughputs(rng, K)
    s["T"] = _walk(rng, T, 200) if case.get("dynamic") else [T]
    s["at"] = 0
    s["params"] = _he_params(layers, gen)
    x = torch.randn((B,) + tuple(in_shape), device="cuda", generator=gen)
    s["x"] = x.to(torch.bfloat16) if dtype == "bf16" else x
    s["labels"] = torch.randint(0, case["classes"], (B,), device="cuda", generator=gen, dtype=torch.int32)
    s["loss_per_worker"] = torch.zeros(K, device="cuda")
    s["loss"] = torch.zeros(1, device="cuda")
    nbytes = omni.net_workspace_bytes(s["net"])
    if kind == "asp":
        # every simulated worker keeps its gradient in a workspace of its own until it pushes
        omni.ctl_set_throughputs(s["ctl"], T)
        s["b"], off = omni.ctl_run(s["ctl"], K)
        s["lr"] = 0.01
        s["ws"] = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for _ in range(K)]
        s["rows"] = [(s["x"][off[k]:off[k + 1]], s["labels"][off[k]:off[k + 1]]) for k in range(K)]
        if dtype == "f32" and (case["inputs"] * 4) % 16:   # the step wants x 16-byte aligned: slices of odd rows are copies
            s["rows"] = [(xk.clone(), yk) for xk, yk in s["rows"]]
        s["g"] = [omni.net_worker_grads(s["net"], ws, 1)[0] for ws in s["ws"]]
        s["losses"] = [torch.zeros(1, device="cuda") for _ in range(K)]
        s["order"] = omni.asp_schedule(T, s["b"], K)[0]
        for k in range(K):
            _asp_gradient(s, k)
        return s
    s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    # Batch norm makes a large rate safe.  The others see thousands of steps on one random batch.
    s["lr"] = dict(resnet=0.1, cnn=0.0002).get(kind, 0.003 if case.get("momentum") else 0.01)
    s["velocity"] = None
    if case.get("momentum"):
        s["velocity"] = torch.zeros_like(s["params"])
        omni.net_set_momentum(s["net"], s["velocity"], 0.9, 5e-4)
    s["g"] = omni.net_worker_grads(s["net"], s["ws"], K) if kind == "cnn" else None
    return s


# ------------------------------------------------------------------ one pass


def _asp_gradient(s, k):
    """Worker k's forward and backward pass on its own rows at the current server model."""
    x, y = s["rows"][k]
    omni.step(s["net"], s["params"], x, y, [0, s["b"][k]], [s["b"][k]], 0.0, s["ws"][k], s["losses"][k], s["loss"],
              omni.STEP_NO_UPDATE)


def run(s):
    kind = s["kind"]
    if kind == "update":
        if s["velocity"] is not None:
            omni.weighted_sgd_momentum(s["params"], s["velocity"], s["grads"], s["b"], 0.01, 0.9, 5e-4, s["shadow"])
        else:
            omni.weighted_sgd(s["params"], s["grads"], s["b"], 0.01, s["shadow"])
        return dict(params=s["params"], velocity=s["velocity"], shadow=s["shadow"])
    if kind == "asp":
        for k in s["order"]:
            omni.asp_update(s["params"], s["params"], s["g"][k], s["lr"], s["b"][k], s["B"], True)
            _asp_gradient(s, k)
        return dict(params=s["params"], losses=s["losses"])
    omni.ctl_set_throughputs(s["ctl"], s["T"][s["at"]])
    s["at"] = (s["at"] + 1) % len(s["T"])
    b, off = omni.ctl_run(s["ctl"], s["K"])
    omni.step(s["net"], s["params"], s["x"], s["labels"], off, b, s["lr"], s["ws"], s["loss_per_worker"], s["loss"])
    return dict(params=s["params"], velocity=s["velocity"], worker_grads=s["g"], loss_per_worker=s["loss_per_worker"],
                loss=s["loss"])


# ------------------------------------------------------------------ what a pass costs and how exact it is


def _net_work(layers, in_shape, dtype, rows, K, momentum, update):
    """Contraction flop of forward, input gradients (none for a layer on the network input) and weight
    gradients; bytes: inputs, labels, parameters (and velocity) in and out, the K gradient rows out."""
    shapes = nets.layer_shapes(layers, in_shape)
    flops = 0.0
    for i, L in enumerate(layers):
        if L["op"] in ("linear", "conv"):
            h, w, c = shapes[i]
            one = 2.0 * rows * h * w * c * L["cin"] * L.get("k", 1) ** 2
            flops += one * (3 if L["src"] >= 0 else 2)
    P = nets.param_count(layers)
    x_bytes = rows * math.prod(in_shape) * (2 if dtype == "bf16" else 4) + rows * 4
    return x_bytes + 4.0 * P * ((4 if momentum else 2 if update else 1) + K), flops


def work(case):
    K = case["K"]
    if case["kind"] == "update":
        P = case["P"]
        return {"bytes": 4.0 * P * (K + (4 if case["momentum"] else 2)) + (2.0 * P if case["shadow"] else 0.0),
                "flops": 2.0 * P * (K + 2)}
    layers, in_shape, dtype = _net_of(case)
    if case["kind"] == "asp":
        # per push: model and gradient read, model written; per gradient: one worker's rows, the model read, the
        # gradient written
        nbytes, flops = _net_work(layers, in_shape, dtype, case["B"], K, False, False)
        P = nets.param_count(layers)
        return {"bytes": nbytes - 4.0 * P + K * 4.0 * P * 4, "flops": flops + 2.0 * K * P}
    nbytes, flops = _net_work(layers, in_shape, dtype, case["B"], K, case.get("momentum", False), True)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Largest relative error of parameters, losses, velocity and (convolutional net) per-worker gradients."""
    kind = case["kind"]
    if kind == "update":
        # fp32 sums of at most 64 terms; the bf16 copy may round a value to the other neighbour
        return {"rel": 2e-3, "max": 1e-2} if case["shadow"] else {"rel": 1e-6, "max": 1e-5}
    if kind == "resnet":
        # Gradients through seventeen ReLU / batch-norm layers are ill-conditioned in bf16 (2 to 5 per cent of the
        # whole when one stored value in ten thousand moves by its last bit; single entries by far more), so they
        # are compared through the update they make, which is 5e-4 to 1e-3 of the parameters in one pass.
        return {"rel": 5e-4, "max": 5e-2}
    if kind == "cnn" or case["dtype"] == "bf16":
        # bf16 operands and stored activations; a pooling or ReLU decision taken the other way re-routes one
        # term of a gradient entry's sum (per-worker gradients and the velocity are among the outputs)
        return {"rel": 2e-2, "max": 0.9}
    if case.get("momentum"):
        # fp32; one ReLU argument within rounding of zero moves a gradient row (the velocity) by one row's share
        return {"rel": 2e-3, "max": 0.5}
    return {"rel": 1e-5, "max": 1e-3}
