"""Large fp32 products, which run on the bf16 matrix instruction with every operand in three pieces (128 x 128 tiles, slabs of 32
reduction elements, weight gradients in chunks of 512 rows of a worker): edges of tiles, slabs and chunks against float64, values
that are not finite, and rows that do not depend on other rows.

Bounds.  An output is the sum of n exact products in float32, whatever the order: pieces of 16 in a matrix instruction, six
times (at most 6 x 16 roundings), n / 32 slabs, the two shares, n / 512 chunks.  A rounding is at most u = 2^-24 of the sum of the
absolute products, and what the six of nine products leave out is at most u of each: element by element the error is within
(100 + n / 32 + n / 512) u of that sum.  A sum of one product is within 3 u of it: what is left out, what the instruction cuts off
where it adds the smaller products to the largest (u), and the rounding of that (u).  In the 2-norm the model of test_gpu_sum_errors holds: pieces of 32 (two slabs of a share)."""
import numpy as np
import pytest

import synth
from gpu_util import GpuRun
from test_gpu_isolation import _isolated
from test_gpu_sum_errors import U, _limit, _rel, _run

pytestmark = pytest.mark.gpu


def _check(got, a, b, n, mask=None, bias=None):
    """got = a b, zero where the mask is; with a bias max(a b + bias, 0) (which moves no further than its argument)"""
    want, size = a @ b, a.abs() @ b.abs()
    if bias is not None:
        want, size = (want + bias).clamp(min=0), size + bias.abs()
    if mask is not None:
        want, size = want * mask, size * mask
    worst = float(((got - want).abs() - (100 + n / 32 + n / 512) * U * size).max())
    assert worst <= 0, worst
    return _rel([(got, want)])


@pytest.mark.parametrize("rows,cin,cout", [
    (3329, 32, 1024),      # one slab; a row tile with one row
    (3300, 33, 1021),      # a second slab of one element, moved back; odd widths, rows off every alignment
    (3300, 63, 1021),
    (3300, 64, 1021),
    (3300, 97, 1021),      # a fourth slab
    (3328, 1024, 1024),
])
def test_forward(rows, cin, cout):
    L = _run([cin, cout, 10], [0, rows], "f32")[0]
    err = _check(L["z"], L["x"], L["w"].T, cin, bias=L["b"])
    assert err <= _limit(32, (cin + 63) // 64, 2)


@pytest.mark.parametrize("rows,cin,cout", [(3329, 1024, 32), (3300, 1021, 33), (3300, 1021, 70), (3300, 1021, 129)])
def test_input_gradients(rows, cin, cout):
    """of the layer cin -> cout: its tiles are over the cin columns"""
    L = _run([24, cin, cout, 10], [0, rows // 3, rows], "f32")[1]
    err = _check(L["dx"], L["dy"], L["w"], cout, (L["x"] > 0).double())
    assert err <= _limit(32, (cout + 63) // 64, 2)


@pytest.mark.parametrize("cin,cout,off", [
    (3400, 1021, [0, 1, 33, 34, 66, 400]),            # workers of one row, of a slab, of a slab and one
    (3400, 1021, [0, 4, 37, 70, 74, 700]),            # (the first of these is not split: workers of fewer than four rows)
    (3400, 1021, [0, 511, 1023, 1536]),               # chunks of 511, 512, and 512 + 1 rows
    (3328, 1024, [0, 1056, 1601]),                    # three chunks, two chunks
    (1021, 3400, [0, 250, 505]),
])
@pytest.mark.parametrize("momentum", [False, True])
def test_weight_gradients(cin, cout, off, momentum):
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.mlp([cin, cout, 10])
    B, K, lr, mu, wd = off[-1], len(off) - 1, 0.05, 0.9, 5e-4
    rng = np.random.default_rng(cin + B)
    params = synth.he_normal_params(layers, 7, False)
    x = rng.standard_normal((B, cin)).astype(np.float32)
    y = rng.integers(0, 10, B).astype(np.int32)
    run = GpuRun(layers, (1, 1, cin), "f32", K, B)
    try:
        vel0 = rng.standard_normal(run.P).astype(np.float32) * 0.01
        if momentum:
            velocity = torch.from_numpy(vel0.copy()).cuda()
            omni.net_set_momentum(run.net, velocity, mu, wd)
        got = run.step(params, x, y, off, lr, keep_g=False)
        dy = omni.net_activation_grad(run.net, run.ws, 0, B, "f32").double().cpu()
        vel = velocity.cpu().numpy() if momentum else None
    finally:
        run.close()
    xt = torch.from_numpy(x).double()
    (s, e), (bs, be) = synth.param_slices(layers)[0]["w"], synth.param_slices(layers)[0]["b"]
    pairs = []
    for k in range(K):
        rows = slice(off[k], off[k + 1])
        n = off[k + 1] - off[k]
        gw = torch.from_numpy(got["worker_grads"][k, s:e].reshape(cout, cin)).double()
        _check(gw, dy[rows].T, xt[rows], n)
        pairs.append((gw, dy[rows].T @ xt[rows]))
        gb = torch.from_numpy(got["worker_grads"][k, bs:be]).double()
        assert float(((gb - dy[rows].sum(0)).abs() - (n / 8 + 8) * U * dy[rows].abs().sum(0)).max()) <= 0
    longest = max(off[k + 1] - off[k] for k in range(K))
    assert _rel(pairs) <= _limit(16, (min(longest, 512) + 31) // 32, 2 + longest // 512)
    # the update from the gradients it wrote: sums of K terms, one rounding each, and a few more
    lam = np.diff(off) / B
    g = (got["worker_grads"].astype(np.float64) * lam[:, None]).sum(0)
    th = params.astype(np.float64)
    if momentum:
        v = mu * vel0 + (g + wd * th)
        assert np.abs(vel - v).max() <= (K + 6) * U * (np.abs(vel0) + np.abs(g) + np.abs(th)).max()
        g = v
    assert np.abs(got["params"] - (th - lr * g)).max() <= (K + 6) * U * (np.abs(th) + lr * np.abs(g)).max()


def _forward_with(x, w, dims):
    layers = synth.mlp(dims)
    B = len(x)
    params = synth.he_normal_params(layers, 4, False)
    s, e = synth.param_slices(layers)[0]["w"]
    params[s:e] = w.reshape(-1)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", 1, B)
    try:
        run.step(params, x, np.zeros(B, np.int32), [0, B], 0.0, keep_g=False)
        return run.activation(0, B)
    finally:
        run.close()


@pytest.mark.parametrize("at", [0, 17, 63, 64, 69])
def test_infinities_and_the_largest_values(at):
    """Column 5's weights are zero but for element `at`: infinite, then so large that its pieces are no numbers.  What
    is not near it keeps its bits."""
    dims, B = [70, 1024, 10], 3329
    rng = np.random.default_rng(at)
    x = (np.abs(rng.standard_normal((B, dims[0]))) + 0.5).astype(np.float32)
    w = (rng.standard_normal((dims[1], dims[0])) * 0.1).astype(np.float32)
    w[5] = 0
    w[5, at] = 1.0
    plain = _forward_with(x, w, dims)
    assert np.array_equal(plain[:, 5], x[:, at])
    w[5, at] = np.inf
    hidden = _forward_with(x, w, dims)
    assert np.all(np.isposinf(hidden[:, 5]))
    assert np.array_equal(np.delete(hidden, 5, axis=1), np.delete(plain, 5, axis=1))
    w[5, at] = np.finfo(np.float32).max
    x[:, at] = np.minimum(x[:, at], 1.0)
    hidden = _forward_with(x, w, dims)
    assert np.array_equal(hidden[:, 5], w[5, at] * x[:, at])


# Powers of two on the two operands: down to numbers of a few bits (the smallest fp32 number is 2^-149), and up to where the pieces
# are no numbers (2^104) or a product of the scaled pieces is none (2^80).
RANGES = [(-124, 20), (20, -124), (-112, -30), (110, -30), (-30, 110), (60, 60)]


@pytest.mark.parametrize("ex,ew", RANGES)
def test_forward_of_small_and_large_operands(ex, ew):
    import torch
    dims, B = [97, 1021, 10], 3300
    rng = np.random.default_rng(7)
    x = np.ldexp(rng.standard_normal((B, dims[0])), ex).astype(np.float32)
    w = np.ldexp(rng.standard_normal((dims[1], dims[0])), ew).astype(np.float32)
    z = torch.from_numpy(_forward_with(x, w, dims)).double()
    want = torch.from_numpy(x).double() @ torch.from_numpy(w).double().T
    size = torch.from_numpy(x).double().abs() @ torch.from_numpy(w).double().abs().T
    # (2^-149: the smallest number, for results that have fewer than 24 bits)
    assert float(((z - want.clamp(min=0)).abs() - 110 * U * size).max()) <= 2.0 ** -149


def _backward_with(dims, off, scale, ex):
    """One step with x times 2^ex and layer i's weights times 2^scale[i]: what the first layers stored, float64"""
    import torch
    import paper_2503_17469_amd as omni
    layers = synth.mlp(dims)
    B, K = off[-1], len(off) - 1
    rng = np.random.default_rng(sum(dims) + B)
    params = synth.he_normal_params(layers, 7, False)
    linear = [i for i, L in enumerate(layers) if L["op"] == "linear"]
    for i, e in zip(linear, scale):
        s, t = synth.param_slices(layers)[i]["w"]
        params[s:t] = np.ldexp(params[s:t].astype(np.float64), e)
    x = np.ldexp(rng.standard_normal((B, dims[0])), ex).astype(np.float32)
    y = rng.integers(0, dims[-1], B).astype(np.int32)
    run = GpuRun(layers, (1, 1, dims[0]), "f32", K, B)
    try:
        got = run.step(params, x, y, off, 0.0, keep_g=False)
        dy = [omni.net_activation_grad(run.net, run.ws, i, B, "f32").double().cpu() for i in linear[:-1]]
        hidden = torch.from_numpy(np.ascontiguousarray(run.activation(0, B))).double()
    finally:
        run.close()
    w = []
    for i, (o, n) in zip(linear, zip(dims[1:], dims)):
        s, t = synth.param_slices(layers)[i]["w"]
        w.append((torch.from_numpy(params[s:t].reshape(o, n)).double(),
                  [torch.from_numpy(got["worker_grads"][k, s:t].reshape(o, n)).double() for k in range(K)]))
    return torch.from_numpy(x).double(), hidden, dy, w


@pytest.mark.parametrize("ea,eb", RANGES)
def test_input_gradients_of_small_and_large_operands(ea, eb):
    """output gradients (through the classifier's weights) times 2^ea, weights times 2^eb"""
    _, hidden, dy, w = _backward_with([24, 1021, 129, 10], [0, 1100, 3300], [min(0, -ea - eb), eb, ea], 0)
    a, b = dy[1], w[1][0]
    assert float(a.abs().max()) > 0
    mask = (hidden > 0).double()
    over = (dy[0] - (a @ b) * mask).abs() - 110 * U * (a.abs() @ b.abs()) * mask
    assert float(over.max()) <= 2.0 ** -149


@pytest.mark.parametrize("ea,eb", RANGES)
def test_weight_gradients_of_small_and_large_operands(ea, eb):
    """output gradients (through the classifier's weights) times 2^ea, inputs times 2^eb"""
    off = [0, 300, 1100]
    x, _, dy, w = _backward_with([3400, 1021, 10], off, [min(0, -ea - eb), ea], eb)
    assert float(dy[0].abs().max()) > 0
    for k in range(2):
        a, b = dy[0][off[k]:off[k + 1]].T, x[off[k]:off[k + 1]]
        over = (w[0][1][k] - a @ b).abs() - 130 * U * (a.abs() @ b.abs())
        assert float(over.max()) <= 2 * 2.0 ** -149      # two chunks of two shares, each rounded to a multiple of 2^-149


def test_sums_of_one_product():
    """One element of every row of x is not zero: 3 u (see above; the smaller products' own errors are below 2^-6 of that), where one
    rounding would be 1 u; root mean square 0.58 u, one rounding's 0.43."""
    dims, B = [97, 1021, 10], 3300
    rng = np.random.default_rng(8)
    x = np.zeros((B, dims[0]), np.float32)
    at = np.arange(B) % dims[0]
    x[np.arange(B), at] = rng.standard_normal(B)
    w = rng.standard_normal((dims[1], dims[0])).astype(np.float32)
    want = x[np.arange(B), at].astype(np.float64)[:, None] * w.T[at].astype(np.float64)
    err = (_forward_with(x, w, dims) / np.where(want > 0, want, 1) - 1)[want > 0]
    assert np.abs(err).max() <= 3 * U * (1 + 2.0 ** -6)
    assert (err ** 2).mean() ** 0.5 <= 0.62 * U


def test_errors_have_no_direction():
    """The matrix instruction rounds down; with the halves of a slab summed in opposite signs the errors of many outputs have no
    mean.  In units of 2^-24 of the sum of the absolute products: -0.03 to -0.09 with one sign, at most 0.001 with both."""
    def mean(got, want, size, where):
        return abs(float(((got - want) / size)[where].mean())) / U

    L = _run([1024, 1021, 10], [0, 3300], "f32")[0]
    z = L["x"] @ L["w"].T
    assert mean(L["z"], z, L["x"].abs() @ L["w"].abs().T, z > 0) <= 0.01
    L = _run([24, 1021, 1024, 10], [0, 1100, 3300], "f32")[1]
    assert mean(L["dx"], L["dy"] @ L["w"], L["dy"].abs() @ L["w"].abs(), L["x"] > 0) <= 0.01
    x, _, dy, w = _backward_with([3400, 1021, 10], [0, 2000], [0, 0], 0)
    size = dy[0].abs().T @ x.abs()
    assert mean(w[0][1][0], dy[0].T @ x, size, size > 0) <= 0.01


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("dims,off,bad", [
    ([40, 1024, 10], [0, 1000, 1003, 3329], 1),            # forward: tiles with rows of three workers
    ([24, 1021, 40, 10], [0, 1000, 1003, 3300], 1),        # and input gradient
    ([3400, 1021, 10], [0, 200, 203, 500], 1),             # weight gradient
    ([3400, 1021, 10], [0, 600, 620, 700], 0),
    ([3400, 1021, 10], [0, 300, 304, 500], 1),
])
def test_workers_do_not_depend_on_each_other(dims, off, bad, value):
    _isolated(synth.mlp(dims), (1, 1, dims[0]), "f32", off, bad, value, sum(dims))


@pytest.mark.parametrize("momentum", [False, True])
@pytest.mark.parametrize("off", [[0, 300, 1100], [0, 600, 1300, 1400]])      # (workers of two chunks, of one)
def test_update_of_sums_formed_again(off, momentum):
    """Some columns of x are 2^110 in some workers' rows (their weights are zero, so that nothing else notices): the pieces of these are
    no numbers, the sums of the whole tile's such columns are formed again on the fp32 instruction, and the update takes them.
    Columns inside a tile, in the last one and in the same 16 bytes as others; rows of the last tile's 125.  Gradients against
    float64, the other columns' as without them, parameters and velocity bit for bit the weighted sum of what was stored."""
    import torch
    import paper_2503_17469_amd as omni
    dims, bad = [3400, 1021, 10], [0, 5, 6, 127, 128, 1030, 3398]
    layers = synth.mlp(dims)
    K, B = len(off) - 1, off[-1]
    b = [off[k + 1] - off[k] for k in range(K)]
    rng = np.random.default_rng(B)
    params = synth.he_normal_params(layers, 7, False)
    s, t = synth.param_slices(layers)[0]["w"]
    params[s:t].reshape(dims[1], dims[0])[:, bad] = 0
    x = rng.standard_normal((B, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], B).astype(np.int32)
    large = x.copy()
    large[off[1] - 7:, bad] *= np.float32(2.0 ** 110)          # (the last rows of the first worker, and the other workers)
    out = []
    for xs in (x, large):
        run = GpuRun(layers, (1, 1, dims[0]), "f32", K, B)
        try:
            p = torch.from_numpy(params).cuda()
            v = torch.randn(p.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) * 0.01
            p0, v0 = p.clone(), v.clone()
            if momentum:
                omni.net_set_momentum(run.net, v, 0.9, 5e-4)
            omni.step(run.net, p, torch.from_numpy(xs).cuda(), torch.from_numpy(y).cuda(), off, b, 0.05, run.ws, run.lpw, run.loss)
            G = omni.net_worker_grads(run.net, run.ws, K)
            full = torch.zeros(K, (params.size + 63) // 64 * 64, device="cuda")
            full[:, :params.size] = G[:, :params.size]
            if momentum:
                omni.weighted_sgd_momentum(p0, v0, full, b, 0.05, 0.9, 5e-4, None)
            else:
                omni.weighted_sgd(p0, full, b, 0.05, None)
            torch.cuda.synchronize()
            assert torch.isfinite(p).all()
            assert torch.equal(p, p0) and torch.equal(v, v0)
            out.append((full.cpu().double().numpy(), omni.net_activation_grad(run.net, run.ws, 0, B, "f32").double().cpu().numpy()))
        finally:
            run.close()
    (clean, dy), (got, dy2) = out
    assert np.array_equal(dy, dy2)
    clean, got = (g[:, s:t].reshape(K, dims[1], dims[0]) for g in (clean, got))
    rest = np.setdiff1d(np.arange(dims[0]), bad)
    assert np.array_equal(got[:, :, rest], clean[:, :, rest])
    for k in range(K):
        a, c = dy[off[k]:off[k + 1]].reshape(b[k], -1).T, large[off[k]:off[k + 1]][:, bad].astype(np.float64)
        assert np.abs(a @ c).max() > 2.0 ** 90
        # (one chain of fp32 products, two at a time)
        assert (np.abs(got[k][:, bad] - a @ c) <= b[k] * U * (np.abs(a) @ np.abs(c))).all()
