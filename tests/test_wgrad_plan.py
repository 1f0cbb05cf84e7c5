"""Which launches the weight gradients of one call become, checked on the host: the library's planning is compiled
against its internal header and asked, nothing is launched."""
import ctypes
import os
import subprocess

import pytest

from paper_2503_17469_amd import binding

CSRC = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")

SHIM = r"""
#include "kernels.h"
using namespace omni;
// layers: n x (hw, cin, cout, stride); out: n x (first_layer, launch, workgroups, reduced, scratch_begin, scratch_end)
extern "C" size_t describe(const int* layers, int n, const int* off, int K, int workgroups, long* out) {
  ConvWgradJob jobs[32] = {};
  for (int i = 0; i < n; ++i) {
    const int hw = layers[4 * i], cin = layers[4 * i + 1], cout = layers[4 * i + 2], s = layers[4 * i + 3];
    ConvGeom g{};
    g.rows = off[K]; g.Hs = g.Ws = hw; g.Cs = (cin + 7) / 8 * 8; g.Hp = g.Wp = hw / s;
    g.ks = 3; g.stride = s; g.pad = 1; g.K = 9 * g.Cs;
    jobs[i].Cout = cout; jobs[i].cin_real = cin; jobs[i].g = g;
  }
  Segments seg{};
  seg.K = K;
  for (int k = 0; k <= K; ++k) seg.off[k] = off[k];
  ConvWgradPlanned p[32];
  conv_wgrad_describe(jobs, n, seg, workgroups, p);
  for (int i = 0; i < n; ++i) {
    const long v[6] = {p[i].first_layer, p[i].launch, p[i].workgroups, p[i].reduced, (long)p[i].scratch_begin,
                       (long)p[i].scratch_end};
    for (int e = 0; e < 6; ++e) out[6 * i + e] = v[e];
  }
  return conv_wgrad_partial_floats();
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    lib_dir = os.path.dirname(binding.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    str(d / "shim.cpp"), "-o", str(d / "shim.so"), "-L" + lib_dir, "-l:libomnistep.so",
                    "-Wl,-rpath," + lib_dir, "-Wl,--allow-shlib-undefined"], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.describe.restype = ctypes.c_size_t
    return lib


FIRST3, FIRST4, MID, S2 = (32, 3, 32, 1), (32, 4, 64, 1), (16, 32, 64, 1), (32, 64, 128, 2)


@pytest.mark.parametrize("layers", [
    [FIRST3], [FIRST3, FIRST3], [FIRST3, FIRST4, MID], [MID, FIRST4, S2, FIRST3], [FIRST3] * 6, [FIRST3] * 8,
    [MID, MID, MID, MID, MID, FIRST3, FIRST3], [MID, S2], [S2],
])
@pytest.mark.parametrize("off", [[0, 1], [0, 5, 6, 37], [0, 256, 512, 768, 1024], [0, 300, 2048]])
@pytest.mark.parametrize("workgroups", [256, 512])
def test_every_layer_is_in_one_launch_that_knows_its_kind(shim, layers, off, workgroups):
    n = len(layers)
    flat = (ctypes.c_int * (4 * n))(*[v for L in layers for v in L])
    offs = (ctypes.c_int * len(off))(*off)
    out = (ctypes.c_long * (6 * n))()
    room = shim.describe(flat, n, offs, len(off) - 1, workgroups, out)
    rows = [tuple(out[6 * i:6 * i + 6]) for i in range(n)]
    for (first, launch, blocks, reduced, lo, hi), L in zip(rows, layers):
        assert first == (L in (FIRST3, FIRST4))
        assert launch >= 0, "in no launch, in two, or in one whose kernel does not know it"
        assert len(off) - 1 <= blocks < 1 << 20      # at least a workgroup per worker
        assert 0 <= lo <= hi <= room
    # layers on the network input share a first stage with nobody
    for i in range(n):
        others = [j for j in range(n) if j != i and rows[j][1] == rows[i][1]]
        assert not (rows[i][0] and others)
        assert all(not rows[j][0] for j in others)
    # layers of one call of six (whose second stage is one launch) keep their partial tiles apart
    for base in range(0, n, 6):
        spans = sorted(r[4:6] for r in rows[base:base + 6] if r[3])
        assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))


@pytest.mark.parametrize("layers,at_least", [
    ([(8, 256, 256, 1), (16, 128, 256, 2)], 384),
    ([(16, 128, 128, 1), (32, 64, 128, 2)], 416),
    ([(4, 512, 512, 1), (8, 256, 512, 2)], 512),
    ([(16, 32, 64, 1), (32, 64, 128, 2)], 128),
])
def test_chains_of_stride_1_layers_beside_others(shim, layers, at_least):
    """1024 images of eight workers in 768 workgroups: the sums of a 3x3 / stride-1 layer beside a stride-2 one run through chains no
    longer than the workgroups that kernel C had would make them (fewer workgroups are longer chains, and larger errors)."""
    flat = (ctypes.c_int * 8)(*[v for L in layers for v in L])
    offs = (ctypes.c_int * 9)(*range(0, 1025, 128))
    out = (ctypes.c_long * 12)()
    shim.describe(flat, 2, offs, 8, 768, out)
    assert out[1] == out[7] and out[2] >= at_least


@pytest.mark.parametrize("workers", [1, 4])
def test_chunks_of_few_images(shim, workers):
    """Twenty images beside a stride-2 layer: chunks of at least four units of 128 positions (smaller ones made second stages twice as
    long as they were)."""
    layers = [(8, 256, 256, 1), (16, 128, 256, 2)]
    flat = (ctypes.c_int * 8)(*[v for L in layers for v in L])
    offs = (ctypes.c_int * (workers + 1))(*[20 * k // workers for k in range(workers + 1)])
    out = (ctypes.c_long * 12)()
    shim.describe(flat, 2, offs, workers, 768, out)
    units = [(offs[k + 1] - offs[k]) * 64 / 128 for k in range(workers)]
    assert out[2] == 16 * sum(-(-u // 4) for u in units)
