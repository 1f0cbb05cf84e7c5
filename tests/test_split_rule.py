"""Which weight gradients of fp32 networks go to the bf16 matrix instruction, asked on the host; nothing is launched."""
import ctypes
import os
import subprocess

import pytest

from paper_2503_17469_amd import binding

CSRC = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")

SHIM = r"""
#include "kernels.h"
extern "C" int split(int cin, int cout, const int* off, int K) {
  omni::LinearWgradJob job{};
  job.cin = cin;
  job.cout = cout;
  omni::Segments seg{};
  seg.K = K;
  for (int k = 0; k <= K; ++k) seg.off[k] = off[k];
  return omni::linear_wgrad_f32_split_shape(&job, 1, seg);
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    lib_dir = os.path.dirname(binding.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    str(d / "shim.cpp"), "-o", str(d / "shim.so"), "-L" + lib_dir, "-l:libomnistep.so",
                    "-Wl,-rpath," + lib_dir, "-Wl,--allow-shlib-undefined"], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    return lambda cin, cout, b: bool(lib.split(cin, cout, (ctypes.c_int * (len(b) + 1))(*[sum(b[:k]) for k in range(len(b) + 1)]),
                                               len(b)))


@pytest.mark.parametrize("b,yes", [
    ([399], False), ([400], True), ([4096], True), ([100] * 4, True), ([99, 100, 100, 100], False),
    ([96] * 8, False), ([100] * 8, True), ([64] * 16, False), ([128] * 16, True),
    ([12] * 32, False), ([32] * 32, False), ([128] * 32, True), ([64] * 64, False),      # many workers: rows in all do not count
    ([400, 4], True), ([400, 3], False), ([1, 4000], False),                             # no sums of fewer than four products
])
def test_rows_per_worker(split, b, yes):
    assert split(3400, 1021, b) == yes


@pytest.mark.parametrize("cin,cout,yes", [(2048, 2048, True), (2048, 2049, False), (1638, 2048, False), (1639, 2048, True), (64, 64, False)])
def test_tiles_fill_rounds_of_the_chip(split, cin, cout, yes):
    assert split(cin, cout, [1000]) == yes
