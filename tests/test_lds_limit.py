"""The dynamic-LDS limit of a kernel under several host threads, against stand-ins for the two runtime calls (no GPU)."""
import os
import subprocess

from paper_2503_17469_amd import binding

CSRC = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "lds_limit.h"

static thread_local int t_device = 0;
static std::atomic<int> limit[2], calls[2];
extern "C" hipError_t hipGetDevice(int* d) { *d = t_device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
  std::this_thread::yield();
  limit[t_device] = bytes;
  ++calls[t_device];
  return hipSuccess;
}

int main() {
  static omni::LdsLimit one;
  std::atomic<int> low{0};
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      t_device = t & 1;
      for (int i = 0; i < 2000; ++i) {
        one.raise(nullptr, omni::kLdsOfComputeUnit);
        if (limit[t_device] != (int)omni::kLdsOfComputeUnit) ++low;   // a launch here would be refused
      }
    });
  for (auto& t : threads) t.join();
  std::printf("%d %d %d\n", low.load(), calls[0].load(), calls[1].load());
}
"""


def test_limit_is_raised_before_every_launch_and_never_lowered(tmp_path):
    (tmp_path / "p.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "p")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    str(tmp_path / "p.cpp"), "-o", exe], check=True)
    for _ in range(20):
        low, c0, c1 = map(int, subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split())
        assert low == 0
        assert 1 <= c0 <= 4 and 1 <= c1 <= 4          # once per device, or once per thread that came first


def test_every_kernel_raises_its_limit_through_it():
    for f in sorted(os.listdir(CSRC)):
        if f != "lds_limit.h":
            assert "hipFuncSetAttribute" not in open(os.path.join(CSRC, f)).read(), f
