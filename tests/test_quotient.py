"""Quotients by a high multiplication, on the host: exact for every number below the stated bound, a division where they would not be."""
import os
import subprocess

from paper_2503_17469_amd import binding

CSRC = os.path.join(os.path.dirname(binding.LIB_PATH), "csrc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "quotient.h"
using namespace omni;

static long wrong = 0, multiplied = 0, divided = 0;
static void check(int d, uint64_t below) {
  const uint32_t by = reciprocal_below(d, below);
  by ? ++multiplied : ++divided;
  auto at = [&](int64_t n) {
    if (n >= 0 && (uint64_t)n < below && n < (1ll << 31) && quotient((int)n, by, d) != (int)n / d) ++wrong;
  };
  const int64_t last = (int64_t)below - 1, q = last / d;
  for (int64_t k : {int64_t(0), int64_t(1), q / 2, q - 1, q})
    for (int64_t n : {k * d - 1, k * d, k * d + 1, (k + 1) * d - 1}) at(n);
  at(last);
}

int main() {
  std::mt19937_64 rng(5);
  auto log_up_to = [&](int bits) { return 1 + (int64_t)(rng() >> (64 - 1 - rng() % bits)); };
  for (int i = 0; i < 2000000; ++i) check((int)std::min<int64_t>(log_up_to(31), INT32_MAX), std::min<int64_t>(log_up_to(31), INT32_MAX));
  for (int d = 1; d <= 4096; ++d) {           // at the bound, and one beyond it
    check(d, (1ull << 32) / d);
    check(d, (1ull << 32) / d + 1);
  }
  for (int d : {1, 2, 3, 7, 36, 255, 1023, 16384})
    for (int n = 0; n < 100000; ++n)
      if (quotient(n, reciprocal_below(d, 100000), d) != n / d) ++wrong;
  // one image of 2080000 x 8 positions, 130000 units: the multiplication alone takes the last units for a second image's
  const uint32_t alone = (uint32_t)(((1ull << 32) + 130000 - 1) / 130000);
  std::printf("%ld %d %d %d %d\n", wrong, multiplied > 100000, divided > 100000, quotient(129999, alone, 130000),
              quotient(129999, reciprocal_below(130000, 130000), 130000));
}
"""


def test_quotients(tmp_path):
    (tmp_path / "p.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "p")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    str(tmp_path / "p.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert out.split() == ["0", "1", "1", "1", "0"]


def test_no_other_reciprocals_of_32_bits():
    for f in sorted(os.listdir(CSRC)):
        if f != "quotient.h":
            src = open(os.path.join(CSRC, f)).read()
            assert "1ull << 32) +" not in src and "1l << 32) +" not in src, f
