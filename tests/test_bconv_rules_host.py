"""Host check of the few-source basis conversion's grid (csrc/bconv_rules.hpp): every
coefficient and every target is covered, none of the grid is empty, up to the largest
call (below 2^32 coefficients).  Compiled with g++ as plain host code."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2410_05934_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "bconv_rules.hpp"
using namespace nttk;
int main() {
  std::vector<uint64_t> totals;
  for (int b = 1; b <= 32; ++b)
    for (int64_t d : {-258, -256, -255, -2, 0, 2, 256})
      if ((int64_t)(1ull << b) + d > 0 && (1ull << b) + d < (1ull << 32)) totals.push_back((1ull << b) + d);
  long n = 0;
  for (uint64_t t : totals)
    for (uint32_t M : {1u, 2u, 3u, 4u, 5u, 7u, 8u, 9u, 36u, 4095u, 4096u}) {
      const FewGrid g = few_grid((uint32_t)t, M);
      const bool coef = g.blocks >= 1 && (uint64_t)g.blocks * kBconvBlock >= t &&
                        (uint64_t)(g.blocks - 1) * kBconvBlock < t;
      const bool targ = g.per >= 1 && g.rows >= 1 && (uint64_t)g.rows * g.per >= M &&
                        (uint64_t)(g.rows - 1) * g.per < M && g.rows <= 65535;
      if (!coef || !targ) {
        std::printf("total %llu M %u: %u blocks, %u rows of %u\n", (unsigned long long)t, M, g.blocks, g.rows, g.per);
        return 1;
      }
      ++n;
    }
  std::printf("ok %ld\n", n);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_few_source_grid_covers_every_call(tmp_path):
    src, exe = tmp_path / "drv.cpp", tmp_path / "drv"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout
