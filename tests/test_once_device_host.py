"""Host check of settings made once per device (csrc/once_device.hpp), from several
threads: no thread goes on before its device has been set, failures are not kept, and
the threads' order never lowers a value.  Compiled with g++ as plain host code."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2410_05934_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "once_device.hpp"
using namespace nttk;
int main() {
  for (int round = 0; round < 200; ++round) {
    OncePerDevice once;
    std::atomic<int> limit[3], calls{0}, bad{0};
    for (auto& l : limit) l = 0;
    std::vector<std::thread> th;
    for (int t = 0; t < 8; ++t)
      th.emplace_back([&, t] {
        for (int i = 0; i < 50; ++i) {
          const int d = (t + i) % 3;
          if (once.run(d, [&] { limit[d] = 100; ++calls; return 0; }) != 0) ++bad;
          if (limit[d] != 100) ++bad;  // a launch of any size up to 100 would be refused
        }
      });
    for (auto& x : th) x.join();
    if (bad || calls < 3 || calls > 24) return std::printf("bad %d calls %d\n", (int)bad, (int)calls), 1;
  }
  OncePerDevice once;
  int n = 0;
  if (once.run(0, [&] { ++n; return 7; }) != 7 || once.run(0, [&] { ++n; return 0; }) != 0 ||
      once.run(0, [&] { ++n; return 7; }) != 0 || n != 2) return std::printf("errors\n"), 1;
  if (once.run(64, [&] { ++n; return 0; }) || once.run(64, [&] { ++n; return 0; }) || n != 4)
    return std::printf("many devices\n"), 1;
  std::printf("ok\n");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_once_per_device(tmp_path):
    src, exe = tmp_path / "drv.cpp", tmp_path / "drv"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", f"-I{CSRC}", str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout
