"""What a kernel needs once per device is done on every device, is tried again after a failure and
not done twice; a host program over the header that the launchers use."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cassert>
#include <thread>
#include <vector>
#include "spa_once.hpp"
int main() {
  spa::OncePerDevice once;
  int calls[100] = {};
  auto act = [&](int d) { ++calls[d]; return true; };
  for (int rep = 0; rep < 3; ++rep)
    for (int d : {0, 1, 7, 63}) assert(once.run(d, act));
  for (int d : {0, 1, 7, 63}) assert(calls[d] == 1);
  assert(!once.run(5, [&](int d) { ++calls[d]; return false; }));   // a failure is not remembered
  assert(once.run(5, act) && once.run(5, act) && calls[5] == 2);
  assert(once.run(64, act) && once.run(64, act) && calls[64] == 2);  // beyond the mask: every time
  std::vector<std::thread> t;
  std::atomic<int> n{0};
  spa::OncePerDevice shared;
  for (int i = 0; i < 8; ++i) t.emplace_back([&, i] { shared.run(i % 4, [&](int) { ++n; return true; }); });
  for (auto &x : t) x.join();
  assert(n >= 4 && n <= 8);
  for (int d = 0; d < 4; ++d) shared.run(d, [&](int) { assert(false); return true; });
}
"""


def test_once_per_device(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "t.cpp").write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_1106_0322_amd", "csrc")
    subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I", inc, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")],
                   check=True, timeout=120)
    subprocess.run([str(tmp_path / "t")], check=True, timeout=60)
