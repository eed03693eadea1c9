"""What the launchers do once for every device of the process
(csrc/per_device.h), compiled for the host: each device gets it, once, a failure
is tried again, and threads may come at the same time."""

import shutil
import subprocess

import pytest

from paper_1904_10584_amd import build

MAIN = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.h"
int main() {
  am::PerDevice p;
  int calls = 0;
  auto fails = [&] { ++calls; return 7; };
  auto works = [&] { ++calls; return 0; };
  if (p.once(0, fails) != 7 || p.once(0, fails) != 7 || calls != 2) { puts("a failure is reported, and tried again"); return 1; }
  if (p.once(0, works) != 0 || p.once(0, works) != 0 || calls != 3) { puts("once on a device"); return 1; }
  if (p.once(5, works) != 0 || calls != 4) { puts("another device has it done too"); return 1; }
  if (p.once(0, fails) != 0 || p.once(5, fails) != 0 || calls != 4) { puts("neither again"); return 1; }
  if (p.once(64, works) != 0 || p.once(64, works) != 0 || calls != 6) { puts("beyond 63: every time"); return 1; }
  am::PerDevice q;
  std::atomic<int> set[8] = {};
  std::atomic<bool> early{false};
  std::vector<std::thread> t;
  for (int k = 0; k < 16; ++k)
    t.emplace_back([&, k] {
      for (int i = 0; i < 2000; ++i) {
        const int d = (i + k) % 8;
        q.once(d, [&] { set[d].store(1); return 0; });
        if (!set[d].load()) early = true;
      }
    });
  for (auto& x : t) x.join();
  if (early) { puts("returned before the device was set"); return 1; }
  puts("ok");
}
"""


def test_per_device(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    p = subprocess.run([gxx, "-O1", "-std=c++17", "-pthread", "-I", build.CSRC, str(tmp_path / "main.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0 and p.stdout.strip() == "ok", p.stdout
