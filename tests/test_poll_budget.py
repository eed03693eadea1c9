"""The bound on the ring's polls (csrc/poll_budget.h), compiled for the host: it
is each wait's own, however many steps a pass has, and after a wait that ran out
no later one waits."""

import os
import shutil
import subprocess

import pytest

from paper_1904_10584_amd import build

MAIN = r"""
#include <cstdio>
#include "poll_budget.h"
// polls of a wait that succeeds after `failing` failed polls, or gives up
static unsigned wait(am::PollBudget<(1u << 22)>& b, unsigned failing, bool* gave_up) {
  b.begin();
  for (unsigned n = 1;; ++n) {
    if (n > failing) { *gave_up = false; return n; }
    if (b.spent()) { *gave_up = true; return n; }
  }
}
int main() {
  constexpr unsigned LIMIT = 1u << 22;
  am::PollBudget<LIMIT> b;
  bool gave_up = false;
  // far more failed polls over the steps than one wait may take
  for (unsigned step = 0; step < 2 * LIMIT; ++step)
    if (wait(b, 3, &gave_up) != 4 || gave_up) { printf("gave up at step %u\n", step); return 1; }
  if (wait(b, LIMIT, &gave_up) != LIMIT + 1 || gave_up) { puts("a wait within the limit"); return 1; }
  if (wait(b, LIMIT + 1, &gave_up) != LIMIT + 1 || !gave_up) { puts("a wait beyond the limit"); return 1; }
  for (int step = 0; step < 3; ++step)
    if (wait(b, 100, &gave_up) != 1 || !gave_up) { puts("a wait after one that ran out"); return 1; }
  if (wait(b, 0, &gave_up) != 1 || gave_up) { puts("a poll that succeeds at once"); return 1; }
  puts("ok");
}
"""


def test_poll_budget(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    p = subprocess.run([gxx, "-O1", "-std=c++17", "-I", build.CSRC, str(tmp_path / "main.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0 and p.stdout.strip() == "ok", p.stdout


def test_ring_polls_within_the_budget():
    src = open(os.path.join(build.CSRC, "lstm_xcd.hip")).read()
    loop = src[src.index("polls.begin();"):]
    assert loop.index("polls.spent()") < loop.index("lds_barrier()")
