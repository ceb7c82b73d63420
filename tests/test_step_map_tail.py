"""Role map of the step launch with and without a tail of fluid blocks (compiled
for the host): every role block is dealt once, and where the launch leaves a
tail, an XCD's last positions hold fluid only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2308_05007_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "step_map.h"
using namespace rwmi;
static int check(const int nb[3], bool xcd, int tail) {
  std::vector<int> seen[3], last_walk(8, -1), last(8, -1);
  for (int r = 0; r < 3; ++r) seen[r].assign(nb[r], 0);
  const int g = step_grid(nb, xcd);
  for (int i = 0; i < g; ++i) {
    int idx = -1;
    const int r = step_role(i, nb, xcd, idx, tail);
    if (r == kRoleNone) continue;
    if (idx < 0 || idx >= nb[r] || seen[r][idx]++) { printf("role %d block %d at %d\n", r, idx, i); return 1; }
    const int x = xcd ? i & 7 : 0;
    last[x] = xcd ? i >> 3 : i;
    if (r == kRoleWalk) last_walk[x] = last[x];
  }
  for (int r = 0; r < 3; ++r)
    for (int k = 0; k < nb[r]; ++k)
      if (seen[r][k] != 1) { printf("role %d block %d dealt %d times\n", r, k, seen[r][k]); return 1; }
  for (int x = 0; x < (xcd ? 8 : 1); ++x) {
    const int cf = xcd ? xcd_count(nb[2], x) : nb[2], t = xcd ? tail : 8 * tail;
    if (last_walk[x] >= 0 && last[x] - last_walk[x] < (cf < t ? cf : t)) { printf("xcd %d: walkers at %d of %d\n", x, last_walk[x], last[x]); return 1; }
  }
  return 0;
}
int main() {
  const int vals[] = {0, 1, 7, 8, 9, 64, 65, 1000, 3584, 3907, 8064};
  for (int a : vals) for (int b : {0, 1, 9, 300}) for (int c : vals) for (int x = 0; x < 2; ++x) for (int t : {0, 1, kTailBlocks}) {
    const int nb[3] = {a, b, c};
    if (check(nb, x != 0, t)) { printf("nb %d %d %d xcd %d tail %d\n", a, b, c, x, t); return 1; }
  }
  printf("ok\n");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_role_map_with_and_without_a_tail(tmp_path):
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as fh:
        fh.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
