"""The host's choice of paired fluid steps (compiled for the host): tiles and
runs of planes, found without a walk over every plane of a long lattice."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2308_05007_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


def _run(tmp_path, program):
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as fh:
        fh.write(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


def test_shape_is_the_cheapest_one(tmp_path):
    """The first of the cheapest numbers of runs, as a search over all of them
    finds it, for lattices of every proportion; and 10000 searches over the
    longest lattices in under a minute."""
    _run(tmp_path, r"""
#include <cstdio>
#include <cstdint>
#include "step_map.h"
using namespace rwmi;
int main() {
  const int vals[] = {1, 2, 3, 7, 8, 9, 16, 33, 63, 64, 65, 100, 128, 171, 250, 256, 500, 1000, 2600, 20011};
  for (int x : vals) for (int y : vals) for (int z : vals) {
    const PairArgs a = pair_shape(x, y, z);
    int64_t best = -1; int at = 0;
    for (int c = 1; c <= (z + 3) / 4; ++c) {
      const int64_t cost = (((int64_t)a.ntx * a.nty * c + 255) / 256) * ((z + c - 1) / c + 2);
      if (best < 0 || cost < best) { best = cost; at = c; }
    }
    if (a.cost != best || a.nzc != at) { printf("%d %d %d: %d runs at %lld, not %d at %lld\n", x, y, z, a.nzc, (long long)a.cost, at, (long long)best); return 1; }
    if (a.tx < 1 || a.tx > kPairTx || a.ty < 1 || a.ty > kPairTy || a.ntx * a.tx < x || (a.ntx - 1) * a.tx >= x || a.nty * a.ty < y || (a.nty - 1) * a.ty >= y) { printf("tiles of %d %d\n", x, y); return 1; }
  }
  int64_t sum = 0;
  for (int k = 0; k < 5000; ++k) sum += pair_shape(1, 1, 50000000 + k).cost + pair_shape(16, 16, 200000 + k).cost;
  printf("ok %lld\n", (long long)sum);
  return 0;
}
""")
