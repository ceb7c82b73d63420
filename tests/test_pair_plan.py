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


def test_pass_time_counts_each_particles_planes(tmp_path):
    """The blocks that a particle slows, against a test of every node, also
    across periodic faces and for reaches beyond the lattice."""
    _run(tmp_path, r"""
#include <cstdio>
#include <random>
#include "pair_plan.h"
using namespace rwmi;
int main() {
  std::mt19937 rng(7);
  auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
  for (int k = 0; k < 300; ++k) {
    const int n[3] = {(int)uni(1, 300), (int)uni(1, 120), (int)uni(1, 200)};
    const PairArgs a = pair_shape(n[0], n[1], n[2]);
    std::vector<PairParticle> ps((size_t)uni(1, 12));
    for (auto& p : ps) p = {{uni(-500, 500), uni(-500, 500), uni(-500, 500)}, uni(0.0, k % 3 ? 30 : 400), (int)uni(1, 64)};
    const double plane = (n[0] % 16 == 0 ? 4.5 : n[0] % 8 == 0 ? 5.1 : 6.1) * (0.25 + 0.75 * a.tx / 64);
    const int nb = a.ntx * a.nty * a.nzc;
    std::vector<double> us(nb);
    for (int b = 0; b < nb; ++b) {
      const int i = b % a.ntx, j = b / a.ntx % a.nty, q = b / (a.ntx * a.nty);
      const int z0 = (int)((int64_t)n[2] * q / a.nzc), z1 = (int)((int64_t)n[2] * (q + 1) / a.nzc);
      us[b] = plane * (z1 - z0 + 2);
      for (auto& p : ps) {
        auto near = [&](int k, int at) {
          const double d = at + 0.5 - p.c[k];
          return std::fabs(d - n[k] * std::floor(d / n[k] + 0.5)) <= p.r;
        };
        int planes = 0; bool x = false, y = false;
        for (int v = z0; v < z1; ++v) planes += near(2, v);
        for (int v = i * a.tx; v < std::min(n[0], (i + 1) * a.tx); ++v) x |= near(0, v);
        for (int v = j * a.ty; v < std::min(n[1], (j + 1) * a.ty); ++v) y |= near(1, v);
        if (x && y) us[b] += 2 * planes * (0.05 + 0.06 * p.nc);
      }
    }
    double end = 0;
    for (int x = 0; x < 8; ++x) {
      std::vector<double> cu(32, 0.0);
      for (int i = 0; i < xcd_count(nb, x); ++i) *std::min_element(cu.begin(), cu.end()) += us[xcd_first(nb, x) + i];
      for (double c : cu) end = std::max(end, c);
    }
    const double got = pair_pass_us(a, n, ps);
    if (!(std::fabs(got - end) <= 1e-9 * end)) { printf("case %d: %g, not %g\n", k, got, end); return 1; }
  }
  printf("ok\n");
  return 0;
}
""")


def test_pairs_are_refused_where_they_are_slower(tmp_path):
    """Measured us per update, single and paired, at 256^3 (random places):
    64 particles of 8 points and reach 10 511, 338; of 60 points and reach 22 546,
    1081; no particles and two walkers per node at 192^3 422, 381; 219x187x241
    300, 308."""
    _run(tmp_path, r"""
#include <cstdio>
#include <random>
#include "pair_plan.h"
using namespace rwmi;
static bool gain(int x, int y, int z, int64_t nw, int np, double r, int nc, double box = 0) {
  std::mt19937 rng(3);
  std::vector<PairParticle> ps(np);
  const int n[3] = {x, y, z};
  for (auto& p : ps) {
    for (int k = 0; k < 3; ++k) p.c[k] = std::uniform_real_distribution<double>(0, box > 0 ? box : n[k])(rng);
    p.r = r;
    p.nc = nc;
  }
  return pairs_gain(pair_shape(x, y, z), n, nw, ps);
}
#define WANT(e) if (!(e)) { printf("not %s\n", #e); return 1; }
int main() {
  WANT(gain(256, 256, 256, 0, 0, 0, 0))
  WANT(gain(256, 256, 256, 10000000, 64, 10, 8))
  WANT(!gain(256, 256, 256, 10000000, 64, 22, 60))
  WANT(!gain(256, 256, 256, 0, 64, 22, 60))
  WANT(!gain(250, 250, 100, 0, 43, 22, 60))
  WANT(gain(192, 192, 192, 2 * 192 * 192 * 192, 0, 0, 0))
  WANT(!gain(192, 192, 192, 2 * 192 * 192 * 192 + 1, 0, 0, 0))
  WANT(!gain(219, 187, 241, 0, 0, 0, 0))
  WANT(gain(250, 250, 250, 0, 20, 10, 8))
  WANT(!gain(256, 256, 256, 0, 64, 10, 8, 20.0))  // all in one corner: a few blocks have all their planes
  const double nan = NAN;
  WANT(!pairs_gain(pair_shape(256, 256, 256), (const int[3]){256, 256, 256}, 0, {{{nan, 0, 0}, 5.0, 3}}))
  printf("ok\n");
  return 0;
}
""")
