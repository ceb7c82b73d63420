// Host side of the choice between paired fluid steps (pair_impl.h) and single
// ones.  No HIP.
#pragma once
#include <algorithm>
#include <cmath>
#include <vector>

#include "step_map.h"

namespace rwmi {

// A particle as the choice sees it: centre, reach of its solid fraction, and
// number of control points.
struct PairParticle {
  double c[3], r;
  int nc;
};

// Microseconds of one pass (two fluid updates of every node) of shape a.  A
// block plane takes 4.5 where rows begin at 64-byte sectors, 5.1 at 32-byte
// ones and 6.1 elsewhere, less in narrow tiles; a plane that meets a particle's
// reach waits for the wave that evaluates its control points, twice, at 0.05 +
// 0.06 per point.  The blocks run in order, 32 of an XCD at a time.  Modelled
// and measured per update: 256^3 292, 295; with 20 small particles 321, 324;
// with 64 of 12 points and radius 17 454, 420; with 64 of 60 points 1088, 1081;
// 250^3 387, 400; 224^3 243, 242; 1000x121x64 with 20 193, 193.
inline double pair_pass_us(const PairArgs& a, const int n[3], const std::vector<PairParticle>& parts) {
  const double sector = n[0] % 16 == 0 ? 4.5 : n[0] % 8 == 0 ? 5.1 : 6.1;
  const double plane = sector * (0.25 + 0.75 * a.tx / kPairTx);
  if (parts.empty()) return plane * (double)a.cost;
  const int nb = a.ntx * a.nty * a.nzc;
  std::vector<double> us(nb);
  auto run0 = [&](int q) { return (int)((int64_t)n[2] * q / a.nzc); };
  for (int b = 0; b < nb; ++b) {
    const int q = b / (a.ntx * a.nty);
    us[b] = plane * (run0(q + 1) - run0(q) + 2);
  }
  for (const PairParticle& p : parts) {
    // nodes of an axis within the reach: `len` of them from `lo` on, around
    // the period
    int64_t lo[3], len[3];
    for (int k = 0; k < 3; ++k) {
      const double c = p.c[k] - n[k] * std::floor(p.c[k] / n[k]), r = std::min(p.r, (double)n[k]);
      if (!(c >= 0.0) || !(r >= 0.0)) return INFINITY;
      const int64_t i0 = (int64_t)std::ceil(c - r - 0.5), i1 = (int64_t)std::floor(c + r - 0.5);
      len[k] = std::min<int64_t>(i1 - i0 + 1, n[k]);
      lo[k] = (i0 % n[k] + n[k]) % n[k];
    }
    // the tiles of an axis that they meet
    auto tiles = [&](int k, int size) {
      std::vector<int> t;
      for (int64_t i = lo[k], end = lo[k] + len[k]; i < end;) {
        const int64_t at = i % n[k];
        t.push_back((int)(at / size));
        i += std::min<int64_t>(n[k], (at / size + 1) * size) - at;
      }
      if (t.size() > 1 && t.front() == t.back()) t.pop_back();  // all the way round
      return t;
    };
    const std::vector<int> tx = tiles(0, a.tx), ty = tiles(1, a.ty);
    for (int q = 0; q < a.nzc; ++q) {
      int64_t planes = 0;  // of the run
      for (int64_t l = lo[2] - n[2]; l <= lo[2]; l += n[2])
        planes += std::max<int64_t>(0, std::min<int64_t>(run0(q + 1), l + len[2]) - std::max<int64_t>(run0(q), l));
      if (planes <= 0) continue;
      for (int j : ty)
        for (int i : tx) us[(q * a.nty + j) * a.ntx + i] += 2.0 * (double)planes * (0.05 + 0.06 * p.nc);
    }
  }
  double end = 0.0;
  for (int x = 0; x < 8; ++x) {
    double cu[32] = {};
    for (int b = xcd_first(nb, x), m = b + xcd_count(nb, x); b < m; ++b) *std::min_element(cu, cu + 32) += us[b];
    end = std::max(end, *std::max_element(cu, cu + 32));
  }
  return end;
}

// Is a fluid update with its walkers faster as half of a pass?  A single update
// takes 30.6 ps per node; walkers run 30-50 us per 1e7 slower apart from the
// fluid (at most two per node have been measured).  The line lies at 0.9
// because the model is up to 13% off.  us per update, single and paired, of
// what it takes: 256^3 509, 295, with 64 particles of reach 10 and 8 points
// 511, 338 and with 1e7 walkers too 700, 583; with the particles within ten
// planes of y 511, 501; 176^3 168, 121, with 20 such particles 169, 155; 250^3
// 479, 400; 192^3 with 1.4e7 walkers 422, 381; 48x48x2600 176, 115.  And of
// what it refuses: 256^3 with 64 particles of 60 points and reach 22 546, 1081,
// with one of 64 points and reach 38 511, 519, with 64 small ones in a corner
// of 20^3 516, 806; 176^3 with 49 of 12 points and reach 18 170, 187, with 20
// and 2.7e6 walkers 222, 225; 219x187x241 300, 308; 200x200x140 with 10
// particles and 5e5 walkers 197, 197; 24x500x500 180, 180; 16x16x21000 159, 205.
inline bool pairs_gain(const PairArgs& a, const int n[3], int64_t nw, const std::vector<PairParticle>& parts) {
  const double N = (double)n[0] * n[1] * n[2];
  if ((double)nw > 2.0 * N) return false;
  auto gain = [&](const std::vector<PairParticle>& p) {
    return 0.5 * pair_pass_us(a, n, p) + 4.0e-6 * (double)nw < 0.9 * 30.6e-6 * N;
  };
  return gain({}) && gain(parts);
}

}  // namespace rwmi
