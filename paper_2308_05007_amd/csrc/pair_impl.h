// Two fluid steps in one pass over the lattice (FP32 storage, two lattices,
// periodic, partially saturated cells with prescribed particles).
//
// A lattice beyond the caches is bound by its 38 words per node and step (the
// single step runs at 5.4 TB/s, 99% of that access pattern's rate), so the pass
// that reads f*(t - 1) carries it to f*(t + 1): 38 words and two velocities for
// two steps.  A block owns a tile of 64 x 8 nodes in x and y and walks up z.
// Each plane, its threads (one per node of the tile and its rim of one node)
// pull and collide step t, leave the plane's post-collision populations in
// LDS, and take from there what streams to their own node of the tile: the
// five directions that go down complete the node of the plane below for step
// t + 1, the nine that stay wait one plane in registers, the five that go up
// two.  The rim is computed twice (66 x 10 for 64 x 8 nodes) and re-read
// through L2, where the neighbouring tiles of an XCD meet; what is written is
// stored non-temporally, so that it does not push those lines out (256^3: 352
// -> 325 us per step with the particles).  The next plane's loads are in flight
// while this one collides, and two LDS planes in turn leave one barrier per
// plane.  One block of 11 waves fills a CU (100 KB LDS, 146 VGPRs), so the
// blocks per pass are chosen to fill whole rounds of the chip (pair_shape).
//
// Measured, us per fluid step without particles, single and paired: 256^3 509 ->
// 295, 224^3 346 -> 242, 192^3 220 -> 136; with particles a block waits at each
// plane for the wave that evaluates their control points, where the single
// step's other waves go on (pairs_gain).  A pass of 256^3 with 64 particles moves
// 1.19 times its own bytes (the rims) at 5.2 TB/s; tiles 32 x 16 352, 32 x 8 423,
// 64 x 12 342 at 256^3, and with 4, 8 runs of planes (2, 4 rounds of blocks)
// instead of 2 the step with particles and walkers 489, 504 instead of 464.
// With 16-bit storage the bytes no longer bound it and it gained nothing (281
// against 275).  The walkers then run in a launch of their own, 142 us per step
// for 1e7 where beside the single step's fluid they add 95: the whole step at
// 256^3 with 1e7 walkers 607 -> 466.
//
// Every node is computed by the functions of the single step (collide_float,
// solid_sum), whose fused multiply-adds are written out, so a run's values do not
// depend on how its steps are paired.
#pragma once
#include "lbm_impl.h"
#include "pro_impl.h"
#include "step_map.h"

namespace rwmi {

// Slots of the populations that wait: the nine that stay in the plane and the
// five that go up.
constexpr int flat_slot(int i) { return i <= 4 ? i : i - 2; }                        // 0..4, 7..10
constexpr int up_slot(int i) { return i == 5 ? 0 : i == 11 ? 1 : i == 14 ? 2 : i == 15 ? 3 : 4; }
static_assert(kEz[5] == 1 && kEz[11] == 1 && kEz[14] == 1 && kEz[15] == 1 && kEz[18] == 1, "directions that go up");

// ALIGNED: a plane is whole tiles of the layout (nx ny a multiple of kTile), so
// that a node's offset within its plane is the same in every plane.
template <bool FORCE, bool ALIGNED>
__global__ void __launch_bounds__(kPairThreads) k_pair(PairArgs a, const DomView* __restrict__ views) {
  __shared__ float lds[2][kQ * kPairRim];
  const DomView& V = views[0];
  // XCD-aware: hardware block i runs on XCD i mod 8, which owns a contiguous
  // run of the blocks (tiles x fastest, then y, then the z chunk)
  const int xcd = (int)blockIdx.x & 7, q = (int)blockIdx.x >> 3;
  const int nb = a.ntx * a.nty * a.nzc;
  if (q >= xcd_count(nb, xcd)) return;  // uniform over the block
  const int b = xcd_first(nb, xcd) + q;
  const int tix = b % a.ntx, tiy = (b / a.ntx) % a.nty, zc = b / (a.ntx * a.nty);
  const int nx = V.n[0], ny = V.n[1], nz = V.n[2];
  const int x0 = tix * a.tx, y0 = tiy * a.ty;
  const int wx = nx - x0 < a.tx ? nx - x0 : a.tx, wy = ny - y0 < a.ty ? ny - y0 : a.ty;
  const int z0 = (int)((int64_t)nz * zc / a.nzc), z1 = (int)((int64_t)nz * (zc + 1) / a.nzc);
  const uint64_t t = step_of(V, a.j);
  const bool lat = source_lattice(V, a.s);
  const auto src = gp((const float*)(lat ? V.fB : V.fA));
  const auto dst = gp((float*)(lat ? V.fA : V.fB));
  const auto u0 = gp((float*)V.u[t & 1ull]);
  const auto u1 = gp((float*)V.u[(t + 1) & 1ull]);
  const int ps0 = pose_slot(t), ps1 = pose_slot(t + 1);
  const uint32_t sxy = (uint32_t)nx * (uint32_t)ny;
  auto wrap = [](int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); };

  // step t: thread i has node i of the tile and its rim, rows of wx + 2
  const int hx = wx + 2, rim = hx * (wy + 2);
  const int tid = threadIdx.x;
  const bool act = tid < rim;
  const int lx = act ? tid % hx : 0, ly = act ? tid / hx : 0;
  const int x = wrap(x0 + lx - 1, nx), y = wrap(y0 + ly - 1, ny);
  const bool inner = act && lx >= 1 && lx <= wx && ly >= 1 && ly <= wy;
  const uint32_t xy = (uint32_t)x + (uint32_t)y * (uint32_t)nx;
  // upstream columns by (ex, ey): node in the plane, or (aligned) its byte
  uint32_t col[3][3];
#pragma unroll
  for (int ey = -1; ey <= 1; ++ey)
#pragma unroll
    for (int ex = -1; ex <= 1; ++ex) {
      const uint32_t n = (uint32_t)wrap(x - ex, nx) + (uint32_t)wrap(y - ey, ny) * (uint32_t)nx;
      col[ey + 1][ex + 1] = ALIGNED ? fnode(true, n) * 4u : n;
    }
  // step t + 1: thread i has node i of the tile
  const bool mine = tid < wx * wy;
  const int ix = mine ? tid % wx : 0, iy = mine ? tid / wx : 0;
  const int rimid = (iy + 1) * hx + ix + 1;
  const uint32_t xy1 = (uint32_t)(x0 + ix) + (uint32_t)(y0 + iy) * (uint32_t)nx;
  const uint32_t byte1 = fnode(true, xy1) * 4u;
  const uint32_t plane = sxy / kTile * (uint32_t)(kQ * kTile);  // elements per plane (aligned)

  // lane p of every wave holds particle p's reach: it meets the wave's rows of
  // a plane where the squared z distance is at most lim (a superset: float,
  // radii enlarged by kCullMargin)
  float cz[2] = {0.0f, 0.0f}, lim[2] = {-1.0f, -1.0f};
  const int lane = tid & 63;
  {
    const int first = tid & ~63, last = first + 63;  // the wave's threads
    const int r0 = first / hx - 1, r1 = (last < rim ? last : rim - 1) / hx - 1;
    const int s0 = first / wx, s1 = (last < wx * wy ? last : wx * wy - 1) / wx;
    if (lane < V.np) {
      const float r = (float)sqrt(V.parts[lane].epscut2) + kCullMargin;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const auto pt = gp((const double*)V.pose[k ? ps1 : ps0]) + kPoseRec * lane;
        const float xa = (float)(k ? x0 : x0 - 1) + 0.5f, xb = (float)(k ? x0 + wx - 1 : x0 + wx) + 0.5f;
        const float ya = (float)(y0 + (k ? s0 : r0)) + 0.5f, yb = (float)(y0 + (k ? s1 : r1)) + 0.5f;
        const float gx = gap_lb(1, (float)nx, 1.0f / (float)nx, xa, xb, (float)pt[0]);
        const float gy = gap_lb(1, (float)ny, 1.0f / (float)ny, ya, yb, (float)pt[1]);
        cz[k] = (float)pt[2];
        lim[k] = r * r - (gx * gx + gy * gy);
      }
    }
  }
  const float Lz = (float)nz, invLz = 1.0f / Lz;
  auto plane_bits = [&](int k, int z) -> unsigned long long {
    const float g = gap_lb(1, Lz, invLz, (float)z + 0.5f, (float)z + 0.5f, cz[k]);
    return __ballot(g * g <= lim[k]);
  };

  auto load = [&](int z, float(&r)[kQ]) {
    const uint32_t zz[3] = {(uint32_t)wrap(z + 1, nz), (uint32_t)z, (uint32_t)wrap(z - 1, nz)};  // by ez + 1
    unroll<0, kQ>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const uint32_t c = col[kEy[i] + 1][kEx[i] + 1];
      if constexpr (ALIGNED) {
        r[i] = *at_byte<const float>(src + ((size_t)i * kTile + zz[kEz[i] + 1] * plane), c);
      } else {
        const uint32_t n = c + zz[kEz[i] + 1] * sxy;
        r[i] = *at_byte<const float>(src + (size_t)i * kTile, fnode(true, n) * 4u);
      }
    });
  };
  float next[kQ];
  float flat[9], up1[5], up2[5];  // populations of step t + 1 that wait
#pragma unroll
  for (int i = 0; i < 9; ++i) flat[i] = 0.0f;
#pragma unroll
  for (int i = 0; i < 5; ++i) up1[i] = up2[i] = 0.0f;
#pragma unroll
  for (int i = 0; i < kQ; ++i) next[i] = 0.0f;
  if (act) load(wrap(z0 - 1, nz), next);
  for (int k = z0 - 1; k <= z1; ++k) {
    const int z = wrap(k, nz);
    float* L = lds[(k - z0 + 1) & 1];
    float f[kQ];
#pragma unroll
    for (int i = 0; i < kQ; ++i) f[i] = next[i];
    if (act && k < z1) load(wrap(k + 1, nz), next);
    // step t on plane k
    const unsigned long long bits0 = V.np > 0 ? plane_bits(0, z) : 0ull;
    if (act) {
      const int nd[3] = {x, y, z};
      float es, un[3], u[3], rho;
      solid_sum(V, ps0, bits0, nd, es, un);
      collide_float(V, f, es, un, FORCE, u, rho, [&](auto ic, float v) {
        L[decltype(ic)::value * kPairRim + tid] = v;
      });
      if (inner && k >= z0 && k < z1) {
        const auto up = at_byte<float>(u0, 12u * (xy + (uint32_t)z * sxy));
#pragma unroll
        for (int c = 0; c < 3; ++c) __builtin_nontemporal_store(u[c], up + c);
      }
    }
    lds_barrier();
    // step t + 1 on plane k - 1
    const int zb = k - 1;
    const bool out = zb >= z0 && zb < z1;
    const unsigned long long bits1 = V.np > 0 && out ? plane_bits(1, zb) : 0ull;
    if (mine) {
      float g[kQ], nflat[9], nup[5];
      unroll<0, kQ>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const float v = L[i * kPairRim + rimid - kEx[i] - kEy[i] * hx];
        if constexpr (kEz[i] == 0) {
          nflat[flat_slot(i)] = v;
          g[i] = flat[flat_slot(i)];
        } else if constexpr (kEz[i] == 1) {
          nup[up_slot(i)] = v;
          g[i] = up1[up_slot(i)];
        } else {
          g[i] = v;
        }
      });
      if (out) {
        const int nd[3] = {x0 + ix, y0 + iy, zb};
        const uint32_t id = xy1 + (uint32_t)zb * sxy;
        const uint32_t ob = ALIGNED ? byte1 : fnode(true, id) * 4u;
        const size_t oe = ALIGNED ? (size_t)((uint32_t)zb * plane) : 0;
        float es, un[3], u[3], rho;
        solid_sum(V, ps1, bits1, nd, es, un);
        collide_float(V, g, es, un, FORCE, u, rho, [&](auto ic, float v) {
          __builtin_nontemporal_store(v, at_byte<float>(dst + ((size_t)decltype(ic)::value * kTile + oe), ob));
        });
        const auto up = at_byte<float>(u1, 12u * id);
#pragma unroll
        for (int c = 0; c < 3; ++c) __builtin_nontemporal_store(u[c], up + c);
        if (a.dens) *at_byte<float>(gp((float*)V.rho), 4u * id) = rho;
      }
#pragma unroll
      for (int i = 0; i < 9; ++i) flat[i] = nflat[i];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        up1[i] = up2[i];
        up2[i] = nup[i];
      }
    }
  }
}

}  // namespace rwmi
