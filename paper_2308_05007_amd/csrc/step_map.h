// Block roles of the fused step launch (host and device).
//
// One launch of a step group carries three kinds of blocks: the walkers of
// step t-1 (fast path, then the block's own near-surface walkers), the fluid
// update of step t and the prologue of step t+1 (particle poses, coarse cull
// mask).  They read only what earlier launches wrote and write disjoint
// buffers (velocity double-buffered by step parity, pose table and mask by
// step mod 3), so they need no ordering among themselves.
//
// Hardware block i runs on XCD i mod 8.  With the XCD-aware map every XCD
// receives a contiguous run of the fluid blocks (neighbouring nodes share its
// L2), its share of the walker blocks interleaved evenly among all but the last
// of them (latency-bound walker work overlaps bandwidth-bound fluid work on
// every CU, and fluid blocks cover the end of the last walkers), and its
// prologue blocks first.  Without it the roles are dealt the same way over the
// whole grid.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define RWMI_HD __host__ __device__
#else
#define RWMI_HD  // plain C++ (host-side tests)
#endif

namespace rwmi {

enum BlockRole { kRoleWalk = 0, kRolePro = 1, kRoleFluid = 2, kRoles = 3, kRoleNone = -1 };

constexpr int kFlagXcd = 1;          // XCD-aware role map
constexpr int kFlagNontemporal = 2;  // non-temporal stores of f* and u
// Set by the host (never by a caller) on the launch that carries the last
// fluid step of a launch group: that step also writes the node densities,
// which only read-outs use.
constexpr int kFlagDensity = 4;
// The domains have two-way coupled particles: the prologue builds the masks
// from the poses the particle update wrote (step_impl.h, pro_impl.h).
constexpr int kFlagDem = 8;
// The domains couple fluid and particles by interpolated bounce-back
// (lbm_impl.h); set by the host.
constexpr int kFlagIbb = 16;

// The group takes fluid steps in pairs: launches without fluid blocks run
// k_walk (step_impl.h); set by the host.
constexpr int kFlagPairs = 32;

// With particles, the last positions of an XCD's run hold fluid blocks only: a
// walker block can end with a chain of near-surface evaluations (up to 10-20 us),
// which would otherwise run on alone after the last fluid blocks.  448 is twice the
// blocks of 256 threads an XCD holds at once (32 CUs, 7 blocks), some 12 us of
// fluid.  us per step with the walkers spread over the whole run, and with the
// last 224, 448 and 896 positions left out: 128^3 FP32 channel 65.9, 62.7,
// 61.5, 65.9; 192^3 FP32 bounce-back 297.4, 293.7, 290.9, 291.3; 80^3 FP32
// 26.1, 23.5, 24.0, 24.0; 97x61x83 FP64 41.6, 35.5, 35.7, 35.7; 256^3 within
// 1%.  (Walkers all first, which the smallest grids get: they fit the chip.)
// Without particles there is no such chain, and with more walkers than nodes the
// fluid left for the end is missed beside the walkers: spread and with 448 left
// out, 96^3 FP32 with 3e6 walkers 56.4, 62.5; with 9e5 35.7, 36.4; 128^3 with 2e6
// 77.2, 76.3, with 3e4 55.6, 54.5; 48^3 with 1e5 8.5, 8.1; 256^3 FP16 with 1e5 297,
// 288.
constexpr int kTailBlocks = 448;
constexpr int kFlagTail = 64;  // the launch has particles, or no more walkers than nodes; set by the host

struct DomView;

// One fused step launch over nd domains (kernel argument).
struct StepArgs {
  const DomView* views;
  const int32_t* boff;  // kRoles maps of nd + 1 block prefixes: walkers, prologue, fluid
  int nd;
  int nb[kRoles];       // blocks per role over all domains
  int flags;            // kFlagXcd | kFlagNontemporal | kFlagDensity
  int inplace;          // every domain of the launch streams its lattice in place
  int32_t j;            // launch index within the group (-1: the prologue-only launch)
  int32_t s;            // lattice swaps of the group before this launch (two lattices)
};

// One launch of two fluid steps (pair_impl.h): tiles of tx x ty nodes (the last
// of a row or column may be smaller), ntx x nty of them, each in nzc runs of
// planes.
constexpr int kPairTx = 64, kPairTy = 8;
constexpr int kPairRim = (kPairTx + 2) * (kPairTy + 2);  // nodes of a tile and its rim
constexpr int kPairThreads = 704;                        // whole waves
static_assert(kPairRim <= kPairThreads, "a thread per node");
struct PairArgs {
  int tx, ty, ntx, nty, nzc;
  int dens;   // store the densities of the second step
  int32_t j;  // the first step's offset within the group
  int32_t s;  // lattice swaps of the group before this launch
  int64_t cost;  // pair_shape's
};

// Tiles and runs of planes of an nx x ny x nz lattice: whole tiles (rows of 64
// floats, so that they begin where lines do; the last of a row or column is
// what is left), and the number of runs whose blocks fill the last round of the
// chip best (256 CUs, one block each; a run of m planes walks m + 2).
// cost: block planes walked one after the other on a CU.
inline PairArgs pair_shape(int nx, int ny, int nz) {
  PairArgs a{};
  a.tx = nx < kPairTx ? nx : kPairTx;
  a.ty = ny < kPairTy ? ny : kPairTy;
  a.ntx = (nx + a.tx - 1) / a.tx;
  a.nty = (ny + a.ty - 1) / a.ty;
  a.cost = -1;
  const int64_t tiles = (int64_t)a.ntx * a.nty;
  for (int c = 1; c <= (nz + 3) / 4; ++c) {
    // no larger c can do better once tiles c / 256 rounds of nz / c + 2 planes
    // are as many (a column of 5e7 planes: 260 steps of the search, not 1e7)
    if (a.cost >= 0 && tiles * (nz + 2ll * c) >= 256 * a.cost) break;
    const int64_t rounds = (tiles * c + 255) / 256;
    const int64_t cost = rounds * ((nz + c - 1) / c + 2);
    if (a.cost < 0 || cost < a.cost) {
      a.cost = cost;
      a.nzc = c;
    }
  }
  return a;
}

// Share of XCD x of n items dealt in contiguous runs: count and first item.
RWMI_HD inline int xcd_count(int n, int x) { return (n >> 3) + (x < (n & 7) ? 1 : 0); }
RWMI_HD inline int xcd_first(int n, int x) { return x * (n >> 3) + (x < (n & 7) ? x : (n & 7)); }

// Grid size for nb[role] blocks per role.
RWMI_HD inline int step_grid(const int nb[3], bool xcd) {
  if (!xcd) return nb[0] + nb[1] + nb[2];
  int g = 0;
  for (int x = 0; x < 8; ++x) {
    const int t = xcd_count(nb[0], x) + xcd_count(nb[1], x) + xcd_count(nb[2], x);
    if (t > g) g = t;
  }
  return 8 * g;
}

// Role of hardware block i and its index among the blocks of that role
// (kRoleNone for the padding blocks of the XCD-aware grid).
RWMI_HD inline int step_role(int i, const int nb[3], bool xcd, int& idx, int tail = kTailBlocks) {
  int g = i, cw = nb[0], cp = nb[1], cf = nb[2], bw = 0, bp = 0, bf = 0;
  if (xcd) {
    const int x = i & 7;
    g = i >> 3;
    cw = xcd_count(nb[0], x);
    cp = xcd_count(nb[1], x);
    cf = xcd_count(nb[2], x);
    bw = xcd_first(nb[0], x);
    bp = xcd_first(nb[1], x);
    bf = xcd_first(nb[2], x);
  }
  if (g < cp) {
    idx = bp + g;
    return kRolePro;
  }
  const int h = g - cp, T = cw + cf;
  if (h >= T) return kRoleNone;
  // walker blocks spread evenly over the first S positions: position h < S is
  // a walker block when floor((h+1) cw / S) > floor(h cw / S)
  if (!xcd) tail *= 8;
  const int S = T - tail > cw ? T - tail : cw;
  if (h >= S) {
    idx = bf + (h - cw);
    return kRoleFluid;
  }
  const int wa = (int)(((int64_t)h * cw) / S);
  const int wb = (int)(((int64_t)(h + 1) * cw) / S);
  if (wb > wa) {
    idx = bw + wa;
    return kRoleWalk;
  }
  idx = bf + (h - wa);
  return kRoleFluid;
}

}  // namespace rwmi
