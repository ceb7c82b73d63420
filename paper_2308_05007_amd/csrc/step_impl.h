// The fused step launch: walker blocks of step t-1, fluid blocks of step t
// and prologue blocks of step t+1 in one grid (roles from step_map.h), t being
// the domain's step counter at the start of the launch group plus the launch
// index j.  A group of n steps is a prologue-only launch (j = -1, prologue of
// t0) and then launches j = 0..n: fluid of t0 + j (j < n), prologue of
// t0 + j + 1 (j < n - 1), walkers of t0 + j - 1 (j >= 1).
//
// No role reads what another role of the same launch writes.  The fluid of
// step t reads f of parity t & 1, the poses of slot t mod 3 and writes f, u of
// parity (t + 1) & 1 and t & 1 (and, on the group's last fluid step, the
// densities, which no role reads); the walkers of step t - 1 read u of parity
// (t - 1) & 1 and the poses/mask of slot (t - 1) mod 3; the prologue writes
// slot (t + 1) mod 3.
#pragma once
#include "lbm_impl.h"
#include "pro_impl.h"
#include "step_map.h"
#include "walk_impl.h"

namespace rwmi {

template <int P, int BS>
union StepLds {
  WalkLds<typename Store<P>::O, BS> walk;
  ProLds pro;
  unsigned long long dem[6 * kMaxParticles];  // fluid blocks with coupled particles
};

// IP: the domains of the launch stream their lattice in place (else: two
// lattices); one instantiation per layout keeps each kernel's registers to
// the paths it can take.
#ifndef RWMI_STEP_WAVES_PER_EU_32
#define RWMI_STEP_WAVES_PER_EU_32 6
#endif
#ifndef RWMI_STEP_WAVES_PER_EU_64
#define RWMI_STEP_WAVES_PER_EU_64 4
#endif
#ifndef RWMI_STEP_WAVES_PER_EU_16
#define RWMI_STEP_WAVES_PER_EU_16 8
#endif
// Waves per SIMD the register allocation must leave room for.  FP32 storage: 6
// (78 VGPRs, no spill); 7 (72, 2 spilled) runs most lattices within 1% of it, 160^3
// with 6e6 walkers in 238 us instead of 233.  16-bit storage: 8, 256^3 413 us
// against 431 at 6.  FP64: 4 (128 VGPRs, 2 spilled); the near-surface rows would
// take 138, those of coupled particles 169, which leaves 3 and 2 waves: 64^3 with
// 1e6 walkers 46.4 us instead of 43.9, coupled particles (120x120x180, 1e6 walkers)
// 294.8 instead of 261.2; the smallest lattices the other way, 32^3 16.2, 16.6.
template <int P, bool IBB = false>
constexpr int step_waves_per_eu() {
  return P == P64 ? RWMI_STEP_WAVES_PER_EU_64 : (P == P32 ? RWMI_STEP_WAVES_PER_EU_32 : RWMI_STEP_WAVES_PER_EU_16);
}

// A launch without fluid blocks of a group that takes fluid steps in pairs (FP32):
// walkers and prologue at 8 waves per SIMD, 142 us for 1e7 walkers.  8 waves leave
// the near-surface rows 13 spilled registers and share the L1 among more walkers,
// so they gain where walkers are dense (the band of the oscillator) and lose where
// they are spread.  us per step of the 256^3 oscillator, 6 waves (k_step) and 8:
// 1e7 walkers in the band 505, 488, without particles 434, 423, with 100 times the
// diffusivity 727, 761; 2e7 667, 632; 1e7 uniform in the box 533, 536; 5e6 460, 468.
// Such launches of other groups (calls of one step, the coupled particles'
// prologue) stay with k_step: 80^3 FP32 40.2, 42.3; 160x96x120 84.8, 88.0; 256^3
// with 5e6 walkers 670, 688; 48^3 FP16 32.0 both; coupled particles in calls of
// many steps 171.6, 173.0.
#ifndef RWMI_WALK_WAVES
#define RWMI_WALK_WAVES 8
#endif
template <int BS>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(RWMI_WALK_WAVES)))
k_walk(StepArgs a, const DomView* __restrict__ views, const int32_t* __restrict__ boff) {
  __shared__ union {
    WalkLds<typename Store<P32>::O, BS> walk;
    ProLds pro;
  } lds;
  int idx = 0;
  const int role = step_role((int)blockIdx.x, a.nb, (a.flags & kFlagXcd) != 0, idx);
  if (role == kRoleNone) return;
  const int32_t* bo = boff + role * (a.nd + 1);
  const int d = find_domain(bo, a.nd, idx);
  const DomView& V = views[d];
  const int lb = idx - bo[d];
  const uint64_t t = step_of(V, a.j);
  if (role == kRoleWalk) walk_block<P32, BS>(V, lb, t - 1, lds.walk);
  else prologue_block(V, lb, t + 1, BS, lds.pro, (a.flags & kFlagDem) != 0);
}

// DEM: the launch's domains have two-way coupled particles (the fluid
// blocks accumulate the hydrodynamic force and torque on them).  IBB: they
// couple fluid and particles by interpolated bounce-back (two lattices).
template <int P, int BS, bool IP, bool DEM = false, bool IBB = false>
__global__ void __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(step_waves_per_eu<P, IBB>())))
k_step(StepArgs a, const DomView* __restrict__ views, const int32_t* __restrict__ boff) {
  // views and boff (the same pointers as in a) are read-only in the launch:
  // as restrict parameters their wave-uniform reads compile to scalar loads
  __shared__ StepLds<P, BS> lds;
  int idx = 0;
  const int role = step_role((int)blockIdx.x, a.nb, (a.flags & kFlagXcd) != 0, idx,
                             (a.flags & kFlagTail) != 0 ? kTailBlocks : 0);
  if (role == kRoleNone) return;
  const int32_t* bo = boff + role * (a.nd + 1);
  const int d = find_domain(bo, a.nd, idx);
  const DomView& V = views[d];
  const int lb = idx - bo[d];
  const uint64_t t = step_of(V, a.j);
  if (role == kRoleWalk) walk_block<P, BS>(V, lb, t - 1, lds.walk);
  else if (role == kRolePro) prologue_block(V, lb, t + 1, BS, lds.pro, (a.flags & kFlagDem) != 0);
  else {
    const bool nt = (a.flags & kFlagNontemporal) != 0, dens = (a.flags & kFlagDensity) != 0;
    if constexpr (!IP) {
      const bool lat = source_lattice(V, a.s);
      fluid_block<P, BS, kTwoLattices, DEM, IBB>(V, (uint32_t)lb, t, lat, nt, dens, lds.dem);
    } else if (t & 1ull) {
      fluid_block<P, BS, kInPlaceOdd, DEM>(V, (uint32_t)lb, t, false, nt, dens, lds.dem);
    } else {
      fluid_block<P, BS, kInPlaceEven, DEM>(V, (uint32_t)lb, t, false, nt, dens, lds.dem);
    }
  }
}

}  // namespace rwmi
