// Walker seeding, occupancy (Eq. 16) and the FP64 moment reductions.
#pragma once
#include "dev_common.h"
#include "lbm_impl.h"
#include "walk_impl.h"

namespace rwmi {

// Seeding at t = 0: walker w tries Philox blocks (w, 0xFFFFFFFF, 16 + a, 0).
// Writes cell, offsets (in the walker precision) and flag[w] = 1 if placed.
template <typename R>
__global__ void k_seed(const DomView* __restrict__ views, int dom, int kind, double cx, double cy, double cz,
                       double sigma, int band_axis, double band_lo, double band_hi, const double* __restrict__ xyz,
                       int64_t n, int attempts, int32_t* __restrict__ cell_out, R* __restrict__ off_out,
                       uint8_t* __restrict__ flag) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= n) return;
  // particle centres at t = 0
  const double centre[3] = {cx, cy, cz};
  bool placed = false;
  int cell[3] = {0, 0, 0};
  double o[3] = {0, 0, 0};
  for (int at = 0; at < attempts && !placed; ++at) {
    double X[3];
    if (kind == 3) {
      X[0] = xyz[3 * w];
      X[1] = xyz[3 * w + 1];
      X[2] = xyz[3 * w + 2];
    } else {
      const U4 r = philox4x32_10((uint32_t)w, 0xFFFFFFFFu, 16u + (uint32_t)at, 0u, V.key0, V.key1);
      if (kind == 1) {
        double z0, z1, z2;
        gauss3(r, z0, z1, z2);
        X[0] = centre[0] + sigma * z0;
        X[1] = centre[1] + sigma * z1;
        X[2] = centre[2] + sigma * z2;
      } else {
        const uint32_t rr[3] = {r.x, r.y, r.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          double lo = V.bc[a] ? 1.0 : 0.0, hi = V.bc[a] ? (double)(V.n[a] - 1) : (double)V.n[a];
          if (kind == 2 && a == band_axis) {
            lo = band_lo;
            hi = band_hi;
          }
          X[a] = lo + unit_open(rr[a]) * (hi - lo);
        }
      }
    }
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double L = (double)V.n[a];
      double x = X[a];
      if (!V.bc[a]) {
        x = x - L * floor(x / L);
        if (x >= L) x = 0.0;
      } else if (x < 1.0 || x >= L - 1.0) {
        ok = false;
      }
      const double k = floor(x);
      cell[a] = (int)k;
      o[a] = (double)(R)(x - k);
    }
    if (!ok) continue;
    // inside a particle at t = 0?
    bool inside = false;
    for (int p = 0; p < V.np && !inside; ++p) {
      const DevParticle& P = V.parts[p];
      double pc[3], pv[3];
      particle_pose(P, 0, pc, pv);
      const double dx = axis_disp<double>(!V.bc[0], V.n[0], cell[0], pc[0], o[0]);
      const double dy = axis_disp<double>(!V.bc[1], V.n[1], cell[1], pc[1], o[1]);
      const double dz = axis_disp<double>(!V.bc[2], V.n[2], cell[2], pc[2], o[2]);
      if ((dx * dx + dy * dy) + dz * dz >= P.maskr * P.maskr) continue;
      // control points as given (seeding happens before the first step, at
      // the initial orientation)
      if (metaball_value<double>(gp(V.ctrl) + 4 * P.ctrl0, P.nc, dx, dy, dz) >= 1.0) inside = true;
    }
    if (inside) continue;
    placed = true;
  }
  flag[w] = placed ? 1 : 0;
  cell_out[w] = (int32_t)lin(V, cell[0], cell[1], cell[2]);
  off_out[w] = (R)o[0];
  off_out[n + w] = (R)o[1];
  off_out[2 * n + w] = (R)o[2];
}

// Scatter the placed walkers (exclusive prefix pos of flag) into the walker
// arrays, keeping their order.
template <typename R>
__global__ void k_seed_scatter(const DomView* __restrict__ views, int dom, int64_t n, const int32_t* __restrict__ cell_in,
                               const R* __restrict__ off_in, const uint8_t* __restrict__ flag,
                               const int32_t* __restrict__ pos, int64_t m) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= n || !flag[w]) return;
  const int64_t k = pos[w];
  R* off = (R*)V.woff;
  V.wcell[k] = cell_in[w];
  off[k] = off_in[w];
  off[m + k] = off_in[n + w];
  off[2 * m + k] = off_in[2 * n + w];
  V.wimg[k] = 0;
  V.wimg[m + k] = 0;
  V.wimg[2 * m + k] = 0;
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_occupancy(const DomView* __restrict__ views, int dom) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w < V.nw)
    __hip_atomic_fetch_add(gp(V.occ) + gp(V.wcell)[w], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- profile
// Concentration profile along one axis (Eq. 16 summed over the two other
// axes): the number of walkers whose cell lies in each layer.  Exact integer
// counts in any order of addition.  Layers up to kProfileLds are counted in
// a block histogram in LDS first, then added to the global counts once per
// block and layer.
constexpr int kProfileLds = 4096;
constexpr int kProfileThreads = 256;
constexpr int kProfilePerThread = 16;

__global__ void __launch_bounds__(kProfileThreads) k_profile(const DomView* __restrict__ views, int dom, int axis,
                                                             uint32_t* __restrict__ counts) {
  __shared__ uint32_t h[kProfileLds];
  const DomView& V = views[dom];
  const int nl = V.n[axis];
  const bool lds = nl <= kProfileLds;
  if (lds)
    for (int i = threadIdx.x; i < nl; i += kProfileThreads) h[i] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kProfileThreads * kProfilePerThread;
  for (int k = 0; k < kProfilePerThread; ++k) {
    const int64_t w = base + (int64_t)k * kProfileThreads + threadIdx.x;
    if (w >= V.nw) break;
    const uint32_t c = (uint32_t)gp(V.wcell)[w];
    const uint32_t q1 = fdiv(c, V.dx);
    uint32_t layer;
    if (axis == 0) layer = c - q1 * (uint32_t)V.n[0];
    else if (axis == 1) layer = q1 - fdiv(q1, V.dy) * (uint32_t)V.n[1];
    else layer = fdiv(q1, V.dy);
    if (lds) __hip_atomic_fetch_add(&h[layer], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_fetch_add(gp(counts) + layer, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (lds)
    for (int i = threadIdx.x; i < nl; i += kProfileThreads)
      if (h[i]) __hip_atomic_fetch_add(gp(counts) + i, h[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- moments
// FP64 reductions whose results do not depend on the launch configuration of
// the stepping kernels, nor on the order of the walkers' slots (which the
// regrouping leaves arbitrary within a bin).
//
// Nodes: chunk k covers nodes [k*4096, (k+1)*4096), one block each; thread j
// of its T threads adds nodes j, j+T, ..., the block's sums are folded in a
// fixed order, and the final kernel adds the chunks the same way.  T is 1024 on
// a small lattice, whose few blocks would leave the chip idle with fewer, and
// 256 on a large one, where a block's other threads wait for the wave that
// culls the particles (launch_moments).
//
// Walkers: every term is rounded to a multiple of 2^-76 and split into three
// integers (ExactSum); the integers' sums are exact, so any order gives the
// same result, and are combined into a double at the end.  Walkers are so read slot by slot,
// coalesced.  In id order (a gather through the id map, 28 scattered bytes a
// walker) the same sums took 1.19 ms for 1e7 walkers, and the map 0.13 ms.
// Displacements whose squares those integers do not hold (2^25.5 lattice units,
// or a reference point that is not finite) or hold in too few bits (2^-11) get
// sums in double, walkers in id order: a read-out with 1e7 walkers then takes
// 1.60 ms instead of 0.26 (in double for all walkers it took 2.83).
constexpr int kRedThreads = 1024;
constexpr int kRedRows = kRedThreads / 16;
constexpr int kRedChunk = 4096;       // nodes per block
constexpr int kWalkChunk = 16384;     // walkers per block
constexpr int kWalkMom = 6;           // sum d[3], sum d^2[3]
constexpr int kWalkWords = 3 * kWalkMom;
constexpr int kNodeMom = 12;          // rho, rho u[3], (1-eps) u[3], (1-eps), eps us[3], eps

// Sum of doubles below 2^51 in magnitude, exact to 2^-76 per term: x = h 2^20
// + m 2^-28 + l 2^-76 with each remainder exact (powers of two only), |h| <=
// 2^31, |m|, |l| <= 2^47.  `carry` brings m and l back to those ranges, so that
// 2^15 terms, or 2^15 carried sums, fit in 64 bits; the h of 2^31 terms always
// do.  A square of 2^-22 or more (a displacement of 5e-4) keeps all its bits,
// so a sum of squares of at least kExactMin per walker is held to half of
// its last place, and the sum of the displacements far better.  (With the last
// digit at 2^-59, 1000 squares of displacements of 1e-6 were off by 1e-8 of
// their sum.  A fourth digit instead of sums in double for such displacements:
// 101 us for 1e7 walkers, with three 85.)
constexpr double kExactMax = 0x1p51;
struct ExactSum {
  long long h = 0, m = 0, l = 0;
  // the nearest integer to t (|t| < 2^51) as the low bits of t + 1.5 2^52
  static __device__ __forceinline__ long long digit(double& t) {
    constexpr double magic = 0x1.8p52;
    const double s = t + magic;
    t = s - magic;
    return __double_as_longlong(s) - __double_as_longlong(magic);
  }
  __device__ __forceinline__ void add(double x) {
    double t = x * 0x1p-20;
    h += digit(t);
    x = x - t * 0x1p20;
    t = x * 0x1p28;
    m += digit(t);
    x = x - t * 0x1p-28;
    t = x * 0x1p76;
    l += digit(t);
  }
  __device__ __forceinline__ void carry() {
    const long long c = (l + (1ll << 47)) >> 48;
    l -= c << 48;
    m += c;
    const long long d = (m + (1ll << 47)) >> 48;
    m -= d << 48;
    h += d;
  }
  __device__ __forceinline__ double value() {
    carry();
    return (double)h * 0x1p20 + ((double)m * 0x1p-28 + (double)l * 0x1p-76);
  }
};

// Value of the lane N places on, around the row of 16 lanes.
template <int N, typename T>
__device__ __forceinline__ T row_ror(T v) {
  static_assert(sizeof(T) == 8, "two words");
  union { T t; int i[2]; } x;
  x.t = v;
#pragma unroll
  for (int k = 0; k < 2; ++k) x.i[k] = __builtin_amdgcn_update_dpp(0, x.i[k], 0x120 + N, 0xf, 0xf, true);
  return x.t;
}
template <typename T>
__device__ __forceinline__ T row_sum(T v) {
  v = v + row_ror<8>(v);
  v = v + row_ror<4>(v);
  v = v + row_ror<2>(v);
  return v + row_ror<1>(v);
}

// Sums over the block of acc[0..K) of every thread, in thread 16 k for k < K.
// The order is fixed: each row of 16 lanes through the DPP network, the rows'
// sums through LDS, thread 16 k + i adding rows i, i + 16, ..., then their row.
template <int THREADS, typename T, int K>
__device__ __forceinline__ T block_sum(T (&acc)[K], T (*sh)[K]) {
  static_assert(16 * K <= THREADS, "a row per sum");
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = row_sum(acc[k]);
  const int tid = threadIdx.x;
  if ((tid & 15) == 0)
#pragma unroll
    for (int k = 0; k < K; ++k) sh[tid >> 4][k] = acc[k];
  __syncthreads();
  T s = (T)0;
  if (tid < 16 * K) {
#pragma unroll
    for (int r = 0; r < THREADS / 256; ++r) s = s + sh[(tid & 15) + 16 * r][tid >> 4];
    s = row_sum(s);
  }
  __syncthreads();
  return s;
}

struct MomRef {
  double x[3];
};

// part[chunk][3 k + digit]: the chunk's carried sums.  range[0] is set where a
// term is beyond ExactSum's range (or is not finite), range[1] where a square is
// below its last digit and not zero.
template <typename R>
__global__ void __launch_bounds__(kRedThreads) k_mom_walkers(const DomView* __restrict__ views, int dom, MomRef ref,
                                                             long long* __restrict__ part, double* __restrict__ range) {
  __shared__ long long sh[kRedRows][kWalkWords];
  const DomView& V = views[dom];
  const auto off = gp((const R*)V.woff);
  const auto img = gp((const int32_t*)V.wimg);
  const auto cell = gp((const int32_t*)V.wcell);
  const int64_t nw = V.nw, base = (int64_t)blockIdx.x * kWalkChunk;
  ExactSum sum[kWalkMom];
  bool beyond = false, below = false;
#pragma unroll 4
  for (int j = 0; j < kWalkChunk / kRedThreads; ++j) {
    const int64_t w = base + (int64_t)j * kRedThreads + threadIdx.x;
    if (w >= nw) break;
    const uint32_t lc = (uint32_t)cell[w];
    const uint32_t q1 = fdiv(lc, V.dx);
    const int cz = (int)fdiv(q1, V.dy);
    const int c[3] = {(int)(lc - q1 * (uint32_t)V.n[0]), (int)q1 - cz * V.n[1], cz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int64_t X = (int64_t)c[a] + (int64_t)img[a * nw + w] * (int64_t)V.n[a];
      const double dv = ((double)X - ref.x[a]) + (double)off[a * nw + w];
      beyond |= !(dv * dv < kExactMax);
      below |= dv != 0.0 && dv * dv < 0x1p-76;
      sum[a].add(dv);
      sum[3 + a].add(dv * dv);
    }
  }
  if (beyond) range[0] = 1.0;  // by as many threads as find it
  if (below) range[1] = 1.0;
  long long acc[kWalkWords];
#pragma unroll
  for (int k = 0; k < kWalkMom; ++k) {
    acc[3 * k] = sum[k].h;
    acc[3 * k + 1] = sum[k].m;
    acc[3 * k + 2] = sum[k].l;
  }
  const long long s = block_sum<kRedThreads>(acc, sh);
  if ((threadIdx.x & 15) == 0 && threadIdx.x < 16 * kWalkWords) sh[0][threadIdx.x >> 4] = s;
  __syncthreads();
  if (threadIdx.x < kWalkMom) {
    ExactSum e;
    e.h = sh[0][3 * threadIdx.x];
    e.m = sh[0][3 * threadIdx.x + 1];
    e.l = sh[0][3 * threadIdx.x + 2];
    e.carry();
    long long* o = part + (int64_t)blockIdx.x * kWalkWords + 3 * threadIdx.x;
    o[0] = e.h;
    o[1] = e.m;
    o[2] = e.l;
  }
}

// The same sums added in double, in an order of the walkers' ids that is fixed:
// for displacements whose squares ExactSum does not hold, or holds badly.  cell, off, img: the
// walkers in id order (k_read_walkers).  Thread j adds walkers j, j + 256, ...
// of its block's chunk, the block folds by halves, k_mom_by_id_final adds the
// chunks in turn.
constexpr int kIdThreads = 256;
template <typename R>
__global__ void __launch_bounds__(kIdThreads) k_mom_walkers_by_id(const DomView* __restrict__ views, int dom,
                                                                  MomRef ref, const int32_t* __restrict__ cell,
                                                                  const R* __restrict__ off,
                                                                  const int32_t* __restrict__ img,
                                                                  double* __restrict__ part) {
  __shared__ double sh[kWalkMom][kIdThreads];
  const DomView& V = views[dom];
  const int64_t nw = V.nw, base = (int64_t)blockIdx.x * kRedChunk;
  const int tid = threadIdx.x;
  double acc[kWalkMom] = {0, 0, 0, 0, 0, 0};
  for (int j = tid; j < kRedChunk; j += kIdThreads) {
    const int64_t w = base + j;
    if (w >= nw) break;
    const uint32_t lc = (uint32_t)gp(cell)[w];
    const uint32_t q1 = fdiv(lc, V.dx);
    const int cz = (int)fdiv(q1, V.dy);
    const int c[3] = {(int)(lc - q1 * (uint32_t)V.n[0]), (int)q1 - cz * V.n[1], cz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int64_t X = (int64_t)c[a] + (int64_t)gp(img)[a * nw + w] * (int64_t)V.n[a];
      const double dv = ((double)X - ref.x[a]) + (double)gp(off)[a * nw + w];
      acc[a] = acc[a] + dv;
      acc[3 + a] = acc[3 + a] + dv * dv;
    }
  }
#pragma unroll
  for (int k = 0; k < kWalkMom; ++k) sh[k][tid] = acc[k];
  __syncthreads();
  for (int h = kIdThreads / 2; h > 0; h >>= 1) {
    if (tid < h) {
#pragma unroll
      for (int k = 0; k < kWalkMom; ++k) sh[k][tid] = sh[k][tid] + sh[k][tid + h];
    }
    __syncthreads();
  }
  if (tid < kWalkMom) part[(int64_t)blockIdx.x * kWalkMom + tid] = sh[tid][0];
}

__global__ void __launch_bounds__(64) k_mom_by_id_final(const double* __restrict__ part, int64_t chunks,
                                                        double* __restrict__ out) {
  const int tid = threadIdx.x;
  if (tid >= kWalkMom) return;
  double s = 0.0;
  for (int64_t b = 0; b < chunks; ++b) s = s + gp(part)[b * kWalkMom + tid];
  out[tid] = s;
}

// range[0..1] is cleared for the walkers' kernel, which runs after this one.
template <typename U, int THREADS>
__global__ void __launch_bounds__(THREADS) k_mom_nodes(const DomView* __restrict__ views, int dom,
                                                       double* __restrict__ part, double* __restrict__ range) {
  __shared__ double sh[THREADS / 16][kNodeMom];
  using C = typename Store<sizeof(U) == 8 ? P64 : P32>::C;
  __shared__ BlockParticles<C> sp;
  const DomView& V = views[dom];
  const uint32_t N = (uint32_t)V.N;
  if (blockIdx.x == 0 && threadIdx.x < 2) range[threadIdx.x] = 0.0;
  const uint32_t base = blockIdx.x * (uint32_t)kRedChunk;
  const uint32_t last = base + kRedChunk - 1 < N ? base + kRedChunk - 1 : N - 1;
  const uint64_t done = V.tstep[0];  // steps completed
  const bool stepped = done > 0;
  // the poses of the last step are still in the table its prologue (or, for
  // coupled particles, the particle update) wrote
  if (stepped && V.np > 0 && !V.ibb) cull_block<C>(V, base, last, done - 1, sp);
  else if (threadIdx.x == 0) sp.cnt = 0;
  __syncthreads();
  double acc[kNodeMom];
#pragma unroll
  for (int k = 0; k < kNodeMom; ++k) acc[k] = 0.0;
  const auto uf = gp((const U*)V.u[stepped ? ((done - 1) & 1ull) : 0]);
  const auto rf = gp((const U*)V.rho);
  for (int j = 0; j < kRedChunk / THREADS; ++j) {
    const uint32_t id = base + (uint32_t)j * THREADS + threadIdx.x;
    if (id >= N) break;
    const uint32_t q1 = fdiv(id, V.dx);
    const int z = (int)fdiv(q1, V.dy);
    const int nd[3] = {(int)(id - q1 * (uint32_t)V.n[0]), (int)q1 - z * V.n[1], z};
    bool wall = false;
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (V.bc[a] && (nd[a] == 0 || nd[a] == V.n[a] - 1)) wall = true;
    if (wall) continue;
    const double u[3] = {(double)uf[3ull * id], (double)uf[3ull * id + 1], (double)uf[3ull * id + 2]};
    const double r = (double)rf[id];
    double es = 0.0, un[3] = {0.0, 0.0, 0.0};
    if (V.ibb) {
      // interpolated bounce-back: a node is solid or fluid; a solid node's
      // stored velocity is its particle's rigid velocity
      if (stepped && (V.smap[(done - 1) & 1ull][id] & kSolidBits)) {
        es = 1.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) un[a] = u[a];
      }
    } else
    for (int k = 0; k < sp.cnt; ++k) {
      C dl[3];
      const double e = (double)node_eps<C>(V, sp, k, nd, dl);
      es = es + e;
      double up[3] = {sp.v[k][0], sp.v[k][1], sp.v[k][2]};
      if (((V.dem_mask >> sp.id[k]) & 1ull) && e > 0.0) {
        const double dd[3] = {(double)dl[0], (double)dl[1], (double)dl[2]};
        rigid_velocity<double>(sp.w[k], dd, up);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) un[a] = un[a] + e * up[a];
    }
    const double eps = es < 1.0 ? es : 1.0;
    acc[0] = acc[0] + r;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double usa = es > 0.0 ? un[a] / es : 0.0;
      acc[1 + a] = acc[1 + a] + r * u[a];
      acc[4 + a] = acc[4 + a] + (1.0 - eps) * u[a];
      acc[8 + a] = acc[8 + a] + eps * usa;
    }
    acc[7] = acc[7] + (1.0 - eps);
    acc[11] = acc[11] + eps;
  }
  const double s = block_sum<THREADS>(acc, sh);
  if ((threadIdx.x & 15) == 0 && threadIdx.x < 16 * kNodeMom)
    part[(int64_t)blockIdx.x * kNodeMom + (threadIdx.x >> 4)] = s;
}

// out: [0..5] walker sums, [6..17] node sums, [18..25] counters, [26] step, and
// range (kMomRange), which the other kernels write.
// One block; one thread adding the chunks in turn took 1.2 ms for the 4096
// chunks of a 256^3 lattice.
__global__ void __launch_bounds__(kRedThreads) k_mom_final(const DomView* __restrict__ views, int dom,
                                                           const long long* __restrict__ pw, int64_t nbw,
                                                           const double* __restrict__ pn, int64_t nbn,
                                                           double* __restrict__ out) {
  __shared__ long long shw[kRedRows][kWalkWords];
  __shared__ double shn[kRedRows][kNodeMom];
  const DomView& V = views[dom];
  const int tid = threadIdx.x;
  long long aw[kWalkWords];
#pragma unroll
  for (int k = 0; k < kWalkWords; ++k) aw[k] = 0;
  for (int64_t b = tid; b < nbw; b += kRedThreads)
#pragma unroll
    for (int k = 0; k < kWalkWords; ++k) aw[k] += gp(pw)[b * kWalkWords + k];
  // up to 2^7 chunks a thread, 2^10 threads: carried in between
#pragma unroll
  for (int k = 0; k < kWalkMom; ++k) {
    ExactSum e;
    e.h = aw[3 * k];
    e.m = aw[3 * k + 1];
    e.l = aw[3 * k + 2];
    e.carry();
    aw[3 * k] = e.h;
    aw[3 * k + 1] = e.m;
    aw[3 * k + 2] = e.l;
  }
  double an[kNodeMom];
#pragma unroll
  for (int k = 0; k < kNodeMom; ++k) an[k] = 0.0;
  for (int64_t b = tid; b < nbn; b += kRedThreads)
#pragma unroll
    for (int k = 0; k < kNodeMom; ++k) an[k] = an[k] + gp(pn)[b * kNodeMom + k];
  const long long sw = block_sum<kRedThreads>(aw, shw);
  if ((tid & 15) == 0 && tid < 16 * kWalkWords) shw[0][tid >> 4] = sw;
  const double sn = block_sum<kRedThreads>(an, shn);
  if ((tid & 15) == 0 && tid < 16 * kNodeMom) out[kWalkMom + (tid >> 4)] = sn;
  __syncthreads();
  if (tid < kWalkMom) {
    ExactSum e;
    e.h = shw[0][3 * tid];
    e.m = shw[0][3 * tid + 1];
    e.l = shw[0][3 * tid + 2];
    out[tid] = e.value();
  } else if (tid >= 64 && tid < 64 + kCounters) {
    out[kWalkMom + kNodeMom + tid - 64] = __longlong_as_double((long long)V.counters[tid - 64]);
  } else if (tid == 64 + kCounters) {
    out[kWalkMom + kNodeMom + kCounters] = __longlong_as_double((long long)V.tstep[0]);
  }
}

// End of a launch group: every domain of the launch has completed n more
// steps, and swapped its two lattices (if it has two) `swaps` times.
__global__ void k_advance(const DomView* __restrict__ views, int nd_count, uint32_t n, uint32_t swaps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nd_count) {
    views[i].tstep[0] += n;
    views[i].tstep[1] += swaps;
  }
}

__global__ void k_normals(uint32_t k0, uint32_t k1, uint32_t t, uint32_t purpose, int64_t n, double* __restrict__ z) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const U4 r = philox4x32_10((uint32_t)i, t, purpose, 0u, k0, k1);
  double a, b, c;
  gauss3(r, a, b, c);
  z[3 * i] = a;
  z[3 * i + 1] = b;
  z[3 * i + 2] = c;
}

// ---------------------------------------------------------------- walker sort
// Walkers are kept grouped by coarse mask block (4^3 nodes) so that the
// walkers of a wavefront gather neighbouring velocities and share mask words.
// A counting sort: rank within the block's bin (wave-aggregated atomics, so
// the order inside a bin is arbitrary), exclusive scan of the bin counts,
// scatter to scratch, copy back.  Every result of the library is independent
// of the slot order (walker ids travel with the walkers; read-outs put them in
// id order and moment sums are the same in any), so the arbitrary order inside a
// bin changes nothing.

__device__ __forceinline__ uint32_t walker_bin(const DomView& V, int32_t cell) {
  const uint32_t lc = (uint32_t)cell;
  const uint32_t q1 = fdiv(lc, V.dx);
  const uint32_t z = fdiv(q1, V.dy);
  const uint32_t y = q1 - z * (uint32_t)V.n[1];
  const uint32_t x = lc - q1 * (uint32_t)V.n[0];
  return x / kMaskBlock + (uint32_t)V.mb[0] * (y / kMaskBlock + (uint32_t)V.mb[1] * (z / kMaskBlock));
}

// Every bin has kSortCopies counters, stored copy-major (counter copy * nbins
// + bin, so the copies of a bin sit in different cache lines); a block uses
// copy blockIdx mod kSortCopies, so that the walkers of a dense bin do not
// all queue on one address.  The starts are then taken bin by bin: bin totals,
// exclusive scan over the bins, then the copies of each bin in order.
constexpr int kSortCopies = 16;

// bin[w] (its counter) and rank[w] (position among the walkers of that
// counter); hist[counter] ends as the count.
__global__ void k_sort_rank(const DomView* __restrict__ views, int dom, uint32_t* __restrict__ hist,
                            uint32_t* __restrict__ bin, uint32_t* __restrict__ rank) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = w < V.nw;
  const uint32_t nbins = (uint32_t)V.mb[0] * (uint32_t)V.mb[1] * (uint32_t)V.mb[2];
  const uint32_t key = active ? (uint32_t)(blockIdx.x % kSortCopies) * nbins + walker_bin(V, gp(V.wcell)[w]) : 0u;
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(active);
  uint32_t r = 0;
  while (todo) {
    // the lowest pending lane's key: one atomic for all lanes holding it
    const int leader = __ffsll((long long)todo) - 1;
    const uint32_t k = __shfl(key, leader);
    const unsigned long long same = __ballot(active && key == k) & todo;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(&hist[k], (uint32_t)__popcll(same));
    base = __shfl(base, leader);
    if ((same >> lane) & 1ull) r = base + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    todo &= ~same;
  }
  if (active) {
    gp(bin)[w] = key;
    gp(rank)[w] = r;
  }
}

// Exclusive scan of n counts in place: tiles of kScanTile counts scanned by
// one block each (every thread a contiguous run of 4, loaded and stored
// coalesced), the tile sums scanned by one block, then added to the tiles.
constexpr int kScanThreads = 1024;
constexpr int kScanTile = 4 * kScanThreads;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s, uint32_t& total) {
  const int tid = threadIdx.x;
  s[tid] = v;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {  // Hillis-Steele inclusive scan
    const uint32_t u = tid >= o ? s[tid - o] : 0u;
    __syncthreads();
    s[tid] += u;
    __syncthreads();
  }
  total = s[kScanThreads - 1];
  return s[tid] - v;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_tiles(uint32_t* __restrict__ a, int64_t n,
                                                             uint32_t* __restrict__ tsum) {
  __shared__ uint32_t s[kScanThreads];
  const int64_t i0 = (int64_t)blockIdx.x * kScanTile + 4 * threadIdx.x;
  const auto g = gp(a);
  uint32_t v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = i0 + k < n ? g[i0 + k] : 0u;
  uint32_t total;
  uint32_t run = block_exclusive_scan((v[0] + v[1]) + (v[2] + v[3]), s, total);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (i0 + k < n) g[i0 + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) gp(tsum)[blockIdx.x] = total;
}

// Exclusive scan of m <= kScanThreads * 64 tile sums, one block.
__global__ void __launch_bounds__(kScanThreads) k_scan_sums(uint32_t* __restrict__ t, int64_t m) {
  __shared__ uint32_t s[kScanThreads];
  const int64_t per = (m + kScanThreads - 1) / kScanThreads;
  const int64_t b = threadIdx.x * per, e = (b + per < m) ? b + per : m;
  uint32_t sum = 0;
  for (int64_t i = b; i < e; ++i) sum += t[i];
  uint32_t total;
  uint32_t run = block_exclusive_scan(sum, s, total);
  for (int64_t i = b; i < e; ++i) {
    const uint32_t c = t[i];
    t[i] = run;
    run += c;
  }
}

__global__ void k_scan_add(uint32_t* __restrict__ a, int64_t n, const uint32_t* __restrict__ tsum) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) gp(a)[i] += gp(tsum)[i / kScanTile];
}

// total[b] = sum over the copies of bin b.
__global__ void k_bin_totals(const uint32_t* __restrict__ cnt, int64_t nbins, uint32_t* __restrict__ total) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  uint32_t s = 0;
#pragma unroll
  for (int c = 0; c < kSortCopies; ++c) s += gp(cnt)[c * nbins + b];
  gp(total)[b] = s;
}

// Counts of the copies of bin b become their starts, from the bin's start.
__global__ void k_bin_starts(uint32_t* __restrict__ cnt, int64_t nbins, const uint32_t* __restrict__ start) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  uint32_t run = gp(start)[b];
#pragma unroll
  for (int c = 0; c < kSortCopies; ++c) {
    const uint32_t k = gp(cnt)[c * nbins + b];
    gp(cnt)[c * nbins + b] = run;
    run += k;
  }
}

// Scatter every walker to slot start[bin] + rank in the scratch arrays.
template <typename R>
__global__ void k_sort_scatter(const DomView* __restrict__ views, int dom, const uint32_t* __restrict__ start,
                               const uint32_t* __restrict__ bin, const uint32_t* __restrict__ rank,
                               int32_t* __restrict__ cell2, R* __restrict__ off2, int32_t* __restrict__ img2,
                               int32_t* __restrict__ wid2) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= V.nw) return;
  const int64_t nw = V.nw;
  const int64_t d = (int64_t)gp(start)[gp(bin)[w]] + gp(rank)[w];
  gp(cell2)[d] = gp(V.wcell)[w];
  gp(wid2)[d] = gp(V.wid)[w];
  const auto off = gp((const R*)V.woff);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gp(off2)[a * nw + d] = off[a * nw + w];
    gp(img2)[a * nw + d] = gp(V.wimg)[a * nw + w];
  }
}

// Copy the sorted scratch back.
template <typename R>
__global__ void k_sort_back(const DomView* __restrict__ views, int dom, const int32_t* __restrict__ cell2,
                            const R* __restrict__ off2, const int32_t* __restrict__ img2,
                            const int32_t* __restrict__ wid2) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= V.nw) return;
  const int64_t nw = V.nw;
  gp(V.wcell)[w] = gp(cell2)[w];
  gp(V.wid)[w] = gp(wid2)[w];
  const auto off = gp((R*)V.woff);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    off[a * nw + w] = gp(off2)[a * nw + w];
    gp(V.wimg)[a * nw + w] = gp(img2)[a * nw + w];
  }
}

// Slot i holds walker i (after seeding).
__global__ void k_ids_identity(const DomView* __restrict__ views, int dom) {
  const DomView& V = views[dom];
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= V.nw) return;
  gp(V.wid)[w] = (int32_t)w;
}

// The walkers in id order, for a read-out, in the sort's scratch (free between
// launches, so that a read-out allocates nothing on the device).  An id out of
// range (a corrupt map) sets *bad, which starts at zero.  Scattered by one host
// thread they took 23 of the 25 ms of a read-out of 1e6 walkers.
template <typename R>
__global__ void __launch_bounds__(256) k_read_walkers(const DomView* __restrict__ views, int dom,
                                                      int32_t* __restrict__ cell, R* __restrict__ off,
                                                      int32_t* __restrict__ img, uint32_t* __restrict__ bad) {
  const DomView& V = views[dom];
  const int64_t nw = V.nw, w = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (w >= nw) return;
  const uint32_t id = (uint32_t)gp(V.wid)[w];
  if (id >= (uint64_t)nw) {
    gp(bad)[0] = 1u;
    return;
  }
  gp(cell)[id] = gp(V.wcell)[w];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gp(off)[a * nw + id] = gp((const R*)V.woff)[a * nw + w];
    gp(img)[a * nw + id] = gp(V.wimg)[a * nw + w];
  }
}

}  // namespace rwmi
