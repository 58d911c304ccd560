// Whole-track transport with one lane per track, persistent over the batch
// (Sec. III.A: a particle is stepped, volume after volume, until it leaves the
// geometry).
//
// The basket regrouping of gv_baskets.h keeps a wavefront's tracks in one
// logical volume by moving 16 bytes of indices per track and step and a
// 64-byte record through HBM.  With the daughter indexes of gv_step.h a step
// evaluates one or two daughter distances in any volume, so the divergence
// the regrouping avoids has become cheaper than the traffic it costs.  The
// form here keeps each track's state in registers for its whole life:
//
//  * coherent order -- the tracks are counting-sorted once by a direction
//    key (the octahedral map of the direction cut into 2^h x 2^h cells,
//    numbered along a Morton curve).  Straight tracks leaving a common region
//    in neighbouring directions cross the same volumes in the same order, so
//    the 64 lanes of a wavefront mostly run the same branch of the step and
//    read the same table entries.  The order changes no result: every track's
//    arithmetic is its own.
//  * persistent workers -- as many workgroups as the device holds at once;
//    each wavefront takes 64 consecutive places of the order from an atomic
//    counter and steps its tracks to the end, then takes the next 64.  The
//    64 tracks of a wavefront start together, so every step is taken by all
//    of its live lanes at once.  (Giving a lane whose track has ended a new
//    track at once was measured 2x slower: the lanes then run different
//    volume classes at every step.)
//
// Every output row is written by the lane that owns the track, so the results
// (sequences, lengths, counts, flags) are independent of the order and the
// grid.
#pragma once
#include "gv_step.h"

namespace gv {

constexpr int kSortMaxBits = 7;  // at most 2^7 x 2^7 direction cells
constexpr int kSortMaxCells = 1 << (2 * kSortMaxBits);

// Interleaves the low 7 bits of x with zeros (bit b to bit 2b).
__device__ __forceinline__ uint32_t spread_bits7(uint32_t x) {
  x &= 0x7Fu;
  x = (x | (x << 4)) & 0x0F0Fu;
  x = (x | (x << 2)) & 0x3333u;
  x = (x | (x << 1)) & 0x5555u;
  return x;
}

// Direction key: the octahedral map of the direction onto [-1, 1]^2 (the
// lower hemisphere folded over the diagonals), cut into 2^h x 2^h cells and
// numbered in Morton order, so that consecutive keys are neighbouring cones.
// Only the order of the work depends on it.
__device__ __forceinline__ uint32_t direction_key(double dx, double dy, double dz, int h) {
  const double a = fabs(dx) + fabs(dy) + fabs(dz);
  double u = dx / a, v = dy / a;
  if (dz < 0.0) {
    const double uu = (1.0 - fabs(v)) * (u < 0.0 ? -1.0 : 1.0), vv = (1.0 - fabs(u)) * (v < 0.0 ? -1.0 : 1.0);
    u = uu;
    v = vv;
  }
  const int side = 1 << h, m = side - 1;
  // a NaN converts to some integer, clamped into the grid: order only
  const uint32_t iu = (uint32_t)min(m, max(0, (int)((u + 1.0) * (0.5 * side))));
  const uint32_t iv = (uint32_t)min(m, max(0, (int)((v + 1.0) * (0.5 * side))));
  return spread_bits7(iu) | (spread_bits7(iv) << 1);
}

// Direction key aligned with the z axis: cos(theta) = dz cut into 2^h
// equal-area bands, the azimuth (pseudo-angle of (dx, dy)) into 2^h sectors,
// bands outermost, so that consecutive keys share a band and neighbouring
// azimuths -- the symmetry of detectors built around the z axis (layers in r,
// modules in phi).  Only the order of the work depends on it.
__device__ __forceinline__ uint32_t direction_key_zaxis(double dx, double dy, double dz, int h) {
  const int side = 1 << h, m = side - 1;
  const uint32_t it = (uint32_t)min(m, max(0, (int)((dz + 1.0) * (0.5 * side))));
  const uint32_t ip = (uint32_t)min(m, max(0, (int)(pseudo_angle(dx, dy) * (0.25 * side))));
  return it << h | ip;
}

// Lane-transport control words (device workspace): cnt[cells] key counts,
// then the running place of each cell during the scatter, and the work
// counter the persistent workers take places from.
struct LaneCtl {
  int32_t* pv0;     // [n] start volume of each track, where the caller gives none
  uint32_t* key;    // [n] direction key of each track
  int32_t* perm;    // [n] track of each place in the coherent order
  uint32_t* cnt;    // [cells] tracks per key
  uint32_t* queue;  // [1] next place to hand out
};

// Geometries with composites: tracks start in several volumes, and a step in
// one that is a composite or holds one costs what the few daughters on its way
// cost (a polycone minus a cone takes 20 us of a wavefront's time).  So the
// tracks are ordered by start volume, then by what their first step will
// evaluate, then by direction, and in each iteration the lanes of one such
// volume step together (8 % of lanes active per VALU instruction without the
// bins, 23 % with them; 500,009 tracks: 990 and 617 us when the bins came;
// basket form 1,867 us, most of it 128 step launches for tracks that take 1.7
// steps).  The volumes that neither are nor hold composites share one start
// group and the step classes of other geometries: with a class and a group for
// each, a detector holding one composite kept 2 x 2 direction cells and stepped
// one layer at a time.
//
// Start group of a track: its LV's first, and in an LV that has several (its
// daughters are found by their boxes) one more than twice the daughter whose box
// it enters first, and whether it enters more than one (0: no daughter box on
// its way).
constexpr int kStartBoxes = 15;  // daughters that have groups of their own
__device__ __forceinline__ uint32_t start_group(const DevGeom& G, int pv, V3 p, V3 d) {
  const int lv = pv_rec(G, pv).lv;
  const uint32_t g0 = (uint32_t)G.lv_key[2 * lv];
  if (G.lv_key[2 * lv + 1] == 1) return g0;
  const LvRec v = lv_rec(G, lv);
  CQ X = G.pv_gxf + 12 * (size_t)pv;
  const V3 pl = to_child_p(X, p), dl = to_child_d(X, d);
  const V3 inv{inv_dir64(dl.x), inv_dir64(dl.y), inv_dir64(dl.z)};
  const V3 pin{-pl.x * inv.x, -pl.y * inv.y, -pl.z * inv.z};
  double best = GV_INF;
  int bk = -1, hits = 0;
  for (int k = 0; k < v.cnt; ++k) {
    const double t = box_entry64(G.dau_box + 6 * (size_t)(v.off + k), inv, pin);
    if (!(t < GV_INF)) continue;
    ++hits;
    if (t < best) {
      best = t;
      bk = k;
    }
  }
  return g0 + (bk < 0 ? 0 : 1 + 2 * (bk % kStartBoxes) + (hits > 1 ? 1 : 0));
}

// Before a transport: zeroes the key counts and the work counter, and locates
// the tracks whose start volume the caller does not give.  With the
// point lookup inside the transport kernel instead, its code took registers
// from the step loop (1.89 against 1.85 ms per 2^20-track detector transport,
// measured before the tubes' closed form);
// here it runs at full occupancy.  groups: also each track's start group, into
// its key.
template <int K>
__global__ void k_ls_begin(DevGeom G, int64_t n, const double* __restrict__ x, const double* __restrict__ y,
                           const double* __restrict__ z, const double* __restrict__ dx,
                           const double* __restrict__ dy, const double* __restrict__ dz,
                           const int32_t* __restrict__ start_pv, int groups, LaneCtl L, int cells) {
  for (int64_t i = gtid(); i < cells; i += gstride()) L.cnt[i] = 0u;
  if (gtid() == 0) *L.queue = 0u;
  if (start_pv && !groups) return;
  for (int64_t i = gtid(); i < n; i += gstride()) {
    const V3 p = ld3(x, y, z, i);
    const int pv = start_pv ? start_pv[i] : locate<K>(G, p);
    if (!start_pv) L.pv0[i] = pv;
    if (groups) L.key[i] = pv >= 0 && pv < G.n_pv ? start_group(G, pv, p, ld3(dx, dy, dz, i)) : 0u;
  }
}

// Key of every track (z-axis or octahedral cell; when groups > 0, below its
// start group, which its key holds on entry) and the per-key counts
// (workgroup histogram in LDS, 4 cells bytes of dynamic LDS, one global
// atomic per workgroup and key).
static __global__ void k_ls_count(int64_t n, const double* __restrict__ dx, const double* __restrict__ dy,
                                  const double* __restrict__ dz, int h, int zaxis, int groups, LaneCtl L) {
  extern __shared__ uint32_t key_hist[];
  const int cells = max(groups, 1) << (2 * h);
  for (int c = threadIdx.x; c < cells; c += blockDim.x) key_hist[c] = 0u;
  __syncthreads();
  for (int64_t i = gtid(); i < n; i += gstride()) {
    uint32_t k = zaxis ? direction_key_zaxis(dx[i], dy[i], dz[i], h) : direction_key(dx[i], dy[i], dz[i], h);
    if (groups > 0) k |= L.key[i] << (2 * h);
    L.key[i] = k;
    atomicAdd(&key_hist[k], 1u);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < cells; c += blockDim.x)
    if (key_hist[c]) atomicAdd(&L.cnt[c], key_hist[c]);
}

// Exclusive scan of the key counts in place (one workgroup of 1024 threads):
// cnt[c] becomes the first place of key c.
static __global__ void __launch_bounds__(1024) k_ls_scan(LaneCtl L, int cells) {
  __shared__ uint32_t part[1024];
  const int t = threadIdx.x;
  const int per = (cells + 1023) / 1024;
  const int c0 = t * per, c1 = min(cells, c0 + per);
  uint32_t s = 0;
  for (int c = c0; c < c1; ++c) s += L.cnt[c];
  part[t] = s;
  __syncthreads();
  // Hillis-Steele inclusive scan over the 1024 partial sums
  for (int o = 1; o < 1024; o <<= 1) {
    const uint32_t v = t >= o ? part[t - o] : 0u;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  uint32_t run = t > 0 ? part[t - 1] : 0u;
  for (int c = c0; c < c1; ++c) {
    const uint32_t v = L.cnt[c];
    L.cnt[c] = run;
    run += v;
  }
}

// Places: each workgroup takes `chunk` consecutive tracks, counts their keys
// in LDS, reserves each key's run of places with one global atomic, and gives
// each of its tracks the next place of its key's run (4 cells bytes of
// dynamic LDS).  The order inside a key depends on the atomics' order, which
// changes no result.
static __global__ void __launch_bounds__(1024) k_ls_scatter(int64_t n, int64_t chunk, int cells, LaneCtl L) {
  extern __shared__ uint32_t key_run[];
  const int64_t a = (int64_t)blockIdx.x * chunk, b = min(n, a + chunk);
  for (int c = threadIdx.x; c < cells; c += blockDim.x) key_run[c] = 0u;
  __syncthreads();
  for (int64_t i = a + threadIdx.x; i < b; i += blockDim.x) atomicAdd(&key_run[L.key[i]], 1u);
  __syncthreads();
  for (int c = threadIdx.x; c < cells; c += blockDim.x)
    if (key_run[c]) key_run[c] = atomicAdd(&L.cnt[c], key_run[c]);
  __syncthreads();
  for (int64_t i = a + threadIdx.x; i < b; i += blockDim.x) L.perm[atomicAdd(&key_run[L.key[i]], 1u)] = (int32_t)i;
}

// One track's state while a lane carries it.
struct LaneTrack {
  V3 p, d;
  double safe;  // physics: distance still to go to the last boundary found
  int64_t i;    // track index
  int pv, k, zero_run;
  int left;     // placement index of the box daughter of pv the track left last (-1: none)
  uint32_t fl;
  uint64_t procs;  // physics, staged outputs: the process codes of the run, byte k % 8 for step k
};

// The arguments of a lane transport.  The kernels read them where they need
// them, through a pointer that the compiler cannot see through (lane_args), so
// that it loads them again instead of holding 60 scalar registers of pointers
// through the step loop, where they were spilled to vector registers.
template <class T>
using GIn = const __attribute__((address_space(1))) T*;
template <class T>
using GOut = __attribute__((address_space(1))) T*;
struct LaneArgs {
  DevGeom G;
  int64_t n;
  GIn<double> x, y, z, dx, dy, dz;
  GIn<int32_t> start_pv, perm;
  GOut<uint32_t> queue;
  GOut<int32_t> out_pv;
  GOut<double> out_step;
  GOut<int32_t> out_nsteps;
  GOut<uint32_t> out_flags;
  GOut<int8_t> out_proc;
  PhysArgs P;
  int max_steps;
};
typedef const __attribute__((address_space(4))) LaneArgs* CLA;
__device__ __forceinline__ CLA lane_args() {
  CLA a = (CLA)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

__device__ __forceinline__ const DevGeom& geom_of(CLA a) { return *(const DevGeom*)&a->G; }

// Starts track i: its volume and entry 0 of its sequence.  Returns false (and
// writes the track's zero count and flags) when it starts outside the world.
__device__ __forceinline__ bool lane_begin(CLA a, LaneTrack& T, int64_t i) {
  T.i = i;
  T.p = V3{a->x[i], a->y[i], a->z[i]};
  T.d = V3{a->dx[i], a->dy[i], a->dz[i]};
  T.fl = 0u;
  T.k = 0;
  T.zero_run = 0;
  T.left = -1;
  T.safe = 0.0;
  T.procs = 0;
  int pv = a->start_pv[i];
  if (pv < -1 || pv >= a->G.n_pv) {
    pv = -1;
    T.fl = kFlagLocateFail;
  }
  T.pv = pv;
  a->out_pv[(size_t)i * (a->max_steps + 1)] = pv;
  if (pv < 0) {
    a->out_nsteps[i] = 0;
    a->out_flags[i] = T.fl;
    return false;
  }
  return true;
}

// A lane's column of its wavefront's output staging in LDS: entry j of the
// column holds the j-th step since the last flush, 64 entries apart (the 64
// lanes write one row of the buffer per step, without bank conflicts).
struct LaneStage {
  double* st;
  int32_t* pv;
};

// What a step found: its length, the next volume, the acting process (physics,
// -1: none), and whether it ends at the mother's exit.
struct LaneStep {
  double st;
  int nx, proc;
  bool exited;
};

// One ComputeStep of a carried track in volume pv (logical volume lv).
template <bool F32, bool PHYS, int K>
__device__ __forceinline__ void lane_compute(const DevGeom& G, LaneTrack& T, int lv, int pv, const PhysArgs& P,
                                             LaneStep& R) {
  NoWork w;
  R.exited = false;
  if (PHYS) {
    R.st = step_physics<F32, K>(G, lv, pv, T.p, T.d, (uint32_t)T.i, T.k, P, T.safe, &R.nx, &R.proc, &T.fl, w, T.left,
                                &R.exited);
  } else {
    R.st = step_culled<F32, K>(G, lv, pv, T.p, T.d, &R.nx, &T.fl, w, T.left, &R.exited);
    T.p = advance(T.p, R.st, T.d);
  }
}

// Records a carried track's step; returns true when the track has ended (left
// the world, stuck, or out of steps), after writing its count and flags.
// With ST > 0 the step length and next volume go to the lane's LDS column
// (and a physics step's process code to a byte of T.procs) and are written
// to the track's rows ST steps at a time (and at its end), so the row stores
// of a lane come in runs of consecutive addresses; all lanes of a wavefront
// that started together write their runs in the same iteration, and a full
// run goes out in 16-byte stores (its process codes in one 8-byte store).
template <bool PHYS, int ST>
__device__ __forceinline__ bool lane_record(CLA a, LaneTrack& T, const LaneStep& R, LaneStage S) {
  static_assert(ST == 0 || ST == 8, "a staged run is 8 steps (the process codes of a run fill 64 bits)");
  constexpr int kRun = ST > 0 ? ST : 1;
  const int nx = R.nx;
  const double st = R.st;
  if (PHYS) {
    if (ST == 0) {
      if (a->out_proc) a->out_proc[(size_t)T.i * a->max_steps + T.k] = (int8_t)R.proc;
    } else {
      T.procs |= (uint64_t)(uint8_t)R.proc << (8 * (T.k % 8));
    }
  }
  // a track that leaves its volume into the mother carries the volume's
  // placement index there (the line does not change, so the volume is behind
  // it); entering a daughter clears it
  if (nx != T.pv) T.left = R.exited ? pv_rec(geom_of(a), T.pv).k : -1;
  if (ST == 0) {
    a->out_step[(size_t)T.i * a->max_steps + T.k] = st;
    a->out_pv[(size_t)T.i * (a->max_steps + 1) + T.k + 1] = nx;
  } else {
    S.st[64 * (T.k % kRun)] = st;
    S.pv[64 * (T.k % kRun)] = nx;
  }
  ++T.k;
  bool end = nx < 0;
  if (!end) {
    T.zero_run = st < kTol ? T.zero_run + 1 : 0;
    if (T.zero_run >= 8) {
      T.fl |= kFlagStuck;
      end = true;
    } else if (T.k == a->max_steps) {
      T.fl |= kFlagOverflow;
      end = true;
    }
  }
  T.pv = nx;
  if (ST > 0 && (end || T.k % kRun == 0)) {
    const int m = (T.k - 1) % kRun + 1, k0 = T.k - m;
    double* rs = (double*)a->out_step + (size_t)T.i * a->max_steps + k0;
    int32_t* rp = (int32_t*)a->out_pv + (size_t)T.i * (a->max_steps + 1) + k0 + 1;
    if (m == ST) {
      double vs[kRun];
      int32_t vp[kRun];
      for (int j = 0; j < ST; ++j) {
        vs[j] = S.st[64 * j];
        vp[j] = S.pv[64 * j];
      }
      __builtin_memcpy(rs, vs, sizeof vs);
      __builtin_memcpy(rp, vp, sizeof vp);
    } else {
      for (int j = 0; j < m; ++j) {
        rs[j] = S.st[64 * j];
        rp[j] = S.pv[64 * j];
      }
    }
    if (PHYS) {
      if (a->out_proc) {
        int8_t* rq = (int8_t*)a->out_proc + (size_t)T.i * a->max_steps + k0;
        if (m == ST) {
          __builtin_memcpy(rq, &T.procs, 8);
        } else {
          for (int j = 0; j < m; ++j) rq[j] = (int8_t)(T.procs >> (8 * j));
        }
      }
      T.procs = 0;
    }
  }
  if (end) {
    a->out_nsteps[T.i] = T.k;
    a->out_flags[T.i] = T.fl;
  }
  return end;
}

// Persistent whole-track transport.  Places 0..n-1 of the order (perm, or the
// identity when perm is NULL) are handed out from *queue, which must be 0 at
// launch: a wavefront takes 64 places at a time and carries their tracks to
// their ends.  WV: waves per SIMD the kernel is built for (its register
// budget); ST: steps staged in LDS per lane before its rows are written (0:
// every step writes its rows at once).  CLS: per-class scheduling -- in each
// iteration only the lanes whose volume is in the step class (the branch of
// the step code: mother solid type and daughter access) that most live lanes
// are in take their step, and the others wait; lanes that fell behind (a
// track that crossed a module is two steps behind one that passed between
// modules) thus catch up before the wavefront moves on, instead of every
// iteration running the branches of every class with partial masks.
// (Taking each step one logical volume at a time with every lane stepping in
// every iteration, was measured 2.3x slower: lanes in different layers then
// run the same branch separately.  Giving a lane whose track has ended the
// next track at once, which let its new track wait for its class like any
// other, was measured slower as well: 2.66 against 2.56 ms.)
template <bool F32, bool PHYS, int K, int WV, int ST, bool CLS = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WV))) k_lane_transport(LaneArgs) {
  constexpr int kStage = ST > 0 ? 4 * ST * 64 : 1;  // 4 wavefronts per workgroup
  __shared__ double stage_st[kStage];
  __shared__ int32_t stage_pv[kStage];
  const int lane = __lane_id();
  const int wbase = ST > 0 ? (int)(threadIdx.x / 64) * ST * 64 + lane : 0;
  const LaneStage S{stage_st + wbase, stage_pv + wbase};
  LaneTrack T;
  for (;;) {
    CLA a = lane_args();
    uint32_t b = 0;
    if (lane == 0) b = atomicAdd((uint32_t*)a->queue, 64u);
    const int64_t base = (int64_t)__shfl(b, 0);
    if (base >= a->n) break;
    const int64_t j = base + lane;
    bool live = false;
    if (j < a->n) live = lane_begin(a, T, a->perm ? a->perm[j] : j);
    LaneStep R;
    if (!CLS) {
      while (live) {
        a = lane_args();
        const DevGeom& G = geom_of(a);
        lane_compute<F32, PHYS, K>(G, T, pv_rec(G, T.pv).lv, T.pv, PhysArgs{a->P.seed, a->P.shortcut}, R);
        live = !lane_record<PHYS, ST>(a, T, R, S);
      }
      continue;
    }
    for (uint64_t lm = __ballot(live); lm; lm = __ballot(live)) {
      a = lane_args();
      const DevGeom& G = geom_of(a);
      const PhysArgs P{a->P.seed, a->P.shortcut};
      int lv = -1, cl = -1;
      if (live) {  // volume and class in one load
        const PvRec v = pv_rec(G, T.pv);
        lv = v.lv;
        cl = v.cls;
      }
      // the class most live lanes are in (few classes are present at once;
      // on equal counts the first found).  Lanes in a composite below the
      // world, or in a volume that holds one, come first: they take the few
      // steps more that it costs and stay near the others; left for last, each
      // went the rest of its way alone (262,144 tracks of the detector with a
      // composite in one kind of module 0.85 and 0.65 ms, 4,099 606 and 305 us;
      // the world as well where it holds the composite: 1.30 and 2.39 ms).
      int best = -1, nbest = 0;
      for (uint64_t rest = lm; rest;) {
        const int c = __builtin_amdgcn_readlane(cl, __ffsll((unsigned long long)rest) - 1);
        const uint64_t m = __ballot(cl == c);
        const int nm = __popcll(m) + (K == kComposites && c > kOwnClass ? 64 : 0);
        if (nm > nbest) {
          nbest = nm;
          best = c;
        }
        rest &= ~m;
      }
      // When every stepping lane is in one logical volume (always in the
      // world, whose volume is unique; in a layer or a module when the
      // wavefront's tracks are all in one), the step runs with that volume
      // (and, for navigation, the placed volume too when shared) as
      // wavefront-uniform values: the volume's tables then come through
      // scalar loads instead of per-lane gathers.
      const bool mine = live && cl == best;
      const int lead = __ffsll((unsigned long long)__ballot(mine)) - 1;
      const int lv0 = __builtin_amdgcn_readlane(lv, lead);
      // (A composite, or a volume that holds one, is a class of its own.)
      constexpr int E = K == kComposites ? kElementary : K;
      const bool uni_lv = __ballot(mine && lv != lv0) == 0;
      const int pv0 = __builtin_amdgcn_readlane(T.pv, lead);
      if (K == kComposites && best >= kOwnClass) {
        if (mine) lane_compute<F32, PHYS, kOneComposite>(G, T, lv0, T.pv, P, R);
      } else if (!PHYS && K != kComposites && uni_lv && __ballot(mine && T.pv != pv0) == 0) {
        if (mine) lane_compute<F32, PHYS, E>(G, T, lv0, pv0, P, R);
      } else if (uni_lv) {
        if (mine) lane_compute<F32, PHYS, E>(G, T, lv0, T.pv, P, R);
      } else if (mine) {
        lane_compute<F32, PHYS, E>(G, T, lv, T.pv, P, R);
      }
      if (mine)
        live = !lane_record<PHYS, ST>(a, T, R, S);
    }
  }
}

}  // namespace gv
