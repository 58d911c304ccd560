// Device-resident geometry tables and per-track navigation (Sec. III.A step
// selection over the Sec. III.B volume hierarchy).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gv_solids.h"

namespace gv {

// What a step reads of a logical volume, a placement and a placed volume, each
// in one aligned record: the fields used to be arrays of their own, and a step
// waited for seven loads of its volume, then for the daughter's, the parent's
// and the child's one after another.
struct LvRec {
  int type, par;    // solid type and offset of its parameters in DevGeom::par
  int off, cnt;     // first daughter placement and number of daughters
  int dtype;        // solid type shared by all daughters, -1 if mixed or none
  int rad, phi;     // first entry of its radial list / first phi mask, -1 without
  int loc;          // how point lookups reach the daughters (kLoc*)
  int boxtube;      // 1 when it and its daughters are boxes and full tubes
  int thin;         // 1 when it has kSafetySectors daughters or more and each phi sector a sixteenth of them or less on
                    // average; all three share a word
};
struct DauRec {
  int lv, par;      // child volume, offset of its solid's parameters
  int ident;        // 1 when the placement is the identity (R = I, t = 0)
  int type;         // the child's solid type; both share a word of the record
  int delta;        // placed volume of this daughter minus its mother's
};
struct PvRec {
  int lv, cls;      // logical volume, step class: branch of the step code (daughter access mode x 8 + solid type)
  int parent, k;    // placed mother (-1: none), placement index among its daughters (-1: the world)
};

// All arrays live in HBM; geom_load fills them once.  Transforms are 12
// doubles: R row-major then t, with x_mother = R x_child + t.
constexpr int kWave = 64;
constexpr int kPhiSectors = 256, kPhiLevels = 8, kSafetySectors = 20;
constexpr int kLvSlots = 1024;  // slots of the LVs in the regrouped kernels
constexpr int kOwnClass = 128;  // an LV that is a composite or holds one has a step class of its own from here on (the world this one)

struct DevGeom {
  int n_lv, n_pv, n_place;
  CQI lv_slot;       // [n_lv] place of each LV in order of step class, then number (scaled into kLvSlots)
  CQI lv_key;        // [n_lv][2] first start group of each LV's tracks (ordering of transports), and the number of groups
  CQ4 lv_rec;        // [n_lv][2] records of LvRec, one 32-byte load
  CQ par;            // derived solid parameters
  CQ dau_xf;         // [n_place][12] placement transform, LV frame
  CQ4 dau_rec;       // [n_place] records of DauRec, one 16-byte load
  CQ dau_box;        // [n_place][6] child's bounding box in the mother frame (lo xyz, hi xyz), padded
  CQ4 pv_rec;        // [n_pv] records of PvRec, one 16-byte load
  CQ pv_gxf;         // [n_pv][12] composed world <- PV transform
  // FP32 screen tables (daughter culling in FP32 with FP64 refinement)
  CQF lv_scr;        // [n_lv] S: max |coordinate| of a point of the LV's solid + 1 mm
  CQF dau_box32;     // [n_place][8] dau_box widened by 128 u (S(mother) + |box|inf), rounded outward; 2 unused
  CQF dau_scr32;     // [n_place][16] R (9), t (3), child a b c (box: dx dy dz; tube: rmin rmax dz), e
  // daughter groups: 8 consecutive daughters of an LV with >= 16 daughters
  CQI lv_grp;        // [n_lv] index of the LV's first group box, -1 without groups
  CQ grp_box;        // [n_grp][6] union of the group's padded daughter boxes (lo xyz, hi xyz)
  CQF grp_box32;     // [n_grp][8] union of the group's FP32 boxes; 2 unused
  // radial order: an LV whose daughters are identity-placed full tubes with
  // disjoint radial ranges lists them by radius
  CQ rad_r2;         // [n_rad][2] rmin^2, rmax^2 in radial order; before an LV's first: its largest z half-length, 0
  CQI rad_k;         // [n_rad] daughter index (placement order) of each entry
  // phi sectors: an LV whose (<= 64) daughters lie around the z axis, each
  // within less than a half turn, has kPhiSectors masks of the daughters
  // whose angular extent (widened) meets each sector of pseudo-angle
  CQL phi_mask;      // [n_phi_lv][kPhiLevels][kPhiSectors]: at level l the union of the 2^l masks from each sector on
  // materials for physics-limited steps (geom_set_materials); n_mat 0 if unset
  int n_mat, n_proc;
  CQ mat_rate;       // [n_mat][n_proc] n sigma = 1 / mean free path, 1/mm
  CQI lv_mat;        // [n_lv] material of each LV
};

__device__ __forceinline__ LvRec lv_rec(const DevGeom& G, int lv) {
  const Int4 a = G.lv_rec[2 * (size_t)lv], b = G.lv_rec[2 * (size_t)lv + 1];
  return LvRec{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w & 3, b.w >> 2 & 1, b.w >> 3};
}
__device__ __forceinline__ DauRec dau_rec(const DevGeom& G, int k) {
  const Int4 a = G.dau_rec[k];
  return DauRec{a.x, a.y, a.z & 1, a.z >> 1, a.w};
}
__device__ __forceinline__ PvRec pv_rec(const DevGeom& G, int pv) {
  const Int4 a = G.pv_rec[pv];
  return PvRec{a.x, a.y, a.z, a.w};
}

__device__ __forceinline__ V3 ld3(const double* x, const double* y, const double* z, int64_t i) {
  return V3{x[i], y[i], z[i]};
}

// x_child = R^T (x_mother - t)
__device__ __forceinline__ V3 to_child_p(CQ X, V3 p) {
  double q0 = p.x - X[9], q1 = p.y - X[10], q2 = p.z - X[11];
  return V3{X[0] * q0 + X[3] * q1 + X[6] * q2, X[1] * q0 + X[4] * q1 + X[7] * q2,
            X[2] * q0 + X[5] * q1 + X[8] * q2};
}
__device__ __forceinline__ V3 to_child_d(CQ X, V3 d) {
  return V3{X[0] * d.x + X[3] * d.y + X[6] * d.z, X[1] * d.x + X[4] * d.y + X[7] * d.z,
            X[2] * d.x + X[5] * d.y + X[8] * d.z};
}

constexpr uint32_t kFlagOverflow = 1u, kFlagStuck = 2u, kFlagLocateFail = 4u;

// Point lookups through the daughter indexes.  lv_loc says how an LV's
// daughters that can hold a point (or, for NavSafety, be nearest to it) are
// found; every candidate then goes through the same solid code as in the loop
// over all daughters, so the answers are the same bit for bit.
enum { kLocPlain = 0, kLocRadial = 1, kLocPhi = 2, kLocBox = 3 };

// The access mode for a point: the indexes take finite coordinates only (a NaN
// or infinity goes through every daughter's own code).
__device__ __forceinline__ int loc_mode(const LvRec& v, V3 p) {
  return p.x * p.x + p.y * p.y + p.z * p.z < 1e200 ? v.loc : kLocPlain;
}

__device__ __forceinline__ int phi_sector32(float a) {
  return min(kPhiSectors - 1, max(0, (int)(a * (kPhiSectors / 4.0f))));
}
__device__ __forceinline__ int phi_sector(double a) {
  return min(kPhiSectors - 1, max(0, (int)(a * (kPhiSectors / 4.0))));
}

// Union of the masks of sectors first..last, going up around the circle: two
// runs of the largest power of two that fits.  (Read one by one, a track moving
// along a layer waited for up to 128 masks, one after another.)
__device__ __forceinline__ uint64_t phi_range(CQL M, int first, int last) {
  const int n = ((last - first) & (kPhiSectors - 1)) + 1, l = min(kPhiLevels - 1, 31 - __clz(n));
  CQL R = M + l * kPhiSectors;
  return R[first] | R[(last + 1 - (1 << l)) & (kPhiSectors - 1)];
}

// Radial entries with rmin^2 <= rho^2 (ascending).  Four at a time while every
// active lane is past them, then one by one until no lane is: lanes that run
// together mostly sit between the same two tubes.
__device__ __forceinline__ int radial_rank(CQ R2, int cnt, double rho2) {
  int m = 0;
  while (m + 4 <= cnt && __ballot(!(R2[2 * (m + 3)] <= rho2)) == 0) m += 4;
  int j = m;
  for (; m < cnt; ++m) {
    const bool past = R2[2 * m] <= rho2;
    if (__ballot(past) == 0) break;
    j += past ? 1 : 0;
  }
  return j;
}

// Index of the first daughter of lv whose Inside code is not outside (-1:
// none).  Radial order: only the tubes whose radial range, widened by more than
// the surface band, holds the point's radius (the ranges are disjoint and
// sorted, so those are neighbours of its rank).  Phi sectors: the daughters of
// the point's sector.  Boxes: the daughters whose padded box holds the point.
// The plain loop made a point in the detector evaluate up to 84 daughters (128
// us per 300,007 points spread over it), the indexes two or three (13 us, most
// of it the call).  With the boxes, first the mask of all that hold the point,
// then those daughters in turn: with each box in front of its daughter a
// wavefront waits for the box and then, as nearly every daughter has a lane in
// its box, for the daughter's tables, one after another (23 spheres, 5,000
// points 21.4 us, by masks 14.1, without boxes 16; 56 polycones, 300,000 points
// 79 and 48).
template <int K>
__device__ __forceinline__ int first_daughter(const DevGeom& G, const LvRec& v, V3 pl) {
  const int off = v.off, cnt = v.cnt;
  if (cnt == 0) return -1;
  const int mode = loc_mode(v, pl);
  auto holds = [&](int k) {
    const DauRec d = dau_rec(G, off + k);
    const V3 pc = to_child_p(G.dau_xf + 12 * (size_t)(off + k), pl);
    return code_of(solid_sgn<K>(d.type, G.par + d.par, pc)) != kOutside;
  };
  if (mode == kLocRadial) {
    const int r0 = v.rad;
    CQ R2 = G.rad_r2 + 2 * (size_t)r0;
    CQI order = G.rad_k + r0;
    const double rho2 = pl.x * pl.x + pl.y * pl.y;
    const int j = radial_rank(R2, cnt, rho2);
    int best = cnt;
    auto test = [&](int m) {
      const int k = order[m];
      if (k < best && code_of(Tubs::sgn(G.par + dau_rec(G, off + k).par, pl)) != kOutside) best = k;
    };
    for (int m = j - 1; m >= 0 && rho2 <= fma(R2[2 * m + 1], 1.0 + 1e-8, 1e-8); --m) test(m);
    for (int m = j; m < cnt && rho2 >= fma(R2[2 * m], 1.0 - 1e-8, -1e-8); ++m) test(m);
    return best < cnt ? best : -1;
  }
  if (mode == kLocPhi && fabs(pl.x) + fabs(pl.y) > 1e-6) {
    uint64_t cand = (G.phi_mask + (size_t)v.phi)[phi_sector(pseudo_angle_fast(pl.x, pl.y))];
    const int type = v.dtype;
    while (cand) {
      const int k = __builtin_ctzll(cand);
      cand &= cand - 1;
      CQ q = G.par + dau_rec(G, off + k).par;
      const V3 pc = to_child_p(G.dau_xf + 12 * (size_t)(off + k), pl);
      if (code_of(type == kBox ? Box::sgn(q, pc) : Tubs::sgn(q, pc)) != kOutside) return k;
    }
    return -1;
  }
  if (mode == kLocBox) {
    for (int c0 = 0; c0 < cnt; c0 += 64) {
      const int m = min(cnt - c0, 64);
      uint64_t cand = 0;
#pragma unroll 4
      for (int j = 0; j < m; ++j) {
        CQ X = G.dau_box + 6 * (size_t)(off + c0 + j);
        const bool in =
            !(pl.x < X[0] || pl.y < X[1] || pl.z < X[2] || pl.x > X[3] || pl.y > X[4] || pl.z > X[5]);
        cand |= (uint64_t)in << j;
      }
      while (cand) {
        const int k = c0 + __builtin_ctzll(cand);
        cand &= cand - 1;
        if (holds(k)) return k;
      }
    }
    return -1;
  }
  for (int k = 0; k < cnt; ++k)
    if (holds(k)) return k;
  return -1;
}

template <int K>
__device__ __forceinline__ int locate(const DevGeom& G, V3 p) {
  LvRec v = lv_rec(G, pv_rec(G, 0).lv);
  if (code_of(solid_sgn<K>(v.type, G.par + v.par, p)) == kOutside) return -1;
  int pv = 0;
  V3 pl = p;
  for (;;) {
    const int k = first_daughter<K>(G, v, pl);
    if (k < 0) return pv;
    const DauRec d = dau_rec(G, v.off + k);
    pl = to_child_p(G.dau_xf + 12 * (size_t)(v.off + k), pl);
    pv += d.delta;
    v = lv_rec(G, d.lv);
  }
}

// NavSafety's part over the daughters of an LV with a radial order or with phi
// sectors of box daughters: lowers s to the smallest SafetyToIn (0 when the
// point is not strictly outside a daughter), visiting only daughters whose
// SafetyToIn can be below s; false when the LV has no such index.  Radial: a
// tube's SafetyToIn is at least rmin - r and r - rmax, which grow away from the
// point's rank.  Phi: the daughters of the point's own sector first; then those
// within the angle beyond which the distance r sin(angle) exceeds sqrt(3) s (a
// box's SafetyToIn, the largest of its three gaps, is at least its distance
// over sqrt(3)), an arc of at most pi/2 sin(angle) in pseudo-angle.  kTolerance
// on top of s keeps rounding of the bounds from mattering.  In the detector two
// or three daughters instead of 20 or 64 (71 against 16 us per 200,003 points).
// Where a sector holds more than a sixteenth of the daughters (boxes all over a
// volume and not on a ring), the loop over all is the faster one: it takes each
// for all lanes at once, while through the sectors each lane takes its own, one
// after another (300,000 points in boxes with up to 33 boxes 77 and 51 us).  The
// same for a few daughters, kSafetySectors: with two rings of 6 and 11 boxes
// 300,000 safeties take 28 us through the sectors and 22 in the loop, with one of
// 18 boxes 33 and 25, among many rings of 8 to 19 boxes 97 and 104, with rings of
// 19 and 13 in thick tubes 24 and 33.
__device__ __forceinline__ bool safety_indexed(const DevGeom& G, const LvRec& v, V3 pl, double& s) {
  const int mode = loc_mode(v, pl);
  if (mode != kLocRadial && !(mode == kLocPhi && v.dtype == kBox && v.thin)) return false;
  const int off = v.off, cnt = v.cnt;
  const double rho2 = pl.x * pl.x + pl.y * pl.y, r = sqrt(rho2);
  auto limit = [&] { return fmax(s, kHalf) + kTol; };
  if (mode == kLocRadial) {
    const int r0 = v.rad;
    CQI order = G.rad_k + r0;
    const int j = radial_rank(G.rad_r2 + 2 * (size_t)r0, cnt, rho2);
    auto eval = [&](CQ q) { s = code_of(Tubs::sgn(q, pl)) == kOutside ? fmin(s, Tubs::safety_in(q, pl)) : 0.0; };
    for (int m = j - 1; m >= 0; --m) {
      CQ q = G.par + dau_rec(G, off + order[m]).par;
      if (r - q[L::TB_RMAX] > limit()) break;
      eval(q);
    }
    for (int m = j; m < cnt; ++m) {
      CQ q = G.par + dau_rec(G, off + order[m]).par;
      if (q[L::TB_RMIN] - r > limit()) break;
      eval(q);
    }
    return true;
  }
  CQL M = G.phi_mask + (size_t)v.phi;
  const uint64_t all = cnt == 64 ? ~0ull : (1ull << cnt) - 1;
  const bool off_axis = fabs(pl.x) + fabs(pl.y) > 1e-6;
  const double a = off_axis ? pseudo_angle_fast(pl.x, pl.y) : 0.0;
  uint64_t cand = off_axis ? M[phi_sector(a)] : all, done = 0;
  for (int pass = 0; pass < 2; ++pass) {
    done |= cand;
    while (cand) {
      const int k = __builtin_ctzll(cand);
      cand &= cand - 1;
      CQ q = G.par + dau_rec(G, off + k).par;
      const V3 pc = to_child_p(G.dau_xf + 12 * (size_t)(off + k), pl);
      s = code_of(Box::sgn(q, pc)) == kOutside ? fmin(s, Box::safety_in(q, pc)) : 0.0;
    }
    if (pass == 1 || done == all) break;
    const double w = 1.5707964 * 1.7320509 * limit() * rcp_fast(r) + 1e-6;  // pi/2 sin(angle)
    if (w < 0.5) {
      const double b0 = a - w, b1 = a + w;
      cand = phi_range(M, phi_sector(b0 < 0.0 ? b0 + 4.0 : b0), phi_sector(b1 >= 4.0 ? b1 - 4.0 : b1));
    } else {
      cand = all;
    }
    cand &= ~done;
  }
  return true;
}

// NavSafety's loop over daughters that are all boxes or all full tubes, that
// solid's code alone: with the choice of solid inside the loop both are worked
// out and waited for (25 boxes, 5,000 points 12.4 and 7.1 us; 300,000 points among
// layers of modules 117 and 72).  Only for geometries of boxes and full tubes:
// where a wavefront also has volumes that take the loop of all types, it runs
// one loop after the other (60 and 70 us).
template <class S>
__device__ __forceinline__ double safety_of_type(const DevGeom& G, const LvRec& v, V3 pl, double s) {
  for (int k = 0; k < v.cnt; ++k) {
    CQ q = G.par + dau_rec(G, v.off + k).par;
    const V3 pc = to_child_p(G.dau_xf + 12 * (size_t)(v.off + k), pl);
    if (code_of(S::sgn(q, pc)) != kOutside) return 0.0;
    s = fmin(s, S::safety_in(q, pc));
  }
  return fmax(s, 0.0);
}

template <int K>
__device__ __forceinline__ double nav_safety(const DevGeom& G, int pv, V3 p) {
  const LvRec v = lv_rec(G, pv_rec(G, pv).lv);
  V3 pl = to_child_p(G.pv_gxf + 12 * (size_t)pv, p);
  CQ q = G.par + v.par;
  if (code_of(solid_sgn<K>(v.type, q, pl)) != kInside) return 0.0;
  double s = solid_safety_out<K>(v.type, q, pl);
  if (safety_indexed(G, v, pl, s)) return fmax(s, 0.0);
  if (K == kBoxTube && v.dtype == kBox) return safety_of_type<Box>(G, v, pl, s);
  if (K == kBoxTube && v.dtype == kTubs) return safety_of_type<FullTubs>(G, v, pl, s);
  for (int k = 0; k < v.cnt; ++k) {
    const DauRec d = dau_rec(G, v.off + k);
    V3 pc = to_child_p(G.dau_xf + 12 * (size_t)(v.off + k), pl);
    CQ qc = G.par + d.par;
    int tc = d.type;
    if (code_of(solid_sgn<K>(tc, qc, pc)) != kOutside) return 0.0;
    s = fmin(s, solid_safety_in<K>(tc, qc, pc));
  }
  return fmax(s, 0.0);
}

}  // namespace gv
