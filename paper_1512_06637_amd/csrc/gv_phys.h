// Physics-limited steps.  Each process i of the current volume's material has
// the mean free path lambda_i = 1 / (n sigma_i) (Sec. III, Eq. (1)); every step,
// each process draws an interaction length by Monte Carlo and the shortest is
// proposed as the physics step (the rates add up, Eqs. (2)-(3)); the navigator
// then takes the border instead when it is nearer (Sec. III.A).
//
// A length is s_i = -ln(u) / (n sigma_i), u in (0, 1) from the counter-based
// generator Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) with counter
// (track, step, process, 0) and key (seed low, seed high): any track's draws
// are reproducible whatever the order in which tracks are processed.
#pragma once
#include "gv_geom.h"

namespace gv {

constexpr int kMaxProc = 16;  // processes per material

// Both halves of a 32-bit product in one instruction (two for the compiler's
// low and high multiplies: 24 against 36 cycles per Philox round and wavefront).
__device__ __forceinline__ uint64_t mul_wide(uint32_t a, uint32_t b) {
  uint64_t p, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, 0" : "=v"(p), "=s"(carry) : "v"(a), "s"(b));
  return p;
}
// One instruction on gfx950 (the compiler makes two of it).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#ifdef __gfx950__
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}

// Philox4x32 with 10 rounds.  A round multiplies words 0 and 2 by the two
// Philox multipliers, and the new words are the high product halves mixed with
// the other words and the round key, and the low product halves; the key
// advances by the two Weyl constants before each round after the first.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += kW0;
      k1 += kW1;
    }
    const uint64_t a = mul_wide(c[0], kM0), b = mul_wide(c[2], kM1);
    const uint32_t n0 = xor3((uint32_t)(b >> 32), c[1], k0), n2 = xor3((uint32_t)(a >> 32), c[3], k1);
    c[0] = n0;
    c[1] = (uint32_t)b;
    c[2] = n2;
    c[3] = (uint32_t)a;
  }
}

// u in (0, 1): the first two output words as a 64-bit integer, its top 53
// bits, centred in their 2^-53 interval.
__host__ __device__ inline double uniform_of(uint64_t w) { return ((double)(w >> 11) + 0.5) * 0x1p-53; }
// The same number in FP32, to one part in 2^24 from 2^-54 up: the 11 low bits go
// and the centre of the interval comes in before the rounding.
__host__ __device__ inline float uniform32(uint32_t hi, uint32_t lo) {
  return fmaf((float)((lo & ~0x7FFu) | 0x400u), 0x1p-64f, (float)hi * 0x1p-32f);
}
__device__ __forceinline__ double length_of(uint64_t w, double rate) { return -log(uniform_of(w)) / rate; }

// Shortest sampled interaction length of the processes of material `mat`
// (rate[mat][i] = n sigma_i precomputed), *proc its process (lowest index on
// equal lengths); +inf and -1 when no process acts.
// Only the winner's logarithm and division are taken in FP64.  The others are
// ruled out in FP32: with L = -log2(u), the hardware logarithm of u rounded to
// FP32 is off by at most 1.2e-7 L (every float in [2^-54, 1) checked) plus 1.9e-7
// for the rounding of u, and the product with 1/rate by a few 6e-8 of itself,
// inside the margins 1e-6 L + 4e-7 below.  Two processes whose intervals overlap
// are compared by their FP64 lengths (about one step in 1e5), so the choice and
// the length are those of the FP64 comparison of all.  Rates beyond 1e+-30 have
// the interval [0, inf].
__device__ __forceinline__ double physics_length(CQ rate, int n_proc, int mat, uint64_t seed, uint32_t track,
                                                 uint32_t step, int* proc) {
  int bp = -1;
  uint64_t bw = 0;
  double br = 1.0;
  float blo = 0.0f, bhi = 0.0f;
  for (int i = 0; i < n_proc; ++i) {
    const double r = rate[mat * n_proc + i];
    if (!(r > 0.0)) continue;
    uint32_t c[4] = {track, step, (uint32_t)i, 0u};
    philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint64_t w = ((uint64_t)c[0] << 32) | c[1];
    const float l = -__builtin_amdgcn_logf(uniform32(c[0], c[1])), e = fmaf(l, 1e-6f, 4e-7f), inv = __builtin_amdgcn_rcpf((float)r);
    const bool sane = r > 1e-30 && r < 1e30;
    const float lo = sane ? (l - e) * inv : 0.0f, hi = sane ? (l + e) * inv : __builtin_huge_valf();
    bool take = bp < 0 || hi < blo;
    if (!take && lo <= bhi) take = length_of(w, r) < length_of(bw, br);
    if (take) {
      bp = i;
      bw = w;
      br = r;
      blo = lo;
      bhi = hi;
    }
  }
  *proc = bp;
  return bp < 0 ? GV_INF : length_of(bw, br);
}

}  // namespace gv
