// Device side of the serving engine: the round's basket table and the fused
// mixed-query kernel that answers a round (host side in gv_serve.h).
#pragma once
#include "gv_step.h"

namespace gv {

enum { kQStep = 0, kQSafety = 1, kQInside = 2 };

// One basket of a round; the fused kernel reads the round's table.
struct SDesc {
  int32_t kind, prec;
  int64_t n;
  int64_t tile0;    // first 64-track tile of the basket within the round
  int64_t in_off;   // byte offset of its inputs in the input arena
  int64_t out_off;  // byte offset of its outputs in the output arena
  int64_t pad;
};
static_assert(sizeof(SDesc) == 48, "SDesc layout");

constexpr int kServeMaxSlots = 1024;

// Bytes of one basket in host layout (gvgeom.h, serving section).
__host__ __device__ inline int64_t serve_in_bytes(int kind, int64_t n) { return (kind == kQStep ? 60 : 28) * n; }
__host__ __device__ inline int64_t serve_out_bytes(int kind, int64_t n) {
  return (kind == kQStep ? 16 : kind == kQSafety ? 8 : 1) * n;
}

// Fused mixed-query kernel: one wavefront answers one tile of 64 tracks of one
// basket, so the query kind and precision are wavefront-uniform; a basket's
// tracks may sit in different volumes (per-lane navigation state).  Composites at
// 2 waves per SIMD, as the single steps (the compiler's choice was 1).
template <int K>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K == kComposites ? 2 : 1))) k_serve(DevGeom G, const SDesc* __restrict__ desc, int nb, int64_t ntiles,
                                               const char* __restrict__ din, char* __restrict__ dout) {
  __shared__ int64_t t0[kServeMaxSlots + 1];
  for (int b = threadIdx.x; b < nb; b += blockDim.x) t0[b] = desc[b].tile0;
  if (threadIdx.x == 0) t0[nb] = ntiles;
  __syncthreads();
  const int lane = __lane_id();
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
  const int64_t nwaves = (int64_t)gridDim.x * blockDim.x / 64;
  for (int64_t t = wave; t < ntiles; t += nwaves) {
    int lo = 0, hi = nb - 1;  // largest b with t0[b] <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (t0[mid] <= t) lo = mid;
      else hi = mid - 1;
    }
    const int b = __builtin_amdgcn_readfirstlane(lo);
    const int kind = desc[b].kind, prec = desc[b].prec;
    const int64_t n = desc[b].n;
    const int64_t i = (t - t0[b]) * 64 + lane;
    if (i >= n) continue;
    const double* X = (const double*)(din + desc[b].in_off);
    char* O = dout + desc[b].out_off;
    const V3 p{X[i], X[n + i], X[2 * n + i]};
    if (kind == kQStep) {
      const V3 d{X[3 * n + i], X[4 * n + i], X[5 * n + i]};
      const double ps = X[6 * n + i];
      const int v = ((const int32_t*)(X + 7 * n))[i];
      uint32_t fl;
      int nx;
      const double st = prec == 0 ? step_query<false, K>(G, v, p, d, ps, &nx, &fl) : step_query<true, K>(G, v, p, d, ps, &nx, &fl);
      double* os = (double*)O;
      int32_t* on = (int32_t*)(os + n);
      uint32_t* of = (uint32_t*)(on + n);
      os[i] = st;
      on[i] = nx;
      of[i] = fl;
    } else {
      const int v = ((const int32_t*)(X + 3 * n))[i];
      const bool ok = v >= 0 && v < G.n_pv;
      if (kind == kQSafety) {
        ((double*)O)[i] = !ok ? 0.0 : prec == 0 ? nav_safety<K>(G, v, p) : nav_safety_screened<K>(G, v, p);
      } else {
        int8_t c = (int8_t)kOutside;
        if (ok) {
          const LvRec m = lv_rec(G, pv_rec(G, v).lv);
          const V3 pl = to_child_p(G.pv_gxf + 12 * (size_t)v, p);
          c = (int8_t)code_of(solid_sgn<K>(m.type, G.par + m.par, pl));
        }
        ((int8_t*)O)[i] = c;
      }
    }
  }
}

}  // namespace gv
