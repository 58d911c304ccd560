// Host check of the FP32 draw that rules physics lengths out: its logarithm
// against the FP64 draw's, over the smallest draws and ordinary ones.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>

#include "../../paper_1512_06637_amd/csrc/gv_phys.h"

int main() {
  double worst = 0.0;
  uint32_t x = 12345u;
  for (uint32_t hi : {0u, 1u, 2u, 7u, 255u, 65535u, 65536u, 0x00FFFFFFu, 0x01000001u, 0x7FFFFFFFu, 0x80000000u, 0xFFFFFF7Fu,
                      0xFFFFFFFFu})
    for (int i = 0; i < 200000; ++i) {
      x = x * 1664525u + 1013904223u;
      const uint32_t lo = i < 5000 ? (uint32_t)i : i < 6000 ? 0xFFFFFFFFu - (uint32_t)(i - 5000) : x >> (i % 24);
      const double u = gv::uniform_of((uint64_t)hi << 32 | lo), v = gv::uniform32(hi, lo);
      const double d = std::fabs(std::log2(v) - std::log2(u));
      if (!(d <= worst)) {
        worst = d;
        if (!(d <= 1.9e-7)) {
          std::printf("hi %u lo %u: log2 differs by %g\n", hi, lo, d);
          return 1;
        }
      }
    }
  std::printf("OK %g\n", worst);
  return 0;
}
