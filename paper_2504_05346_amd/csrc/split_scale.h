// Scales of the two-way fp16 split (gemm_tile_h2.h).  Plain C++ but for the qualifiers: the host tests compile
// it by itself.
#pragma once
#include <cstdint>

namespace thanos {

// The power of two that brings values of magnitude up to `bound` into [2^14, 2^15); finite for every bound.
// Its biased exponent (1 .. 253), which is all that a table of scales needs to hold, ...
__host__ __device__ inline uint32_t h2_exponent(float bound) {
  uint32_t u;
  __builtin_memcpy(&u, &bound, 4);
  const int e = (int)((u >> 23) & 255u);                  // biased exponent of the bound
  const int t = e == 0 ? 254 : 127 + 14 + 127 - e;        // biased exponent of the scale
  return (uint32_t)(t < 1 ? 1 : t > 253 ? 253 : t);
}
// ... and the scale itself.
__host__ __device__ inline float exponent_scale(uint32_t e) {
  const uint32_t v = e << 23;
  float s;
  __builtin_memcpy(&s, &v, 4);
  return s;
}
__host__ __device__ inline float h2_scale(float bound) { return exponent_scale(h2_exponent(bound)); }

// The power of two that brings a column whose largest magnitude is m into [1/2, 1); within 2^+-100 for every
// m (magnitudes of U are: they are 1 / sqrt of what fp32 holds), and 1 for a column of zeros.
__host__ __device__ inline float col_scale(float m) {
  uint32_t u;
  __builtin_memcpy(&u, &m, 4);
  const int e = (int)((u >> 23) & 255u), t = 253 - e;
  const uint32_t v = (uint32_t)(e == 0 ? 127 : t < 27 ? 27 : t > 227 ? 227 : t) << 23;
  float s;
  __builtin_memcpy(&s, &v, 4);
  return s;
}

}  // namespace thanos
