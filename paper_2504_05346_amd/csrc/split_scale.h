// Scales of the two-way fp16 split (gemm_tile_h2.h).  Plain C++ but for the qualifiers: the host tests compile
// it by itself.
#pragma once
#include <cstdint>

namespace thanos {

// The power of two that brings values of magnitude up to `bound` into [2^14, 2^15); finite for every bound.
__host__ __device__ inline float h2_scale(float bound) {
  uint32_t u;
  __builtin_memcpy(&u, &bound, 4);
  const int e = (int)((u >> 23) & 255u);                  // biased exponent of the bound
  const int t = e == 0 ? 254 : 127 + 14 + 127 - e;        // biased exponent of the scale
  const uint32_t v = (uint32_t)(t < 1 ? 1 : t > 253 ? 253 : t) << 23;
  float s;
  __builtin_memcpy(&s, &v, 4);
  return s;
}

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
