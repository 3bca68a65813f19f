// 128x128 fp32 tile product on the CDNA4 fp16 matrix cores with two-way operand splitting, for
// operands whose range is known.
//
// With a power of two s that brings the operand below 2^15, x s = x1 + x2 with x1 = fp16(x s) and
// x2 = fp16(x s - x1).  The remainder is exact in fp32 and has 12 significant bits left, one more than
// fp16 holds when it is in the upper half of its range: a quarter of the values lose their last bit,
// 2^-24 of the value in the root mean square (an fp32 rounding: 2^-24.8), as long as |x s| >= 2^-3;
// smaller values have an absolute error of at most 2^-25 / s.  The product is
//     a1 b1 + (a1 b2 + a2 b1),
// exact in the fp32 accumulator of v_mfma_f32_32x32x16_f16; a2 b2 (2^-23.6 |a||b| in the root mean
// square) is dropped.  Three MFMAs where the three-way bf16 split of gemm_tile_x3.h, which needs no
// range, takes six: what is dropped is made up for by half as many roundings of the running sum.
// 2048 x 2048 products of normal operands against float64, three-way -> two-way: K = 128 1.63 -> 1.43e-7,
// 512 3.4 -> 2.6e-7, 1024 4.9 -> 3.6e-7, 4096 10 -> 7.1e-7; equal signs, equal operands and rows whose
// values span e^6 also get better.  Rates, read-modify-write of C included: 10752^2 at K = 512 160 -> 230
// TFLOP/s, 8192^2 at K = 1024 184 -> 273, K = 4096 198 -> 303.
//
// Same division of labour as in gemm_tile_x3.h (four multiplying, four splitting wavefronts, two
// workgroups per compute unit); four planes instead of six in LDS, 5 instead of 11 vector instructions
// per pair of values.
#pragma once
#include "gemm_tile_x3.h"

namespace thanos {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// LDS view: operand {a, b} x plane {x1, x2}
__device__ __forceinline__ char* h2_plane(char* smem, int operand, int plane) {
  return smem + (operand * 2 + plane) * kXPlane;
}
static_assert(4 * (size_t)kXPlane <= kXSmemBytes, "the staged tile is the larger use of the LDS");

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

__device__ __forceinline__ void split2_h2(float x0, float x1, float s0, float s1, uint32_t (&packed)[2]) {
  const f32x2 v = {x0 * s0, x1 * s1};
  const f16x2 h = __builtin_convertvector(v, f16x2);
  const f32x2 r = {fmaf(x0, s0, -(float)h[0]), fmaf(x1, s1, -(float)h[1])};
  const f16x2 l = __builtin_convertvector(r, f16x2);
  packed[0] = __builtin_bit_cast(uint32_t, h);
  packed[1] = __builtin_bit_cast(uint32_t, l);
}

// Scale of an operand: one for all of it, or (rows) one per row m of the tile, which only an operand with
// A[m * ld + k] can have.
struct ScaleH2 {
  float all;
  float row[8];  // of the rows (u >> 3) + 16 q of this thread's pieces
};

template <bool KMAJOR, bool MASKED, bool ROWS>
__device__ __forceinline__ void slab_store_h2(char* smem, int operand, const SlabRegsX3& rin,
                                              const ScaleH2& sc, int u) {
  SlabRegsX3 r = rin;
  if (MASKED) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (!((r.ok >> q) & 1)) r.v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  char* pl[2] = {h2_plane(smem, operand, 0), h2_plane(smem, operand, 1)};
  if (KMAJOR) {
    const int m4 = 4 * (u & 31), kb = 16 * (u >> 5);
#pragma unroll
    for (int mm = 0; mm < 4; ++mm) {
      float c[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        c[q] = mm == 0 ? r.v[q].x : mm == 1 ? r.v[q].y : mm == 2 ? r.v[q].z : r.v[q].w;
      u32x4 o[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t pk[2];
        split2_h2(c[2 * e], c[2 * e + 1], sc.all, sc.all, pk);
        o[0][e] = pk[0];
        o[1][e] = pk[1];
      }
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<u32x4*>(pl[p] + (m4 + mm) * kXRow + kb) = o[p];
    }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float s = ROWS ? sc.row[q] : sc.all;
      uint32_t lo2[2], hi2[2];
      split2_h2(r.v[q].x, r.v[q].y, s, s, lo2);
      split2_h2(r.v[q].z, r.v[q].w, s, s, hi2);
      const int off = ((u >> 3) + 16 * q) * kXRow + 8 * (u & 7);
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<uint2*>(pl[p] + off) = make_uint2(lo2[p], hi2[p]);
    }
  }
}

// The producers of gemm_tile_x3.h with the two-way split.
template <bool KMAJOR, bool ROWS>
__device__ __forceinline__ void h2_produce4(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                            int ext, int kbeg, const ScaleH2& sc, int u) {
  SlabSrcX3 src;
  slab_src_x3<KMAJOR>(src, P, ld, ext, kbeg, u);
  SlabRegsX3 r0, r1;
  slab_load_x3<KMAJOR, true>(r0, src, 0, 4 * kXK, P);
  slab_load_x3<KMAJOR, true>(r1, src, 1, 3 * kXK, P);
  slab_store_h2<KMAJOR, false, ROWS>(smem, operand, r0, sc, u);
  slab_load_x3<KMAJOR, true>(r0, src, 2, 2 * kXK, P);
  __syncthreads();
  __syncthreads();
  slab_store_h2<KMAJOR, false, ROWS>(smem, operand, r1, sc, u);
  slab_load_x3<KMAJOR, true>(r1, src, 3, kXK, P);
  __syncthreads();
  __syncthreads();
  slab_store_h2<KMAJOR, false, ROWS>(smem, operand, r0, sc, u);
  __syncthreads();
  __syncthreads();
  slab_store_h2<KMAJOR, false, ROWS>(smem, operand, r1, sc, u);
  __syncthreads();
  __syncthreads();
}

template <bool KMAJOR, bool FAST, bool MASKED, bool ROWS>
__device__ __forceinline__ void h2_produce(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                           int ext, int kbeg, int kend, int nslab, const ScaleH2& sc,
                                           int u) {
  SlabSrcX3 src;
  slab_src_x3<KMAJOR>(src, P, ld, ext, kbeg, u);
  const int klen = kend - kbeg;
  SlabRegsX3 r;
  slab_load_x3<KMAJOR, FAST>(r, src, 0, klen, P);
  for (int it = 0; it < nslab; ++it) {
    slab_store_h2<KMAJOR, MASKED, ROWS>(smem, operand, r, sc, u);
    slab_load_x3<KMAJOR, FAST>(r, src, it + 1, klen - (it + 1) * kXK, P);
    __syncthreads();  // slab it is in LDS
    __syncthreads();  // consumers are done with it
  }
}

template <bool KMAJOR, bool ROWS>
__device__ __forceinline__ void h2_producer(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                            int ext, int kbeg, int kend, bool vec, const ScaleH2& sc, int u) {
  const int nslab = (kend - kbeg + kXK - 1) / kXK;
  const bool fast = vec && (KMAJOR ? ext % 4 == 0 : (kend - kbeg) % 4 == 0);
  const bool whole = ext == 128 && (kend - kbeg) % kXK == 0;
  if (fast && whole && kend - kbeg == 4 * kXK) h2_produce4<KMAJOR, ROWS>(smem, operand, P, ld, ext, kbeg, sc, u);
  else if (fast && whole) h2_produce<KMAJOR, true, false, ROWS>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u);
  else if (fast) h2_produce<KMAJOR, true, true, ROWS>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u);
  else h2_produce<KMAJOR, false, false, ROWS>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u);
}

// acc += (sa A)[0:128, kbeg:kend] (sb B)[kbeg:kend, 0:128]; otherwise as gemm_tile_x3().  arows: 128 scales
// of the rows of A instead of sa (LDS or global), read for rows < m_ext only.
template <bool A_KMAJOR, bool B_KMAJOR, bool A_ROWS = false>
__device__ __forceinline__ void gemm_tile_h2(TileAcc& acc, char* smem, const float* __restrict__ A,
                                             int64_t lda, int m_ext, float sa, const float* arows,
                                             const float* __restrict__ B, int64_t ldb, int n_ext, float sb,
                                             int kbeg, int kend, bool vec_a, bool vec_b) {
  static_assert(!(A_KMAJOR && A_ROWS), "row scales need A[m * ld + k]");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (kend <= kbeg) return;
  const int nslab = (kend - kbeg + kXK - 1) / kXK;
  ScaleH2 sc;
  const int u = tid & 127;
  sc.all = wave >= 6 ? sb : sa;
  if (A_ROWS && wave >= 4 && wave < 6) {
#pragma unroll
    for (int q = 0; q < 8; ++q) sc.row[q] = arows[min((u >> 3) + 16 * q, m_ext - 1)];
  }
  __syncthreads();  // previous users of the LDS buffers are done
  if (wave >= 6) {
    h2_producer<B_KMAJOR, false>(smem, 1, B, ldb, n_ext, kbeg, kend, vec_b, sc, u);
  } else if (wave >= 4) {
    h2_producer<A_KMAJOR, A_ROWS>(smem, 0, A, lda, m_ext, kbeg, kend, vec_a, sc, u);
  } else {
    const int wm = wave >> 1, wn = wave & 1;
    const int lo = lane & 31, hi = lane >> 5;
    const int a_off = (wm * 64 + lo) * kXRow + 16 * hi;
    const int b_off = (wn * 64 + lo) * kXRow + 16 * hi;
    for (int it = 0; it < nslab; ++it) {
      __syncthreads();  // slab it is in LDS
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        f16x8 af[2][2], bf[2][2];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            af[f][p] = *reinterpret_cast<const f16x8*>(h2_plane(smem, 0, p) + a_off + f * 32 * kXRow + 32 * ks);
            bf[f][p] = *reinterpret_cast<const f16x8*>(h2_plane(smem, 1, p) + b_off + f * 32 * kXRow + 32 * ks);
          }
        // small partial products first; consecutive MFMAs go to different accumulators
        constexpr int pa[3] = {1, 0, 0};
        constexpr int pb[3] = {0, 1, 0};
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int g = 0; g < 2; ++g)
              acc.v[f][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[f][pa[t]], bf[g][pb[t]], acc.v[f][g],
                                                                   0, 0, 0);
      }
      __syncthreads();  // done with it
    }
  }
}

}  // namespace thanos
