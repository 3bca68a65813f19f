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
// values span e^6 also get better.  Shorter sums round less often, and the three-way split is the more accurate
// one (16: 3.4 against 8.5e-8, 64: 1.10 against 1.13e-7, equal near 72): the sweep's update stays there up to 64
// (kShortK), the lowest merges of the inverse and k_gemm_direct take a2 b2 as well.  The products of 32 x 32
// tiles inside the tiled solver (tile32.h) are parts of sums of up to 256 values and drop it.
// The bound has to be near the values: from 2^-17 of it down an operand loses a bit per power of two.
// Rates, read-modify-write of C included: 10752^2 at K = 512 160 -> 230 TFLOP/s, 8192^2 at K = 1024 184 -> 273,
// K = 4096 198 -> 303.
//
// Same division of labour as in gemm_tile_x3.h (four multiplying, four splitting wavefronts, two
// workgroups per compute unit); four planes instead of six in LDS, 5 instead of 11 vector instructions
// per pair of values.  A slab is 40 KB, so two buffers and two workgroups fill the LDS exactly, and the
// splitting can run one slab ahead of the multiplying with one barrier per slab (NBUF = 2): 10752^2 at
// K = 512 221 -> 238 TFLOP/s, 16384^2 at K = 128 126 -> 139, 8192^2 at K = 4096 305 -> 312, the factorisation
// of 11008 columns 7.01 -> 6.74 ms.  One buffer and two barriers where a workgroup has to fit beside one that
// takes 84 KB (the factorisation next to the row losses: 5120 columns 5.23 against 5.40 ms).
#pragma once
#include "gemm_tile_x3.h"
#include "split_scale.h"

namespace thanos {

// LDS view of a buffer: operand {a, b} x plane {x1, x2}
__device__ __forceinline__ char* h2_plane(char* buf, int operand, int plane) {
  return buf + (operand * 2 + plane) * kXPlane;
}
constexpr int kH2Buf = 4 * kXPlane;                 // one slab
constexpr size_t kH2SmemBytes = 2 * (size_t)kH2Buf;  // half of a compute unit's LDS (NBUF = 1: kXSmemBytes)
static_assert(kH2SmemBytes >= kXSmemBytes && 2 * kH2SmemBytes <= 160 * 1024, "staged tile fits, two per unit");
static_assert(kH2Buf <= kXSmemBytes, "one buffer fits where the tile is staged");

constexpr float kWideH2 = 0x1p11f;

// 1 / s for a power of two between 2^-126 and 2^126
__device__ __forceinline__ float pow2_inv(float s) { return __uint_as_float((254u << 23) - __float_as_uint(s)); }

// WIDE: the second term is 2^11 times as large.
template <bool WIDE = false>
__device__ __forceinline__ void split2_h2(float x0, float x1, float s0, float s1, uint32_t (&packed)[2]) {
  const f32x2 v = {x0 * s0, x1 * s1};
  const f16x2 h = __builtin_convertvector(v, f16x2);
  f32x2 r = {fmaf(x0, s0, -(float)h[0]), fmaf(x1, s1, -(float)h[1])};
  if (WIDE) r *= kWideH2;
  const f16x2 l = __builtin_convertvector(r, f16x2);
  packed[0] = __builtin_bit_cast(uint32_t, h);
  packed[1] = __builtin_bit_cast(uint32_t, l);
}

// eight values of a lane, in the order in which the MFMA takes them
__device__ __forceinline__ void split8_h2(const f32x4& x, const f32x4& y, float s, f16x8& hi, f16x8& lo) {
  u32x4 h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t pk[2];
    split2_h2(e < 2 ? x[2 * e] : y[2 * e - 4], e < 2 ? x[2 * e + 1] : y[2 * e - 3], s, s, pk);
    h[e] = pk[0];
    l[e] = pk[1];
  }
  hi = __builtin_bit_cast(f16x8, h);
  lo = __builtin_bit_cast(f16x8, l);
}

// Scales of the columns of B as biased exponents, n rows (>= 1) of them of stride ld: a column takes the
// smallest.  Read four at a time at any alignment.
struct ColScalesH2 {
  const uint8_t* e;
  int64_t ld;
  int n;
};
// Scale of an operand: one for all of it, or (rows) that times one per row of A or column of B.
struct ScaleH2 {
  float all;
  float row[8];  // of this thread's pieces: rows (u >> 3) + 16 q of A, columns 4 (u & 31) + 0 .. 3 of B
  ColScalesH2 cols;
  uint32_t first[4];
};
template <bool TOPS>
__device__ __forceinline__ void load_rows_h2(ScaleH2& sc, const float* __restrict__ rows, int ext, int u) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float v = rows[min((u >> 3) + 16 * q, ext - 1)];
    sc.row[q] = TOPS ? h2_scale(v) : sc.all * v;
  }
}
// TOPS, columns of B: from their largest magnitudes (n_ext of them).
__device__ __forceinline__ void load_col_tops_h2(ScaleH2& sc, const float* __restrict__ tops, int n_ext, int u) {
#pragma unroll
  for (int q = 0; q < 4; ++q) sc.row[q] = h2_scale(tops[min(4 * (u & 31) + q, n_ext - 1)]);
}
// In two steps, so that the requests for the first slab go out in between: the first four rows of exponents are
// requested, ...
typedef uint32_t u32u __attribute__((aligned(1)));
__device__ __forceinline__ void load_cols_h2(ScaleH2& sc, const ColScalesH2& c, int ext4, int u) {
  sc.cols = c;
  sc.cols.e += min(4 * (u & 31), ext4 - 4);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    sc.first[k] = *reinterpret_cast<const u32u*>(sc.cols.e + (int64_t)min(k, c.n - 1) * c.ld);
}
// ... and made into scales, with the others if there are more.
__device__ __forceinline__ void finish_cols_h2(ScaleH2& sc) {
  uint32_t lo[4] = {253u, 253u, 253u, 253u};
  auto take = [&](uint32_t v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) lo[q] = min(lo[q], (v >> (8 * q)) & 255u);
  };
#pragma unroll
  for (int k = 0; k < 4; ++k) take(sc.first[k]);
  for (int t = 4; t < sc.cols.n; t += 4) {
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      v[k] = *reinterpret_cast<const u32u*>(sc.cols.e + (int64_t)min(t + k, sc.cols.n - 1) * sc.cols.ld);
#pragma unroll
    for (int k = 0; k < 4; ++k) take(v[k]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) sc.row[q] = exponent_scale(lo[q]);
}

// KF: the k-values of a row-major operand are multiplied by kf first (this thread's four of the slab).
template <bool KMAJOR, bool MASKED, bool ROWS, bool KF, bool WIDE>
__device__ __forceinline__ void slab_store_h2(char* smem, int operand, const SlabRegsX3& rin,
                                              const ScaleH2& sc, int u, const f32x4& kf) {
  SlabRegsX3 r = rin;
  if (KF) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      r.v[q] = make_float4(r.v[q].x * kf[0], r.v[q].y * kf[1], r.v[q].z * kf[2], r.v[q].w * kf[3]);
  }
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
        const float s = ROWS ? sc.row[mm] : sc.all;
        split2_h2(c[2 * e], c[2 * e + 1], s, s, pk);
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
      split2_h2<WIDE>(r.v[q].x, r.v[q].y, s, s, lo2);
      split2_h2<WIDE>(r.v[q].z, r.v[q].w, s, s, hi2);
      const int off = ((u >> 3) + 16 * q) * kXRow + 8 * (u & 7);
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<uint2*>(pl[p] + off) = make_uint2(lo2[p], hi2[p]);
    }
  }
}

// Between two slabs: with two buffers the barrier says that slab it is in LDS and that slab it - 1 has been
// read; with one the second says that slab it has been read.
template <int NBUF>
__device__ __forceinline__ void h2_handover() {
  __syncthreads();
  if (NBUF == 1) __syncthreads();
}

// Reciprocals of this thread's four k-values' divisors in slab it (KF).
template <bool KF>
__device__ __forceinline__ f32x4 slab_factors_h2(const float* __restrict__ kd, int it, int klen, int u) {
  f32x4 f{};
  if (!KF) return f;
  const int k = it * kXK + 4 * (u & 7);
  if ((klen & 3) == 0) {
    f = *reinterpret_cast<const f32x4u*>(kd + min(k, klen - 4));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = kd[min(k + e, klen - 1)];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = pow2_inv(f[e]);
  return f;
}

// The producers of gemm_tile_x3.h with the two-way split; slab it goes to buffer it % NBUF.
template <bool KMAJOR, bool ROWS, int NBUF, bool TOPS, bool KF>
__device__ __forceinline__ void h2_produce4(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                            int ext, int kbeg, ScaleH2& sc, int u, const float* __restrict__ kd) {
  SlabSrcX3 src;
  slab_src_x3<KMAJOR>(src, P, ld, ext, kbeg, u);
  SlabRegsX3 r0, r1;
  slab_load_x3<KMAJOR, true>(r0, src, 0, 4 * kXK, P);
  slab_load_x3<KMAJOR, true>(r1, src, 1, 3 * kXK, P);
  f32x4 f[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) f[it] = slab_factors_h2<KF>(kd, it, 4 * kXK, u);
  if (KMAJOR && ROWS && !TOPS) finish_cols_h2(sc);
  char* const second = smem + (NBUF - 1) * kH2Buf;
  slab_store_h2<KMAJOR, false, ROWS, KF, TOPS && !KF && !KMAJOR>(smem, operand, r0, sc, u, f[0]);
  slab_load_x3<KMAJOR, true>(r0, src, 2, 2 * kXK, P);
  h2_handover<NBUF>();
  slab_store_h2<KMAJOR, false, ROWS, KF, TOPS && !KF && !KMAJOR>(second, operand, r1, sc, u, f[1]);
  slab_load_x3<KMAJOR, true>(r1, src, 3, kXK, P);
  h2_handover<NBUF>();
  slab_store_h2<KMAJOR, false, ROWS, KF, TOPS && !KF && !KMAJOR>(smem, operand, r0, sc, u, f[2]);
  h2_handover<NBUF>();
  slab_store_h2<KMAJOR, false, ROWS, KF, TOPS && !KF && !KMAJOR>(second, operand, r1, sc, u, f[3]);
  h2_handover<NBUF>();
}

template <bool KMAJOR, bool FAST, bool MASKED, bool ROWS, int NBUF, bool TOPS, bool KF>
__device__ __forceinline__ void h2_produce(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                           int ext, int kbeg, int kend, int nslab, ScaleH2& sc, int u,
                                           const float* __restrict__ kd) {
  SlabSrcX3 src;
  slab_src_x3<KMAJOR>(src, P, ld, ext, kbeg, u);
  const int klen = kend - kbeg;
  SlabRegsX3 r;
  slab_load_x3<KMAJOR, FAST>(r, src, 0, klen, P);
  f32x4 f = slab_factors_h2<KF>(kd, 0, klen, u);
  if (KMAJOR && ROWS && !TOPS) finish_cols_h2(sc);
  for (int it = 0; it < nslab; ++it) {
    if (operand == 0 && u < 64) TL_MARK(8 + 4 * it);
    slab_store_h2<KMAJOR, MASKED, ROWS, KF, TOPS && !KF && !KMAJOR>(smem + (NBUF == 2 ? (it & 1) * kH2Buf : 0), operand, r, sc, u, f);
    slab_load_x3<KMAJOR, FAST>(r, src, it + 1, klen - (it + 1) * kXK, P);
    f = slab_factors_h2<KF>(kd, it + 1, klen, u);
    if (operand == 0 && u < 64) TL_MARK(8 + 4 * it + 1);
    h2_handover<NBUF>();
  }
}

template <bool KMAJOR, bool ROWS, int NBUF, bool PIECES, bool TOPS, bool KF>
__device__ __forceinline__ void h2_producer(char* smem, int operand, const float* __restrict__ P, int64_t ld,
                                            int ext, int kbeg, int kend, ScaleH2& sc, int u,
                                            const float* __restrict__ kd) {
  const int nslab = (kend - kbeg + kXK - 1) / kXK;
  const bool fast = (KMAJOR ? ext : kend - kbeg) % 4 == 0;
  const bool whole = ext == 128 && (kend - kbeg) % kXK == 0;
  if (fast && whole && kend - kbeg == 4 * kXK) h2_produce4<KMAJOR, ROWS, NBUF, TOPS, KF>(smem, operand, P, ld, ext, kbeg, sc, u, kd);
  else if (fast && whole) h2_produce<KMAJOR, true, false, ROWS, NBUF, TOPS, KF>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u, kd);
  else if (PIECES || fast) h2_produce<KMAJOR, true, true, ROWS, NBUF, TOPS, KF>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u, kd);
  else h2_produce<KMAJOR, false, false, ROWS, NBUF, TOPS, KF>(smem, operand, P, ld, ext, kbeg, kend, nslab, sc, u, kd);
}

// acc += (sa A)[0:128, kbeg:kend] (sb B)[kbeg:kend, 0:128]; otherwise as gemm_tile_x3().  A_ROWS: further
// scales of the m_ext rows of A.  B_COLS: of the columns of B, instead of sb; their reciprocals end in
// inv[0:128] (LDS beyond the buffers' use after the product), complete after the next barrier.
// B_PIECES: the extents of B are multiples of 4.  TOPS: what arows and btops (n_ext values) hold are the largest
// magnitudes of the rows and columns, not their scales.  KF: column k of A is divided by kd[k], a power of two
// (arows belongs to the result).  TOPS without KF: the values of a row of A may lie further apart than those of B.
// Their second terms are 2^11 times as large, which would be subnormal from 2^-17 of the row's largest value down (now
// from 2^-28), and meet first terms of B that are as much smaller: 4096 x 1366 times 1366 x 2730 125 -> 128 us.
template <bool A_KMAJOR, bool B_KMAJOR, int NBUF, bool A_ROWS = false, bool B_COLS = false, bool B_PIECES = false,
          bool TOPS = false, bool KF = false>
__device__ __forceinline__ void gemm_tile_h2(TileAcc& acc, char* smem, const float* __restrict__ A,
                                             int64_t lda, int m_ext, float sa, const float* arows,
                                             const float* __restrict__ B, int64_t ldb, int n_ext, float sb,
                                             const ColScalesH2& bcols, float* inv, int kbeg, int kend,
                                             const float* btops = nullptr, const float* kd = nullptr) {
  static_assert(!A_ROWS || !A_KMAJOR, "rows of A");
  static_assert(!B_COLS || (B_KMAJOR && (B_PIECES || TOPS)), "columns of B, four at a time");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (kend <= kbeg) return;
  const int nslab = (kend - kbeg + kXK - 1) / kXK;
  ScaleH2 sc;
  const int u = tid & 127;
  sc.all = wave >= 6 ? sb : sa;
  if (A_ROWS && wave >= 4 && wave < 6) load_rows_h2<TOPS>(sc, arows, m_ext, u);
  if (B_COLS && wave >= 6) {
    if (TOPS) load_col_tops_h2(sc, btops, n_ext, u);
    else load_cols_h2(sc, bcols, n_ext, u);
  }
  __syncthreads();  // previous users of the LDS buffers are done
  if (wave >= 6) {
    h2_producer<B_KMAJOR, B_COLS, NBUF, B_PIECES, TOPS, false>(smem, 1, B, ldb, n_ext, kbeg, kend, sc, u, nullptr);
  } else if (wave >= 4) {
    h2_producer<A_KMAJOR, A_ROWS, NBUF, false, TOPS, KF>(smem, 0, A, lda, m_ext, kbeg, kend, sc, u, KF ? kd + kbeg : nullptr);
  } else {
    const int wm = wave >> 1, wn = wave & 1;
    const int lo = lane & 31, hi = lane >> 5;
    const int a_off = (wm * 64 + lo) * kXRow + 16 * hi;
    const int b_off = (wn * 64 + lo) * kXRow + 16 * hi;
    for (int it = 0; it < nslab; ++it) {
      __syncthreads();  // slab it is in LDS
      if (wave == 0) TL_MARK(8 + 4 * it + 2);
      char* const buf = smem + (NBUF == 2 ? (it & 1) * kH2Buf : 0);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        f16x8 af[2][2], bf[2][2];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            af[f][p] = *reinterpret_cast<const f16x8*>(h2_plane(buf, 0, p) + a_off + f * 32 * kXRow + 32 * ks);
            bf[f][p] = *reinterpret_cast<const f16x8*>(h2_plane(buf, 1, p) + b_off + f * 32 * kXRow + 32 * ks);
          }
        f16x8 b1[2] = {bf[0][0], bf[1][0]};
        if (TOPS && !KF) {
#pragma unroll
          for (int g = 0; g < 2; ++g) b1[g] *= (_Float16)(1.f / kWideH2);
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
              acc.v[f][g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[f][pa[t]], t == 0 ? b1[g] : bf[g][pb[t]],
                                                                   acc.v[f][g], 0, 0, 0);
      }
      if (wave == 0) TL_MARK(8 + 4 * it + 3);
      if (NBUF == 1) __syncthreads();
    }
  }
  if (NBUF == 2) __syncthreads();  // the LDS is free
  if (B_COLS && wave == 6 && u < 32) {
#pragma unroll
    for (int q = 0; q < 4; ++q) inv[4 * u + q] = pow2_inv(sc.row[q]);
  }
}

}  // namespace thanos
