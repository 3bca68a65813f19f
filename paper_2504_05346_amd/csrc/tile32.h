// 32x32 tiles in the registers of one wavefront: layouts, LDS form, products and the elimination of a
// diagonal tile, on v_mfma_f32_32x32x2_f32.  Used by the per-row solvers and by the factorisation.
//
// ACCUMULATOR layout: register r of lane (lo, hi) = X[tl_row(r, hi)][lo].
// OPERAND layout:     register r of lane (lo, hi) = X[lo][tl_row(r, hi)], i.e. the accumulator layout of
// X^T.  It is what either operand of an MFMA over the columns looks like (both sides take the
// k-values in the same permuted order), and an accumulator tile is a second operand over its rows.
// In LDS a tile in operand layout is [k / 4][row][k % 4] with kRsGroup floats per group: a lane's 16
// values are four 16-byte pieces, consecutive lanes are 16 bytes apart, and the 4-byte accesses
// of the transposed view (lane <-> k) are 4 floats apart from group to group.
#pragma once
#include "common.h"

namespace thanos {

// The value of lane (l & 31) for every lane l: the lower half of the wavefront broadcast to the
// upper half (one v_permlane32_swap, no trip through LDS).
__device__ __forceinline__ float lower_half(float v) {
  const unsigned int u = __float_as_uint(v);
  return __uint_as_float(__builtin_amdgcn_permlane32_swap(u, u, false, false)[0]);
}

__device__ __forceinline__ int tl_row(int r, int hi) { return 8 * (r >> 2) + 4 * hi + (r & 3); }
// Original row of row x of a tile loaded in elimination order (see tl_eliminate).
__device__ __forceinline__ int tl_nat(int x) { return (x & ~7) + 2 * (x & 3) + ((x >> 2) & 1); }

constexpr int kRsGroup = 132;
constexpr int kRsTile = 8 * kRsGroup;

__device__ __forceinline__ void rs_store(float* tile, const f32x16& v, int lo, int hi) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[4 * g + e];
    *reinterpret_cast<f32x4*>(tile + (2 * g + hi) * kRsGroup + 4 * lo) = x;
  }
}
// the transposed view of a tile in LDS: element (tl_row(r, hi), k = lo) is at rs_col()[rs_step(r)]
__device__ __forceinline__ int rs_col(int lo, int hi) {
  return (lo >> 2) * kRsGroup + (lo & 3) + 16 * hi;
}
__device__ __forceinline__ constexpr int rs_step(int r) { return 32 * (r >> 2) + 4 * (r & 3); }
// acc += A B^T (NEG: -=), A in LDS, B in LDS or in registers.  The operands come 16 bytes at a time:
// with whole tiles of them the kernels that use this do not fit 128 registers.
__device__ __forceinline__ f32x4 rs_piece(const float* tile, int g, int lo, int hi) {
  return *reinterpret_cast<const f32x4*>(tile + (2 * g + hi) * kRsGroup + 4 * lo);
}
template <bool NEG>
__device__ __forceinline__ void rs_mma(f32x16& acc, const float* a, const float* b, int lo, int hi) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = rs_piece(a, g, lo, hi), y = rs_piece(b, g, lo, hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(NEG ? -x[e] : x[e], y[e], acc, 0, 0, 0);
  }
}
template <bool NEG>
__device__ __forceinline__ void rs_mma(f32x16& acc, const float* a, const f32x16& b, int lo, int hi) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = rs_piece(a, g, lo, hi);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(NEG ? -x[e] : x[e], b[4 * g + e], acc, 0, 0, 0);
  }
}

// ---- products on the fp16 matrix cores ----
// x = x1 + x2 in fp16 for |x| < 2^15 (gemm_tile_h2.h), a1 b1 + a1 b2 + a2 b1 (a2 b2 is dropped although a tile is
// 32 values deep: an element sums up to seven such products and then goes through an elimination; what one
// block adds to the weights is off float64 by 4.8 and 6.4e-7 at 128 and 256 unknowns, 5.1 and 7.0 with fp32 MFMAs,
// by 10.5 against 10.9 for independent channels): six MFMAs of 32 cycles for the
// 32 k-values of two tiles instead of sixteen of 64.  An operand-layout tile's registers 8 m .. 8 m + 7 are
// the k-values of MFMA m, the same ones in both operands.  In LDS a split tile is four 16-byte pieces per
// lane (x1, x2 of m = 0, then of m = 1), in the lanes' order: kRsTile floats hold it.
struct RsSplit {
  f16x8 x1[2], x2[2];
};
__device__ __forceinline__ RsSplit rs_split_h2(const f32x16& v) {
  RsSplit s;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    u32x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x2 x = {v[8 * m + 2 * e], v[8 * m + 2 * e + 1]};
      const f16x2 x1 = __builtin_convertvector(x, f16x2);
      const f32x2 r = {x[0] - (float)x1[0], x[1] - (float)x1[1]};
      h[e] = __builtin_bit_cast(uint32_t, x1);
      l[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
    }
    s.x1[m] = __builtin_bit_cast(f16x8, h);
    s.x2[m] = __builtin_bit_cast(f16x8, l);
  }
  return s;
}
__device__ __forceinline__ void rs_store_h2(float* tile, const RsSplit& s, int lane) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    *reinterpret_cast<f16x8*>(tile + 256 * (2 * m) + 4 * lane) = s.x1[m];
    *reinterpret_cast<f16x8*>(tile + 256 * (2 * m + 1) + 4 * lane) = s.x2[m];
  }
}
// acc += A A^T, A in registers; the same sums as rs_mma_h2
__device__ __forceinline__ void rs_mma_h2(f32x16& acc, const RsSplit& a) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.x2[m], a.x1[m], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.x1[m], a.x2[m], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.x1[m], a.x1[m], acc, 0, 0, 0);
  }
}
// acc += A B^T, both split tiles in LDS
__device__ __forceinline__ void rs_mma_h2(f32x16& acc, const float* a, const float* b, int lane) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const f16x8 a1 = *reinterpret_cast<const f16x8*>(a + 256 * (2 * m) + 4 * lane);
    const f16x8 a2 = *reinterpret_cast<const f16x8*>(a + 256 * (2 * m + 1) + 4 * lane);
    const f16x8 b1 = *reinterpret_cast<const f16x8*>(b + 256 * (2 * m) + 4 * lane);
    const f16x8 b2 = *reinterpret_cast<const f16x8*>(b + 256 * (2 * m + 1) + 4 * lane);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b1, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b2, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b1, acc, 0, 0, 0);
  }
}

// The power of two that brings a normal uniform d > 0, from a v_readlane, to [2, 4), on the vector unit (the detour through
// the scalar unit takes 14 cycles of a chain).  Scaling by it is exact, and keeps the determinants of pairs of pivots in
// the range of fp32 whenever the pivots are.  exponents: 0x7f800000 in a register.  d comes in a vector register: a
// vector instruction may read what v_readlane has written only two wait states later, which the compiler sees to for
// its own move, not for an instruction in here.  (With the scalar register and s_nop 1 in here the same times.)
__device__ __forceinline__ float pivot_scale(float d, float exponents) {
  float ps;
  asm("v_bfi_b32 %0, %1, 0, %2" : "=v"(ps) : "v"(d), "v"(exponents));
  return ps;
}

// Eliminates the symmetric tile D (accumulator layout), F F^T = D, and applies the same row
// operations to E: E = I becomes T = F^{-1}, E = A^T becomes F^{-1} A^T = (A F^{-T})^T, the tile of
// the factor next to D.  One wavefront.  aux: 32 floats of LDS.  Returns the pivot of column lo (not
// positive: not positive definite).  KEEP_F: U becomes F in operand layout.
//
// Two pivots per MFMA.  In the accumulator layout rows k and k + 4 (k mod 8 < 4) sit in the same
// register, in the lower and in the upper half of the wavefront: exactly where the two
// reduction slots of v_mfma_f32_32x32x2_f32 take their operands from.  The pivots are therefore
// taken in the order 0,4,1,5,2,6,3,7,8,12,...: with u1 = row k and u2 = row k + 4 AFTER the
// elimination of k (u2 = D[k+4] - (D[k][k+4] / d1) u1; the lower half's row is fetched with one
// cross-lane read), D -= u1 u1^T / d1 + u2 u2^T / d2 is one MFMA instead of two half-empty
// ones.  F is the Cholesky factor in that pivot order: a row-permuted triangle, or a triangle if
// the tile was loaded with its rows and columns in the order tl_nat.
// mid() is called half way.
struct TlNothing {
  __device__ __forceinline__ void operator()() const {}
};
template <bool KEEP_F, typename Mid = TlNothing>
__device__ __forceinline__ float tl_eliminate(f32x16 D, f32x16& E, f32x16& U, float* aux, int lo,
                                              int hi, const Mid& mid = Mid()) {
  // place of column lo in the order of elimination, one less in the upper half: what a half of the second operand
  // keeps; and the column whose pivot the half takes, shifted to k1
  const int rank = 2 * (4 * (lo >> 3) + (lo & 3)) + ((lo >> 2) & 1) - hi, own = lo - 4 * hi;
  float exponents = __uint_as_float(0x7f800000u);
  asm volatile("" : "+v"(exponents));
  float dl = 1.f;                             // pivot of column lo, in the half that takes it
#pragma unroll
  for (int t = 0; t < 16; ++t) {              // pair t: rows k1 and k2 = k1 + 4, both in D[t]
    if (t == 8) mid();
    const int k1 = 8 * (t >> 2) + (t & 3), k2 = k1 + 4;
    const float v = D[t];                     // lower half: D[k1][lo], upper half: D[k2][lo]
    const float x = lower_half(v);            // D[k1][lo] in both halves
    const float d1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k1));
    const float c12 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k2));
    const float d2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32 + k2));
    // 1 / d1 and 1 / d2' (d2' = d2 - c12^2 / d1, the pivot of k2 after the elimination of k1)
    // from two INDEPENDENT reciprocals, of d1 and of det = d1 d2 - c12^2: d2' = det / d1, row k1
    // scaled to a pivot e1 = ps d1 near one.  The wavefront is alone on this chain, so its length is
    // what counts: every instruction is 4 cycles, an MFMA 64 (the wavefront's own vector instructions wait for it).
    const float ps = pivot_scale(d1, exponents);
    const float e1 = ps * d1, e12 = ps * c12;
    const float cc = e12 * c12;
    const float det = fmaf(e1, d2, -cc) - fmaf(e12, c12, -cc);
    const float q1 = __builtin_amdgcn_rcpf(e1);
    const float qd = __builtin_amdgcn_rcpf(det);
    const float re = fmaf(fmaf(-e1, q1, 1.f), q1, q1);
    const float rd = fmaf(fmaf(-det, qd, 1.f), qd, qd);
    const float m = e12 * re;
    const float d2p = det * re;
    const float r1 = ps * re;
    const float r2 = e1 * rd;
    const float mh = hi ? m : 0.f;
    // second operands: u1 in the lower half, u2 in the upper half; columns eliminated by
    // earlier pairs are zero, and so is column k1 of u2
    float bop = fmaf(-mh, x, v);
    bop = rank >= 2 * t ? bop : 0.f;
    const float aop = bop * (hi ? -r2 : -r1);
    D = __builtin_amdgcn_mfma_f32_32x32x2f32(aop, bop, D, 0, 0, 0);
    if (KEEP_F) U[t] = bop;
    // the same row operations on E: row k1 as it is, row k2 after the operation of k1; the
    // pivot rows themselves stay
    const float ev = E[t];
    const float xe = lower_half(ev);
    const float be = fmaf(-mh, xe, ev);
    const bool mine = own == k1;
    const float a2 = mine ? 0.f : aop;
    dl = mine ? (hi ? d2p : d1) : dl;
    E = __builtin_amdgcn_mfma_f32_32x32x2f32(a2, be, E, 0, 0, 0);
  }
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(dl), __float_as_uint(dl), false, false);
  dl = __uint_as_float((lo >> 2) & 1 ? halves[1] : halves[0]);
  float isd = __builtin_amdgcn_rsqf(dl);
  isd = fmaf(0.5f * isd, fmaf(-dl * isd, isd, 1.f), isd);
  aux[lo] = isd;  // both halves write the same value
#pragma unroll
  for (int r = 0; r < 16; ++r) {  // rows of E, columns of F: / sqrt(d)
    E[r] *= aux[tl_row(r, hi)];
    if (KEEP_F) U[r] *= aux[tl_row(r, hi)];
  }
  return dl;
}

}  // namespace thanos
