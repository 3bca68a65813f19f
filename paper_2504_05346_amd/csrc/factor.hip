// thanos_factor: damping, diagonal extraction and the upper factor U of the inverse of the
// damped Hessian, H_d^{-1} = U^T U.
//
// Why one factor is enough.  Alg. 1 of the paper re-inverts the residual Hessian
// H_d[j:, j:] after every block (O(b^4/B), App. G.6).  With V upper triangular and
// H_d = V V^T, the trailing sub-matrix is H_d[j:, j:] = V[j:, j:] V[j:, j:]^T, so with
// U = V^{-1} (also upper triangular) inv(H_d[j:, j:]) = U[j:, j:]^T U[j:, j:] for every j.
//
// How U is computed.  Reversing the index order turns H_d = V V^T into an ordinary Cholesky
// factorisation: with J the reversal, A' = J H_d J = L L^T (L lower), V = J L J and
// U = J L^{-1} J.  So: (1) reversed, zero/identity-padded copy A' (ld = bp, a multiple of the
// factor block NB = 128); (2) right-looking blocked Cholesky: diagonal block in one workgroup
// (which also produces the inverse of the diagonal block), panel = product with that inverse,
// trailing update on the matrix cores, two-level (rank NB inside an outer block of 4 factor
// blocks, rank 4 NB for everything right of it) while many block rows are left, then one launch per step (k_chol_step); (3) L^{-1} by recursive doubling over
// block pairs, X21 = -Linv22 * (L21 * Linv11), two products per level; (4) U = J L^{-1} J.
// Storage and chains are fp32; the products split their operands into two fp16 values (below).
//
// Ranges.  The copy of step (1) is D A' D with D diagonal, powers of two that bring the diagonal into
// [1, 4): every value of the factorisation is then the unscaled one times a power of two, so nothing
// changes in it, but |L_ij| <= 2 whatever the scales of the channels are (a row of L has the norm
// sqrt(A'_ii)), and the products can split their operands into two fp16 values (gemm_tile_h2.h)
// instead of three bf16 ones.  L^{-1} is bounded by what is written: every diagonal block and every
// merge leaves the largest magnitude of its block column in `bounds`.  Step (4) takes D out again.
#include <algorithm>

#include "factor_plan.h"
#include "gemm_tile_h2.h"
#include "tile32.h"

namespace thanos {

constexpr int NB = kFactorNB;
// ------------------------------------------------------------------------------------------
// xnorm2[j] = H[j][j];  lam = damping * mean_j H[j][j]  (sum in fp64, fixed order);  d[j] = the scale of
// channel j, d0[j] = that of the row losses (LOSSES; without the damping).  Also clears the n_bounds bounds.  One
// workgroup of 1024 threads.
template <bool LOSSES>
__global__ __launch_bounds__(1024) void k_diag_stats(const float* __restrict__ H, int64_t b,
                                                     float damping, float* __restrict__ xnorm2,
                                                     float* __restrict__ lam_out, float* __restrict__ d_out,
                                                     float* __restrict__ d0,
                                                     float* __restrict__ bounds, int n_bounds,
                                                     int32_t* __restrict__ info) {
  __shared__ double part[1024];
  double s = 0.0;
  for (int e = threadIdx.x; e < n_bounds; e += 1024) bounds[e] = 0.f;
  // eight loads in flight (each touches a page of its own); added in order
  float d[8];
  int64_t last = 0;  // what d holds: threadIdx.x + last + 1024 e
  for (int64_t j0 = threadIdx.x; j0 < b; j0 += 8 * 1024) {
    last = j0 - threadIdx.x;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t j = min(j0 + 1024 * e, b - 1);
      d[e] = H[j * b + j];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (j0 + 1024 * e < b) {
        xnorm2[j0 + 1024 * e] = d[e];
        s += (double)d[e];
      }
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  const float lam = (float)((double)damping * (part[0] / (double)b));
  if (threadIdx.x == 0) {
    *lam_out = lam;
    *info = 0;
  }
  for (int64_t j = threadIdx.x; j < last; j += 1024) {  // its own writes
    d_out[j] = diag_scale(xnorm2[j] + lam);
    if (LOSSES) d0[j] = loss_scale(xnorm2[j]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t j = threadIdx.x + last + 1024 * e;
    if (j < b) {
      d_out[j] = diag_scale(d[e] + lam);
      if (LOSSES) d0[j] = loss_scale(d[e]);
    }
  }
}

// *bound <- max(*bound, largest of the wavefronts' m), m >= 0 (NaN counts as large)
__device__ __forceinline__ void raise_bound(float* bound, float m) {
  uint32_t u = __float_as_uint(m);
  for (int off = 32; off > 0; off >>= 1) u = max(u, (uint32_t)__shfl_xor((int)u, off, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(reinterpret_cast<unsigned int*>(bound), u);
}

// Split tiles right of the diagonal (see k_chol_step): offset of piece e of tile (r, kt) from the first element of its block;
// ld: the matrix's.  A piece is two rows of 512 bytes; lane (lo, hi) has its 16 bytes hi * ld + 4 * lo further on.
__device__ __forceinline__ int64_t st_parked(int r, int kt, int e, int64_t ld) { return (8 * (4 * r + kt) + 2 * e) * ld; }

// A'[i][j] = (D H_d D)[b-1-i][b-1-j] for i >= j (read from the lower triangle of H as
// H[b-1-j][b-1-i]); identity on the padding; its mirror image above the diagonal of the 64x64 tiles on it
// (cd_load_op reads whole tiles), zero in the rest of a diagonal block.  What lies right of the diagonal blocks is room for
// the split tiles of the steps and is written by them; of a factorisation that begins with steps (parked), what
// belongs below the first diagonal block is left there in that form and not in its place.  64x64 tiles through LDS so that
// both the read of H and the write of A' are coalesced, sixteen loads per thread in flight: 11008 columns 270 -> 135 us
// (before: 32x32 tiles, zeros in the whole upper triangle).  R rows of threads: with few columns, where the launch waits for
// its own loads, 16 rows of them have four loads and stores each instead of sixteen: 128 columns 35.0 and 33.5 us for the
// factorisation, 512 179.3 and 177.8, 1024 389.7 and 389; 2048 equal.
constexpr int kRpT = 64;
constexpr int64_t kRpFew = 1024;
template <int R>
__global__ __launch_bounds__(64 * R) void k_reverse_pad(const float* __restrict__ H, int64_t b,
                                                        const float* __restrict__ lam_p,
                                                        const float* __restrict__ d, float* __restrict__ Ap,
                                                        int64_t bp, int parked) {
  __shared__ float t[kRpT][kRpT + 1];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x R
  const int64_t i0 = (int64_t)blockIdx.y * kRpT, j0 = (int64_t)blockIdx.x * kRpT;
  if (j0 >= (i0 / NB + 1) * NB) return;
  // A'[i0+r][j0+cidx] = H[b-1-(j0+cidx)][b-1-(i0+r)]: source rows are indexed by cidx,
  // source columns by r.  Load with lanes along r (source columns, contiguous, descending).
  const int64_t sc = b - 1 - (i0 + tx);
  float v[kRpT / R], di[kRpT / R];
#pragma unroll
  for (int e = 0; e < kRpT / R; ++e) {
    const int64_t sr = b - 1 - (j0 + ty + R * e);
    v[e] = H[max(sr, (int64_t)0) * b + max(sc, (int64_t)0)];
  }
#pragma unroll
  for (int e = 0; e < kRpT / R; ++e) di[e] = d[max(b - 1 - (i0 + ty + R * e), (int64_t)0)];
  const float lam = *lam_p;
  const int64_t j = j0 + tx;
  const float dj = d[max(b - 1 - j, (int64_t)0)];
#pragma unroll
  for (int e = 0; e < kRpT / R; ++e) {
    const int64_t sr = b - 1 - (j0 + ty + R * e);
    t[ty + R * e][tx] = (sc >= 0 && sr >= sc) ? v[e] : 0.f;  // t[cidx][r]; only the lower triangle is valid
  }
  if (parked && j0 < NB && i0 >= NB) {  // below the first diagonal block
    __syncthreads();
    __shared__ float ds[2 * kRpT];  // scales of the tile's rows, then of its columns; zero on the padding
    if (ty < 2) {
      const int64_t at = b - 1 - ((ty == 0 ? i0 : j0) + tx);
      ds[kRpT * ty + tx] = at >= 0 ? d[at] : 0.f;
    }
    __syncthreads();
    float* const block = Ap + (i0 / NB) * NB;
    const float sa = h2_scale(kBoundA);
    for (int v = threadIdx.x; v < kRpT * kRpT / 8; v += 64 * R) {  // pieces of 16 bytes: eight values of a row
      const int lo = v & 31, hi = (v >> 5) & 1, m = (v >> 6) & 1, kt = (v >> 7) & 1, rt = v >> 8;
      const int r = 32 * rt + lo;
      f32x4 x[2];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 32 * kt + tl_row(8 * m + e, hi);
        x[e >> 2][e & 3] = t[k][r] * (ds[r] * ds[kRpT + k]);
      }
      f16x8 h, l;
      split8_h2(x[0], x[1], sa, h, l);
      float* const at = block + st_parked((int)(i0 % NB) / 32 + rt, (int)j0 / 32 + kt, 2 * m, bp) + (hi * bp + 4 * lo);
      *reinterpret_cast<f16x8*>(at) = h;
      *reinterpret_cast<f16x8*>(at + 2 * bp) = l;
    }
    return;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kRpT / R; ++e) {
    const int r = ty + R * e;
    const int64_t i = i0 + r;
    float o;
    if (j > i) o = i0 == j0 && j < b ? t[r][tx] * (di[e] * dj) : 0.f;
    else if (i >= b) o = (i == j) ? 1.f : 0.f;
    else o = (t[tx][r] + ((i == j) ? lam : 0.f)) * (di[e] * dj);
    Ap[i * bp + j] = o;
  }
}

// ------------------------------------------------------------------------------------------
// Cholesky factor and inverse of one NB x NB diagonal block, one workgroup of 8 wavefronts.
//   in : A'[kb*NB .. , kb*NB ..], of its diagonal 32-tiles both triangles, of the others the lower ones
//   out: L_kk in the same place (its diagonal 32-tiles with zeros above the diagonal, the tiles above
//        them untouched), Linv diagonal block = L_kk^{-1} (full square, zeros above the diagonal).
//
// The whole chip waits for this kernel, so what counts is the length of its chain: four phases of
// 32 pivots.  The block is a 4 x 4 grid of 32x32 tiles, all arithmetic is on them (tile32.h, rows and
// columns of a tile in elimination order, so that pairs of pivots leave a true triangle).
//   Wavefronts 0..3 (one per SIMD, raised priority) run the chain.  In phase j each holds a copy of
//     the diagonal tile (j, j) and eliminates it with two pivots per MFMA; the same row operations
//     turn a second tile into T_j = L_jj^{-1} (wavefront 0, from I) and into L_ij (wavefront i - j,
//     from A_ij).  Between phases each applies L_*j to its copy of the next diagonal tile and to its
//     next tile: registers in, registers out, one barrier per phase.
//   Wavefronts 4..7 do the rest beside it: the trailing tiles two or more columns ahead, the stores
//     of what is final, and the inverse by rows,
//         X_ij = -T_i V_ij,  V_ij = sum_{j <= k < i} L_ik X_kj,  X_jj = T_j,
//     with V of tile row i formed in phase i (before T_i is known), X of it in phase i + 1.
// 17.5 us per block by itself, 14.5 inside k_chol_step.  Four unrolled phases, fp32 MFMAs between them and the most
// products beside the longest chain: 23.5.  With one pivot per MFMA, LDS round trips of the tiles between the phases and the
// inverse after them (four wavefronts): 34.5.
constexpr int kCdL = 0, kCdT = 10, kCdA = 14, kCdTiles = 17;  // LDS tiles: L (i, j), T_j, A_22 A_32 A_33
constexpr int kCdB = 9, kCdB1 = 8, kCdB2 = 5;  // A_11 A_21 A_31, in the place of L tiles of phases 2 and 3
constexpr size_t kCholDiagSmem = ((size_t)kCdTiles * kRsTile + 4 * 32) * sizeof(float);

__device__ __forceinline__ constexpr int cd_l(int i, int j) { return kCdL + i * (i + 1) / 2 + j; }

// Global tile (p = its first element) <-> registers, rows and columns in elimination order.
// nl = tl_nat(lo).
__device__ __forceinline__ void cd_swap(float& a, float& b) {  // upper half of a <-> lower half of b
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(s[0]);
  b = __uint_as_float(s[1]);
}
// operand layout (of a symmetric tile: accumulator layout); a lane reads 16-byte pieces of its row, whose even (odd)
// columns belong to the lower (upper) half of the wavefront
__device__ __forceinline__ void cd_load_rows(f32x4 (&x)[4], const float* p, int64_t ld, int nl, int hi) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
    x[g] = *reinterpret_cast<const f32x4*>(p + 8 * g + ((uint32_t)nl * (uint32_t)ld + 4 * hi));
}
__device__ __forceinline__ void cd_from_rows(f32x16& v, const f32x4 (&x)[4]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float a = x[g][2 * e], b = x[g][2 * e + 1];
      cd_swap(a, b);
      v[4 * g + e] = a;
      v[4 * g + e + 2] = b;
    }
  }
}
__device__ __forceinline__ void cd_load_op(f32x16& v, const float* p, int64_t ld, int nl, int hi) {
  f32x4 x[4];
  cd_load_rows(x, p, ld, nl, hi);
  cd_from_rows(v, x);
}
__device__ __forceinline__ void cd_store_op(float* p, int64_t ld, const float* tile, int lo, int hi) {
  const int nl = tl_nat(lo);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 v = rs_piece(tile, g, lo, hi);
    f32x4 f;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float a = v[e], b = v[e + 2];
      cd_swap(a, b);
      f[2 * e] = a;
      f[2 * e + 1] = b;
    }
    *reinterpret_cast<f32x4*>(p + (int64_t)nl * ld + 8 * g + 4 * hi) = f;
  }
}
// accumulator layout; top: largest magnitude stored so far
__device__ __forceinline__ void cd_store_acc(float* p, int64_t ld, const f32x16& v, int nl, int hi, uint32_t& top) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    p[(int64_t)(8 * (r >> 2) + 2 * (r & 3) + hi) * ld + nl] = v[r];
    top = max(top, __float_as_uint(fabsf(v[r])));
  }
}
__device__ __forceinline__ f32x16 cd_get(const float* tile, int lo, int hi) {
  f32x16 v;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = rs_piece(tile, g, lo, hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * g + e] = x[e];
  }
  return v;
}
__device__ __forceinline__ f32x16 cd_zero() {
  f32x16 v;
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = 0.f;
  return v;
}
// -T V for T in LDS (stored transposed, as it leaves the elimination) and V in accumulator layout
__device__ __forceinline__ f32x16 cd_minus_tv(const float* T, const f32x16& V, int lo, int hi) {
  f32x16 acc = cd_zero();
  const float* t = T + rs_col(lo, hi);
#pragma unroll
  for (int r = 0; r < 16; ++r)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(-t[rs_step(r)], V[r], acc, 0, 0, 0);
  return acc;
}

// v -= A B^T for tiles of L in LDS, on the two-way split (|L| <= kBoundL), which is made here: a tile is read
// by three products at most.  Eight MFMAs of 32 cycles and 112 vector instructions where 16 fp32 MFMAs take 64 each.
// The operands have 22 bits or more here instead of 24; all four partial products are summed in fp32, in eight MFMAs of 16
// values instead of 16 of two.  Whole factors against float64 with fp32 MFMAs here and with these, damping 1e-2: 64
// columns 1.69 and 1.42e-7, 128 2.90 and 1.86, 512 3.42 and 3.07, 1024 4.12 and 3.83, 4096 6.93 and 6.81, 5120 28.6 both; with
// channels 100 times as large and damping 1e-4 128 columns 2.86 and 1.79, 1024 4.32 and 4.12, 4096 7.21 and 7.10; no size
// from 33 to 5120 columns was further off.  128 columns 29.1 and 27.3 us, 512 130.5 and 124.7, 4096 1093 and 1067.
struct CdSplit {
  f16x8 h[2], l[2];
};
__device__ __forceinline__ CdSplit cd_split(const float* tile, int lo, int hi) {
  CdSplit t;
#pragma unroll
  for (int m = 0; m < 2; ++m)
    split8_h2(rs_piece(tile, 2 * m, lo, hi), rs_piece(tile, 2 * m + 1, lo, hi), h2_scale(kBoundL), t.h[m], t.l[m]);
  return t;
}
__device__ __forceinline__ void cd_sub(f32x16& v, const CdSplit& a, const CdSplit& b) {
  f32x16 acc = cd_zero();
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.l[m], b.l[m], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.l[m], b.h[m], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h[m], b.l[m], acc, 0, 0, 0);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h[m], b.h[m], acc, 0, 0, 0);
  const float f = -pow2_inv(h2_scale(kBoundL)) * pow2_inv(h2_scale(kBoundL));
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = fmaf(f, acc[r], v[r]);
}

// The block itself: A, Li point at it in A' and in the inverse.  sym(v, i) and op(v, i, j) give tile (i, i) in
// accumulator and tile (i, j) in operand layout; all_have() is reached by every wavefront once it has its first ones (by
// the chain in the middle of phase 0), before anything is written to LDS.
template <typename Sym, typename Op, typename All>
__device__ __forceinline__ void cd_block(float* cd_smem, float* A, float* Li, int64_t bp, int kb_glob, int64_t b,
                                         float* bound, int32_t* info, const Sym& sym, const Op& op,
                                         const All& all_have) {
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5, nl = tl_nat(lo);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  auto S = [&](int t) { return cd_smem + t * kRsTile; };
  auto Ag = [&](int i, int j) { return A + (int64_t)(32 * i) * bp + 32 * j; };
  auto Xg = [&](int i, int j) { return Li + (int64_t)(32 * i) * bp + 32 * j; };

  if (wave < 4) {  // ------------------------------------------------------------------ chain
    __builtin_amdgcn_s_setprio(3);
    float* aux = cd_smem + kCdTiles * kRsTile + 32 * wave;
    auto ident = [&]() {
      f32x16 v;
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = (tl_row(r, hi) == lo) ? 1.f : 0.f;
      return v;
    };
    f32x16 D, E, U;
    sym(D, 0);
    if (wave == 0) E = ident();
    else op(E, wave, 0);
    int bad = -1;
    // a loop, not four copies: the code of an elimination is 6 KB, and a copy that is met for the first time waits
    // for its instructions (2000 of 8000 cycles)
#pragma clang loop unroll(disable)
    for (int j = 0; j < 4; ++j) {
      if (wave + j < 4) {
        if (j > 0) {  // copies of the diagonal tile, and the next tile
          const float* Lj = S(cd_l(j, j - 1));
          D = cd_get(S(j == 1 ? kCdB : j == 2 ? kCdA : kCdA + 2), lo, hi);
          const CdSplit x = cd_split(Lj, lo, hi);
          cd_sub(D, x, x);
          if (wave == 0) {
            E = ident();
          } else {
            E = cd_get(S(j == 2 ? kCdA + 1 : wave == 1 ? kCdB1 : kCdB2), lo, hi);  // j = 2: tile (3, 2)
            cd_sub(E, x, cd_split(S(cd_l(j + wave, j - 1)), lo, hi));
          }
        }
        const float dl = tl_eliminate<true>(D, E, U, aux, lo, hi, [&] {
          if (j == 0) all_have();
        });
        rs_store(S(wave == 0 ? kCdT + j : cd_l(j + wave, j)), E, lo, hi);
        if (wave == 0) {
          rs_store(S(cd_l(j, j)), U, lo, hi);
          // first non-positive pivot in the order of elimination (what follows it is garbage)
          const float dn = __shfl(dl, (lo & ~7) + ((lo & 7) >> 1) + 4 * (lo & 1), 64);
          const unsigned long long m = __ballot(!(dn > 0.f)) & 0xffffffffull;
          if (m && bad < 0) bad = 32 * j + __ffsll((long long)m) - 1;
        }
      }
      __syncthreads();
    }
    if (bad >= 0 && lane == 0) {
      const int64_t orig = b - ((int64_t)kb_glob * NB + bad);  // 1-based original column
      atomicCAS(info, 0, (int32_t)(orig > 0 ? orig : 1));
    }
    return;
  }

  // --------------------------------------------------------------------------------- beside it
  // Wavefront 4 shares its SIMD with the longest chain and has the fewest products; what needs most of them is
  // where the chains end first (wavefront 7, then 6).
  f32x16 X, V, Y;
  uint32_t top = 0;
  if (wave == 4) {
    sym(X, 3);
  } else if (wave == 5) {
    op(Y, 2, 1);
    op(X, 3, 2);
  } else if (wave == 6) {
    sym(Y, 1);
    sym(X, 2);
  } else {
    op(Y, 3, 1);
  }
  all_have();
  if (wave == 6) rs_store(S(kCdB), Y, lo, hi);
  if (wave == 5) rs_store(S(kCdB1), Y, lo, hi);
  if (wave == 7) rs_store(S(kCdB2), Y, lo, hi);
  if (wave == 4) {
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 24; ++q) {  // zeros of the inverse: tiles (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
      const int t = q >> 2, i = t < 3 ? 0 : t < 5 ? 1 : 2, j = t < 3 ? t + 1 : t < 5 ? t - 1 : 3;
      *reinterpret_cast<float4*>(Xg(i, j) + (int64_t)(8 * (q & 3) + (lane >> 3)) * bp + 4 * (lane & 7)) = z;
    }
  }
  __syncthreads();  // ---- phase 1: column 0 of L and T_0 are there
  if (wave == 4) {
    const CdSplit x = cd_split(S(cd_l(3, 0)), lo, hi);
    cd_sub(X, x, x);
    cd_store_op(Ag(3, 0), bp, S(cd_l(3, 0)), lo, hi);
  } else if (wave == 5) {
    cd_sub(X, cd_split(S(cd_l(2, 0)), lo, hi), cd_split(S(cd_l(3, 0)), lo, hi));
    rs_store(S(kCdA + 1), X, lo, hi);
    cd_store_op(Ag(1, 0), bp, S(cd_l(1, 0)), lo, hi);
    cd_store_op(Ag(2, 0), bp, S(cd_l(2, 0)), lo, hi);
  } else if (wave == 6) {
    const CdSplit x = cd_split(S(cd_l(2, 0)), lo, hi);
    cd_sub(X, x, x);
    rs_store(S(kCdA), X, lo, hi);
    cd_store_acc(Xg(0, 0), bp, cd_get(S(kCdT), lo, hi), nl, hi, top);
    cd_store_op(Ag(0, 0), bp, S(cd_l(0, 0)), lo, hi);
  } else {
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(1, 0)), S(kCdT), lo, hi);  // V_10
  }
  __syncthreads();  // ---- phase 2: column 1 of L and T_1
  if (wave == 4) {
    const CdSplit x = cd_split(S(cd_l(3, 1)), lo, hi);
    cd_sub(X, x, x);
    rs_store(S(kCdA + 2), X, lo, hi);
  } else if (wave == 5) {
    cd_store_acc(Xg(1, 1), bp, cd_get(S(kCdT + 1), lo, hi), nl, hi, top);
    cd_store_op(Ag(1, 1), bp, S(cd_l(1, 1)), lo, hi);
    cd_store_op(Ag(2, 1), bp, S(cd_l(2, 1)), lo, hi);
    cd_store_op(Ag(3, 1), bp, S(cd_l(3, 1)), lo, hi);
  } else if (wave == 6) {
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(2, 1)), S(kCdT + 1), lo, hi);  // V_21
  } else {
    X = cd_minus_tv(S(kCdT + 1), V, lo, hi);  // X_10
    cd_store_acc(Xg(1, 0), bp, X, nl, hi, top);
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(2, 0)), S(kCdT), lo, hi);
    rs_mma<false>(V, S(cd_l(2, 1)), X, lo, hi);  // V_20
  }
  __syncthreads();  // ---- phase 3: column 2 of L and T_2
  if (wave == 4) {
    cd_store_acc(Xg(2, 2), bp, cd_get(S(kCdT + 2), lo, hi), nl, hi, top);
    cd_store_op(Ag(2, 2), bp, S(cd_l(2, 2)), lo, hi);
    cd_store_op(Ag(3, 2), bp, S(cd_l(3, 2)), lo, hi);
  } else if (wave == 5) {
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(3, 2)), S(kCdT + 2), lo, hi);  // V_32
  } else if (wave == 6) {
    Y = cd_minus_tv(S(kCdT + 2), V, lo, hi);  // X_21
    cd_store_acc(Xg(2, 1), bp, Y, nl, hi, top);
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(3, 1)), S(kCdT + 1), lo, hi);
    rs_mma<false>(V, S(cd_l(3, 2)), Y, lo, hi);  // V_31
  } else {
    Y = cd_minus_tv(S(kCdT + 2), V, lo, hi);  // X_20
    cd_store_acc(Xg(2, 0), bp, Y, nl, hi, top);
    V = cd_zero();
    rs_mma<false>(V, S(cd_l(3, 0)), S(kCdT), lo, hi);
    rs_mma<false>(V, S(cd_l(3, 1)), X, lo, hi);
    rs_mma<false>(V, S(cd_l(3, 2)), Y, lo, hi);  // V_30
  }
  __syncthreads();  // ---- L_33 and T_3
  if (wave == 4) {
    cd_store_acc(Xg(3, 3), bp, cd_get(S(kCdT + 3), lo, hi), nl, hi, top);
    cd_store_op(Ag(3, 3), bp, S(cd_l(3, 3)), lo, hi);
  } else {  // wavefronts 7, 6, 5: X_30, X_31, X_32
    cd_store_acc(Xg(3, 7 - wave), bp, cd_minus_tv(S(kCdT + 3), V, lo, hi), nl, hi, top);
  }
  raise_bound(bound, __uint_as_float(top));
}

// 512 threads at 128 registers: half of a compute unit's registers, so that the workgroup finds
// room beside one workgroup of the matrix products.
__global__ __launch_bounds__(512, 4) void k_chol_diag(float* __restrict__ Ap, float* __restrict__ Linv, int64_t bp,
                                                      int kb_glob, int64_t b, float* __restrict__ bound,
                                                      int32_t* __restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) float cd_smem[];
  const int lane = threadIdx.x & 63, nl = tl_nat(lane & 31), hi = lane >> 5;
  float* A = Ap + ((int64_t)kb_glob * NB) * bp + (int64_t)kb_glob * NB;
  float* Li = Linv + ((int64_t)kb_glob * NB) * bp + (int64_t)kb_glob * NB;
  cd_block(
      cd_smem, A, Li, bp, kb_glob, b, bound, info,
      [&](f32x16& v, int i) { cd_load_op(v, A + (int64_t)(32 * i) * (bp + 1), bp, nl, hi); },
      [&](f32x16& v, int i, int j) { cd_load_op(v, A + (int64_t)(32 * i) * bp + 32 * j, bp, nl, hi); }, [] {});
}

// ------------------------------------------------------------------------------------------
// A whole step of the factorisation in one launch, for the last block rows: workgroup 0 goes from block
// column k to the next diagonal block,
//     L_{k+1,k} = A_{k+1,k} Linv_kk^T,  A_{k+1,k+1} -= L_{k+1,k} L_{k+1,k}^T,  cd_block(k + 1),
// and every other workgroup updates one tile right of it, A_ij -= L_ik L_jk^T (i >= j > k), with L_ik and L_jk worked
// out for itself: the tiles of a step need no launch between panel and update, and with up to 32 block rows they take hardly
// longer than the diagonal block.  A step is 22.5 us (2.5 for its first loads, 2.3 panel, 2.5 update, 14.5 block); as
// separate launches it was 41 (block 23.5, panel 8.5, update 8.5), and 22 to 31 more for the strip of every fourth:
// whole factorisations 512 columns 174 -> 125 us, 2048 818 -> 485, 4096 1696 -> 1037.  128 registers, so that two
// workgroups share a compute unit when there are many tiles; 25 are spilled for it (STORED: 34).
//
// What a launch reads of A_ik no workgroup of it may overwrite, so tiles of the column that comes next (j = k + 1) do not
// go to their place in A', which takes L_ij in the next launch, but to block (j, i), right of the diagonal, where
// nothing else lives; and in the form that their only reader wants: split into fp16 pairs in the layout of the
// operands (512 consecutive bytes per half wavefront and load).  STORED: the first launch behind two-level updates, whose
// panel is in A'; of a factorisation that begins with steps, k_reverse_pad leaves the first column like that (the launch of its
// panel, 7 to 9 us, is gone).
//
// Products as in k_gemm_direct: two-way split, all four partial products, two partial sums.
struct StepArgs {
  float *Ap, *Linv;
  int64_t bp, b;
  int k, nb;
  float* bound_inv;
  int32_t* info;
};
struct SplitTile {  // 32 x 32 in operand layout: x1 and x2 of registers 0 .. 7, then of 8 .. 15
  u32x4 p[4];
};
__device__ __forceinline__ SplitTile st_split(const f32x4 (&x)[4], float s) {
  SplitTile t;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    f16x8 h, l;
    split8_h2(x[2 * m], x[2 * m + 1], s, h, l);
    t.p[2 * m] = __builtin_bit_cast(u32x4, h);
    t.p[2 * m + 1] = __builtin_bit_cast(u32x4, l);
  }
  return t;
}
// rows of a matrix <-> operand layout; p is uniform, at = lo * ld + 4 * hi the lane's offset (32 bits: one register)
__device__ __forceinline__ void st_rows(f32x4 (&x)[4], const float* p, uint32_t at) {
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = *reinterpret_cast<const f32x4*>(p + 8 * q + at);
}
__device__ __forceinline__ void st_rows_out(float* p, const f32x4 (&x)[4], uint32_t at) {
#pragma unroll
  for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(p + 8 * q + at) = x[q];
}
// A split tile in LDS, 4 KB, pieces in the order of the lanes.  First the ten of the inverse; the tiles (r, 2) and (r, 3)
// of L_jk behind them, as soon as they are there, (r, 0) and (r, 1) in their place.
constexpr int kStTile = 1024;
__device__ __forceinline__ int st_slot(int r, int n) { return (n >= 2 ? 10 + 2 * r : 2 * r) + (n == 1 || n == 2 ? 1 : 0); }
constexpr size_t kStepSmem = 18 * kStTile * sizeof(float);
static_assert(kStepSmem >= kCholDiagSmem, "the diagonal block is done in the same launch");
__device__ __forceinline__ void st_put(float* t, const SplitTile& v, int lane) {
#pragma unroll
  for (int e = 0; e < 4; ++e) *reinterpret_cast<u32x4*>(t + 256 * e + 4 * lane) = v.p[e];
}
__device__ __forceinline__ SplitTile st_get(const float* t, int lane) {
  SplitTile v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v.p[e] = *reinterpret_cast<const u32x4*>(t + 256 * e + 4 * lane);
  return v;
}
__device__ __forceinline__ SplitTile st_fetch(const float* p, int r, int kt, int64_t ld, uint32_t at) {
  SplitTile v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v.p[e] = *reinterpret_cast<const u32x4*>(p + st_parked(r, kt, e, ld) + at);
  return v;
}
// 16 of the 32 columns of a split tile: of one in LDS, of one in registers
struct SplitHalf {
  f16x8 h, l;
};
__device__ __forceinline__ SplitHalf st_half(const float* t, int m, int lane) {
  return {*reinterpret_cast<const f16x8*>(t + 512 * m + 4 * lane),
          *reinterpret_cast<const f16x8*>(t + 512 * m + 256 + 4 * lane)};
}
__device__ __forceinline__ SplitHalf st_half(const SplitTile& t, int m) {
  return {__builtin_bit_cast(f16x8, t.p[2 * m]), __builtin_bit_cast(f16x8, t.p[2 * m + 1])};
}
// (acc + acc2)[x][y] = sum over 32 KT values k of a[x][k] b[y][k]; in registers x, y the lane.  a(kt, m), b(kt, m):
// halves of the operands' tiles, fetched a tile at a time (all of them at once are spilled).
template <int KT, typename A, typename B>
__device__ __forceinline__ void st_product(f32x16& acc, f32x16& acc2, const A& a, const B& b) {
  acc = cd_zero();
  acc2 = cd_zero();
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const SplitHalf x = a(kt, m), y = b(kt, m);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.l, y.l, acc2, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.h, y.l, acc2, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.h, y.h, acc, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(x.l, y.h, acc2, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}
// L tile from its rows of A (split, k-tiles 0 .. n) and tile row n of the inverse in LDS
template <int KT>
__device__ __forceinline__ void st_panel(f32x4 (&x)[4], const SplitTile (&R)[4], const float* inv, float f, int lane) {
  constexpr int n = KT - 1;
  f32x16 acc, acc2;
  st_product<KT>(
      acc, acc2, [&](int kt, int m) { return st_half(inv + (n * (n + 1) / 2 + kt) * kStTile, m, lane); },
      [&](int kt, int m) { return st_half(R[kt], m); });
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[q][e] = f * (acc[4 * q + e] + acc2[4 * q + e]);
}

template <bool STORED>
__global__ __launch_bounds__(512, 4) void k_chol_step(StepArgs g) {
  extern __shared__ __attribute__((aligned(16))) float cd_smem[];
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t bp = g.bp;
  const int k = g.k;
  // tile 0 is the diagonal block; column by column behind it
  int i = (int)blockIdx.x, j = k + 1;
  for (; i >= g.nb - j; ++j) i -= g.nb - j;
  i += j;
  const bool diag = blockIdx.x == 0, next = j == k + 1;
  auto blk = [&](int r, int c) { return g.Ap + (int64_t)r * NB * bp + (int64_t)c * NB; };
  const float sl = h2_scale(kBoundL);
  const int r = wave >> 1, half = wave & 1;
  const uint32_t at_row = (uint32_t)lo * (uint32_t)bp + 4 * hi, at_parked = (uint32_t)hi * (uint32_t)bp + 4 * lo;

  // ---- L_jk into LDS as split tiles [row tile][k-tile]; a wavefront makes two of a row, five k-tiles in all
  f32x4 x[4];
  SplitTile p1;
  const int n0 = half ? 2 : 3, n1 = half ? 1 : 0;
  float fp = 0.f;
  // a line of the next diagonal block per thread: its tiles come from the L2 later on (its loads in front of
  // their products waited 2 us for memory)
  float touch = 0.f;
  if (diag) touch = blk(j, j)[(int64_t)(threadIdx.x >> 2) * bp + 32 * (threadIdx.x & 3)];
  if constexpr (STORED) {
    const float* Lj = blk(j, k) + (int64_t)(32 * r) * bp;
    f32x4 y[4];
    st_rows(x, Lj + 32 * n0, at_row);
    st_rows(y, Lj + 32 * n1, at_row);
    st_put(cd_smem + st_slot(r, n0) * kStTile, st_split(x, sl), lane);
    p1 = st_split(y, sl);
  } else {
    const float sa = h2_scale(kBoundA), si = h2_scale(g.bound_inv[k]);
    fp = pow2_inv(sa) * pow2_inv(si);
    const float* Li = g.Linv + (int64_t)k * NB * (bp + 1);
    const float* Rj = blk(k, j);
    SplitTile R[4];
    // the inverse's tiles, in rows: 0 | 1 2 | 3 4 5 | 6 7 8 9
    const int e0 = wave, t0 = e0 < 1 ? 0 : e0 < 3 ? 1 : e0 < 6 ? 2 : 3, c0 = e0 - t0 * (t0 + 1) / 2;
    f32x4 y[4];
    st_rows(x, Li + (int64_t)(32 * t0) * bp + 32 * c0, at_row);
    if (wave < 2) st_rows(y, Li + (int64_t)96 * bp + 32 * (2 + wave), at_row);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
      if (kt <= n0) R[kt] = st_fetch(Rj, r, kt, bp, at_parked);
    st_put(cd_smem + e0 * kStTile, st_split(x, si), lane);
    if (wave < 2) st_put(cd_smem + (8 + wave) * kStTile, st_split(y, si), lane);
    __syncthreads();
    float* Lj = blk(j, k) + (int64_t)(32 * r) * bp;
    auto keep = [&](int n) {
      if (diag) st_rows_out(Lj + 32 * n, x, at_row);
    };
    if (half == 0) {
      st_panel<4>(x, R, cd_smem, fp, lane);
      keep(3);
      st_put(cd_smem + st_slot(r, n0) * kStTile, st_split(x, sl), lane);
      st_panel<1>(x, R, cd_smem, fp, lane);
      keep(0);
    } else {
      st_panel<3>(x, R, cd_smem, fp, lane);
      keep(2);
      st_put(cd_smem + st_slot(r, n0) * kStTile, st_split(x, sl), lane);
      st_panel<2>(x, R, cd_smem, fp, lane);
      keep(1);
    }
    p1 = st_split(x, sl);
  }
  auto put_panel = [&]() {
    if (!STORED) __syncthreads();  // the inverse has been read
    st_put(cd_smem + st_slot(r, n1) * kStTile, p1, lane);
    __syncthreads();
  };
  const float fl = -pow2_inv(sl) * pow2_inv(sl);

  if (diag) {
    float* A = blk(j, j);
    const int nl = tl_nat(lo), lp = nl + 32 * hi;  // rows in elimination order
    asm volatile("" ::"v"(touch));
    put_panel();
    auto minus = [&](f32x16& v, int ti, int tj) {
      f32x4 old[4];
      cd_load_rows(old, A + (int64_t)(32 * ti) * bp + 32 * tj, bp, nl, hi);
      f32x16 acc, acc2;
      st_product<4>(
          acc, acc2, [&](int kt, int m) { return st_half(cd_smem + st_slot(tj, kt) * kStTile, m, lp); },
          [&](int kt, int m) { return st_half(cd_smem + st_slot(ti, kt) * kStTile, m, lp); });
      cd_from_rows(v, old);
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] += fl * (acc[e] + acc2[e]);
      __builtin_amdgcn_sched_barrier(0);
    };
    cd_block(
        cd_smem, A, g.Linv + (int64_t)j * NB * (bp + 1), bp, j, g.b, g.bound_inv + j, g.info,
        [&](f32x16& v, int t) { minus(v, t, t); }, [&](f32x16& v, int ti, int tj) { minus(v, ti, tj); },
        [] { __syncthreads(); });
    return;
  }

  // ---- tile (i, j): a wavefront has 32 rows of it and two of the column tiles; L_ik of its rows in registers
  SplitTile P[4];
  if (i != j) {
    if constexpr (STORED) {
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        st_rows(x, blk(i, k) + (int64_t)(32 * r) * bp + 32 * n, at_row);
        P[n] = st_split(x, sl);
      }
    } else {
      const float* Ri = blk(k, i);
      SplitTile R[4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) R[kt] = st_fetch(Ri, r, kt, bp, at_parked);
      float* Lik = blk(i, k) + (int64_t)(32 * r) * bp;
      auto keep = [&](int n) {  // the tiles of the next column have all rows; two k-tiles per wavefront
        if (next && (n >> 1) == half) st_rows_out(Lik + 32 * n, x, at_row);
      };
      st_panel<4>(x, R, cd_smem, fp, lane);
      keep(3);
      P[3] = st_split(x, sl);
      st_panel<3>(x, R, cd_smem, fp, lane);
      keep(2);
      P[2] = st_split(x, sl);
      st_panel<2>(x, R, cd_smem, fp, lane);
      keep(1);
      P[1] = st_split(x, sl);
      st_panel<1>(x, R, cd_smem, fp, lane);
      keep(0);
      P[0] = st_split(x, sl);
    }
  }
  put_panel();
  if (i == j) {
#pragma unroll
    for (int n = 0; n < 4; ++n) P[n] = st_get(cd_smem + st_slot(r, n) * kStTile, lane);
  }
  float* C = blk(i, j) + (int64_t)(32 * r) * bp;
  float* parked = blk(j, i);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = 2 * half + h;
    f32x16 acc, acc2;
    st_product<4>(
        acc, acc2, [&](int n, int m) { return st_half(cd_smem + st_slot(c, n) * kStTile, m, lane); },
        [&](int n, int m) { return st_half(P[n], m); });
    st_rows(x, C + 32 * c, at_row);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[q][e] += fl * (acc[4 * q + e] + acc2[4 * q + e]);
    if (next) {
      const SplitTile t = st_split(x, h2_scale(kBoundA));
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<u32x4*>(parked + st_parked(r, c, e, bp) + at_parked) = t.p[e];
    } else {
      st_rows_out(C + 32 * c, x, at_row);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Inverse of the block lower-triangular L by recursive doubling.  At level S (in blocks) the
// matrix is cut into pairs of S-block halves; for each pair
//     Tbuf21 = L21 * Linv11        (Linv11 lower triangular: k-blocks >= column block)
//     Linv21 = -Linv22 * Tbuf21    (Linv22 lower triangular: k-blocks <= row block)
struct TrinvArgs {
  const float* L;
  float* Linv;
  float* T;
  int64_t bp;
  int nb, S;
  int p0, c0;  // this launch: pairs from p0 (blockIdx.z), tile columns of a pair from c0 (blockIdx.x)
  // Largest magnitudes by block column, nb each: of L^{-1} so far, of Tbuf at this level.  A launch reads
  // what earlier launches of its stream have left and raises others: equal calls give equal bits.
  // What the lowest level leaves has an array of its own: its workgroups read the others' block.
  float *bound_inv, *bound_T, *bound_first;
};
__device__ __forceinline__ uint32_t inv_bound(const TrinvArgs& a, int j) {
  return max(__float_as_uint(a.bound_inv[j]), __float_as_uint(a.bound_first[j]));
}

// Whole tile: C = scale * acc, and its largest magnitude into *bound.
__device__ __forceinline__ void write_tile_bound(const TileAcc& acc, char* smem, float* C, int64_t ldc,
                                                 float scale, float* bound) {
  raise_bound(bound, x3_write_tile(acc, smem, C, ldc, scale));
}

template <int NBUF>
__global__ __launch_bounds__(kXThreads, 4) void k_trinv_T(TrinvArgs a) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  const int tj = a.c0 + blockIdx.x, ti = blockIdx.y, p = a.p0 + blockIdx.z;
  const int base = 2 * p * a.S;
  const int gi = base + a.S + ti, gj = base + tj;
  if (gi >= a.nb) return;
  const float* A = a.L + ((int64_t)gi * NB) * a.bp + (int64_t)base * NB;   // [m][k]
  const float* B = a.Linv + ((int64_t)base * NB) * a.bp + (int64_t)gj * NB;  // [k][n]
  TileAcc acc;
  acc_zero(acc);
  const float sa = h2_scale(kBoundL), sb = h2_scale(__uint_as_float(inv_bound(a, gj)));
  gemm_tile_h2<false, true, NBUF>(acc, sm, A, a.bp, NB, sa, nullptr, B, a.bp, NB, sb, {}, nullptr, tj * NB, a.S * NB);
  write_tile_bound(acc, sm, a.T + ((int64_t)gi * NB) * a.bp + (int64_t)gj * NB, a.bp,
                   (1.f / sa) * (1.f / sb), a.bound_T + gj);
}

template <int NBUF>
__global__ __launch_bounds__(kXThreads, 4) void k_trinv_X(TrinvArgs a) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  const int tj = a.c0 + blockIdx.x, ti = blockIdx.y, p = a.p0 + blockIdx.z;
  const int base = 2 * p * a.S;
  const int gi = base + a.S + ti, gj = base + tj;
  if (gi >= a.nb) return;
  const float* A = a.Linv + ((int64_t)gi * NB) * a.bp + (int64_t)(base + a.S) * NB;  // [m][k]
  const float* B = a.T + ((int64_t)(base + a.S) * NB) * a.bp + (int64_t)gj * NB;     // [k][n]
  TileAcc acc;
  acc_zero(acc);
  uint32_t ba = 0;  // bound of the part of Linv22 that this tile row reads
  for (int e = threadIdx.x & 63; e <= ti; e += 64) ba = max(ba, inv_bound(a, base + a.S + e));
  for (int off = 32; off > 0; off >>= 1) ba = max(ba, (uint32_t)__shfl_xor((int)ba, off, 64));
  const float sa = h2_scale(__uint_as_float(ba)), sb = h2_scale(a.bound_T[gj]);
  gemm_tile_h2<false, true, NBUF>(acc, sm, A, a.bp, NB, sa, nullptr, B, a.bp, NB, sb, {}, nullptr, 0, (ti + 1) * NB);
  write_tile_bound(acc, sm, a.Linv + ((int64_t)gi * NB) * a.bp + (int64_t)gj * NB, a.bp,
                   -(1.f / sa) * (1.f / sb), a.bound_inv + gj);
}

// The same products where a launch has few tiles, as in k_gemm_direct: a wavefront owns 32 x 32 of the result and
// fetches its operands straight into the registers that the MFMAs read them from, 64 k-values ahead.  For the last
// merges of a factorisation, which have nothing beside them: a layer of 512 columns 393 -> 388 us, 5120 4997 -> 4957.
template <bool SECOND>
__global__ __launch_bounds__(256, 2) void k_trinv_direct(TrinvArgs a) {
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  const int tj = a.c0 + blockIdx.x, ti = blockIdx.y >> 2, p = a.p0 + blockIdx.z;
  const int base = 2 * p * a.S;
  const int gi = base + a.S + ti, gj = base + tj;
  if (gi >= a.nb) return;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t i0 = (int64_t)gi * NB + 32 * (blockIdx.y & 3), j0 = (int64_t)gj * NB + 32 * w;
  const int kb = SECOND ? base + a.S : base;  // factor block where the reduction index starts
  const float* pa = (SECOND ? a.Linv : a.L) + (i0 + lo) * a.bp + (int64_t)kb * NB + 4 * hi;
  const float* pb = (SECOND ? a.T : a.Linv) + (int64_t)kb * NB * a.bp + j0;  // uniform; the lane's offset has 32 bits
  const uint32_t ob = (uint32_t)(4 * hi) * (uint32_t)a.bp + (uint32_t)lo;
  const int kbeg = SECOND ? 0 : tj * NB, kend = SECOND ? (ti + 1) * NB : a.S * NB;
  f32x4 x[2][8], y[2][8];
  auto load = [&](int buf, int k) {
    const float* pk = pb + k * a.bp;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      x[buf][q] = *reinterpret_cast<const f32x4*>(pa + k + 8 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e, pk += a.bp) y[buf][q][e] = pk[ob];
      pk += 4 * a.bp;
    }
  };
  uint32_t ba = SECOND && lane <= ti ? inv_bound(a, base + a.S + lane) : 0;  // the part of Linv22 that is read
  load(0, kbeg);
  load(1, kbeg + 64);
  if (SECOND)
    for (int off = 32; off > 0; off >>= 1) ba = max(ba, (uint32_t)__shfl_xor((int)ba, off, 64));
  const float sa = SECOND ? h2_scale(__uint_as_float(ba)) : h2_scale(kBoundL);
  const float sb = SECOND ? h2_scale(a.bound_T[gj]) : h2_scale(__uint_as_float(inv_bound(a, gj)));
  f32x16 acc, acc2;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = acc2[r] = 0.f;
  auto multiply = [&](int buf) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f16x8 a1, a2, b1, b2;
      split8_h2(x[buf][2 * m], x[buf][2 * m + 1], sa, a1, a2);
      split8_h2(y[buf][2 * m], y[buf][2 * m + 1], sb, b1, b2);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b2, acc2, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b1, acc2, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b1, acc, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b2, acc2, 0, 0, 0);
    }
  };
#pragma clang loop unroll(disable)
  for (int k = kbeg + 128; k < kend; k += 128) {
    multiply(0);
    __builtin_amdgcn_sched_barrier(0);
    load(0, k);
    multiply(1);
    __builtin_amdgcn_sched_barrier(0);
    load(1, k + 64);
  }
  multiply(0);
  multiply(1);
  const float f = (SECOND ? -1.f : 1.f) * pow2_inv(sa) * pow2_inv(sb);
  float* out = (SECOND ? a.Linv : a.T) + (i0 + 4 * hi) * a.bp + j0 + lo;
  uint32_t top = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = f * (acc[r] + acc2[r]);
    out[(int64_t)(8 * (r >> 2) + (r & 3)) * a.bp] = v;
    top = max(top, __float_as_uint(fabsf(v)));
  }
  raise_bound((SECOND ? a.bound_inv : a.bound_T) + gj, __uint_as_float(top));
}
// Up to 1024 tiles as in direct_ok (gemm_f32.hip), reductions of up to 1024: the factor of 1152 columns 328 us with up to
// 512, 320 with up to 1024, of 2048 495 and 484, of 4096 1072 and 1062.
constexpr int kTriDirectTiles = 1024, kTriDirectS = 8;

// The lowest level (S = 1) in one launch: Linv21 = -Linv22 (L21 Linv11) for 128x128 blocks, of which each
// product by itself is mostly launch and latency.  A workgroup owns 32 columns of a pair, a wavefront 32
// rows: operands straight into the registers of the MFMAs as in k_gemm_direct, split there; the strip of
// L21 Linv11 is in the layout of a second operand as it leaves the first product, and goes round through
// LDS.  Its bound needs no look at it: rows of L have norms of at most 2, columns of Linv11 at most
// sqrt(128) times their largest value.  Two launches 15 us, this one 9.
__global__ __launch_bounds__(256, 2) void k_trinv_first(TrinvArgs a) {
  __shared__ float strip[4][16][64];
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int gj = 2 * (a.p0 + (int)blockIdx.z), gi = gj + 1, n0 = 32 * blockIdx.x;
  if (gi >= a.nb) return;
  const float* L21 = a.L + ((int64_t)gi * NB + 32 * w + lo) * a.bp + (int64_t)gj * NB + 4 * hi;
  const float* I11 = a.Linv + ((int64_t)gj * NB + 4 * hi) * a.bp + (int64_t)gj * NB + n0 + lo;
  const float* I22 = a.Linv + ((int64_t)gi * NB + 32 * w + lo) * a.bp + (int64_t)gi * NB + 4 * hi;
  f32x4 x[16], y[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {  // k = 8 q + 4 hi + c
    x[q] = *reinterpret_cast<const f32x4*>(L21 + 8 * q);
#pragma unroll
    for (int c = 0; c < 4; ++c) y[q][c] = I11[(int64_t)(8 * q + c) * a.bp];
  }
  const float bound = a.bound_inv[gj];
  const float sl = h2_scale(kBoundL), si = h2_scale(bound);
  f32x16 acc, acc2;
  auto multiply = [&](float sx, float sy) {  // acc + acc2 = sx sy x y
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = acc2[r] = 0.f;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      f16x8 a1, a2, b1, b2;
      split8_h2(x[2 * m], x[2 * m + 1], sx, a1, a2);
      split8_h2(y[2 * m], y[2 * m + 1], sy, b1, b2);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b2, acc2, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b1, acc2, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b1, acc, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b2, acc2, 0, 0, 0);
    }
  };
  multiply(sl, si);
  const float f = pow2_inv(sl) * pow2_inv(si);
#pragma unroll
  for (int r = 0; r < 16; ++r) strip[w][r][lane] = f * (acc[r] + acc2[r]);
#pragma unroll
  for (int q = 0; q < 16; ++q) x[q] = *reinterpret_cast<const f32x4*>(I22 + 8 * q);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) y[q][c] = strip[q >> 2][4 * (q & 3) + c][lane];
  const float s2 = h2_scale(a.bound_inv[gi]), st = h2_scale(32.f * bound);
  multiply(s2, st);
  const float g = -pow2_inv(s2) * pow2_inv(st);
  float* out = a.Linv + ((int64_t)gi * NB + 32 * w + 4 * hi) * a.bp + (int64_t)gj * NB + n0 + lo;
  uint32_t top = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = g * (acc[r] + acc2[r]);
    out[(int64_t)(8 * (r >> 2) + (r & 3)) * a.bp] = v;
    top = max(top, __float_as_uint(fabsf(v)));
  }
  raise_bound(a.bound_first + gj, __uint_as_float(top));
}

// U[i][j] = Linv[b-1-i][b-1-j] d[j] for j >= i, else 0, and the largest magnitude of each column.  A thread
// takes `rows` rows of a column, kOutRows of them in flight; columns whose maximum is already as large (a
// stale value is a smaller one) are left alone.
constexpr int kOutRows = 8;
__global__ __launch_bounds__(256) void k_reverse_out(const float* __restrict__ Linv, int64_t bp,
                                                     const float* __restrict__ d, float* __restrict__ U,
                                                     int64_t b, int rows, float* __restrict__ umax) {
  const int64_t i0 = (int64_t)blockIdx.y * rows, i1 = min(b, i0 + rows);
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= b) return;
  if (j < i0) {
    for (int64_t i = i0; i < i1; ++i) U[i * b + j] = 0.f;
    return;
  }
  const float dj = d[j];
  uint32_t top = 0;
  for (int64_t r = i0; r < i1; r += kOutRows) {
    float v[kOutRows];
#pragma unroll
    for (int e = 0; e < kOutRows; ++e) v[e] = Linv[(b - 1 - min(r + e, j)) * bp + (b - 1 - j)];
#pragma unroll
    for (int e = 0; e < kOutRows; ++e) {
      const float u = r + e <= j ? v[e] * dj : 0.f;
      if (r + e < i1) U[(r + e) * b + j] = u;
      top = max(top, __float_as_uint(fabsf(u)));
    }
  }
  if (__float_as_uint(umax[j]) < top) atomicMax(reinterpret_cast<unsigned int*>(umax) + j, top);
}

static inline int64_t padded(int64_t b) { return ceil_div(b, NB) * NB; }

const float* factor_L(const void* ws, int64_t b, int64_t* ld) {
  *ld = padded(b);
  return reinterpret_cast<const float*>(reinterpret_cast<const char*>(ws) + 256);
}

// The scales and the bounds live in the first 128 rows of the inverse's temporary, which no merge writes
// (its tile rows belong to second halves): bp scales, nb bounds of L^{-1}, nb bounds of Tbuf per level
// (level 0: of what the lowest merges leave), the largest magnitudes of U's bp columns, the scales of the row losses: at
// most 10 values per block of 128 columns beside three times 128, and there are 128 x 128.
static inline float* scales(const void* ws, int64_t bp) {
  return reinterpret_cast<float*>(const_cast<char*>(reinterpret_cast<const char*>(ws)) + 256) + 2 * bp * bp;
}
static inline int merge_levels(int nb) {
  int n = 0;
  for (int S = 1; S < nb; S *= 2) ++n;
  return n;
}
static inline int n_bounds(int nb) { return nb * (1 + merge_levels(nb)); }
const float* factor_scale(const void* ws, int64_t b) { return scales(ws, padded(b)); }
const float* factor_umax(const void* ws, int64_t b) {
  const int64_t bp = padded(b);
  return scales(ws, bp) + bp + n_bounds((int)(bp / NB));
}

const float* factor_loss_scale(const void* ws, int64_t b) { return factor_umax(ws, b) + padded(b); }

size_t factor_workspace_bytes(int64_t b) {
  const int64_t bp = padded(b);
  return 3 * (size_t)bp * bp * sizeof(float) + 256;
}

thanos_status factor_begin(hipStream_t s, const float* H, int64_t b, float damping, float* xnorm2,
                           void* ws, int32_t* info, bool losses) {
  const int64_t bp = padded(b);
  float* lam = reinterpret_cast<float*>(ws);
  float* Ap = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + 256);
  const int nb = (int)(bp / NB);
  float* d = scales(ws, bp);
  hipLaunchKernelGGL(losses ? k_diag_stats<true> : k_diag_stats<false>, dim3(1), dim3(1024), 0, s, H, b, damping, xnorm2,
                     lam, d, d + 2 * bp + n_bounds(nb), d + bp, n_bounds(nb) + (int)bp, info);
  THANOS_LAUNCH_CHECK();
  const dim3 tiles((unsigned)(bp / kRpT), (unsigned)(bp / kRpT));
  const int parked = factor_first_step(nb) == 0 ? 1 : 0;
  if (b <= kRpFew) hipLaunchKernelGGL(k_reverse_pad<16>, tiles, dim3(1024), 0, s, H, b, lam, d, Ap, bp, parked);
  else hipLaunchKernelGGL(k_reverse_pad<4>, tiles, dim3(256), 0, s, H, b, lam, d, Ap, bp, parked);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

thanos_status factor(hipStream_t s, const float* H, int64_t b, float damping, float* U,
                     float* xnorm2, void* ws, int32_t* info, bool single_stream, bool begun,
                     bool company) {
  const int64_t bp = padded(b);
  const int nb = (int)(bp / NB);
  float* Ap = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + 256);
  float* Linv = Ap + bp * bp;
  float* Tb = Linv + bp * bp;
  const float* d = scales(ws, bp);
  float* bound_inv = scales(ws, bp) + bp;
  float* bound_first = bound_inv + nb;  // the array of level 0, whose products share a launch
  if (!begun) THANOS_CHECK(factor_begin(s, H, b, damping, xnorm2, ws, info, false));

  // Two-level blocking: inside an outer block of kOuter factor blocks the trailing update of a
  // step only reaches the columns of that outer block (narrow, K = NB); everything to the right
  // gets one update per outer block with K = kOuter*NB, which reads and writes the trailing
  // matrix kOuter times less often and runs the matrix cores on long reductions.
  // That wide update is split in two: the column strip of the NEXT outer block stays on the
  // caller's stream (the next diagonal block needs it), the rest runs on a second stream next
  // to the latency-bound diagonal / panel chain of the next outer block.  Column ranges of the
  // two streams are disjoint until the next strip, which waits for the previous rest.
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_chol_diag),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kCholDiagSmem));
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_chol_step<true>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepSmem));
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_chol_step<false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepSmem));
  const int first_step = factor_first_step(nb);
  AuxStream aux(s, 2 * factor_rests(nb), single_stream);
  if (!aux.ok) return THANOS_ERR_HIP;

  // The inverse of L (recursive doubling, see k_trinv_T / k_trinv_X) does not wait for the end
  // of the factorisation: the merge of two halves at level S needs, for its first product
  // L21 * Linv11, only the column blocks of the FIRST half (final once their panels are
  // solved), and for its second product the inverse of the second half.  After every outer
  // block the merges that have become possible are queued on a third stream, lowest level
  // first and the first product before the second at each level (the order of their
  // dependencies); they fill the compute units that the chain of diagonal blocks leaves idle.
  // Regions written by different merges are disjoint, and none overlaps what the
  // factorisation still writes.
  auto* const kern_T = company ? k_trinv_T<1> : k_trinv_T<2>;
  auto* const kern_X = company ? k_trinv_X<1> : k_trinv_X<2>;
  const size_t tri_smem = company ? kXSmemBytes : kH2SmemBytes;
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_trinv_T<1>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXSmemBytes));
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_trinv_X<1>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXSmemBytes));
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_trinv_T<2>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kH2SmemBytes));
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_trinv_X<2>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kH2SmemBytes));
  const int n_batches = factor_tri_batches(nb);
  AuxStream tri(s, n_batches > 0 ? n_batches + 1 : 0, single_stream);
  if (!tri.ok) return THANOS_ERR_HIP;
  int tri_done = -1;  // blocks 0..tri_done have been handed to the inversion
  int tri_batches = 0;
  constexpr int tri_cap = 512;  // workgroups of one launch while the factorisation runs (256 or 384 measured the same,
                                // 192 and fewer slower, next to two-level updates; not measured next to steps)
  auto trinv_upto = [&](int kdone) -> thanos_status {
    // blocks <= kdone: diagonal inverse known, panel below solved (recorded on s by the caller)
    // The last batch runs on the caller's stream, behind the earlier ones: one hop between streams
    // (about 10 us) instead of two, none where there were no earlier ones.
    hipStream_t ts = tri.stream;
    if (kdone == nb - 1) {
      if (tri_batches > 0) {
        THANOS_CHECK(tri.record(n_batches));
        THANOS_CHECK(tri.join(n_batches));
      }
      ts = s;
    } else {
      THANOS_CHECK(tri.fork(tri_batches));
      ++tri_batches;
    }
    int level = 0;
    for (int S = 1; S < nb; S *= 2, ++level) {
      for (int second = S == 1 ? 1 : 0; second < 2; ++second) {  // one launch does both products of S = 1
        int p_lo = -1, p_hi = -1;
        for (int p = 0; 2 * p * S + S < nb; ++p) {
          const int e = second ? std::min(2 * p * S + 2 * S, nb) - 1 : 2 * p * S + S - 1;
          if (e > tri_done && e <= kdone) {
            if (p_lo < 0) p_lo = p;
            p_hi = p;
          }
        }
        if (p_lo < 0) continue;
        const int np = p_hi - p_lo + 1;
        if (S == 1) {
          TrinvArgs a{Ap, Linv, Tb, bp, nb, S, p_lo, 0, bound_inv, nullptr, bound_first};
          hipLaunchKernelGGL(k_trinv_first, dim3(NB / 32, 1, (unsigned)np), dim3(256), 0, ts, a);
          THANOS_LAUNCH_CHECK();
          continue;
        }
        // rows of the second half that exist (the last pair of a level may be cut short)
        const int rows = std::min(S, nb - (2 * p_hi * S + S));
        const int rows_all = np > 1 ? S : rows;
        // while the factorisation runs, a launch takes at most tri_cap workgroups (one round of
        // the chip's workgroup slots), so that the short kernels of the chain are not queued
        // behind thousands of long-running tiles
        const bool last = kdone == nb - 1;
        if (last && S <= kTriDirectS && 16 * S * rows_all * np <= kTriDirectTiles) {
          const TrinvArgs a{Ap, Linv, Tb, bp, nb, S, p_lo, 0, bound_inv, bound_inv + (1 + level) * nb, bound_first};
          const dim3 grid((unsigned)S, 4u * (unsigned)rows_all, (unsigned)np);
          hipLaunchKernelGGL(second ? k_trinv_direct<true> : k_trinv_direct<false>, grid, dim3(256), 0, ts, a);
          THANOS_LAUNCH_CHECK();
          continue;
        }
        int cols = S;
        if (!last) cols = std::max(1, std::min(S, tri_cap / (rows_all * np)));
        for (int c0 = 0; c0 < S; c0 += cols) {
          TrinvArgs a{Ap, Linv, Tb, bp, nb, S, p_lo, c0, bound_inv, bound_inv + (1 + level) * nb, bound_first};
          dim3 grid((unsigned)std::min(cols, S - c0), (unsigned)rows_all, (unsigned)np);
          if (second)
            hipLaunchKernelGGL(kern_X, grid, dim3(kXThreads), tri_smem, ts, a);
          else
            hipLaunchKernelGGL(kern_T, grid, dim3(kXThreads), tri_smem, ts, a);
          THANOS_LAUNCH_CHECK();
        }
      }
    }
    tri_done = kdone;
    return THANOS_OK;
  };
  int pending_join = -1;  // event index recorded on the aux stream after the last "rest"
  for (int k = 0; k <= first_step; ++k) {
    hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(512), kCholDiagSmem, s, Ap, Linv, bp, k, b, bound_inv + k,
                       info);
    THANOS_LAUNCH_CHECK();
    if (first_step == 0) break;  // the first panel waits where a step looks for it (k_reverse_pad)
    const int64_t rem = bp - (int64_t)(k + 1) * NB;
    float* panel = Ap + ((int64_t)(k + 1) * NB) * bp + (int64_t)k * NB;
    const float* dinv = Linv + ((int64_t)k * NB) * bp + (int64_t)k * NB;
    // L_ik = A_ik * Linv_kk^T  (in place, all rows below the diagonal block)
    thanos_status st = gemm_bounded(s, rem, NB, NB, 1.f, panel, bp, kBoundA, dinv, bp, 0.f, bound_inv + k,
                                    0.f, panel, bp, false, company);
    if (st != THANOS_OK) return st;
    if (k == first_step) break;
    if ((k + 1) % kOuter == 0) {
      st = trinv_upto(k);
      if (st != THANOS_OK) return st;
    }
    const int ob = k / kOuter;
    const int ob_begin = ob * kOuter;
    const int ob_end = ob_begin + kOuter;  // at least a step's rows follow (factor_first_step), also behind the next one
    // narrow: A_ij -= L_ik L_jk^T for block columns k < j < ob_end, lower tiles
    const int64_t ncols = (int64_t)(ob_end - (k + 1)) * NB;
    if (ncols > 0) {
      float* trail = Ap + ((int64_t)(k + 1) * NB) * bp + (int64_t)(k + 1) * NB;
      st = gemm_bounded(s, rem, ncols, NB, -1.f, panel, bp, kBoundL, panel, bp, kBoundL, nullptr, 1.f, trail,
                        bp, true, company);
      if (st != THANOS_OK) return st;
    }
    // wide: after the last step of an outer block, everything right of it
    if (k + 1 == ob_end) {
      const int next_end = ob_end + kOuter;
      const int64_t kk = (int64_t)(ob_end - ob_begin) * NB;
      const float* lp = Ap + ((int64_t)ob_end * NB) * bp + (int64_t)ob_begin * NB;
      // The strip of the next outer block first: it is on the critical path (the next diagonal
      // block waits for it) and gets the chip to itself for the ~25 us it needs; launched behind
      // the rest, it shared the compute units with that much larger product and took 80-100 us.
      // It was last written by the previous rest.
      if (pending_join >= 0) THANOS_CHECK(aux.join(pending_join));
      pending_join = -1;
      {
        const int64_t rows = bp - (int64_t)ob_end * NB;
        const int64_t cols = (int64_t)(next_end - ob_end) * NB;
        float* cs = Ap + ((int64_t)ob_end * NB) * bp + (int64_t)ob_end * NB;
        st = gemm_bounded(s, rows, cols, kk, -1.f, lp, bp, kBoundL, lp, bp, kBoundL, nullptr, 1.f, cs, bp,
                          true, company);
        if (st != THANOS_OK) return st;
      }
      // fork: the rest (rows and columns >= next_end) on the second stream, next to the
      // latency-bound chain of the next outer block (the fork point lies behind the strip, which
      // costs the rest nothing: the two write disjoint columns)
      THANOS_CHECK(aux.fork(2 * ob));
      const int64_t rest = bp - (int64_t)next_end * NB;
      const float* lr = lp + ((int64_t)(next_end - ob_end) * NB) * bp;
      float* cr = Ap + ((int64_t)next_end * NB) * bp + (int64_t)next_end * NB;
      st = gemm_bounded(aux.stream, rest, rest, kk, -1.f, lr, bp, kBoundL, lr, bp, kBoundL, nullptr, 1.f, cr,
                        bp, true, company);
      if (st != THANOS_OK) return st;
      THANOS_CHECK(aux.record(2 * ob + 1));
      pending_join = 2 * ob + 1;
    }
  }
  if (pending_join >= 0) THANOS_CHECK(aux.join(pending_join));
  // the last block rows: one launch per step, every tile updated in every step
  for (int k = first_step; k + 1 < nb; ++k) {
    const StepArgs a{Ap, Linv, bp, b, k, nb, bound_inv, info};
    const int rows = nb - 1 - k;
    hipLaunchKernelGGL(k == first_step && first_step > 0 ? k_chol_step<true> : k_chol_step<false>,
                       dim3((unsigned)(rows * (rows + 1) / 2)), dim3(512), kStepSmem, s, a);
    THANOS_LAUNCH_CHECK();
    if ((k + 1) % kOuter == 0 && k + 2 < nb) THANOS_CHECK(trinv_upto(k));
  }
  THANOS_CHECK(trinv_upto(nb - 1));

  // few columns: enough workgroups; many: few updates of the maxima.  Whole factorisation, 8 rows and 64 per
  // thread: 128 columns 36.3 and 42.0 us, 512 180.6 and 185.8, 1024 391 and 397, 1365 545.5 and 546, 2048 831 and
  // 825, 4096 1710 and 1705.
  const int out_rows = b <= 1024 ? kOutRows : 8 * kOutRows;
  hipLaunchKernelGGL(k_reverse_out, dim3((unsigned)ceil_div(b, 256), (unsigned)ceil_div(b, out_rows)),
                     dim3(256), 0, s, Linv, bp, d, U, b, out_rows, scales(ws, bp) + bp + n_bounds(nb));
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

}  // namespace thanos
