// fp32 matrix product on the 16-bit matrix cores: split bf16 for operands of any range
// (gemm_tile_x3.h: sweep, fp32 Hessian accumulation), split fp16 where the range is known (gemm_tile_h2.h: the
// factorisation, row losses, structured update; the sweep's update has a kernel of its own).
#include <algorithm>

#include "gemm_tile_h2.h"

namespace thanos {

struct GemmArgs {
  const float* A;
  const float* B;
  float* C;
  int64_t lda, ldb, ldc;
  int M, N, K;
  float alpha, beta;
  int lower_only;
  int vec_a, vec_b;  // 16-byte aligned rows (k_gemm_direct)
  float sa, sb;          // H2: scales of the operands ...
  const float* bound_b;  // ... of B from a bound on the device instead, unless nullptr
};

// NBUF: two-way split with that many LDS buffers (0: three-way)
template <bool AK, bool BK, int NBUF = 0>
__global__ __launch_bounds__(kXThreads, 4) void k_gemm_f32(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  const int tn = blockIdx.x, tm = blockIdx.y;
  if (g.lower_only && tn > tm) return;
  const int m0 = tm * kTM, n0 = tn * kTN;
  const int m_ext = min(kTM, g.M - m0), n_ext = min(kTN, g.N - n0);
  const float* A = AK ? g.A + m0 : g.A + (int64_t)m0 * g.lda;
  const float* B = BK ? g.B + n0 : g.B + (int64_t)n0 * g.ldb;
  TileAcc acc;
  acc_zero(acc);
  if constexpr (NBUF > 0) {
    const float sb = g.bound_b ? h2_scale(*g.bound_b) : g.sb;
    gemm_tile_h2<AK, BK, NBUF>(acc, sm, A, g.lda, m_ext, g.sa, nullptr, B, g.ldb, n_ext, sb, {}, nullptr, 0, g.K);
    g.alpha *= (1.f / g.sa) * (1.f / sb);
  } else {
    gemm_tile_x3<AK, BK>(acc, sm, A, g.lda, m_ext, B, g.ldb, n_ext, 0, g.K);
  }
  const float* T = x3_stage_tile(acc, sm);
  // row pass: wavefront w takes rows w, w + 8, ..., lane l the columns 2l, 2l + 1
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c0 = 2 * lane;
  float* Cg = g.C + (int64_t)m0 * g.ldc + n0 + c0;
  if (m_ext == kTM && n_ext == kTN) {  // whole tile: pairs of columns, of any alignment
    f32x2u old[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      old[i] = g.beta != 0.f ? *reinterpret_cast<const f32x2u*>(Cg + (int64_t)(wave + 8 * i) * g.ldc)
                             : f32x2u{0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float2 t = *reinterpret_cast<const float2*>(T + (wave + 8 * i) * kXCLd + c0);
      *reinterpret_cast<f32x2u*>(Cg + (int64_t)(wave + 8 * i) * g.ldc) =
          f32x2u{g.beta * old[i].x + g.alpha * t.x, g.beta * old[i].y + g.alpha * t.y};
    }
  } else {
    for (int i = 0; i < 16; ++i) {
      const int row = wave + 8 * i;
      if (row >= m_ext) break;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (c0 + e < n_ext) {
          float* p = Cg + (int64_t)row * g.ldc + e;
          const float o = g.beta != 0.f ? *p : 0.f;
          *p = g.beta * o + g.alpha * T[row * kXCLd + c0 + e];
        }
      }
    }
  }
}

// C = A B (B[k*ldb + n]) on the two-way split, the scales from the largest magnitudes of the rows of A and, of B, from
// those of its columns (not triangular) or from a bound (triangular).  Lower triangle: A diag(kd)^-1 in the place of
// A.  row_top: the largest magnitudes of the rows of C are raised there, unless nullptr.
struct ToppedArgs {
  const float *A, *B;
  float* C;
  int64_t lda, ldb, ldc;
  int M, N, K;
  const float *a_top, *b_top, *kd;
  float sb, *row_top;
};
constexpr size_t kToppedInv = kXSmemBytes;  // reciprocal scales of the columns, behind the staged tile
static_assert(kToppedInv + kTN * sizeof(float) <= kH2SmemBytes, "both fit");
template <TriB TRI>
__global__ __launch_bounds__(kXThreads, 4) void k_gemm_topped(ToppedArgs g) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  // Triangular B: tiles differ in the length of their reduction, and the longest go first (a
  // whole column of tiles at a time), so that the short ones fill the last round: 4096^3, lower
  // triangle, 619 -> 392 us against tiles in row order (three-way split).
  const int tn = TRI == kTriNone ? blockIdx.x : TRI == kTriLower ? blockIdx.y : gridDim.y - 1 - blockIdx.y;
  const int tm = TRI == kTriNone ? blockIdx.y : blockIdx.x;
  const int m0 = tm * kTM, n0 = tn * kTN;
  const int m_ext = min(kTM, g.M - m0), n_ext = min(kTN, g.N - n0);
  const int kbeg = TRI == kTriLower ? n0 : 0;
  const int kend = TRI == kTriUpper ? min(g.K, n0 + kTN) : g.K;
  float* const inv = reinterpret_cast<float*>(sm + kToppedInv);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  TileAcc acc;
  acc_zero(acc);
  float a_top[16];  // of the rows that this wavefront writes out: scalar loads, done by then
#pragma unroll
  for (int i = 0; i < 16; ++i) a_top[i] = g.a_top[m0 + min(wave + 8 * i, m_ext - 1)];
  constexpr bool kCols = TRI == kTriNone;
  gemm_tile_h2<false, true, 2, true, kCols, false, true, TRI == kTriLower>(
      acc, sm, g.A + (int64_t)m0 * g.lda, g.lda, m_ext, 1.f, g.a_top + m0, g.B + n0, g.ldb, n_ext, g.sb, {}, inv, kbeg,
      kend, g.b_top + n0, g.kd);
  // Lower triangle: the row losses, whose H' need not be bounded (elements from 16 on are infinite in the split, and
  // every sum they enter is infinite or NaN).  Such a tile is computed again on the three-way split: calls with one
  // such element 4096 x 4096 3375 us, without 3360.
  constexpr bool kAgain = TRI == kTriLower;
  uint32_t* const bad = reinterpret_cast<uint32_t*>(inv);  // a word of each multiplying wavefront
  if (kAgain && wave < 4) {
    bool b = false;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 16; ++r) b = b || !(fabsf(acc.v[f][h][r]) < INFINITY);
    const uint32_t any = __any(b) ? 1u : 0u;
    if (lane == 0) bad[wave] = any;
  }
  const float* T = x3_stage_tile(acc, sm);
  bool again = false;
  if (kAgain && (bad[0] | bad[1] | bad[2] | bad[3]) != 0u) {
    again = true;
    acc_zero(acc);
    gemm_tile_x3<false, true, true>(acc, sm, g.A + (int64_t)m0 * g.lda, g.lda, m_ext, g.B + n0, g.ldb, n_ext, kbeg, kend,
                                    g.kd);
    T = x3_stage_tile(acc, sm);
  }
  const int c0 = 2 * lane;
  const float f0 = kCols ? inv[c0] : again ? 1.f : pow2_inv(g.sb), f1 = kCols ? inv[c0 + 1] : f0;
  float* Cg = g.C + (int64_t)m0 * g.ldc + n0 + c0;
  const bool ok0 = c0 < n_ext, ok1 = c0 + 1 < n_ext;
  uint32_t u[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = wave + 8 * i;
    const float fr = again ? 1.f : pow2_inv(h2_scale(a_top[i]));
    const float2 t = *reinterpret_cast<const float2*>(T + row * kXCLd + c0);
    const float o0 = t.x * fminf(fr, f0) * fmaxf(fr, f0), o1 = t.y * fminf(fr, f1) * fmaxf(fr, f1);
    u[i] = max(ok0 ? __float_as_uint(fabsf(o0)) : 0u, ok1 ? __float_as_uint(fabsf(o1)) : 0u);
    float* p = Cg + (int64_t)row * g.ldc;
    if (row < m_ext) {
      if (ok1) *reinterpret_cast<f32x2u*>(p) = f32x2u{o0, o1};
      else if (ok0) *p = o0;
    }
  }
  if (!g.row_top) return;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = max(u[i], (uint32_t)__shfl_xor((int)u[i], off, 64));
  uint32_t mine = u[0];  // lane i has row wave + 8 i
#pragma unroll
  for (int i = 1; i < 16; ++i) mine = lane == i ? u[i] : mine;
  if (lane < 16 && wave + 8 * lane < m_ext)
    atomicMax(reinterpret_cast<unsigned int*>(g.row_top) + m0 + wave + 8 * lane, mine);
}

// C = beta C + alpha A B^T, reduction a multiple of 128: panel, narrow and strip updates of the
// factorisation while few rows are left.  These launches stand in the factorisation's chain, and the
// pipelined kernel above needs 6 us for four slabs (1.7 for every further one) that it cannot overlap
// with anything.  Here a wavefront owns 32 x 32 of C and fetches its operands straight into the
// registers the MFMAs read them from (lane (lo, hi) holds k = 8 q + 4 hi + c of its row: both
// operands in the same order), 64 k-values ahead of the fp32 MFMAs on the 64 before: no LDS.  A
// workgroup is a strip of 32 rows x 128 columns, so that C may be A (N = K = 128): every wavefront
// has its rows before one stores.  H2 (operands of known range): every lane splits its values into fp16
// pairs (gemm_tile_h2.h), 16 MFMAs of 32 cycles and 160 vector instructions per 64 k-values instead of 32
// MFMAs of 64.  All four partial products here: the reductions are short, and the matrix pipes are idle.
// Factor: 1365 columns 566 -> 557 us, 4096 1.759 -> 1.731 ms; errors of U 512 4.0 -> 3.5e-7, 1365 9.3 -> 6.2e-7.
template <bool H2>
__global__ __launch_bounds__(256, 2) void k_gemm_direct(GemmArgs g) {
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  const int m0 = 32 * blockIdx.y, n0 = kTN * blockIdx.x + 32 * (threadIdx.x >> 6);
  if (g.lower_only && (int)blockIdx.x > m0 / kTM) return;  // same tiles as k_gemm_f32
  const float* pa = g.A + (int64_t)(m0 + lo) * g.lda + 4 * hi;
  const float* pb = g.B + (int64_t)(n0 + lo) * g.ldb + 4 * hi;
  float* pc = g.C + (int64_t)(m0 + 4 * hi) * g.ldc + n0 + lo;
  f32x4 a[2][8], b[2][8];
  auto load = [&](int buf, int k) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      a[buf][q] = *reinterpret_cast<const f32x4*>(pa + k + 8 * q);
      b[buf][q] = *reinterpret_cast<const f32x4*>(pb + k + 8 * q);
    }
  };
  load(0, 0);
  load(1, 64);
  f32x16 old, acc, acc2;  // two partial sums: a chain half as long, and half of its rounding
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    old[r] = g.beta != 0.f ? pc[(int64_t)(8 * (r >> 2) + (r & 3)) * g.ldc] : 0.f;
    acc[r] = acc2[r] = 0.f;
  }
  float sa = 1.f, sb = 1.f;
  if (H2) {
    sa = g.sa;
    sb = g.bound_b ? h2_scale(*g.bound_b) : g.sb;
    g.alpha *= pow2_inv(sa) * pow2_inv(sb);
  }
  auto multiply = [&](int buf) {
    if constexpr (H2) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {  // k = 16 m + 8 (0, 1) + 4 hi + c in both operands
        f16x8 a1, a2, b1, b2;
        split8_h2(a[buf][2 * m], a[buf][2 * m + 1], sa, a1, a2);
        split8_h2(b[buf][2 * m], b[buf][2 * m + 1], sb, b1, b2);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b2, acc2, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a2, b1, acc2, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b1, acc, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b2, acc2, 0, 0, 0);
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int c = 0; c < 4; c += 2) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][q][c], b[buf][q][c], acc, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][q][c + 1], b[buf][q][c + 1], acc2, 0, 0, 0);
      }
  };
  for (int k = 128; k < g.K; k += 128) {
    multiply(0);
    load(0, k);
    multiply(1);
    load(1, k + 64);
  }
  multiply(0);
  multiply(1);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r)
    pc[(int64_t)(8 * (r >> 2) + (r & 3)) * g.ldc] = g.beta * old[r] + g.alpha * (acc[r] + acc2[r]);
}
// One 32 x 32 tile of C per SIMD.  K = 128: 8.5 us instead of 10 to 11.5, at 1488 tiles 15.2 against
// 11.9.  K = 512: 22 instead of 29, at 1792 tiles 36 against 31.  The whole factor with a limit of 512, 1024
// and 2048: 1244, 1217 and 1242 us at 2944 columns, 1839, 1801 and 1817 at 4096, 5097, 4989 and 5058 at 8192.
constexpr int64_t kDirectTiles = 1024;

// A product beside the factorisation's chain takes more than half of a compute unit's LDS, so that one
// workgroup runs per unit, and leaves room for a diagonal block (72 KB) and half of the registers.
// Two per unit kept the chain's kernels waiting for whole tiles: its first step took 670 us next to
// the 690 us product of 5120 columns (now 40).
constexpr size_t kBesideSmemBytes = 84 * 1024;
static_assert(kBesideSmemBytes >= kXSmemBytes && kBesideSmemBytes >= kH2SmemBytes, "the products themselves fit");

static inline bool vec_ok(const float* p, int64_t ld) {
  return (reinterpret_cast<uintptr_t>(p) % 16 == 0) && (ld % 4 == 0);
}

static inline bool direct_ok(const GemmArgs& g) {
  return g.K > 0 && g.K % 128 == 0 && g.K <= 512 && g.M % 32 == 0 && g.N % kTN == 0 && g.vec_a && g.vec_b &&
         (int64_t)(g.M / 32) * (g.N / 32) <= kDirectTiles;
}
template <bool H2>
static thanos_status launch_direct(hipStream_t s, const GemmArgs& g) {
  hipLaunchKernelGGL(k_gemm_direct<H2>, dim3((unsigned)(g.N / kTN), (unsigned)(g.M / 32)), dim3(256), 0, s, g);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

thanos_status gemm_bounded(hipStream_t s, int64_t M, int64_t N, int64_t K, float alpha, const float* A,
                           int64_t lda, float bound_a, const float* B, int64_t ldb, float bound_b,
                           const float* bound_b_dev, float beta, float* C, int64_t ldc, bool lower_only,
                           bool company) {
  if (M <= 0 || N <= 0) return THANOS_OK;
  GemmArgs g{A, B, C, lda, ldb, ldc, (int)M, (int)N, (int)K, alpha, beta, lower_only ? 1 : 0,
             vec_ok(A, lda) ? 1 : 0, vec_ok(B, ldb) ? 1 : 0,
             h2_scale(bound_a), h2_scale(bound_b), bound_b_dev};
  if (direct_ok(g)) return launch_direct<true>(s, g);
  // two buffers unless the workgroup has to fit beside a larger one
  const dim3 grid((unsigned)ceil_div(N, kTN), (unsigned)ceil_div(M, kTM));
  if (company) {
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_f32<false, false, 1>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXSmemBytes));
    hipLaunchKernelGGL((k_gemm_f32<false, false, 1>), grid, dim3(kXThreads), kXSmemBytes, s, g);
  } else {
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_f32<false, false, 2>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kH2SmemBytes));
    hipLaunchKernelGGL((k_gemm_f32<false, false, 2>), grid, dim3(kXThreads), kH2SmemBytes, s, g);
  }
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

thanos_status gemm_topped(hipStream_t s, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                          const float* a_top, const float* B, int64_t ldb, const float* b_top, float bound_b,
                          float* C, int64_t ldc, TriB b_tri, const float* kd, float* row_top, bool beside) {
  if (M <= 0 || N <= 0) return THANOS_OK;
  if ((b_tri == kTriLower) != (kd != nullptr) || (b_tri == kTriNone) != (b_top != nullptr))
    return THANOS_ERR_UNSUPPORTED;  // no caller
  const ToppedArgs g{A, B, C, lda, ldb, ldc, (int)M, (int)N, (int)K, a_top, b_top, kd, h2_scale(bound_b), row_top};
  dim3 grid((unsigned)ceil_div(N, kTN), (unsigned)ceil_div(M, kTM));
  if (b_tri != kTriNone) std::swap(grid.x, grid.y);
  auto* const kern = b_tri == kTriLower ? k_gemm_topped<kTriLower>
                     : b_tri == kTriUpper ? k_gemm_topped<kTriUpper> : k_gemm_topped<kTriNone>;
  // the limit belongs to the kernel, not to the launch: the same value whoever sets it, or another thread's
  // launch could find it lowered
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBesideSmemBytes));
  hipLaunchKernelGGL(kern, grid, dim3(kXThreads), beside ? kBesideSmemBytes : kH2SmemBytes, s, g);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

thanos_status gemm_f32(hipStream_t s, bool a_kmajor, bool b_kmajor, int64_t M, int64_t N,
                       int64_t K, float alpha, const float* A, int64_t lda, const float* B,
                       int64_t ldb, float beta, float* C, int64_t ldc, bool lower_only) {
  if (M <= 0 || N <= 0) return THANOS_OK;
  GemmArgs g{A, B, C, lda, ldb, ldc, (int)M, (int)N, (int)K, alpha, beta, lower_only ? 1 : 0,
             vec_ok(A, lda) ? 1 : 0, vec_ok(B, ldb) ? 1 : 0, 1.f, 1.f, nullptr};
  if (!a_kmajor && !b_kmajor && direct_ok(g)) return launch_direct<false>(s, g);
  const dim3 grid((unsigned)ceil_div(N, kTN), (unsigned)ceil_div(M, kTM));
  void (*kern)(GemmArgs);
  if (!a_kmajor && !b_kmajor) kern = k_gemm_f32<false, false>;
  else if (!a_kmajor) kern = k_gemm_f32<false, true>;
  else if (b_kmajor) kern = k_gemm_f32<true, true>;
  else return THANOS_ERR_UNSUPPORTED;  // no caller
  THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kXSmemBytes));
  hipLaunchKernelGGL(kern, grid, dim3(kXThreads), kXSmemBytes, s, g);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

}  // namespace thanos
