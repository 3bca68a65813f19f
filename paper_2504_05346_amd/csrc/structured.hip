// Structured pruning (Alg. 2, Sec. 4.7): s = ceil(p b / (1 - alpha)) whole columns are removed
// from every non-outlier row in one shot,
//     W_R <- W_R - W_{R,Q} (Hinv[Q,Q])^{-1} Hinv[Q,:],      Hinv = (H + damping)^{-1},
// Q = the s columns of smallest loss v_j = (sum_{i in R} W_ij^2) H_jj, R = all rows but the
// ceil(alpha c) of largest loss h_i = W_i H W_i^T.
//
// How it is computed.  With sigma the ascending order of (v_j, j) and H' = H[sigma, sigma], the
// removed columns are the first s of the permuted problem, and with U' from the factorisation
// of H' (H'_d^{-1} = U'^T U'):
//     Hinv'[0:s, :]   = U'_ss^T U'[0:s, :],      Hinv'[0:s, 0:s] = U'_ss^T U'_ss,
//     Delta'          = -(W'_Q U'_ss^{-1}) U'[0:s, :],
// and U'_ss^{-1} is the index-reversed trailing s x s block of the Cholesky factor L the
// factorisation leaves in its workspace (U' = J L^{-1} J).  So: two rankings, one symmetric
// gather, the factorisation, two matrix products, one scatter.  Nothing of W is permuted in
// place; sigma only addresses columns.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace thanos {

constexpr int64_t kRowLds = 32 * 1024;  // columns of a row that goes through LDS: 128 KB
constexpr int64_t kFewCols = 1024;      // a row is a wavefront's work, four go through LDS at a time

// Column losses v[j] = H[j][j] * sum over non-skipped rows of W[i][j]^2, in two steps: fp64
// partial sums over chunks of rows (blockIdx.y), then the sum of the partials in chunk order.
__global__ __launch_bounds__(256) void k_col_loss_part(const float* __restrict__ W, int64_t c,
                                                       int64_t b, int64_t rows_per_chunk,
                                                       const uint8_t* __restrict__ skip,
                                                       double* __restrict__ part) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= b) return;
  const int64_t i0 = (int64_t)blockIdx.y * rows_per_chunk, i1 = min(c, i0 + rows_per_chunk);
  double acc = 0.0;
  // eight rows in flight, added in row order: one load at a time, behind the test of the row,
  // took 75 us at 4096 x 4096 (now 25)
  for (int64_t i = i0; i < i1; i += 8) {
    float w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = W[min(i + e, i1 - 1) * b + j];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (i + e < i1 && !(skip && skip[i + e])) acc += (double)w[e] * (double)w[e];
  }
  part[(int64_t)blockIdx.y * b + j] = acc;
}

__global__ __launch_bounds__(256) void k_col_loss_fin(const double* __restrict__ part,
                                                      const float* __restrict__ H, int64_t b,
                                                      int nchunk, float* __restrict__ v) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= b) return;
  double acc = 0.0;
  for (int c0 = 0; c0 < nchunk; c0 += 16) {  // sixteen in flight, added in order
    double p[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) p[e] = part[(int64_t)min(c0 + e, nchunk - 1) * b + j];
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if (c0 + e < nchunk) acc += p[e];
  }
  v[j] = (float)(acc * (double)H[j * b + j]);
}

// sigma = the columns in ascending (v, j) order, rank its inverse; one wavefront per column.
__global__ __launch_bounds__(256) void k_col_rank(const float* __restrict__ v, int64_t b,
                                                  int* __restrict__ rank, int* __restrict__ sigma) {
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= b) return;
  const int64_t r = wave_rank(v, b, j);
  if ((threadIdx.x & 63) == 0) {
    rank[j] = (int)r;
    sigma[r] = (int)j;
  }
}

// S = the symmetric matrix whose lower triangle is H's, in 64 x 64 tiles on and below the diagonal: a tile goes out
// as it is and transposed.
__global__ __launch_bounds__(256) void k_mirror(const float* __restrict__ H, int64_t b, float* __restrict__ S) {
  __shared__ float t[64][65];
  if (blockIdx.x > blockIdx.y) return;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t i0 = 64 * (int64_t)blockIdx.y, j0 = 64 * (int64_t)blockIdx.x;
  const bool diag = i0 == j0;
  float v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {  // never above the diagonal
    const int64_t i = min(i0 + ty + 4 * e, b - 1), j = min(j0 + tx, b - 1);
    v[e] = H[max(i, j) * b + min(i, j)];
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t i = i0 + ty + 4 * e, j = j0 + tx;
    if (i < b && j < b) S[i * b + j] = v[e];
    t[ty + 4 * e][tx] = v[e];
  }
  if (diag) return;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t i = j0 + ty + 4 * e, j = i0 + tx;
    if (i < b && j < b) S[i * b + j] = t[tx][ty + 4 * e];
  }
}

// Hp[x][y] = S[sigma[x]][sigma[y]] for y <= x, one workgroup per row, which goes through LDS (staged).  Taken from
// the lower triangle of H, half of the values are columns of it, a cache line each: 4096 columns 82 us, with the
// mirroring 45.  Few columns (S = H, whole = 0) fit the caches and save a launch.
__global__ __launch_bounds__(256) void k_permute_sym(const float* __restrict__ S, int64_t b,
                                                     const int* __restrict__ sigma, float* __restrict__ Hp,
                                                     int whole, int staged) {
  extern __shared__ float row_lds[];
  const int64_t x = blockIdx.x, sx = sigma[x];
  const float* row = S + sx * b;
  if (staged) {
    for (int64_t j = threadIdx.x; j < b; j += 8 * 256) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = row[min(j + 256 * e, b - 1)];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (j + 256 * e < b) row_lds[j + 256 * e] = v[e];
    }
    __syncthreads();
  }
  for (int64_t y = threadIdx.x; y <= x; y += 256) {
    const int64_t sy = sigma[y];
    Hp[x * b + y] = staged ? row_lds[sy] : whole || sx >= sy ? row[sy] : S[sy * b + sx];
  }
}

// WQ[i][x] = W[i][sigma[x]] / d[x], x < s, zeros up to sp, and the largest magnitude of each row (d powers of two:
// exact); clears z_top.  TPR threads per row: 256, or 64 for rows of up to kFewCols columns.  staged: the row goes
// through LDS, which takes any order of columns at its own rate: 4096 x 1365 of 4096 47 -> 22 us.
template <int TPR>
__global__ __launch_bounds__(256) void k_gather_cols(const float* __restrict__ W, int64_t c, int64_t b,
                                                     const int* __restrict__ sigma, const float* __restrict__ d,
                                                     int64_t s, int64_t sp, float* __restrict__ WQ,
                                                     float* __restrict__ q_top, float* __restrict__ z_top, int staged) {
  extern __shared__ float row_lds[];
  __shared__ uint32_t tops[4];
  const int t = threadIdx.x & (TPR - 1), sub = (int)threadIdx.x / TPR;
  const int64_t i = (int64_t)blockIdx.x * (256 / TPR) + sub, ic = min(i, c - 1);
  const float* row = W + ic * b;
  float* lds = row_lds + sub * b;
  if (staged) {
    for (int64_t j = t; j < b; j += 8 * TPR) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = row[min(j + TPR * e, b - 1)];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (j + TPR * e < b) lds[j + TPR * e] = v[e];
    }
    __syncthreads();
  }
  uint32_t u = 0;
  if (i < c)
    for (int64_t x = t; x < sp; x += TPR) {
      const int col = sigma[x];  // sp <= b
      const float v = x < s ? (staged ? lds[col] : row[col]) / d[x] : 0.f;
      WQ[i * sp + x] = v;
      u = max(u, __float_as_uint(fabsf(v)));
    }
  for (int off = 32; off > 0; off >>= 1) u = max(u, (uint32_t)__shfl_xor((int)u, off, 64));
  if (TPR > 64) {
    if ((threadIdx.x & 63) == 0) tops[threadIdx.x >> 6] = u;
    __syncthreads();
    u = max(max(tops[0], tops[1]), max(tops[2], tops[3]));
  }
  if (t == 0 && i < c) {
    q_top[i] = __uint_as_float(u);
    z_top[i] = 0.f;
  }
}

// M[x][y] = L[b-1-x][b-1-y] for x <= y < s, else 0 (sp x sp): the inverse of U'_ss times d[x] in its rows (L is the factor
// of the matrix scaled by d).
__global__ __launch_bounds__(256) void k_rev_L(const float* __restrict__ L, int64_t ld, int64_t b, int64_t s,
                                               int64_t sp, float* __restrict__ M) {
  const int64_t y = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t x = blockIdx.y;
  if (y >= sp) return;
  M[x * sp + y] = (x <= y && y < s) ? L[(b - 1 - x) * ld + (b - 1 - y)] : 0.f;
}

// Non-skipped rows: column j sits at position pos = rank[j] of the permuted order;
// W[i][j] = 0 for pos < s, else -= T[i][pos]; mask accordingly, and the result in the layer's type
// where the caller wants it (cast).  Threads run over the natural columns: W, mask and cast are
// written in whole rows, four columns per thread (vec: rows and pointers aligned for it); only T is
// gathered.
template <typename O>
__global__ __launch_bounds__(256) void k_struct_apply(float* __restrict__ W,
                                                      const float* __restrict__ T, int64_t b,
                                                      const int* __restrict__ rank, int64_t s,
                                                      const uint8_t* __restrict__ skip,
                                                      uint8_t* __restrict__ mask,
                                                      O* __restrict__ cast, int vec) {
  const int64_t j = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  const int64_t i = blockIdx.y;
  if (j >= b) return;
  const int64_t idx = i * b + j;
  const bool keep_row = skip && skip[i];
  const int cnt = (int)min((int64_t)4, b - j);
  Quad<float> w{};
  if (vec) w = *reinterpret_cast<const Quad<float>*>(W + idx);
  else
    for (int e = 0; e < cnt; ++e) w.v[e] = W[idx + e];
  Quad<uint8_t> m{};
  if (!keep_row) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e >= cnt) break;
      const int64_t pos = rank[j + e];
      if (pos < s) {
        w.v[e] = 0.f;
        m.v[e] = 1;
      } else if (s > 0) {
        w.v[e] -= T[i * b + pos];
      }
    }
  }
  Quad<O> o;
#pragma unroll
  for (int e = 0; e < 4; ++e) from_f32(w.v[e], o.v[e]);
  if (vec) {
    if (!keep_row) *reinterpret_cast<Quad<float>*>(W + idx) = w;
    *reinterpret_cast<Quad<uint8_t>*>(mask + idx) = m;
    if (cast) *reinterpret_cast<Quad<O>*>(cast + idx) = o;
  } else {
    for (int e = 0; e < cnt; ++e) {
      if (!keep_row) W[idx + e] = w.v[e];
      mask[idx + e] = m.v[e];
      if (cast) cast[idx + e] = o.v[e];
    }
  }
}
template <typename O>
static void launch_struct_apply(hipStream_t st, float* W, const float* T, int64_t c, int64_t b,
                                const int* rank, int64_t s, const uint8_t* skip, uint8_t* mask,
                                void* cast) {
  const int vec = b % 4 == 0 && reinterpret_cast<uintptr_t>(W) % sizeof(Quad<float>) == 0 &&
                  reinterpret_cast<uintptr_t>(mask) % sizeof(Quad<uint8_t>) == 0 &&
                  reinterpret_cast<uintptr_t>(cast) % sizeof(Quad<O>) == 0;
  hipLaunchKernelGGL(k_struct_apply<O>, dim3((unsigned)ceil_div(b, 1024), (unsigned)c), dim3(256), 0,
                     st, W, T, b, rank, s, skip, mask, (O*)cast, vec);
}

static char* carve(char*& p, size_t bytes) {
  char* q = p;
  p += align_up(bytes, 256);
  return q;
}

size_t structured_workspace_bytes(int64_t c, int64_t b) {
  size_t n = 0;
  n += align_up((size_t)b * b * 4, 256);      // HB: symmetric H, then H', then U'_ss^{-1}
  n += align_up((size_t)c * b * 4, 256);      // T: W H, then the update in permuted order
  n += align_up((size_t)c * b * 4, 256);      // WQ
  n += align_up((size_t)c * b * 4, 256);      // Z
  n += align_up((size_t)b * b * 4, 256);      // U'
  n += 2 * align_up((size_t)b * 4, 256);      // v, xnorm2'
  n += 2 * align_up((size_t)b * 4, 256);      // sigma and its inverse
  n += align_up((size_t)c * 4, 256);          // h
  n += align_up((size_t)c, 256);              // row_skip
  n += align_up(factor_workspace_bytes(b), 256);
  return n;
}

thanos_status structured(hipStream_t st, const void* W_in, thanos_dtype wdt, int64_t c, int64_t b,
                         const float* H, float damping, long long s_cols, long long n_out,
                         float* W, void* W_cast, uint8_t* mask, void* ws, int32_t* info,
                         bool single_stream) {
  char* p = reinterpret_cast<char*>(ws);
  float* HB = reinterpret_cast<float*>(carve(p, (size_t)b * b * 4));
  float* T = reinterpret_cast<float*>(carve(p, (size_t)c * b * 4));
  float* WQ = reinterpret_cast<float*>(carve(p, (size_t)c * b * 4));
  float* Z = reinterpret_cast<float*>(carve(p, (size_t)c * b * 4));
  float* U = reinterpret_cast<float*>(carve(p, (size_t)b * b * 4));
  float* v = reinterpret_cast<float*>(carve(p, (size_t)b * 4));
  float* xn2 = reinterpret_cast<float*>(carve(p, (size_t)b * 4));
  int* sigma = reinterpret_cast<int*>(carve(p, (size_t)b * 4));
  int* rank = reinterpret_cast<int*>(carve(p, (size_t)b * 4));
  float* h = reinterpret_cast<float*>(carve(p, (size_t)c * 4));
  uint8_t* skip = reinterpret_cast<uint8_t*>(carve(p, (size_t)c));
  void* fws = p;

  THANOS_CHECK(convert_in(st, W_in, wdt, W, c * b));

  const uint8_t* skip_c = nullptr;
  if (n_out > 0) {
    thanos_status e = row_outliers(st, W, H, c, b, n_out, HB, T, h, nullptr, v, skip);
    if (e != THANOS_OK) return e;
    skip_c = skip;
  }
  const unsigned bb = (unsigned)ceil_div(b, 256);
  {
    // chunks for about 1024 workgroups, 32 at least (17664 x 128 54 -> 28 us); the partial sums live in the
    // (still unused) buffer of U': nchunk * b doubles <= b * b floats
    const int64_t want = std::max<int64_t>(32, 1024 / bb);
    int nchunk = (int)std::max<int64_t>(1, std::min<int64_t>(want, c / 64));
    nchunk = (int)std::min<int64_t>(nchunk, std::max<int64_t>(1, b / 2));
    const int64_t rpc = ceil_div(c, nchunk);
    double* part = reinterpret_cast<double*>(U);
    hipLaunchKernelGGL(k_col_loss_part, dim3(bb, (unsigned)nchunk), dim3(256), 0, st, W, c, b, rpc,
                       skip_c, part);
    hipLaunchKernelGGL(k_col_loss_fin, dim3(bb), dim3(256), 0, st, part, H, b, nchunk, v);
    hipLaunchKernelGGL(k_col_rank, dim3((unsigned)ceil_div(b, 4)), dim3(256), 0, st, v, b, rank,
                       sigma);
    THANOS_LAUNCH_CHECK();
  }
  const int staged = b <= kRowLds ? 1 : 0;
  if (b <= kFewCols) {
    hipLaunchKernelGGL(k_permute_sym, dim3((unsigned)b), dim3(256), 0, st, H, b, sigma, HB, 0, 0);
  } else {
    const unsigned t64 = (unsigned)ceil_div(b, 64);  // into the buffer of U', which the factorisation writes last
    hipLaunchKernelGGL(k_mirror, dim3(t64, t64), dim3(256), 0, st, H, b, U);
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_permute_sym),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kRowLds * sizeof(float))));
    hipLaunchKernelGGL(k_permute_sym, dim3((unsigned)b), dim3(256), staged ? (size_t)b * sizeof(float) : 0, st, U, b,
                       sigma, HB, 1, staged);
  }
  THANOS_LAUNCH_CHECK();
  thanos_status e = factor(st, HB, b, damping, U, xn2, fws, info, single_stream);
  if (e != THANOS_OK) return e;
  if (s_cols > 0 && s_cols < b) {  // (no kept column: nothing to update)
    const int64_t s = s_cols;
    // reductions in whole slabs of 32, where that leaves a column of W_Q's buffer free
    const int64_t s32 = ceil_div(s, 32) * 32, sp = s32 < b ? s32 : s;
    int64_t ldL = 0;
    const float* L = factor_L(fws, b, &ldL);
    hipLaunchKernelGGL(k_rev_L, dim3((unsigned)ceil_div(sp, 256), (unsigned)sp), dim3(256), 0, st, L,
                       ldL, b, s, sp, HB);
    THANOS_LAUNCH_CHECK();
    float* const z_top = WQ + c * sp;
    if (b <= kFewCols) {
      hipLaunchKernelGGL(k_gather_cols<64>, dim3((unsigned)ceil_div(c, 4)), dim3(256), (size_t)b * 4 * sizeof(float), st,
                         W, c, b, sigma, factor_scale(fws, b), s, sp, WQ, h, z_top, staged);
    } else {
      THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_gather_cols<256>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(kRowLds * sizeof(float))));
      hipLaunchKernelGGL(k_gather_cols<256>, dim3((unsigned)c), dim3(256), staged ? (size_t)b * sizeof(float) : 0, st,
                         W, c, b, sigma, factor_scale(fws, b), s, sp, WQ, h, z_top, staged);
    }
    THANOS_LAUNCH_CHECK();
    // Z = W_Q U'_ss^{-1}  (c x s), T = Z U'[0:s, :]  (c x b), on the two-way split: W_Q without the scales of the
    // factorisation, which are in U'_ss^{-1} (4096 x 4096, 1366 removed, 363 -> 197 us).  The first s columns of T are the
    // removed ones, which become exact zeros: only the tiles that hold a kept column are computed.
    // Short reductions stay on the three-way split, which is the more accurate one there (gemm_tile_h2.h): what 300
    // rows of 128 columns gain, 39 removed, is off float64 by 8.67e-7 and 8.74e-7 with the two-way one.
    const int64_t n0 = s / 128 * 128;
    if (sp <= kShortK) {
      THANOS_CHECK(gemm_f32(st, false, true, c, sp, sp, 1.f, WQ, sp, HB, sp, 0.f, Z, sp, false));
      THANOS_CHECK(gemm_f32(st, false, true, c, b - n0, sp, 1.f, Z, sp, U + n0, b, 0.f, T + n0, b, false));
    } else {
      THANOS_CHECK(gemm_topped(st, c, sp, sp, WQ, sp, h, HB, sp, nullptr, kBoundL, Z, sp, kTriUpper, nullptr, z_top, false));
      THANOS_CHECK(gemm_topped(st, c, b - n0, sp, Z, sp, z_top, U + n0, b, factor_umax(fws, b) + n0, 0.f, T + n0, b,
                               kTriNone, nullptr, nullptr, false));
    }
  }
  const int64_t s = s_cols;
  if (wdt == THANOS_F32)
    launch_struct_apply<float>(st, W, T, c, b, rank, s, skip_c, mask, W_cast);
  else if (wdt == THANOS_F16)
    launch_struct_apply<__half>(st, W, T, c, b, rank, s, skip_c, mask, W_cast);
  else
    launch_struct_apply<__hip_bfloat16>(st, W, T, c, b, rank, s, skip_c, mask, W_cast);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

}  // namespace thanos
