// Column-block sweep of thanos_prune_layer: mask selection, per-row solve, trailing update.
//
// Per block [j1, j2) of B columns, with U the factor of thanos_factor (H_d^{-1} = U^T U):
//   P_k   = U[j1:j2, j1:j2]^T * U[j1:j2, j1:b]      first (j2-j1) rows of inv(H_d[j1:, j1:]),
//                                                   i.e. every row "R" of Sec. 4.1 can need
//   G     = P_k[:, 0:j2-j1]                          so that R_hat = G[q, q]
//   lambda R_hat = u, u = W[i, j1+q]                 per-row solve (eq. (R_hat), (u))
//   Lam[i, q] = lambda, 0 elsewhere                  scattered multipliers
//   W[:, j1:b] -= Lam * P_k                          == -u R_hat^{-1} R for every row at once
// All P_k are produced by one batched launch before the sweep.
//
// Scaled coordinates.  With sc[j] the power of two that brings the largest magnitude of column j of U into
// [1/2, 1), the sweep works with P' = S P S and u' = u S, which gives lambda' = lambda S^{-1}: the same
// values times powers of two, so nothing changes in them, but no column of P' can outweigh the others, and with
// the largest |lambda'| of each row (rsc) and the largest |P'| of each column of a block (pexp) at hand the
// products can split their operands into two fp16 values (gemm_tile_h2.h).  W stays as it is: the update takes
// the scales out again.
#include <algorithm>

#include <cmath>

#include "gemm_tile_h2.h"
#include "lam_layout.h"
#include "select_plan.h"
#include "solve_plan.h"
#include "tile32.h"

namespace thanos {

// Orders LDS traffic between the lanes of ONE wavefront (no instruction beyond a wait).
#define WAVE_SYNC()                                        \
  do {                                                     \
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); \
    __builtin_amdgcn_wave_barrier();                       \
  } while (0)

// ------------------------------------------------------------------------------------------
// Inverses of the blocks' G matrices, for rows that lose more than half of a block.
// With G = P_k[:, :bw] = U_bb^T U_bb (U_bb the diagonal block of the factor), K = G^{-1} =
// V_bb V_bb^T, where V = U^{-1} is the reverse Cholesky factor the factorisation leaves behind
// (V[x][y] = L[b-1-x][b-1-y], L = its workspace's lower factor of the index-reversed matrix), and
// the diagonal block of the inverse of a triangular matrix is the inverse of its diagonal block:
// no inversion is computed.  Kc[blk][a][j] = sum_{m >= max(a, j)} V[j1+a][j1+m] V[j1+j][j1+m],
// row stride B.  One workgroup per 32 x 32 tile (a0, c0) of a block, in the launch of k_block_rows, beside
// which it takes no time of its own (in a launch of its own 11 us: 512x512 layer 434 -> 422 us).  L is the factor of a scaled matrix: row
// b-1-x of it is d[x] times that of the matrix itself; Kc is in the scaled coordinates of the sweep.
struct CompArgs {
  const float* L;  // nullptr: none wanted
  int64_t ldL;
  const float* d;
  float* Kc;
  int nt, nz;      // tiles of 32 per side of a block; blockIdx.z from nz on
};
__device__ __forceinline__ void comp_tile(const CompArgs& a, const float* __restrict__ sc, int64_t b, int B,
                                          int64_t blk, int a0, int c0, char* sm) {
  float (*Va)[33] = reinterpret_cast<float (*)[33]>(sm);
  float (*Vj)[33] = Va + 32;
  const int64_t j1 = blk * B;
  const int bw = (int)min((int64_t)B, b - j1);
  if (a0 >= bw || c0 >= bw) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // ty 0..15
  float acc[2] = {0.f, 0.f};
  // block-local indices, zero outside the upper triangle; loads from clamped addresses, a tile ahead
  auto at = [&](int x, int y) {
    return a.L[(b - 1 - (j1 + min(x, bw - 1))) * a.ldL + (b - 1 - (j1 + max(min(y, bw - 1), min(x, bw - 1))))];
  };
  auto V = [&](float v, int x, int y) { return (x >= bw || y >= bw || y < x) ? 0.f : v; };
  float va[2], vj[2];
  auto load = [&](int m0) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      va[e] = at(a0 + ty + 16 * e, m0 + tx);
      vj[e] = at(c0 + ty + 16 * e, m0 + tx);
    }
  };
  int m0 = max(a0, c0);
  load(m0);
  for (; m0 < bw; m0 += 32) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      Va[ty + 16 * e][tx] = V(va[e], a0 + ty + 16 * e, m0 + tx);
      Vj[ty + 16 * e][tx] = V(vj[e], c0 + ty + 16 * e, m0 + tx);
    }
    if (m0 + 32 < bw) load(m0 + 32);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float t = acc[e];
#pragma unroll
      for (int m = 0; m < 32; ++m) t = fmaf(Va[ty + 16 * e][m], Vj[tx][m], t);
      acc[e] = t;
    }
    __syncthreads();
  }
  float* out = a.Kc + blk * B * B;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int x = a0 + ty + 16 * e, y = c0 + tx;
    if (x < bw && y < bw) out[(int64_t)x * B + y] = acc[e] / (a.d[j1 + x] * sc[j1 + x]) / (a.d[j1 + y] * sc[j1 + y]);
  }
}

// ------------------------------------------------------------------------------------------
// P[(j1+m)*b + col] = sc[j1+m] sc[col] sum_k U[j1+k][j1+m] * U[j1+k][col], col in [j1, b), for every block.
struct BlockRowsArgs {
  const float* U;
  float* P;
  const float* sc;
  uint8_t* pexp;  // scales of the update's product as biased exponents, by column and 128 rows of a block
  int64_t b;
  int B;
  CompArgs comp;
};

// Rows of pexp: block by block, a block's row tiles in order.
constexpr int64_t block_row_tiles(int B) { return (B + kTM - 1) / kTM; }

constexpr size_t kBlockRowsSmem = kXSmemBytes + (kTM + 8 * kTN) * sizeof(float);
__global__ __launch_bounds__(kXThreads, 4) void k_block_rows(BlockRowsArgs a) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  if (a.comp.L && (int)blockIdx.z >= a.comp.nz) {
    const int t = ((int)blockIdx.z - a.comp.nz) * (int)gridDim.x + (int)blockIdx.x;
    if (t < a.comp.nt * a.comp.nt)
      comp_tile(a.comp, a.sc, a.b, a.B, blockIdx.y, 32 * (t / a.comp.nt), 32 * (t % a.comp.nt), sm);
    return;
  }
  const int64_t j1 = (int64_t)blockIdx.y * a.B;
  const int bw = (int)min((int64_t)a.B, a.b - j1);
  const int64_t col0 = j1 + (int64_t)blockIdx.x * kTN;
  const int mrow0 = (int)blockIdx.z * kTM;  // row tile inside the block (B may exceed 128)
  if (col0 >= a.b || mrow0 >= bw) return;
  const int n_ext = (int)min((int64_t)kTN, a.b - col0);
  const int m_ext = min(kTM, bw - mrow0);
  const float* A = a.U + j1 * a.b + j1 + mrow0;  // (m,k) at A[k*b + m]
  const float* Bm = a.U + j1 * a.b + col0;       // (k,n) at B[k*b + n]
  TileAcc acc;
  acc_zero(acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float s0 = a.sc[min(col0 + 2 * lane, a.b - 1)], s1 = a.sc[min(col0 + 2 * lane + 1, a.b - 1)];
  const float mine = a.sc[min(j1 + mrow0 + ((int)threadIdx.x & (kTM - 1)), a.b - 1)];
  gemm_tile_x3<true, true>(acc, sm, A, a.b, m_ext, Bm, a.b, n_ext, 0, bw);
  float* const sr = reinterpret_cast<float*>(sm + kXSmemBytes);  // scales of the rows, behind the tile
  if (threadIdx.x < kTM) sr[threadIdx.x] = mine;  // a barrier follows in the staging
  const float* T = x3_stage_tile(acc, sm);
  float* Pg = a.P + (j1 + mrow0) * a.b + col0;
  const bool whole = m_ext == kTM && n_ext == kTN;
  uint32_t top0 = 0, top1 = 0;  // largest magnitudes as bits: NaN counts as large
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = wave + 8 * i;
    const float2 t = *reinterpret_cast<const float2*>(T + row * kXCLd + 2 * lane);
    const f32x2u o = {t.x * sr[row] * s0, t.y * sr[row] * s1};
    if (row < m_ext) {
      top0 = max(top0, __float_as_uint(fabsf(o.x)));
      top1 = max(top1, __float_as_uint(fabsf(o.y)));
    }
    if (whole) {
      *reinterpret_cast<f32x2u*>(Pg + (int64_t)row * a.b + 2 * lane) = o;
    } else if (row < m_ext) {
      if (2 * lane < n_ext) Pg[(int64_t)row * a.b + 2 * lane] = o.x;
      if (2 * lane + 1 < n_ext) Pg[(int64_t)row * a.b + 2 * lane + 1] = o.y;
    }
  }
  if (!a.pexp) return;
  uint32_t* const tops = reinterpret_cast<uint32_t*>(sr + kTM);
  tops[wave * kTN + 2 * lane] = top0;
  tops[wave * kTN + 2 * lane + 1] = top1;
  __syncthreads();
  const int col = threadIdx.x;
  if (col >= n_ext) return;
  uint32_t top = tops[col];
#pragma unroll
  for (int v = 1; v < 8; ++v) top = max(top, tops[v * kTN + col]);
  const int64_t at = blockIdx.y * block_row_tiles(a.B) + blockIdx.z;
  a.pexp[at * a.b + col0 + col] = (uint8_t)h2_exponent(__uint_as_float(top));
}

// sc from a given factor (own factors bring the largest magnitudes of their columns along): 16 threads per
// column, eight loads in flight.
__global__ __launch_bounds__(1024) void k_col_scales(const float* __restrict__ U, int64_t b, int B,
                                                     float* __restrict__ sc) {
  __shared__ float part[16][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * 64 + tx, jc = min(j, b - 1);
  const int64_t rows = min(b, ((int64_t)blockIdx.x * 64 + 63) / B * B + B);  // all that k_block_rows reads
  float top = 0.f;
  for (int64_t i = ty; i < rows; i += 8 * 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = fabsf(U[min(i + 16 * e, rows - 1) * b + jc]);
      top = v > top ? v : top;
    }
  }
  part[ty][tx] = top;
  __syncthreads();
  if (ty != 0 || j >= b) return;
  for (int e = 1; e < 16; ++e) top = fmaxf(top, part[e][tx]);
  sc[j] = col_scale(top);
}

// ------------------------------------------------------------------------------------------
// Unstructured selection: exact r-th smallest metric over the residual W[:, j1:b] by a radix
// select on the fp32 bit pattern (11 + 11 + 10 bits), all state on the device.
//
// ONE launch per block (k_select), at most one workgroup per compute unit so that all of them
// are resident at once.  The threshold of a block is predicted from the previous block's: the
// update that writes the new weights also histograms a window of 2048 bins (of 16 to 64 keys)
// around the previous tau, counts what lies below it, and every update workgroup lists the keys of its
// tile that fall inside the window (with their rows).  Every workgroup of k_select works out for
// itself, from the same data, whether the wanted rank falls inside the window.
//   * It does (every block after the first on all data tried): the bin gives all but the last
//     4 to 6 bits of tau.
//     The workgroups go through the per-tile lists in parallel and hand the keys of that bin to
//     workgroup 0, which resolves the last bits and the ties from them: no pass over the
//     weights, and no device-wide fence (on this chip a release fence at device scope writes the
//     L2 of a compute die back, ~20 us after an update has filled it; the hand-over uses atomic
//     stores, loads and counters only, which are coherent across the dies by themselves).
//   * It does not (first block, a threshold that moved out of the window, a full list): all
//     workgroups run the three radix passes over the residual, separated by grid-wide barriers.
// Every wait is bounded: a wait that does not end within kSpinMax polls ends the kernel and
// reports kInfoSelectTimeout through info, so no wave can spin for ever.  Waiting workgroups
// poll a word of their own (or, for the one counter workgroup 0 waits on, are alone in polling):
// hundreds of pollers on one address make every access to that cache line take microseconds.
// The counters of a launch (arrivals, barrier, bin list) are cleared by the update that runs
// between two launches, never by k_select itself, so no workgroup can meet a counter that
// another one has already reset.
struct SelState {
  long long r_rem;      // weights still to remove (before the current block)
  long long need_eq;    // how many keys equal to tau are removed (ties, in (row, col) order)
  int ties_all;         // every key equal to tau is removed: no ranking of ties (need_eq = 2^62)
  int deferred;         // 1: some row of the block was left to the second solver launch
  unsigned int tau;     // r-th smallest key
  int none;             // 1: nothing left to remove
  unsigned int win_lo;  // first bin (key >> win_shift) of the window of the NEXT block
  int win_shift;        // keys per bin of that window = 2^win_shift (kWinShiftMin .. kWinShiftMax)
  int pred_try;         // 1: a window was counted for this block
  int cand_overflow;    // an update workgroup found more window keys than it can list
  // counters of the current k_select launch
  unsigned int arrived; // workgroups that have handed over their part
  unsigned int nbin;    // keys of the threshold's bin handed to workgroup 0
  unsigned int bar;     // arrivals at the grid barriers
};

constexpr int32_t kInfoSelectTimeout = -0x7ffffff0;  // info: a bounded wait of k_select ran out
constexpr int kSelThreads = 64 * kSelRows;
constexpr unsigned int kSpinMax = 1u << 21;
constexpr int kCandStage = 384;       // window keys one update workgroup can list (two update
                                      // workgroups still fit the LDS of a compute unit)
constexpr int kBinCap = 4096;         // keys of the threshold's bin that k_select can resolve
// The window has 2048 bins of 2^shift keys, 1024 on either side of the last threshold.  The bin
// width follows the drift of the threshold from block to block (at least 8 times the last step
// must fit into half the window): 16 keys per bin (+- 0.2 % of tau) while the threshold moves
// little, up to 64 (+- 0.8 %) when it moves more; the lists of window keys grow in proportion,
// which is what bounds the width.
constexpr int kWinShiftMin = 4, kWinShiftMax = 6;

__device__ __forceinline__ unsigned int metric_key(float w, float sx) {
  return __float_as_uint(fabsf(w) * sx);
}

// Workgroup of NT threads: the bin of hist[0 .. nbins) (nbins = 16, 1024 or 2048) that holds
// the rank-th smallest key, the number of keys in the bins before it and inside it.  bin = -1
// if rank is not in 1 .. total.
struct BinSel {
  int bin;
  unsigned int count;
  long long before;
};
// FRESH: the counts come from this launch's own atomics (read past the caches).
template <int NT, bool FRESH = false>
__device__ __forceinline__ BinSel block_select_bin(const unsigned int* hist, int nbins, long long rank) {
  __shared__ long long wtot[NT / 64];
  __shared__ BinSel res;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = nbins >= NT ? nbins / NT : 1;  // at most 8
  unsigned int loc[8];
  long long s = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int idx = tid * per + e;
    loc[e] = !(e < per && idx < nbins) ? 0u
             : FRESH ? __hip_atomic_load(hist + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                     : hist[idx];
    s += loc[e];
  }
  long long incl = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const long long t = __shfl_up(incl, off, 64);
    if (lane >= off) incl += t;
  }
  if (lane == 63) wtot[wave] = incl;
  if (tid == 0) res.bin = -1;
  __syncthreads();
  long long before = incl - s;
  for (int v = 0; v < wave; ++v) before += wtot[v];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (rank > 0 && before < rank && rank <= before + loc[e]) {
      res.bin = tid * per + e;
      res.count = loc[e];
      res.before = before;
    }
    before += loc[e];
  }
  __syncthreads();
  const BinSel r = res;
  __syncthreads();  // res and wtot are free for the next call
  return r;
}

// Sum of one value per thread over a workgroup of NT threads (all threads get it).
template <int NT>
__device__ __forceinline__ long long block_sum(long long v) {
  __shared__ long long wsum[NT / 64];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  long long t = 0;
  for (int w = 0; w < NT / 64; ++w) t += wsum[w];
  __syncthreads();
  return t;
}

// PASS 0: bin = key >> 21.  PASS 1: keys with key>>21 == prefix, bin = (key>>10) & 2047.
// PASS 2: keys with key>>10 == prefix, bin = the low 10 bits; also counts those keys (cand).
template <int PASS>
__device__ __forceinline__ void sel_count(unsigned int* h, unsigned int key, unsigned int prefix,
                                          int& cand) {
  if (PASS == 0) {
    atomicAdd(&h[key >> 21], 1u);
  } else if (PASS == 1) {
    if ((key >> 21) == prefix) atomicAdd(&h[(key >> 10) & 2047u], 1u);
  } else {
    if ((key >> 10) == prefix) {
      atomicAdd(&h[key & 1023u], 1u);
      ++cand;
    }
  }
}

struct SelectArgs {
  const float* W;
  const float* sx;
  SelState* st;
  unsigned int* hist;              // window histogram, then the three radix passes (4 x 2048)
  const unsigned int* below_part;  // keys below the window, one count per update workgroup
  int n_part;                      // update workgroups (tiles) of the previous block
  const unsigned int* cand_n;      // per tile: keys inside the window
  const uint2* cand;               // per tile: cand_cap x (key, row)
  int cand_cap;
  unsigned long long* binlist;     // kBinCap x (row << 32 | key): the threshold's bin
  const int* row_cnt;              // weights the previous block removed from each row
  int* row_cand;                   // per row: keys sharing the bits resolved before the last pass
  int* row_eq;                     // per row: keys equal to tau, then their exclusive prefix
  float* tau_out;                  // optional: threshold of this block
  int32_t* info;
  int64_t c, b, j1;
  int first;                       // first block: no window exists
  int vec;                         // 16-byte loads of the row segments are aligned
  unsigned int seq;                // block sequence number, >= 1
  // One word per workgroup, each in a cache line of its own (stride kFlagStride), through which
  // a grid barrier releases it.  Values only grow: 8 * seq + k after barrier k of block seq.
  unsigned int* wgflag;
};
constexpr int kFlagStride = 32;  // words (128 bytes)

// Thread 0 of the calling workgroup waits until *f has reached `want` (bounded).
__device__ __forceinline__ unsigned int wait_word(const unsigned int* f, unsigned int want) {
  unsigned int n = 0, v = 0;
  for (;;) {
    v = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v >= want || ++n >= kSpinMax) break;
    __builtin_amdgcn_s_sleep(8);
  }
  return v;
}

// One radix pass of the calling workgroup over its rows (one wavefront per row; lanes stride
// over the residual columns, 16 bytes per lane when aligned, four loads in flight).  The
// workgroup's LDS histogram is added to hist_out at the end.  It has kSelCopies copies, dealt to the
// lanes: the first pass counts exponents, a few bins for all keys, and one copy would take the 64
// lanes of an instruction one after the other.
constexpr int kSelCopies = 4;
template <int PASS>
__device__ __forceinline__ void sel_pass(const SelectArgs& a, unsigned int* h, unsigned int prefix,
                                         unsigned int* __restrict__ hist_out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < kSelCopies * 2048; e += kSelThreads) h[e] = 0u;
  __syncthreads();
  unsigned int* mine = h + 2048 * (lane & (kSelCopies - 1));
  constexpr int RW = kSelThreads / 64;  // rows per workgroup and step
  for (int64_t i = (int64_t)blockIdx.x * RW + wave; i < a.c; i += (int64_t)gridDim.x * RW) {
    const float* row = a.W + i * a.b;
    int cand = 0;
    if (a.vec) {
      const int64_t nvec = (a.b - a.j1) >> 2;
      for (int64_t v0 = lane; v0 < nvec; v0 += 4 * 64) {
        float4 w4[4], s4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t j = a.j1 + 4 * min(v0 + 64 * u, nvec - 1);
          w4[u] = *reinterpret_cast<const float4*>(row + j);
          s4[u] = *reinterpret_cast<const float4*>(a.sx + j);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (v0 + 64 * u < nvec) {
            sel_count<PASS>(mine, metric_key(w4[u].x, s4[u].x), prefix, cand);
            sel_count<PASS>(mine, metric_key(w4[u].y, s4[u].y), prefix, cand);
            sel_count<PASS>(mine, metric_key(w4[u].z, s4[u].z), prefix, cand);
            sel_count<PASS>(mine, metric_key(w4[u].w, s4[u].w), prefix, cand);
          }
      }
      for (int64_t j = a.j1 + 4 * nvec + lane; j < a.b; j += 64)
        sel_count<PASS>(mine, metric_key(row[j], a.sx[j]), prefix, cand);
    } else {
      for (int64_t j = a.j1 + lane; j < a.b; j += 64)
        sel_count<PASS>(mine, metric_key(row[j], a.sx[j]), prefix, cand);
    }
    if (PASS == 2) {
      for (int off = 32; off > 0; off >>= 1) cand += __shfl_down(cand, off, 64);
      if (lane == 0)
        __hip_atomic_store(a.row_cand + i, cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  for (int e = tid; e < 2048; e += kSelThreads) {
    unsigned int n = 0;
#pragma unroll
    for (int u = 0; u < kSelCopies; ++u) n += h[2048 * u + e];
    if (n) atomicAdd(&hist_out[e], n);
  }
}

// All workgroups of the launch have arrived at barrier `phase` (1, 2, ...) of this block: each
// adds itself to a counter, and the one that completes the count releases every workgroup
// through its own word.  No fence at device scope: what crosses the barrier (histograms, counts per
// row) is written with atomics or atomic stores, which are complete when a wavefront's vmcnt is zero,
// and read with atomic loads.  Such fences on both sides, one per wavefront behind the barrier, wrote
// the L2s back thousands of times: three passes over 4096 x 4096 took 310 us, and 200 over the last
// 128 columns (now 67 and 30).  Returns false if the wait ran out.
__device__ __forceinline__ bool grid_barrier(const SelectArgs& a, unsigned int phase) {
  __shared__ int ok, last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(&a.st->bar, 1u) + 1u == phase * gridDim.x ? 1 : 0;
  __syncthreads();
  const unsigned int want = 8u * a.seq + phase;
  if (last)
    for (unsigned int w = threadIdx.x; w < gridDim.x; w += kSelThreads)
      __hip_atomic_store(a.wgflag + (size_t)w * kFlagStride, want, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 0)
    ok = wait_word(a.wgflag + (size_t)blockIdx.x * kFlagStride, want) >= want ? 1 : 0;
  __syncthreads();
  return ok != 0;
}

// Exclusive prefix sum of row_eq over the rows by one workgroup, in place: afterwards row_eq[i]
// = number of keys equal to tau in the rows before row i (ties are taken in (row, column) order).
__device__ __forceinline__ void tie_prefix(int* row_eq, int64_t c) {
  __shared__ long long wtot[kSelThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t per = (c + kSelThreads - 1) / kSelThreads;
  const int64_t lo = tid * per, hi = min(c, lo + per);
  long long s = 0;
  auto count = [&](int64_t i) {
    return __hip_atomic_load(row_eq + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int64_t i = lo; i < hi; ++i) s += count(i);
  long long incl = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const long long t = __shfl_up(incl, off, 64);
    if (lane >= off) incl += t;
  }
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  long long run = incl - s;
  for (int v = 0; v < wave; ++v) run += wtot[v];
  for (int64_t i = lo; i < hi; ++i) {
    const int v = count(i);
    row_eq[i] = (int)min(run, (long long)0x7fffffff);
    run += v;
  }
}

// Workgroup 0, at the end of the launch: the state later kernels read.  tau_valid: a threshold
// was found (else nothing is left to remove).
__device__ __forceinline__ void publish(const SelectArgs& a, long long r_rem, bool tau_valid,
                                        unsigned int tau, long long rank_eq, bool all) {
  SelState* st = a.st;
  for (int e = threadIdx.x; e < 2048; e += kSelThreads) a.hist[e] = 0u;  // window: consumed
  if (threadIdx.x != 0) return;
  st->r_rem = r_rem;
  st->none = tau_valid ? 0 : 1;
  st->deferred = 0;
  st->cand_overflow = 0;
  if (!tau_valid) {
    if (a.tau_out) *a.tau_out = -1.f;
    return;
  }
  // bin width of the next window from the step the threshold has just taken
  int shift = kWinShiftMin;
  if (!a.first && st->tau != 0u) {
    const unsigned int prev = st->tau;
    const unsigned int step = tau > prev ? tau - prev : prev - tau;
    while (shift < kWinShiftMax && (1024u << shift) < 8u * (unsigned long long)step) ++shift;
  }
  st->tau = tau;
  if (a.tau_out) *a.tau_out = __uint_as_float(tau);
  st->need_eq = all ? (1ll << 62) : rank_eq;
  st->ties_all = all ? 1 : 0;
  const unsigned int pb = tau >> shift;
  st->pred_try = tau != 0u ? 1 : 0;
  st->win_shift = shift;
  st->win_lo = pb > 1024u ? pb - 1024u : 0u;
}

__global__ __launch_bounds__(kSelThreads) void k_select(SelectArgs a) {
  // workgroup 0, window hit: the threshold's bin; otherwise the histograms of the radix passes
  __shared__ unsigned long long bins[kBinCap];
  static_assert(sizeof(bins) == kSelCopies * 2048 * sizeof(unsigned int), "both uses fit");
  unsigned int* h = reinterpret_cast<unsigned int*>(bins);
  __shared__ unsigned int h16[1 << kWinShiftMax];  // counts of the bin's keys by their low bits
  __shared__ unsigned int s_ok;
  SelState* st = a.st;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int RW = kSelThreads / 64;

  // ---- every workgroup: r <- r - ||M||_F^2 of the previous block (Alg. 1), the keys below the
  //      window, and whether the window holds the wanted rank.  Nothing read here is written
  //      before all workgroups have handed over (workgroup 0 writes the state at the very end).
  long long sum = 0, bsum = 0;
  if (!a.first) {
    for (int64_t i = tid; i < a.c; i += kSelThreads) sum += a.row_cnt[i];
    for (int e = tid; e < a.n_part; e += kSelThreads) bsum += a.below_part[e];
  }
  const long long r_old = st->r_rem;
  const bool pred_try = !a.first && st->pred_try != 0 && st->cand_overflow == 0;
  const unsigned int win_lo = st->win_lo;
  const int wsh = st->win_shift;
  const long long r_rem = r_old - block_sum<kSelThreads>(sum);
  const long long below = block_sum<kSelThreads>(bsum);
  const bool none = r_rem <= 0;
  BinSel r;
  r.bin = -1;
  r.count = 0;
  r.before = 0;
  if (!none && pred_try) r = block_select_bin<kSelThreads>(a.hist, 2048, r_rem - below);
  const bool hit = r.bin >= 0 && r.count <= (unsigned int)kBinCap;

  if (none || hit) {
    if (hit) {
      // ---- the keys of the threshold's bin: one wavefront per tile list; the list of a tile
      //      holds at most kCandStage entries, i.e. up to 6 independent loads per lane ----
      const unsigned int prefix28 = win_lo + (unsigned int)r.bin;
      for (int t = (int)blockIdx.x * RW + wave; t < a.n_part; t += (int)gridDim.x * RW) {
        const unsigned int n = min(a.cand_n[t], (unsigned int)a.cand_cap);
        const uint2* list = a.cand + (size_t)t * a.cand_cap;
        uint2 kr[kCandStage / 64];
#pragma unroll
        for (int u = 0; u < kCandStage / 64; ++u) kr[u] = list[min(64 * u + lane, a.cand_cap - 1)];
#pragma unroll
        for (int u = 0; u < kCandStage / 64; ++u)
          if ((unsigned int)(64 * u + lane) < n && (kr[u].x >> wsh) == prefix28) {
            const unsigned int slot = atomicAdd(&st->nbin, 1u);
            if (slot < (unsigned int)kBinCap)
              __hip_atomic_store(a.binlist + slot,
                                 ((unsigned long long)kr[u].y << 32) | kr[u].x, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          }
      }
    }
    // hand over: this workgroup's entries have left before it counts itself in
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    if (tid == 0) atomicAdd(&st->arrived, 1u);
    if (blockIdx.x != 0) return;

    // ---- workgroup 0: wait for the others (it is the only one polling this counter) ----
    if (tid == 0) s_ok = wait_word(&st->arrived, gridDim.x) >= gridDim.x ? 1u : 0u;
    __syncthreads();
    if (!s_ok) {
      if (tid == 0) atomicCAS(a.info, 0, kInfoSelectTimeout);
      return;
    }
    if (none) {
      publish(a, r_rem, false, 0u, 0, true);
      return;
    }
    const unsigned int nbin = __hip_atomic_load(&st->nbin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (nbin != r.count) {  // the lists and the histogram disagree: cannot happen
      if (tid == 0) atomicCAS(a.info, 0, kInfoSelectTimeout);
      return;
    }
    const unsigned int nlow = 1u << wsh;
    if (tid < (int)nlow) h16[tid] = 0u;
    __syncthreads();
    for (unsigned int e = tid; e < nbin; e += kSelThreads) {
      const unsigned long long v =
          __hip_atomic_load(a.binlist + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bins[e] = v;
      atomicAdd(&h16[(unsigned int)v & (nlow - 1u)], 1u);
    }
    __syncthreads();
    long long rank = r_rem - below - r.before;  // 1-based rank inside the bin
    unsigned int low = 0, cnt_eq = 0;
    for (unsigned int v = 0; v < nlow; ++v) {   // uniform: every thread walks the counts
      if (rank <= (long long)h16[v]) {
        low = v;
        cnt_eq = h16[v];
        break;
      }
      rank -= h16[v];
    }
    const unsigned int prefix28 = win_lo + (unsigned int)r.bin;
    const unsigned int tau = (prefix28 << wsh) | low;
    const bool all = rank == (long long)cnt_eq;
    if (!all) {
      // ties to rank (some, not all, keys equal to tau are removed), in (row, column) order:
      // row_eq[i] = keys equal to tau in the rows before row i, counted from the bin in LDS
      for (int64_t i = tid; i < a.c; i += kSelThreads) {
        int before = 0;
        for (unsigned int e = 0; e < nbin; ++e)
          before += ((unsigned int)bins[e] == tau && (unsigned int)(bins[e] >> 32) < (unsigned int)i) ? 1 : 0;
        a.row_eq[i] = before;
      }
    }
    publish(a, r_rem, true, tau, rank, all);
    return;
  }

  // ---- radix passes over the residual, all workgroups (the histograms of the passes were
  //      cleared by the update, or by the fill at the start of the sweep) ----
  unsigned int* hist_a = a.hist + 2048;
  unsigned int* hist_b = a.hist + 2 * 2048;
  unsigned int* hist_c = a.hist + 3 * 2048;
  bool ok = true;
  sel_pass<0>(a, h, 0u, hist_a);
  ok = grid_barrier(a, 1u);
  const BinSel r0 = block_select_bin<kSelThreads, true>(hist_a, 2048, r_rem);
  const unsigned int prefix1 = (unsigned int)r0.bin;
  const long long rank1 = r_rem - r0.before;
  if (ok) {
    sel_pass<1>(a, h, prefix1, hist_b);
    ok = grid_barrier(a, 2u);
  }
  const BinSel r1 = block_select_bin<kSelThreads, true>(hist_b, 2048, rank1);
  const unsigned int prefix2 = (prefix1 << 11) | (unsigned int)r1.bin;
  const long long rank2 = rank1 - r1.before;
  if (ok) {
    sel_pass<2>(a, h, prefix2, hist_c);
    ok = grid_barrier(a, 3u);
  }
  if (!ok) {
    if (tid == 0) atomicCAS(a.info, 0, kInfoSelectTimeout);
    return;
  }
  // The last pass resolves the key completely, so the chosen bin counts the keys equal to tau:
  // if all of them are removed (the usual case: one key at the threshold) their order does not
  // matter and nothing is ranked.
  const BinSel r2 = block_select_bin<kSelThreads, true>(hist_c, 1024, rank2);
  const unsigned int tau = (prefix2 << 10) | (unsigned int)r2.bin;
  const long long rank_eq = rank2 - r2.before;  // keys equal to tau that are removed
  const bool all = rank_eq == (long long)r2.count;
  if (all) {
    if (blockIdx.x == 0) publish(a, r_rem, true, tau, rank_eq, true);
    return;
  }
  // rows that hold candidates (keys sharing the 22 bits resolved before the last pass) count
  // their keys equal to tau over the residual row; other rows have none
  for (int64_t i = (int64_t)blockIdx.x * RW + wave; i < a.c; i += (int64_t)gridDim.x * RW) {
    int n = 0;
    if (__hip_atomic_load(a.row_cand + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      const float* row = a.W + i * a.b;
      if (a.vec) {
        const int64_t nvec = (a.b - a.j1) >> 2;
        for (int64_t v = lane; v < nvec; v += 64) {
          const int64_t j = a.j1 + 4 * v;
          const float4 w4 = *reinterpret_cast<const float4*>(row + j);
          const float4 s4 = *reinterpret_cast<const float4*>(a.sx + j);
          n += (metric_key(w4.x, s4.x) == tau) + (metric_key(w4.y, s4.y) == tau) +
               (metric_key(w4.z, s4.z) == tau) + (metric_key(w4.w, s4.w) == tau);
        }
        for (int64_t j = a.j1 + 4 * nvec + lane; j < a.b; j += 64)
          n += (metric_key(row[j], a.sx[j]) == tau) ? 1 : 0;
      } else {
        for (int64_t j = a.j1 + lane; j < a.b; j += 64)
          n += (metric_key(row[j], a.sx[j]) == tau) ? 1 : 0;
      }
      for (int off = 32; off > 0; off >>= 1) n += __shfl_down(n, off, 64);
    }
    if (lane == 0) __hip_atomic_store(a.row_eq + i, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!grid_barrier(a, 4u)) {
    if (tid == 0) atomicCAS(a.info, 0, kInfoSelectTimeout);
    return;
  }
  if (blockIdx.x == 0) {
    tie_prefix(a.row_eq, a.c);
    publish(a, r_rem, true, tau, rank_eq, false);
  }
}

// Ties before row i; row_eq is stale (and not read) when no tie needs ranking.
__device__ __forceinline__ long long ties_before(const SelState* __restrict__ st,
                                                 const int* __restrict__ row_eq, int64_t i) {
  return (st->none || st->ties_all) ? 0 : (long long)row_eq[i];
}

// ------------------------------------------------------------------------------------------
// Mask + per-row solve (Alg. 1, loop over the rows of W; Sec. 4.1, eqs. (R_hat), (u)):
// lambda R_hat = u with R_hat = G[q, q], G the block's rows of the residual inverse, q the
// removed columns of the row (Sec. 4.5), u the removed weights.  Three kernels share the
// arguments below and differ in how many unknowns they hold and where.
// SEL_PICKED: k_pick has chosen the block's mask (mask_out, row_cnt) and k_lam_rows turns what the rows
// solved through the complement leave in Z into multipliers.
enum { SEL_NM = 0, SEL_THRESHOLD = 1, SEL_GIVEN = 2, SEL_PICKED = 3 };

struct SolveArgs {
  const float* W;        // c x b, current weights
  const float* P;        // b x b, block rows of the residual inverses
  const float* sx;       // sqrt(xnorm2)
  const float* sc;       // scales of the columns
  float* rsc;            // per row: scale of its multipliers for the update (the smallest of a super-block)
  int rsc_first;         // first block of a super-block
  const uint8_t* mask_in;
  uint8_t* mask_out;     // c x b
  float* Lam;            // c x ldl
  const SelState* st;    // SEL_THRESHOLD
  SelState* st_rw;
  const int* row_eq;     // exclusive tie prefix per row (k_select; see ties_before)
  int* row_cnt;          // SEL_THRESHOLD: number of weights removed from row i in this block
  const uint8_t* row_skip;  // optional, c bytes: 1 = row is left untouched (outlier row)
  int32_t* info;
  int64_t c, b, j1;
  int bw, ldl, n, m;
  int nt_lo, nt_max;     // k_solve_tiled: rows with nt_lo <= ceil(s/32) <= nt_max; LDS holds nt_max
  int s_min;             // k_solve_wide: rows with s < s_min belong to another launch
  float* tile_scratch;   // k_solve_tiled<.., BIG>: tile grids in global memory, one slot per workgroup
  int64_t slot_floats;
  const float* Kc;       // k_solve_tiled: inverse of this block's G (bw x bw, row stride ldk), or
  int ldk;               // nullptr; rows that lose more than half of the block are solved through it
  int defer_large;       // k_solve_mfma: rows with more unknowns than it holds belong to another launch
  float* Z;              // SEL_PICKED: c x ldz, w~ on entry, (w~ - y~) of the complement rows on return
  const float* WK;       // SEL_PICKED: c x ldz, w~ K
  int ldz;
};

// rsc of row i, for m = the largest |lambda'| that the calling lane has written: by the one wavefront that
// writes the row, or (rsc_clear before a barrier, then rsc_lower by every wavefront) by several.
__device__ __forceinline__ float wave_max(float m) {  // m >= 0; in registers: the row waits for it
  uint32_t u = __float_as_uint(m);
#define ROW_STEP(ctrl) u = max(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, ctrl, 0xf, 0xf, false))
  ROW_STEP(0x121);  // rotations within 16 lanes, by 1, 2, 4, 8
  ROW_STEP(0x122);
  ROW_STEP(0x124);
  ROW_STEP(0x128);
#undef ROW_STEP
  auto h = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  u = max((uint32_t)h[0], (uint32_t)h[1]);
  h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(max((uint32_t)h[0], (uint32_t)h[1]));
}
__device__ __forceinline__ float rsc_old(const SolveArgs& a, int64_t i) {
  return a.rsc_first ? h2_scale(0.f) : a.rsc[i];
}
__device__ __forceinline__ void rsc_set(const SolveArgs& a, int64_t i, float m, float old) {
  const float s = h2_scale(wave_max(m));
  if ((threadIdx.x & 63) == 0) a.rsc[i] = fminf(old, s);
}
__device__ __forceinline__ void rsc_clear(const SolveArgs& a, int64_t i) {
  if (a.rsc_first) __hip_atomic_store(a.rsc + i, h2_scale(0.f), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void rsc_lower(const SolveArgs& a, int64_t i, float m) {
  const float s = h2_scale(wave_max(m));
  if ((threadIdx.x & 63) == 0)  // positive floats compare as their bits
    atomicMin(reinterpret_cast<unsigned int*>(a.rsc + i), __float_as_uint(s));
}

// ------------------------------------------------------------------------------------------
// Mask + per-row solve for systems of up to SMAX = 128 or 256 unknowns: one workgroup of SMAX
// threads (2 or 4 wavefronts) per row of W, thread t <-> block column t <-> row t of R_hat
// (SMAX registers).
// Symmetric Gauss-Jordan elimination (no back-substitution: after s steps lambda_k = u_k / d_k)
// in its square-root-free form  A[rho][j] -= (A[rho][k] / d) * A[j][k],  so that the broadcast
// column needs no scaling; after every panel of 4 pivots the registers are renamed (column j
// moves to register j - 4), which keeps all register indices static.  The pivot column travels
// through LDS (one barrier per pivot).
// Only the registers that still hold live columns (j < s - 4*panel) are touched, in chunks of
// 16, so a system of s unknowns costs ~s^2/2 fused multiply-adds per thread, not s*128.
template <int SEL, int SMAX>
__global__ __launch_bounds__(SMAX, (SMAX == 128 ? 3 : 1)) void k_solve_wide(SolveArgs a) {
  constexpr int NWV = SMAX / 64;
  __shared__ __attribute__((aligned(16))) float col[2][4][SMAX + 32];  // tail stays zero
  __shared__ float ukb[2][4];
  __shared__ float wrow[SMAX];
  __shared__ float key[SMAX];
  __shared__ int q[SMAX];
  __shared__ int cnt[NWV];
  __shared__ int eqc[NWV];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t i = blockIdx.x;
  const float* wrow_g = a.W + i * a.b + a.j1;
  // second launch of a block (s_min > 0): nothing to do unless the first one left rows behind
  if (SEL == SEL_THRESHOLD && a.s_min > 0 && a.st->deferred == 0) return;

  const float w = (tid < a.bw) ? wrow_g[tid] : 0.f;
  wrow[tid] = (tid < a.bw) ? w * a.sc[a.j1 + tid] : 0.f;
  for (int e = tid; e < 2 * 4 * (SMAX + 32); e += SMAX) (&col[0][0][0])[e] = 0.f;
  bool sel = false;
  if (SEL == SEL_GIVEN) {
    sel = (tid < a.bw) && a.mask_in[i * a.b + a.j1 + tid] != 0;
  } else if (SEL == SEL_NM) {
    key[tid] = (tid < a.bw) ? fabsf(w) * a.sx[a.j1 + tid] : 0.f;
    __syncthreads();
    if (tid < a.bw) {
      const int g0 = (tid / a.m) * a.m;
      const float mine = key[tid];
      int rank = 0;
      for (int e = 0; e < a.m; ++e) {
        const float o = key[g0 + e];
        rank += (o < mine || (o == mine && g0 + e < tid)) ? 1 : 0;
      }
      sel = rank < a.n;
    }
    if (a.row_skip && a.row_skip[i]) sel = false;
  } else {  // SEL_THRESHOLD
    const bool none = a.st->none != 0;
    const unsigned int tau = a.st->tau;
    const long long need_eq = a.st->need_eq;
    const bool in = (tid < a.bw) && !none;
    const unsigned int kk = in ? metric_key(w, a.sx[a.j1 + tid]) : 0xffffffffu;
    const bool lt = in && kk < tau;
    const bool eq = in && kk == tau;
    const unsigned long long eqb = __ballot(eq);
    if (lane == 0) eqc[wave] = __popcll(eqb);
    __syncthreads();
    int eq_before = 0;
    for (int v = 0; v < wave; ++v) eq_before += eqc[v];
    const long long my = ties_before(a.st, a.row_eq, i) + eq_before +
                         __popcll(eqb & ((1ull << lane) - 1ull));
    sel = lt || (eq && my < need_eq);
  }
  const unsigned long long bal = __ballot(sel);
  if (lane == 0) cnt[wave] = __popcll(bal);
  __syncthreads();
  int s = 0, sel_before = 0;
  for (int v = 0; v < NWV; ++v) {
    if (v < wave) sel_before += cnt[v];
    s += cnt[v];
  }
  if (s < a.s_min) return;  // solved by the launch for smaller systems
  const int myrank = sel_before + __popcll(bal & ((1ull << lane) - 1ull));
  if (sel) q[myrank] = tid;
  if (tid < a.bw) a.mask_out[i * a.b + a.j1 + tid] = sel ? 1 : 0;
  if (SEL == SEL_THRESHOLD) {
    if (tid == 0) a.row_cnt[i] = s;  // summed at the start of the next block
  }
  float* lam_g = a.Lam + i * a.ldl;
  if (tid == 0) rsc_clear(a, i);
  if (s == 0) {
    if (tid < a.bw) lam_g[tid] = 0.f;
    return;
  }
  __syncthreads();

  // ---- gather R_hat: A[j] = G[q_j][q_rho] (= G[q_rho][q_j]) ----
  const float* G = a.P + a.j1 * a.b + a.j1;
  const int rho = tid;
  const int qr = (rho < s) ? q[rho] : 0;
  float u = (rho < s) ? wrow[qr] : 0.f;
  float dinv = 0.f;
  float A[SMAX];
  // Loads are issued unconditionally, 16 at a time, from clamped (valid) indices and masked
  // afterwards: a conditional load, or a select right behind a load, makes the compiler wait for
  // every outstanding load, i.e. one memory round trip per element.  q * b < 2^31.
  {
    const unsigned int bb = (unsigned int)a.b, qc = (unsigned int)qr;
#pragma unroll
    for (int c16 = 0; c16 < SMAX / 16; ++c16) {
      if (16 * c16 < s) {
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
          const int j = 16 * c16 + jj;
          A[j] = G[(unsigned int)q[min(j, s - 1)] * bb + qc];
        }
      } else {
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) A[16 * c16 + jj] = 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < SMAX; ++j) A[j] = (j < s && rho < s) ? A[j] : 0.f;
  }

  // ---- elimination ----
  bool bad = false;
  const int npanel = (s + 3) >> 2;
  for (int pnl = 0; pnl < npanel; ++pnl) {
    const int k0 = 4 * pnl;
    const int wact = s - k0;  // live registers: columns k0 .. s-1
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = k0 + t;
      float* cb = col[pnl & 1][t];
      cb[rho] = A[t];
      if (rho == k) ukb[pnl & 1][t] = u;
      __syncthreads();
      const float d = cb[k];
      const float uk = ukb[pnl & 1][t];
      float rd = 0.f;
      if (k < s) {
        if (d > 0.f) rd = 1.f / d;
        else bad = true;
      }
      float m = A[t] * rd;
      if (rho == k) {
        dinv = rd;
        m = 0.f;  // the pivot row itself is not modified
      }
      u = fmaf(-m, uk, u);
      const f32x4* cv = reinterpret_cast<const f32x4*>(&cb[k0]);  // register j <-> column k0 + j
      if (t < 3) {
#pragma unroll
        for (int c16 = 0; c16 < SMAX / 16; ++c16) {
          if (16 * c16 < wact) {
#pragma unroll
            for (int j4 = 4 * c16; j4 < 4 * c16 + 4; ++j4) {
              const f32x4 lb = cv[j4];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int j = 4 * j4 + e;
                if (j > t) A[j] = fmaf(-m, lb[e], A[j]);
              }
            }
          }
        }
      } else {
#pragma unroll
        for (int c16 = 0; c16 < SMAX / 16; ++c16) {
          if (16 * c16 < wact + 4) {
#pragma unroll
            for (int j4 = 4 * c16; j4 < 4 * c16 + 4; ++j4) {
              if (j4 >= 1) {
                const f32x4 lb = cv[j4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const int j = 4 * j4 + e;
                  A[j - 4] = fmaf(-m, lb[e], A[j]);
                }
              }
            }
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) A[SMAX - 4 + e] = 0.f;
      }
    }
  }
  if (bad && tid == 0) atomicCAS(a.info, 0, -(int32_t)min(i + 1, (int64_t)0x7fffffff));

  // ---- lambda row: zeros except lambda_k = u_k / d_k at column q_k ----
  __syncthreads();
  wrow[tid] = 0.f;
  __syncthreads();
  if (rho < s) wrow[qr] = u * dinv;
  __syncthreads();
  if (tid < a.bw) lam_g[tid] = wrow[tid];
  rsc_lower(a, i, fabsf(wrow[tid]));
}

// Lanes l .. l + 7 (constants) of v <- the bits s[0 .. 7], uniform.  (The wait is for the v_readlane that has just
// produced the last of them, which the compiler does not look for inside the asm; one wait for each of them was a third
// of a sweep.)
#define set_lanes8(v, s, l)                                                                                        \
  asm volatile(                                                                                                    \
      "s_nop 1\n\tv_writelane_b32 %0, %1, %9\n\tv_writelane_b32 %0, %2, %10\n\tv_writelane_b32 %0, %3, %11\n\t"        \
      "v_writelane_b32 %0, %4, %12\n\tv_writelane_b32 %0, %5, %13\n\tv_writelane_b32 %0, %6, %14\n\t"                  \
      "v_writelane_b32 %0, %7, %15\n\tv_writelane_b32 %0, %8, %16"                                                 \
      : "+v"(v)                                                                                                    \
      : "s"(s[0]), "s"(s[1]), "s"(s[2]), "s"(s[3]), "s"(s[4]), "s"(s[5]), "s"(s[6]), "s"(s[7]), "i"(l), "i"((l) + 1), \
        "i"((l) + 2), "i"((l) + 3), "i"((l) + 4), "i"((l) + 5), "i"((l) + 6), "i"((l) + 7))

// ------------------------------------------------------------------------------------------
// Mask + per-row solve on the matrix cores for systems of up to 32 NTR unknowns (NTR = 2 or 3,
// block width <= 128): one wavefront per row of W.  R_hat is held in the accumulator layout of
// v_mfma_f32_32x32x2_f32 as the lower triangle of a grid of 32x32 tiles (identity on the unused
// part): diagonal tiles as they are, tile (i, j), i > j, transposed (register r of lane (lo, hi)
// = R_hat[32 i + lo][32 j + row(r, hi)]), so that column k of a tile below the pivot tile is
// again row k of the register tile.  Symmetric elimination, square-root free (R_hat = L~ D L~^T):
// row k of a symmetric tile in that layout is at once both operands of its rank-1 update, and
// rows k and k + 4 share a register (lower / upper half of the wavefront), so a PAIR of pivots
// of tile row p costs one MFMA per live tile (i, j), p <= j <= i; the cross-lane traffic is the
// broadcast of the pivots and one cross-lane read per tile row (the second pivot's row must
// first see the elimination of the first).  The columns of -L~ go to LDS, and L~ y = u,
// L~^T lambda = D^-1 y are solved afterwards by sweeps over them.
// NTR = 2 serves n:m at B = 128 (s = 64 for 2:4 and 4:8), and the unstructured mode at B = 128, where s scatters around
// 64, for more rows than NTR = 3 can run at once: rows with more than 64 go through the complement.
// A row waits for itself most of its 27000 cycles, so what counts for many rows is how many a compute unit holds: 8 KB
// of LDS each and at most 102 registers, sixteen or twenty.  4096 rows at 50 %: 35 us per block instead of 53 (NTR = 3, eight).
template <int NTR>
struct SolveMfmaSmem {
  static constexpr int N = 32 * NTR;
  // strict lower triangle of L~, packed by rows, and room for the lanes that have nothing to store (16) and for what the
  // sweeps over it read past its end, for lanes that are final: of the last row a whole wavefront's values;
  // before the elimination and after the back-substitution the first 256 floats hold the row's
  // weights (then lambda) and metric
  static constexpr int kLen = N * (N - 1) / 2 + (NTR == 2 ? 16 : 48);
  static_assert((N - 1) * (N - 2) / 2 + 64 * ((N - 2) / 64) + 63 < kLen, "the sweeps read L up to here");
  float L[kLen];
  alignas(4) unsigned char q[NTR == 2 ? 64 : 128];
};

static_assert(sizeof(SolveMfmaSmem<2>) == 8192, "five rows to a quarter of a compute unit's LDS");

// FULL: the host knows that every row has either no unknown or exactly 32 NTR (n:m on a whole
// block): the padding logic folds away.
template <int SEL, int WPB, int NTR, bool FULL = false>
__global__ __launch_bounds__(64 * WPB, NTR == 2 ? 5 : 3) void k_solve_mfma(SolveArgs a) {
  constexpr int CPL = 2;  // block width <= 128
  constexpr int NZ = (NTR + 1) / 2;  // registers holding y / d: rows 64 z + lane
  extern __shared__ __attribute__((aligned(16))) char solve_smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SolveMfmaSmem<NTR>& sm = reinterpret_cast<SolveMfmaSmem<NTR>*>(solve_smem)[wave];
  float* const wrow = sm.L;
  float* const key = sm.L + 128;
  const int lo = lane & 31, hi = lane >> 5;
  const int64_t i = (int64_t)blockIdx.x * WPB + wave;
  if (i >= a.c) return;
  const float* wrow_g = a.W + i * a.b + a.j1;
  const float old_rsc = rsc_old(a, i);

  // ---- selection of the block mask row M_i ----
  bool sel[CPL];
  float wv[CPL], us[CPL];  // weights, and in scaled coordinates
#pragma unroll
  for (int r = 0; r < CPL; ++r) {
    const int col = lane + 64 * r;
    wv[r] = (col < a.bw) ? wrow_g[col] : 0.f;
    us[r] = (col < a.bw) ? wv[r] * a.sc[a.j1 + col] : 0.f;
    wrow[col] = us[r];
    sel[r] = false;
  }
  if (SEL == SEL_GIVEN) {
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      sel[r] = (col < a.bw) && a.mask_in[i * a.b + a.j1 + col] != 0;
    }
  } else if (SEL == SEL_NM) {
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      key[col] = (col < a.bw) ? fabsf(wv[r]) * a.sx[a.j1 + col] : 0.f;
    }
    WAVE_SYNC();
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      if (col < a.bw) {
        const int g0 = (col / a.m) * a.m;
        const float mine = key[col];
        int rank = 0;
        for (int e = 0; e < a.m; ++e) {
          const float o = key[g0 + e];
          rank += (o < mine || (o == mine && g0 + e < col)) ? 1 : 0;
        }
        sel[r] = rank < a.n;
      }
    }
    if (a.row_skip && a.row_skip[i]) {
#pragma unroll
      for (int r = 0; r < CPL; ++r) sel[r] = false;
    }
  } else {  // SEL_THRESHOLD: key < tau, or key == tau and among the first need_eq ties
    const bool none = a.st->none != 0;
    const unsigned int tau = a.st->tau;
    const long long need_eq = a.st->need_eq;
    long long tie_rank = ties_before(a.st, a.row_eq, i);
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      const bool in = (col < a.bw) && !none;
      const unsigned int mk = in ? metric_key(wv[r], a.sx[a.j1 + col]) : 0xffffffffu;
      const bool lt = in && mk < tau;
      const bool eq = in && mk == tau;
      const unsigned long long eqb = __ballot(eq);
      const long long my = tie_rank + __popcll(eqb & ((1ull << lane) - 1ull));
      sel[r] = lt || (eq && my < need_eq);
      tie_rank += __popcll(eqb);
    }
  }

  // ---- q = phi(M_i) (ascending column indices) and s ----
  int s = 0;
  int myrank[CPL];
#pragma unroll
  for (int r = 0; r < CPL; ++r) {
    const unsigned long long bal = __ballot(sel[r]);
    myrank[r] = s + __popcll(bal & ((1ull << lane) - 1ull));
    s += __popcll(bal);
  }
  // A row with more unknowns than the tile grid holds (s > 32 NTR; rare): with the inverse K of
  // the block's G at hand it is solved here through the complement, a system of bw - s < 32
  // unknowns (see k_solve_tiled for the identity); without K it is left to the launch for
  // larger systems.
  bool comp = false;
  if (s > 32 * NTR && a.defer_large) {
    if (FULL || a.Kc == nullptr) {
      if (SEL == SEL_THRESHOLD && lane == 0) a.st_rw->deferred = 1;
      return;
    }
    comp = true;
  }
  const int ns = comp ? a.bw - s : s;  // unknowns of the system solved below
  // ---- tile grid: nt tile rows, and the PARTIAL tile comes first.  Matrix index m < 32 - pad
  //      is unknown m, 32 - pad <= m < 32 is padding (identity, never eliminated), m >= 32 is
  //      unknown m - pad.  A pivot costs one MFMA per live tile, most in the first tile row
  //      (NTR (NTR + 1) / 2 of them): with the short tile row in front, a system of 66 unknowns
  //      costs 2 * 6 + 32 * 3 + 32 MFMAs instead of 32 * 6 + 32 * 3 + 2. ----
  const int nt = FULL ? NTR : (ns + 31) >> 5;
  const int pad = FULL ? 0 : 32 * nt - ns;
  auto valid = [&](int m) { return FULL || m < 32 - pad || (m >= 32 && m - pad < ns); };
  // whether positions k .. k + 7 (k a multiple of 8; the same indices) are eliminated: asked of the first tile row only
  auto eliminated = [&](int k) { return FULL || k >= 32 || k < 32 - pad; };
  // q[m] = block column of matrix index m (column 0 where there is none: what it fetches is in
  // bounds and masked or never used), four of them to a word
  if (!FULL) {
    if (lane < (int)sizeof(sm.q) / 4) reinterpret_cast<unsigned int*>(sm.q)[lane] = 0u;
    WAVE_SYNC();
  }
  if (comp) {  // the removed columns as a list, with their weights; then the KEPT columns of the block
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      key[lane + 64 * r] = 0.f;
      reinterpret_cast<unsigned char*>(wrow)[lane + 64 * r] = 0;
    }
    WAVE_SYNC();
#pragma unroll
    for (int r = 0; r < CPL; ++r)
      if (sel[r]) {
        key[myrank[r]] = us[r];
        reinterpret_cast<unsigned char*>(wrow)[myrank[r]] = (unsigned char)(lane + 64 * r);
      }
    int before = 0;
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      const bool kept = col < a.bw && !sel[r];
      const unsigned long long bal = __ballot(kept);
      myrank[r] = before + __popcll(bal & ((1ull << lane) - 1ull));
      before += __popcll(bal);
    }
  }
#pragma unroll
  for (int r = 0; r < CPL; ++r) {
    const int col = lane + 64 * r;
    if (comp ? (col < a.bw && !sel[r]) : (sel[r] && s <= 32 * NTR))
      sm.q[myrank[r] < 32 - pad ? myrank[r] : myrank[r] + pad] = (unsigned char)col;
    if (col < a.bw) a.mask_out[i * a.b + a.j1 + col] = sel[r] ? 1 : 0;
  }
  if (SEL == SEL_THRESHOLD) {
    if (lane == 0) a.row_cnt[i] = s;  // summed at the start of the next block
  }
  float* lam_g = a.Lam + i * a.ldl;
  // s > 32 NTR (or, if FULL, anything but 32 NTR) cannot happen for a launch chosen by the host
  if (s == 0 || (s > 32 * NTR && !comp) || (FULL && s != 32 * NTR)) {
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      if (col < a.bw) lam_g[col] = 0.f;
    }
    rsc_set(a, i, 0.f, old_rsc);
    return;
  }
  // (y[0], y[1]) = sum over e < n of x[e] K[idx[e]][2 lane, 2 lane + 1], x and idx in LDS, filled up with zeros to a
  // multiple of 16; sixteen rows of K in flight.  A complement row reads every row of K once: the removed ones for w~ K, the
  // kept ones for y~ K.  (All rows for both, 32 in flight: 4096 x 4096 at 50 % 8.53 ms; rows found bit by bit in the
  // masks 8.83.)
  auto matvec_k = [&](const float* x, const unsigned char* idx, int n) {
    const unsigned int at = min(2 * lane, (a.bw - 1) & ~1);  // at the end of an odd block one value past it is read
    f32x2 y = {0.f, 0.f};
#pragma clang loop unroll(disable)
    for (int e0 = 0; e0 < n; e0 += 16) {
      f32x2 k[16];
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const unsigned int i4 = reinterpret_cast<const unsigned int*>(idx + e0)[e4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          k[4 * e4 + e] = *reinterpret_cast<const f32x2u*>(
              a.Kc + (__umul24((i4 >> (8 * e)) & 255u, (unsigned int)a.ldk) + at));
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        y[0] = fmaf(x[e0 + e], k[e][0], y[0]);
        y[1] = fmaf(x[e0 + e], k[e][1], y[1]);
      }
    }
    return y;
  };
  f32x2 wk = {0.f, 0.f};  // w~ K, columns 2 lane and 2 lane + 1
  if (comp) {
    // right-hand side (w~ K)_k: w~ = the row's weights on the removed columns, zero elsewhere
    WAVE_SYNC();
    wk = matvec_k(key, reinterpret_cast<const unsigned char*>(wrow), s);
    WAVE_SYNC();
    wrow[2 * lane] = wk[0];  // gathered below through q
    wrow[2 * lane + 1] = wk[1];
    WAVE_SYNC();
    if (ns == 0) {  // the whole block goes: lambda = w~ K
      float top = 0.f;
#pragma unroll
      for (int r = 0; r < CPL; ++r) {
        const int col = lane + 64 * r;
        if (col < a.bw) {
          lam_g[col] = wrow[col];
          top = fmaxf(top, fabsf(wrow[col]));
        }
      }
      rsc_set(a, i, top, old_rsc);
      return;
    }
  }
  WAVE_SYNC();

  // ---- gather R_hat = G[q, q] into the tiles (all loads unconditional, masked afterwards: only
  //      the first tile row holds padding); right-hand side distributed by row ----
  const float* G = comp ? a.Kc : a.P + a.j1 * a.b + a.j1;  // R_hat = G[q, q], or K[k, k]
  const char* Gc = reinterpret_cast<const char*>(G);  // byte offsets of 32 bits: 128 rows of at most
  const unsigned int bb = 4u * (comp ? (unsigned int)a.ldk : (unsigned int)a.b);  // 65535 columns
  f32x16 T[NTR][NTR];
  unsigned int qcol[NTR];
#pragma unroll
  for (int ti = 0; ti < NTR; ++ti) qcol[ti] = 4u * sm.q[32 * ti + lo];
#pragma unroll
  for (int tj = 0; tj < NTR; ++tj) {
    if (tj < nt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {  // tile rows held in registers 4 g .. 4 g + 3
        const unsigned int q4 = reinterpret_cast<const unsigned int*>(sm.q)[8 * tj + 2 * g + hi];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned int off = __umul24((q4 >> (8 * e)) & 255u, bb);
#pragma unroll
          for (int ti = tj; ti < NTR; ++ti) 
            T[ti][tj][4 * g + e] = *reinterpret_cast<const float*>(Gc + (off + qcol[ti]));
        }
      }
    }
  }
  if (!FULL) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 8 * (r >> 2) + 4 * hi + (r & 3);
      const bool in = row < 32 - pad;
      T[0][0][r] = (in && lo < 32 - pad) ? T[0][0][r] : (row == lo ? 1.f : 0.f);
#pragma unroll
      for (int ti = 1; ti < NTR; ++ti) T[ti][0][r] = in ? T[ti][0][r] : 0.f;
    }
  }
  // Two pivots per MFMA: rows k1 and k2 = k1 + 4 (k1 mod 8 < 4) of a tile sit in the same
  // register, in the lower and in the upper half of the wavefront, where the two reduction slots
  // of v_mfma_f32_32x32x2_f32 take their operands.  The pivots of a tile are therefore taken in
  // the order 0,4,1,5,2,6,3,7,8,12,...; pair t = (k1, k2) holds POSITIONS 2t and 2t + 1 of that
  // order.  L~ (unit lower triangular in elimination order), d, y and lambda are indexed by
  // position; mrow() maps a position back to its matrix index.
  const int pl = 8 * (lo >> 3) + 2 * (lo & 3) + ((lo >> 2) & 1);  // position of index lo in a tile
  auto mrow = [](int P) { return (P & ~7) + ((P & 7) >> 1) + 4 * (P & 1); };
  float u[NZ];  // right-hand side by position 64 z + lane
#pragma unroll
  for (int z = 0; z < NZ; ++z) {
    const int m = mrow(64 * z + lane);
    u[z] = (m < 32 * nt && valid(m)) ? wrow[sm.q[m & 127]] : 0.f;
  }
  // where this lane's element of a column of -L~ goes: the packed row of its position; lanes
  // whose element is on / above the diagonal write to scratch
  float* rowp[NTR];
#pragma unroll
  for (int ti = 0; ti < NTR; ++ti) rowp[ti] = &sm.L[(32 * ti + pl) * (32 * ti + pl - 1) / 2];
  float exponents = __uint_as_float(0x7f800000u);
  asm volatile("" : "+v"(exponents));
  float* const junk = &sm.L[32 * NTR * (32 * NTR - 1) / 2 + (lo & 15)];
  float dd[NZ];
#pragma unroll
  for (int z = 0; z < NZ; ++z) dd[z] = 1.f;

#pragma unroll
  for (int p = 0; p < NTR; ++p) {
    if (p < nt) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        // four pairs at a time: pivots of padding rows change nothing, and a branch for every pair costs more
        if (p > 0 || eliminated(8 * g))
#pragma unroll
        for (int t = 4 * g; t < 4 * g + 4; ++t) {
          const int k1 = 8 * (t >> 2) + (t & 3), k2 = k1 + 4;
          const float v = T[p][p][t];   // lower half: row k1 of the reduced tile, upper half: row k2
          const float x = lower_half(v);
          const float d1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k1));
          const float c12 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k2));
          const float d2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32 + k2));
          // 1 / d1 and 1 / d2', d2' = d2 - c12^2 / d1 = det / d1 the pivot of k2 after the elimination
          // of k1, from two independent reciprocals (see tl_eliminate)
          const float ps = pivot_scale(d1, exponents);
          const float e1 = ps * d1, e12 = ps * c12;
          const float cc = e12 * c12;
          const float det = fmaf(e1, d2, -cc) - fmaf(e12, c12, -cc);
          const float q1 = __builtin_amdgcn_rcpf(e1);
          const float qd = __builtin_amdgcn_rcpf(det);
          const float re = fmaf(fmaf(-e1, q1, 1.f), q1, q1);
          const float rd = fmaf(fmaf(-det, qd, 1.f), qd, qd);
          const float m = e12 * re;
          const float mh = hi ? m : 0.f;
          const float rh = hi ? -(e1 * rd) : -(ps * re);
          // pivots by position (64 z + lane)
          const float dp = lane & 1 ? det * re : d1;
          dd[p >> 1] = (lane >> 1) == 16 * (p & 1) + t ? dp : dd[p >> 1];
          // u1 (lower half) and u2 = row k2 after the elimination of k1 (upper half).  Columns
          // eliminated earlier hold rounding residue instead of zero; it is not masked, because
          // a product with it only ever lands in eliminated rows and columns of the tiles.
          const float bop = fmaf(-mh, x, v);
          const float aop = bop * rh;
          T[p][p] = __builtin_amdgcn_mfma_f32_32x32x2f32(aop, bop, T[p][p], 0, 0, 0);
          // column 2t + hi of -L~ within the tile: rows at later positions
          *(pl > 2 * t + hi ? rowp[p] + 32 * p + hi + 2 * t : junk) = aop;
          float e2[NTR], be[NTR];
#pragma unroll
          for (int ti = p + 1; ti < NTR; ++ti) {
            if (ti < nt) {
              // R_hat[32 ti + lo][32 p + k1] (lower half) and [..][32 p + k2] (upper half)
              const float ev = T[ti][p][t];
              const float xe = lower_half(ev);
              e2[ti] = fmaf(-mh, xe, ev);
              be[ti] = rh * e2[ti];
              T[ti][p] = __builtin_amdgcn_mfma_f32_32x32x2f32(bop, be[ti], T[ti][p], 0, 0, 0);
              (rowp[ti] + 32 * p + hi)[2 * t] = be[ti];
#pragma unroll
              for (int tj = p + 1; tj <= ti; ++tj) {
                // transposed storage: the first operand runs over the rows of tile row tj
                T[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(be[tj], e2[ti], T[ti][tj], 0, 0, 0);
              }
            }
          }
        }
      }
    }
  }
  WAVE_SYNC();

  // ---- L~ y = u, then L~^T lambda = D^-1 y.  A sweep reads one unknown off its lane (y_k or lambda_k,
  //      final by then) and adds its column of -L~ (row of -L~^T) to all others; lanes that are
  //      already final get rubbish, their value was put aside.  The LDS reads of eight unknowns
  //      are fetched together, eight unknowns ahead of the dependent chain: of a column every lane reads its own
  //      packed row (whose starts, triangular numbers, fall on different banks), of a row
  //      consecutive lanes read consecutive elements.  64 unknowns 2000 and 2900 cycles of a row's 27000, of rows of any
  //      size 2900 and 3000 (5800 and 5300 with a branch and a wait for each unknown).
  //      Carrying u through the elimination instead cost 19 vector instructions per pair of pivots
  //      in a kernel that is bound by their number. ----
  float y[NZ];
  int pofs[NZ];
#pragma unroll
  for (int z = 0; z < NZ; ++z) {
    const int P = min(64 * z + lane, 32 * NTR - 1);
    pofs[z] = P * (P - 1) / 2;
    y[z] = 0.f;
  }
  float ahead[2][8][NZ];
  auto load_cols = [&](float (&col)[8][NZ], int k8) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int z = 0; z < NZ; ++z) col[t][z] = (64 * z + 63 > k8 + t) ? sm.L[pofs[z] + k8 + t] : 0.f;
  };
  load_cols(ahead[0], 0);
#pragma unroll
  for (int k8 = 0; k8 < 32 * NTR; k8 += 8) {
    float (&col)[8][NZ] = ahead[(k8 >> 3) & 1];
    __builtin_amdgcn_sched_barrier(0);  // sixteen ahead, not all of them: registers
    if (k8 + 8 < 32 * NTR) load_cols(ahead[((k8 >> 3) & 1) ^ 1], k8 + 8);
    __builtin_amdgcn_sched_barrier(0);
    if (k8 < 32 * nt && eliminated(k8)) {
      int ys[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int k = k8 + t;
        ys[t] = __builtin_amdgcn_readlane(__float_as_int(u[k >> 6]), k & 63);
#pragma unroll
        for (int z = 0; z < NZ; ++z)
          if (64 * z + 63 > k) u[z] = fmaf(col[t][z], __int_as_float(ys[t]), u[z]);
      }
      set_lanes8(y[k8 >> 6], ys, k8 & 63);
    }
  }
  bool bad = false;
  float lam[NZ];
#pragma unroll
  for (int z = 0; z < NZ; ++z) {
    const int P = 64 * z + lane;
    const bool in = P < 32 * nt && valid(mrow(P));
    bad = bad || (in && !(dd[z] > 0.f));
    const float q0 = __builtin_amdgcn_rcpf(dd[z]);
    const float q1 = fmaf(fmaf(-dd[z], q0, 1.f), q0, q0);
    u[z] = in ? y[z] * q1 : 0.f;
    lam[z] = 0.f;
  }
  if (__ballot(bad) != 0ull && lane == 0)
    atomicCAS(a.info, 0, -(int32_t)min(i + 1, (int64_t)0x7fffffff));
  auto load_rows = [&](float (&row)[8][NZ], int k8) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int z = 0; z < NZ; ++z)
        row[t][z] = (64 * z < k8 + t) ? sm.L[(k8 + t) * (k8 + t - 1) / 2 + 64 * z + lane] : 0.f;
  };
  load_rows(ahead[(4 * NTR - 1) & 1], 32 * NTR - 8);
#pragma unroll
  for (int k8 = 32 * NTR - 8; k8 >= 0; k8 -= 8) {
    float (&row)[8][NZ] = ahead[(k8 >> 3) & 1];
    __builtin_amdgcn_sched_barrier(0);
    if (k8 > 0) load_rows(ahead[((k8 >> 3) & 1) ^ 1], k8 - 8);
    __builtin_amdgcn_sched_barrier(0);
    if (k8 < 32 * nt && eliminated(k8)) {
      int ls[8];
#pragma unroll
      for (int t = 7; t >= 0; --t) {
        const int k = k8 + t;
        ls[t] = __builtin_amdgcn_readlane(__float_as_int(u[k >> 6]), k & 63);
#pragma unroll
        for (int z = 0; z < NZ; ++z)
          if (64 * z < k) u[z] = fmaf(row[t][z], __int_as_float(ls[t]), u[z]);
      }
      set_lanes8(lam[k8 >> 6], ls, k8 & 63);
    }
  }

  if (comp) {
    // what has been solved for is y on the kept columns: lambda = ((w~ - y~) K)_q
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
      const int m = mrow(64 * z + lane);
      if (m < 32 * NTR) wrow[m] = m < 32 * nt && valid(m) ? lam[z] : 0.f;
    }
    WAVE_SYNC();
    const f32x2 yk = matvec_k(wrow, sm.q, 32 * nt);
    key[2 * lane] = wk[0] - yk[0];
    key[2 * lane + 1] = wk[1] - yk[1];
    WAVE_SYNC();
    float top = 0.f;
#pragma unroll
    for (int r = 0; r < CPL; ++r) {
      const int col = lane + 64 * r;
      const float l = sel[r] ? key[col] : 0.f;
      if (col < a.bw) lam_g[col] = l;
      top = fmaxf(top, fabsf(l));
    }
    rsc_set(a, i, top, old_rsc);
    return;
  }
  // ---- lambda row: zeros except lambda_l at column q_l ----
#pragma unroll
  for (int r = 0; r < CPL; ++r) wrow[lane + 64 * r] = 0.f;
  WAVE_SYNC();
#pragma unroll
  for (int z = 0; z < NZ; ++z)
    if (64 * z + lane < 32 * nt && valid(mrow(64 * z + lane)))
      wrow[sm.q[mrow(64 * z + lane)]] = lam[z];
  WAVE_SYNC();
  float top = 0.f;
#pragma unroll
  for (int r = 0; r < CPL; ++r) {
    const int col = lane + 64 * r;
    const float l = wrow[col];  // zero past the block
    if (col < a.bw) lam_g[col] = l;
    top = fmaxf(top, fabsf(l));
  }
  rsc_set(a, i, top, old_rsc);
}

// ------------------------------------------------------------------------------------------
// Mask + per-row solve for systems of up to 256 unknowns (block width <= 512) and beyond: one
// workgroup of NW wavefronts per row of W.  R_hat = G[q, q], padded with the identity past s, is
// factored tile by tile (32x32) with a right-looking blocked Cholesky, R_hat = L L^T, 32 columns
// per step:
//   1. one wavefront eliminates the diagonal tile with rank-1 MFMAs on its accumulator-layout
//      copy (row k of a symmetric tile is both operands of D -= u u^T / d; two pivots per
//      MFMA, see tl_eliminate) and carries a second tile that starts as I along, which ends as
//      T = L_pp^{-1} for a factor L_pp L_pp^T of the tile;
//   2. the tiles below it become L_ip = A_ip T^T (one 32x32x32 product each), y_p = T u_p;
//   3. the tiles right of the panel get A_il -= L_ip L_lp^T, the right-hand side u_i -= L_ip y_p;
//      meanwhile one wavefront updates the next diagonal tile and runs step 1 on it (look-ahead:
//      the elimination is a chain of dependent instructions, the rest is throughput work).
// L^T lambda = y is then solved from the last tile row upwards with the same T tiles.
// Products are fp32 MFMAs (v_mfma_f32_32x32x2_f32), those of step 3 without BIG fp16 ones (tile32.h).
//
// !BIG: the tiles live in the registers of the wavefronts that own them from the gather to the
// back-substitution; LDS only carries T and the current panel.  What bounds a row is the chain of
// eliminations (2.7 us per tile by itself), so the number of rows in flight per compute unit is what
// counts: a row of 256 unknowns takes 41 KB of LDS and half of the registers, two run at once;
// with the tiles in LDS (152 KB) a row filled the unit.  Panel tiles go to LDS split into fp16 pairs, once
// for the up to seven products that read each: 6 MFMAs of 32 cycles instead of 16 of 64.  4096 rows of 256
// unknowns: 890 -> 530 (registers) -> 460 -> 426 us.  Rows of up to 128 unknowns: five per unit instead of three.
// BIG: tiles in global memory.
constexpr int kTlLd = 33;          // LDS row stride of a tile (conflict-free rows and columns)
constexpr int kTlSz = 32 * kTlLd;  // floats per tile
constexpr int kTlSmax = 256;       // largest system
constexpr int kTlBw = 512;         // widest block

__host__ __device__ inline int tl_ntiles(int nt) { return nt * (nt + 1) / 2; }
__device__ __forceinline__ float* tl_tile(float* tiles, int i, int j) {
  return tiles + (i * (i + 1) / 2 + j) * kTlSz;
}
// acc += sign * A * Bn^T for 32x32 tiles, A[m][k] at pa[m*kTlLd + k], Bn[n][k] at pb[n*kTlLd + k]
__device__ __forceinline__ void tl_mma(f32x16& acc, const float* pa, const float* pb, float sign,
                                       int lo, int hi) {
  float av[16], bv[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    av[e] = pa[lo * kTlLd + 2 * e + hi];
    bv[e] = pb[lo * kTlLd + 2 * e + hi];
  }
#pragma unroll
  for (int e = 0; e < 16; ++e)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(sign * av[e], bv[e], acc, 0, 0, 0);
}
// The same with T written to the tile Dt (row stride kTlLd).
__device__ __forceinline__ bool tl_pivots(const f32x16& D, float* Dt, float* aux, int lo, int hi) {
  f32x16 E;
#pragma unroll
  for (int r = 0; r < 16; ++r) E[r] = (tl_row(r, hi) == lo) ? 1.f : 0.f;
  const float dl = tl_eliminate<false>(D, E, E, aux, lo, hi);
  const bool bad = __ballot(!(dl > 0.f)) != 0ull;
#pragma unroll
  for (int r = 0; r < 16; ++r) Dt[tl_row(r, hi) * kTlLd + lo] = E[r];
  return bad;
}

// ---- tiles in registers (!BIG) -------------------------------------------------------------
// A tile below the diagonal is held by one wavefront in operand layout (tile32.h):
// L_ip^T = T A_ip^T and A_il^T -= L_lp L_ip^T go from registers to registers.
// The tiles hold -A: then L' = (-A) T^T = -L, the trailing update is -A += L' L'^T without a
// negation of an operand, u_i += L' y_p and y_j += L'^T lambda_p.
// Tiles (row << 4 | column) below the diagonal owned by each wavefront, one per byte, 0xff = none;
// wavefront w also owns the diagonal tile w.  A wavefront never owns a tile whose column is at
// or right of its diagonal tile (wavefront 0 apart, whose elimination comes first): when it runs
// ahead on its diagonal tile it has no other trailing tile to update.  Of eight, the first of a wavefront's
// tiles is the one left of its diagonal tile: what that tile adds to the diagonal one goes from registers to registers, in
// front of the barrier that the others wait for (4096 rows of 256 unknowns 430 -> 420 us; of four, with five rows per
// compute unit, 8192 rows of about 102 222 -> 229: the others wait for that wavefront).  Within that, the tiles are dealt so that the four SIMDs have about the same number
// of products in every step.
__device__ const uint32_t kRsOwn8[8] = {0x75746031u, 0xffffff10u, 0xff705021u, 0x41402032u,
                                        0x62513043u, 0x63614254u, 0x72645365u, 0x73715276u};
__device__ const uint32_t kRsOwn4[4] = {0xffff3221u, 0xffffff20u, 0xffffff30u, 0xffff3110u};

template <int NW>
constexpr size_t rs_smem_floats() {  // panel + T, wrow, key, u, lambda, q, pivot scratch, counters
  return (size_t)NW * kRsTile + 2 * kTlBw + 3 * 32 * NW + 64 + 2 * 8;
}
// sum over all 32 values of tl_row(r, hi) of t[r] * v[tl_row(r, hi)], v in LDS (16-byte aligned);
// every lane gets the sum of its column lo
__device__ __forceinline__ float rs_sum_halves(float s) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}
__device__ __forceinline__ float rs_dot(const f32x16& t, const float* v, int hi) {
  float s = 0.f;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(v + 8 * g + 4 * hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(t[4 * g + e], x[e], s);
  }
  return rs_sum_halves(s);
}

// Solves lambda R_hat = u for one row: nt tile rows, ns unknowns, R_hat[a][c] = G[q[a] * ldg + q[c]].
// u and q (32 nt values, zero past ns): u is overwritten, lam[0 : 32 nt] times the returned scale is the result.
// The matrix is scaled by a power of two that brings its largest diagonal element to [2^28, 2^29): no
// element of the factor then exceeds 2^14.5, and the trailing products, which are most of the work, take
// two fp16 values per operand (tile32.h).  tiles: NW * kRsTile
// floats (and 2 * kTlBw more behind them that may be overwritten).  Called by all NW wavefronts,
// u and q complete; barriers inside, lam is complete on return.  bad: a pivot was not positive.
template <int NW>
__device__ __forceinline__ float rs_solve(const float* __restrict__ G, unsigned int ldg, const int* q, int ns,
                                          int nt, float* tiles, float* u, float* lam, float* aux, bool& bad) {
  constexpr int SL = NW == 8 ? 4 : 2;  // tiles below the diagonal per wavefront
  constexpr bool kOwnLeft = NW == 8;   // the first of them is the one left of the diagonal tile
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  // the wavefronts' parts rotate with the row, so that the eliminations of the rows that run on a
  // compute unit at the same time do not meet on one SIMD
  const int w = (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) + (int)blockIdx.x) & (NW - 1);
  const uint32_t own = (uint32_t)__builtin_amdgcn_readfirstlane((int)(NW == 8 ? kRsOwn8[w] : kRsOwn4[w]));
  int ti[SL], tj[SL];
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    ti[s] = (own >> (8 * s + 4)) & 15;
    tj[s] = (own >> (8 * s)) & 15;
  }
  float* Tt = tiles + (NW - 1) * kRsTile;

  // ---- gather (all loads unconditional, of column 0 past ns, masked afterwards) ----
  f32x16 off[SL], dg;
  auto fetch = [&](f32x16& v, int i, int j) {  // v[r] = G[q[32 j + row]][q[32 i + lo]]
    const unsigned int qc = (unsigned int)q[32 * i + lo];
#pragma unroll
    for (int g = 0; g < 4; ++g) {  // 512 columns of at most 65535: the offset fits 32 bits, its factors 24
      const u32x4 rows = *reinterpret_cast<const u32x4*>(q + 32 * j + 8 * g + 4 * hi);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * g + e] = G[__umul24(rows[e], ldg) + qc];
    }
  };
  if (w < nt) fetch(dg, w, w);
#pragma unroll
  for (int s = 0; s < SL; ++s)
    if (ti[s] < nt) fetch(off[s], ti[s], tj[s]);
  if (w < nt) {  // largest diagonal element of the tile; lam is free until the end
    float top = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) top = (tl_row(r, hi) == lo && 32 * w + lo < ns) ? fmaxf(top, dg[r]) : top;
    top = wave_max(top);
    if (lane == 0) lam[w] = top;
  }
  __syncthreads();  // the maxima are there, `tiles` is free (its previous contents have been read)
  float top = lam[0];
  for (int t = 1; t < nt; ++t) top = fmaxf(top, lam[t]);
  const int te = 127 + 28 + 127 - (int)(__float_as_uint(top) >> 23);
  const float scale = __uint_as_float((uint32_t)min(max(te, 1), 253) << 23);
  if (w < nt) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool in = 32 * w + lo < ns && 32 * w + tl_row(r, hi) < ns;
      dg[r] = in ? -scale * dg[r] : (tl_row(r, hi) == lo ? -1.f : 0.f);
    }
  }
#pragma unroll
  for (int s = 0; s < SL; ++s)
    if (ti[s] < nt) {
#pragma unroll
      for (int r = 0; r < 16; ++r) off[s][r] = (32 * ti[s] + lo < ns) ? -scale * off[s][r] : 0.f;
    }

  bad = false;
  for (int p = 0; p < nt; ++p) {
    int l = lo, h = hi;  // not known to be the same in every step: keeps lane masks and LDS addresses,
    asm volatile("" : "+v"(l), "+v"(h));  // an instruction each, out of registers that outlive the step
    // The owner of diagonal tile p eliminates it while the others are still in the trailing update
    // of step p - 1 below (no barrier in between): T replaces the tile, in its registers and in LDS.
    if (w == p) {
      __builtin_amdgcn_s_setprio(3);  // the chain of eliminations is what the row waits for
      f32x16 D;
#pragma unroll
      for (int r = 0; r < 16; ++r) D[r] = -dg[r];
#pragma unroll
      for (int r = 0; r < 16; ++r) dg[r] = (tl_row(r, h) == l) ? 1.f : 0.f;
      bad = __ballot(!(tl_eliminate<false>(D, dg, dg, aux, l, h) > 0.f)) != 0ull;
      float* Tc = Tt + rs_col(l, hi);
#pragma unroll
      for (int r = 0; r < 16; ++r) Tc[rs_step(r)] = dg[r];
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();  // T_p is there; the panel of step p - 1 has been read
#pragma unroll
    for (int s = 0; s < SL; ++s)
      if (tj[s] == p && ti[s] < nt) {
        f32x16 C;
#pragma unroll
        for (int r = 0; r < 16; ++r) C[r] = 0.f;
        rs_mma<false>(C, Tt, off[s], l, h);
        off[s] = C;
        const RsSplit x = rs_split_h2(C);
        rs_store_h2(tiles + (ti[s] - 1) * kRsTile, x, l + 32 * h);
        if (kOwnLeft && s == 0 && w == p + 1) rs_mma_h2(dg, x);  // the next diagonal tile
      }
    if (w == p) {  // u_p -= L_p,p-1 y_p-1, left over from the step before; y_p = T u_p
      if (kOwnLeft && p > 0) {
        const float d = rs_dot(off[0], u + 32 * (p - 1), h);
        if (lane < 32) u[32 * p + lane] += d;
        WAVE_SYNC();
      }
      float y = 0.f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 t = rs_piece(Tt, g, l, h);
        const f32x4 x = *reinterpret_cast<const f32x4*>(u + 32 * p + 8 * g + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) y = fmaf(t[e], x[e], y);
      }
      y = rs_sum_halves(y);
      if (lane < 32) u[32 * p + lane] = y;
    }
    __syncthreads();  // panel and y_p are there
    if (p + 1 == nt) break;
    if (w > (kOwnLeft ? p + 1 : p) && w < nt)
      rs_mma_h2(dg, tiles + (w - 1) * kRsTile, tiles + (w - 1) * kRsTile, l + 32 * h);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      if (ti[s] < nt && tj[s] > p)
        rs_mma_h2(off[s], tiles + (tj[s] - 1) * kRsTile, tiles + (ti[s] - 1) * kRsTile, l + 32 * h);
      if (ti[s] < nt && tj[s] == p && !(kOwnLeft && s == 0 && w == p + 1)) {  // u_i -= L_ip y_p (one tile per i in a step)
        const float d = rs_dot(off[s], u + 32 * p, h);
        if (lane < 32) u[32 * ti[s] + lane] += d;
      }
    }
  }

  // ---- L^T lambda = y, last tile row first.  The tiles are turned to lane <-> column first,
  //      each wavefront through its own piece of LDS ----
  {
    float* mine = tiles + (threadIdx.x >> 6) * kRsTile;
#pragma unroll
    for (int s = 0; s < SL; ++s)
      if (ti[s] < nt) {
        rs_store(mine, off[s], lo, hi);
        WAVE_SYNC();
#pragma unroll
        for (int r = 0; r < 16; ++r) off[s][r] = mine[rs_col(lo, hi) + rs_step(r)];
        WAVE_SYNC();
      }
  }
  for (int p = nt - 1; p >= 0; --p) {
    if (w == p) {  // lambda_p = T^T y_p
      const float l = rs_dot(dg, u + 32 * p, hi);
      if (lane < 32) lam[32 * p + lane] = l;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < SL; ++s)
      if (ti[s] == p) {  // y_j -= L_pj^T lambda_p
        const float d = rs_dot(off[s], lam + 32 * p, hi);
        if (lane < 32) u[32 * tj[s] + lane] += d;
      }
    __syncthreads();
  }
  return scale;
}

// y[j] = sum_a x[a] * K[a * ldk + j], j < bw (bw a multiple of 4, K 16-byte aligned rows), for a
// workgroup of NW wavefronts; x and y in LDS.  Rows with x[a] == 0 are skipped (uniform test).
// !BIG (bw <= 512): the wavefronts split the rows a, each lane holds up to two groups of four
// columns, partial sums meet in part[NW][bw] (LDS) and are added in a fixed order.
// BIG: every wavefront owns column groups and walks all rows; no partial sums.
// Barriers inside; x must be complete on entry, y is complete on return.
template <int NW, bool BIG>
__device__ __forceinline__ void tl_matvec(const float* x, int bw, const float* __restrict__ K,
                                          int ldk, float* y, float* part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ng = bw >> 2;
  if (BIG) {
    for (int g = 64 * wave + lane; g < ng; g += 64 * NW) {
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
      for (int a = 0; a < bw; ++a) {
        const float xa = x[a];
        const float4 k4 = *reinterpret_cast<const float4*>(K + (int64_t)a * ldk + 4 * g);
        acc.x = fmaf(xa, k4.x, acc.x);
        acc.y = fmaf(xa, k4.y, acc.y);
        acc.z = fmaf(xa, k4.z, acc.z);
        acc.w = fmaf(xa, k4.w, acc.w);
      }
      *reinterpret_cast<float4*>(y + 4 * g) = acc;
    }
    __syncthreads();
    return;
  }
  const int per = (bw + NW - 1) / NW;
  const int alo = wave * per, ahi = min(bw, alo + per);
  float4 acc[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
  const int g0 = min(lane, ng - 1), g1 = min(lane + 64, ng - 1);  // clamped: loads stay in bounds
#pragma unroll 4
  for (int a = alo; a < ahi; ++a) {
    const float xa = x[a];
    if (xa == 0.f) continue;
    const float4 k0 = *reinterpret_cast<const float4*>(K + (int64_t)a * ldk + 4 * g0);
    const float4 k1 = *reinterpret_cast<const float4*>(K + (int64_t)a * ldk + 4 * g1);
    acc[0].x = fmaf(xa, k0.x, acc[0].x);
    acc[0].y = fmaf(xa, k0.y, acc[0].y);
    acc[0].z = fmaf(xa, k0.z, acc[0].z);
    acc[0].w = fmaf(xa, k0.w, acc[0].w);
    acc[1].x = fmaf(xa, k1.x, acc[1].x);
    acc[1].y = fmaf(xa, k1.y, acc[1].y);
    acc[1].z = fmaf(xa, k1.z, acc[1].z);
    acc[1].w = fmaf(xa, k1.w, acc[1].w);
  }
  if (lane < ng) *reinterpret_cast<float4*>(part + wave * bw + 4 * lane) = acc[0];
  if (lane + 64 < ng) *reinterpret_cast<float4*>(part + wave * bw + 4 * (lane + 64)) = acc[1];
  __syncthreads();
  for (int j = tid; j < bw; j += 64 * NW) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += part[w * bw + j];
    y[j] = t;
  }
  __syncthreads();
}

// BIG = false: one workgroup per row (grid = c), systems of up to 32 NW unknowns in blocks of up to
// 512 columns (rs_solve).  BIG = true: systems of up to kBigSmax unknowns in blocks of up to kBigBw
// columns (the large blocks of the paper's block-size ablation): the tile grid of a row no longer
// fits a compute unit and lives in global memory, one slot per workgroup (a.tile_scratch,
// a.slot_floats; the slot of a workgroup stays in the caches of its compute unit's XCD), and the
// gridDim.x workgroups walk the rows (row = blockIdx.x, blockIdx.x + gridDim.x, ...).  The row's
// right-hand side, multipliers, indices and the block's weights stay in LDS.
constexpr int kBigSmax = 2048;
constexpr int kBigBw = 4096;
static inline size_t tl_big_smem_bytes() {
  return ((size_t)2 * kBigBw + 3 * kBigSmax + 128 + 2 * 8 * (kBigBw / 512)) * sizeof(float);
}

template <int SEL, int NW, bool BIG = false>
__global__ __launch_bounds__(64 * NW, (BIG ? 2 : (NW == 8 ? 4 : 5))) void k_solve_tiled(SolveArgs a) {
  constexpr int NT = 64 * NW;       // threads
  constexpr int SMAX = BIG ? kBigSmax : 32 * NW;
  constexpr int BW = BIG ? kBigBw : kTlBw;
  constexpr int CH = BW / NT;       // block columns per thread
  constexpr int RPT = 1024 / NT;    // tile elements per thread
  constexpr int NC = NW * CH;       // (wavefront, column chunk) pairs
  extern __shared__ __attribute__((aligned(16))) char solve_smem[];
  float* tiles;
  float *wrow, *key, *xtra;
  if (BIG) {
    tiles = a.tile_scratch + (int64_t)blockIdx.x * a.slot_floats;
    wrow = reinterpret_cast<float*>(solve_smem);
    key = wrow + BW;
    xtra = key + BW;
  } else {
    tiles = reinterpret_cast<float*>(solve_smem);
    wrow = tiles + NW * kRsTile;
    key = wrow + BW;
    xtra = key + BW;
  }
  float* u = xtra;                    // right-hand side, then y
  float* lam = xtra + SMAX;
  int* q = reinterpret_cast<int*>(xtra + 2 * SMAX);
  float* aux = xtra + 3 * SMAX;
  int* cnt = reinterpret_cast<int*>(aux + (BIG ? 128 : 64));  // per wavefront and chunk: selected, ties
  int* eqc = cnt + NC;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = lane & 31, hi = lane >> 5;
  for (int64_t i = blockIdx.x; i < a.c; i += gridDim.x) {  // !BIG: gridDim.x == c, one pass
  if (BIG) __syncthreads();  // the previous row's LDS and slot contents are dead
  const float* wrow_g = a.W + i * a.b + a.j1;

  // ---- selection of the block mask row M_i: column col = tid + NT * ch ----
  bool sel[CH];
  float wv[CH], us[CH];  // weights, and in scaled coordinates
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    const int col = tid + NT * ch;
    wv[ch] = (col < a.bw) ? wrow_g[col] : 0.f;
    us[ch] = (col < a.bw) ? wv[ch] * a.sc[a.j1 + col] : 0.f;
    wrow[col] = us[ch];
    sel[ch] = false;
  }
  if (SEL == SEL_GIVEN) {
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      sel[ch] = (col < a.bw) && a.mask_in[i * a.b + a.j1 + col] != 0;
    }
  } else if (SEL == SEL_PICKED) {
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      sel[ch] = (col < a.bw) && a.mask_out[i * a.b + a.j1 + col] != 0;
    }
  } else if (SEL == SEL_NM) {
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      key[col] = (col < a.bw) ? fabsf(wv[ch]) * a.sx[a.j1 + col] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      if (col < a.bw) {
        const int g0 = (col / a.m) * a.m;
        const float mine = key[col];
        int rank = 0;
        for (int e = 0; e < a.m; ++e) {
          const float o = key[g0 + e];
          rank += (o < mine || (o == mine && g0 + e < col)) ? 1 : 0;
        }
        sel[ch] = rank < a.n;
      }
    }
    if (a.row_skip && a.row_skip[i]) {
#pragma unroll
      for (int ch = 0; ch < CH; ++ch) sel[ch] = false;
    }
  } else {  // SEL_THRESHOLD: key < tau, or key == tau and among the first need_eq ties
    const bool none = a.st->none != 0;
    const unsigned int tau = a.st->tau;
    const long long need_eq = a.st->need_eq;
    bool lt[CH], eq[CH];
    unsigned long long eqb[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      const bool in = (col < a.bw) && !none;
      const unsigned int kk = in ? metric_key(wv[ch], a.sx[a.j1 + col]) : 0xffffffffu;
      lt[ch] = in && kk < tau;
      eq[ch] = in && kk == tau;
      eqb[ch] = __ballot(eq[ch]);
      if (lane == 0) eqc[NW * ch + wave] = __popcll(eqb[ch]);
    }
    __syncthreads();
    const long long ties0 = ties_before(a.st, a.row_eq, i);
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      long long my = ties0;
      for (int v = 0; v < NW * ch + wave; ++v) my += eqc[v];
      my += __popcll(eqb[ch] & ((1ull << lane) - 1ull));
      sel[ch] = lt[ch] || (eq[ch] && my < need_eq);
    }
  }

  // ---- q = phi(M_i) (ascending column indices) and s ----
  unsigned long long bal[CH];
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    bal[ch] = __ballot(sel[ch]);
    if (lane == 0) cnt[NW * ch + wave] = __popcll(bal[ch]);
  }
  __syncthreads();
  int s = 0;
#pragma unroll
  for (int v = 0; v < NC; ++v) s += cnt[v];
  // A row that loses more than half of the block is solved through the complement: with
  // K = G^{-1}, kept set k of the block and w~ = (u on q, 0 on k),
  //     (G_qq)^{-1} = K_qq - K_qk (K_kk)^{-1} K_kq,   so   lambda = ((w~ - y~) K)_q
  // with y~ = (0 on q, y on k), y K_kk = (w~ K)_k: a system of bw - s unknowns instead of s,
  // and never more than half a block.  (Same accuracy: K is formed from the factor directly.)
  const bool comp = a.Kc != nullptr && 2 * s > a.bw;  // uniform per workgroup
  const int ns = comp ? a.bw - s : s;                  // unknowns of this row's system
  if (SEL == SEL_THRESHOLD) {
    if (tid == 0) a.row_cnt[i] = s;  // summed at the start of the next block
  }
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    const int col = tid + NT * ch;
    if (SEL != SEL_PICKED && col < a.bw) a.mask_out[i * a.b + a.j1 + col] = sel[ch] ? 1 : 0;
  }
  // A block may be solved by two launches with different numbers of wavefronts per row: this one
  // takes the rows with nt_lo <= ceil(ns/32) <= nt_max and leaves the others untouched.
  const int nt = (ns + 31) >> 5;
  const bool fits = ns <= SMAX;
  if (fits ? (nt < a.nt_lo || nt > a.nt_max) : (32 * a.nt_max < (BIG ? SMAX : kTlSmax))) {
    if (BIG) continue;
    return;
  }
  // the solved set: removed columns, or kept columns of the block when solving the complement
  bool ins[CH];
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) ins[ch] = comp ? (tid + NT * ch < a.bw && !sel[ch]) : sel[ch];
  if (comp) {
    __syncthreads();  // all counts of the removed set have been read
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      bal[ch] = __ballot(ins[ch]);
      if (lane == 0) cnt[NW * ch + wave] = __popcll(bal[ch]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    const int col = tid + NT * ch;
    int before = 0;
    for (int v = 0; v < NW * ch + wave; ++v) before += cnt[v];
    if (ins[ch] && fits) q[before + __popcll(bal[ch] & ((1ull << lane) - 1ull))] = col;
  }
  float* lam_g = a.Lam + i * a.ldl;
  if (SEL != SEL_PICKED && tid == 0) rsc_clear(a, i);  // k_pick has done it
  if (s == 0 || !fits) {  // !fits cannot happen for a launch chosen by the host
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      if (col < a.bw) lam_g[col] = 0.f;
    }
    if (!fits && tid == 0) atomicCAS(a.info, 0, -(int32_t)min(i + 1, (int64_t)0x7fffffff));
    if (BIG) continue;
    return;
  }
  __syncthreads();
  // partial sums of the complement's matrix-vector products: in the tile area (NW * 1056 floats,
  // of which they take NW * 512)
  float* part = BIG ? nullptr : tiles;
  for (int t = ns + tid; t < 32 * nt; t += NT) q[t] = 0;
  if (!comp) {
    for (int t = tid; t < 32 * nt; t += NT) u[t] = (t < s) ? wrow[q[t]] : 0.f;
  } else if (SEL == SEL_PICKED) {
    for (int t = tid; t < 32 * nt; t += NT) u[t] = (t < ns) ? a.WK[i * a.ldz + q[t]] : 0.f;
  } else {
    // right-hand side (w~ K)_k: x = w~ in `key`, the product lands in `wrow` (the row's weights
    // stay in registers)
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) key[tid + NT * ch] = sel[ch] ? us[ch] : 0.f;
    __syncthreads();
    tl_matvec<NW, BIG>(key, a.bw, a.Kc, a.ldk, wrow, part);
    for (int t = tid; t < 32 * nt; t += NT) u[t] = (t < ns) ? wrow[q[t]] : 0.f;
  }
  __syncthreads();

  bool bad = false;
  float ls = 1.f;  // what lam is to be multiplied by
  // R_hat = G[q, q], or K[k, k] for the complement
  const float* G = comp ? a.Kc : a.P + a.j1 * a.b + a.j1;
  const int64_t ldg = comp ? (int64_t)a.ldk : a.b;
  if constexpr (!BIG) {
    if (ns > 0) ls = rs_solve<NW>(G, (unsigned int)ldg, q, ns, nt, tiles, u, lam, aux, bad);
  } else {
  // ---- gather R_hat into the tiles: thread <-> (rows tid/32 + (NT/32)e, column tid%32) of a tile;
  //      up to four tiles of a tile row are fetched together, all loads unconditional from
  //      clamped (valid) indices and masked when stored ----
  if (ns > 0) {
    const int tr = tid >> 5, tc = tid & 31;
    for (int ti = 0; ti < nt; ++ti) {
      const float* grow[RPT];
#pragma unroll
      for (int e = 0; e < RPT; ++e)
        grow[e] = G + (int64_t)q[min(32 * ti + tr + (NT / 32) * e, ns - 1)] * ldg;
      for (int tj0 = 0; tj0 <= ti; tj0 += 4) {
        float v[4][RPT];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int tj = min(tj0 + t, ti);
          const int qc = q[min(32 * tj + tc, ns - 1)];
#pragma unroll
          for (int e = 0; e < RPT; ++e) v[t][e] = grow[e][qc];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int tj = tj0 + t;
          if (tj <= ti) {
            float* T = tl_tile(tiles, ti, tj);
            const int cc = 32 * tj + tc;
#pragma unroll
            for (int e = 0; e < RPT; ++e) {
              const int rr = 32 * ti + tr + (NT / 32) * e;
              const float ident = (rr == cc) ? 1.f : 0.f;
              T[(tr + (NT / 32) * e) * kTlLd + tc] = (rr < ns && cc < ns) ? v[t][e] : ident;
            }
          }
        }
      }
    }
  }
  __syncthreads();

  // ---- blocked Cholesky with look-ahead, forward substitution carried along.  The wavefront
  //      that eliminates a diagonal tile rotates, so that concurrent workgroups of a compute
  //      unit do not run this latency-bound step on the same SIMD. ----
  if (nt > 0 && wave == ((int)blockIdx.x & (NW - 1))) {
    f32x16 D;
#pragma unroll
    for (int r = 0; r < 16; ++r) D[r] = tiles[tl_row(r, hi) * kTlLd + lo];
    bad = tl_pivots(D, tiles, aux, lo, hi);
  }
  __syncthreads();
  for (int p = 0; p < nt; ++p) {
    float* Tp = tl_tile(tiles, p, p);
    {  // panel: L_ip = A_ip T^T
      for (int ii = p + 1 + wave; ii < nt; ii += NW) {
        float* Aip = tl_tile(tiles, ii, p);
        f32x16 C;
#pragma unroll
        for (int r = 0; r < 16; ++r) C[r] = 0.f;
        tl_mma(C, Aip, Tp, 1.f, lo, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) Aip[tl_row(r, hi) * kTlLd + lo] = C[r];
      }
      if (wave == NW - 1 && lane < 32) {  // y_p = T u_p
        float row[32], acc = 0.f;
#pragma unroll
        for (int k = 0; k < 32; ++k) row[k] = Tp[lane * kTlLd + k];
        __builtin_amdgcn_sched_barrier(0);  // all requests first, as in the substitution below
#pragma unroll
        for (int k = 0; k < 32; ++k) acc = fmaf(row[k], u[32 * p + k], acc);
        u[32 * p + lane] = acc;
      }
    }
    __syncthreads();
    if (p + 1 == nt) break;
    // One wavefront brings the next diagonal tile up to date and eliminates it at once (the
    // tile stays in registers); the others apply panel p to the rest of the trailing
    // matrix, the tiles of column p+1 first, and to the right-hand side.
    const int pw = (p + 1 + (int)blockIdx.x) & (NW - 1);
    if (wave == pw) {
      float* Dn = tl_tile(tiles, p + 1, p + 1);
      const float* Lp = tl_tile(tiles, p + 1, p);
      f32x16 D;
#pragma unroll
      for (int r = 0; r < 16; ++r) D[r] = Dn[tl_row(r, hi) * kTlLd + lo];
      tl_mma(D, Lp, Lp, -1.f, lo, hi);
      bad = tl_pivots(D, Dn, aux, lo, hi) || bad;
    } else {
      const int widx = wave - (wave > pw ? 1 : 0);  // 0..NW-2
      int t = 0, mine = widx;
      auto upd = [&](int ii, int l) {
        float* Ail = tl_tile(tiles, ii, l);
        f32x16 C;
#pragma unroll
        for (int r = 0; r < 16; ++r) C[r] = Ail[tl_row(r, hi) * kTlLd + lo];
        tl_mma(C, tl_tile(tiles, ii, p), tl_tile(tiles, l, p), -1.f, lo, hi);
#pragma unroll
        for (int r = 0; r < 16; ++r) Ail[tl_row(r, hi) * kTlLd + lo] = C[r];
      };
      for (int ii = p + 2; ii < nt; ++ii, ++t)
        if (t == mine) {
          upd(ii, p + 1);
          mine += NW - 1;
        }
      for (int l = p + 2; l < nt; ++l)
        for (int ii = l; ii < nt; ++ii, ++t)
          if (t == mine) {
            upd(ii, l);
            mine += NW - 1;
          }
      for (int row = 32 * (p + 1) + 64 * widx + lane; row < 32 * nt; row += 64 * (NW - 1)) {
        // u_i -= L_ip y_p
        const float* Lr = tl_tile(tiles, row >> 5, p) + (row & 31) * kTlLd;
        float acc = u[row];
#pragma unroll
        for (int k = 0; k < 32; ++k) acc = fmaf(-Lr[k], u[32 * p + k], acc);
        u[row] = acc;
      }
    }
    __syncthreads();
  }

  // ---- L^T lambda = y, last tile row first ----
  for (int p = nt - 1; p >= 0; --p) {
    const float* Tp = tl_tile(tiles, p, p);
    if (wave == 0 && lane < 32) {  // lambda_p = T^T y_p
      float col[32], acc = 0.f;
#pragma unroll
      for (int k = 0; k < 32; ++k) col[k] = Tp[k * kTlLd + lane];
      // all requests first: under register pressure the compiler takes them one by one, 32 round trips to the L2
      // in a step that the row waits for (512 unknowns: 11.6 instead of 10.4 ms per block of 4096 rows)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 32; ++k) acc = fmaf(col[k], u[32 * p + k], acc);
      lam[32 * p + lane] = acc;
    }
    __syncthreads();
    for (int t = tid; t < 32 * p; t += NT) {  // y_j -= L_pj^T lambda_p for the tile rows above
      const float* Lc = tl_tile(tiles, p, t >> 5) + (t & 31);
      float acc = u[t];
#pragma unroll
      for (int r = 0; r < 32; ++r) acc = fmaf(-Lc[r * kTlLd], lam[32 * p + r], acc);
      u[t] = acc;
    }
    __syncthreads();
  }
  }  // BIG
  if (bad && lane == 0) atomicCAS(a.info, 0, -(int32_t)min(i + 1, (int64_t)0x7fffffff));

  // ---- lambda row: zeros except lambda_k at column q_k ----
  if (!comp) {
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) wrow[tid + NT * ch] = 0.f;
    __syncthreads();
    for (int t = tid; t < s; t += NT) wrow[q[t]] = ls * lam[t];
    __syncthreads();
    float top = 0.f;
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      const float l = wrow[col];  // zero past the block
      if (col < a.bw) lam_g[col] = l;
      top = fmaxf(top, fabsf(l));
    }
    rsc_lower(a, i, top);
  } else if (SEL == SEL_PICKED) {  // w~ - y~: -y on the kept columns, w~ is there
    for (int t = tid; t < ns; t += NT) a.Z[i * a.ldz + q[t]] = -ls * lam[t];
  } else {
    // lambda = ((w~ - y~) K)_q: x = w on the removed columns, -y on the kept ones
    __syncthreads();
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) key[tid + NT * ch] = sel[ch] ? us[ch] : 0.f;
    __syncthreads();
    for (int t = tid; t < ns; t += NT) key[q[t]] = -ls * lam[t];
    __syncthreads();
    tl_matvec<NW, BIG>(key, a.bw, a.Kc, a.ldk, wrow, part);
    float top = 0.f;
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) {
      const int col = tid + NT * ch;
      const float l = sel[ch] ? wrow[col] : 0.f;  // nothing is removed past the block
      if (col < a.bw) lam_g[col] = l;
      top = fmaxf(top, fabsf(l));
    }
    rsc_lower(a, i, top);
  }
  if (!BIG) return;  // one row per workgroup
  }  // rows of this workgroup
}

// ------------------------------------------------------------------------------------------
// Complement form for many rows.  Its two products of every row with the block's K, w~ K before the
// solve and (w~ - y~) K after it, are matrix products over all rows: the row solver, where each row
// fetches K twice (512 KB at 256 columns), spent half of its time on them.
//   k_pick       mask of the block, s per row, Z = w~ (removed weights, zero elsewhere)
//   gemm_f32     WK = Z K
//   k_solve_tiled<SEL_PICKED>   complement rows: Z = w~ - y~; the others: Lam
//   k_lam_rows   complement rows: Lam = (Z K) on the removed columns, zero elsewhere
// 8192 rows of 256 columns, 60 %: 400 -> 305 us per block.
__global__ __launch_bounds__(256) void k_pick(SolveArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= a.c) return;
  const bool none = a.st->none != 0;
  const unsigned int tau = a.st->tau;
  const long long need_eq = a.st->need_eq;
  long long tie_rank = ties_before(a.st, a.row_eq, i);
  int s = 0;
  for (int c0 = 0; c0 < a.bw; c0 += 64) {  // key < tau, or key == tau and among the first need_eq ties
    const int col = c0 + lane;
    const float w = col < a.bw ? a.W[i * a.b + a.j1 + col] : 0.f;
    const bool in = col < a.bw && !none;
    const unsigned int key = in ? metric_key(w, a.sx[a.j1 + col]) : 0xffffffffu;
    const bool eq = in && key == tau;
    const unsigned long long eqb = __ballot(eq);
    const bool sel = (in && key < tau) ||
                     (eq && tie_rank + __popcll(eqb & ((1ull << lane) - 1ull)) < need_eq);
    tie_rank += __popcll(eqb);
    s += __popcll(__ballot(sel));
    if (col < a.bw) {
      a.mask_out[i * a.b + a.j1 + col] = sel ? 1 : 0;
      a.Z[i * a.ldz + col] = sel ? w * a.sc[a.j1 + col] : 0.f;
    }
  }
  if (lane == 0) {
    a.row_cnt[i] = s;
    rsc_clear(a, i);
  }
}

__global__ __launch_bounds__(kXThreads, 4) void k_lam_rows(SolveArgs a) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  const int n0 = blockIdx.x * kTN;
  const int64_t m0 = (int64_t)blockIdx.y * kTM;
  const int m_ext = (int)min((int64_t)kTM, a.c - m0), n_ext = min(kTN, a.bw - n0);
  TileAcc acc;
  acc_zero(acc);
  // K is symmetric: its rows serve as columns
  gemm_tile_x3<false, false>(acc, sm, a.Z + m0 * a.ldz, a.ldz, m_ext, a.Kc + (int64_t)n0 * a.ldk, a.ldk,
                             n_ext, 0, a.bw);
  const float* T = x3_stage_tile(acc, sm);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int r = wave; r < m_ext; r += 8) {
    const int64_t i = m0 + r;
    if (2 * a.row_cnt[i] <= a.bw) continue;  // solved directly
    float top = 0.f;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int col = lane + 64 * e;
      if (col < n_ext) {
        const float l = a.mask_out[i * a.b + a.j1 + n0 + col] ? T[r * kXCLd + col] : 0.f;
        a.Lam[i * a.ldl + n0 + col] = l;
        top = fmaxf(top, fabsf(l));
      }
    }
    rsc_lower(a, i, top);
  }
}

// ------------------------------------------------------------------------------------------
// W[:, j1:b] -= Lam * P[j1:j2, j1:b]; removed weights of the block become exact zeros.
// W[:, col0:col_end] -= Lam[:, 0:K] * P[prow0:prow0+K, col0:col_end]; entries of the column
// range [zj1, zj2) whose mask byte is set are written as exact zeros.
struct UpdateArgs {
  float* W;
  const float* Lam;     // c x K multipliers, row stride ldl
  const float* P;
  const uint8_t* mask;
  int64_t c, b;
  int64_t prow0;        // first row of P (= first reduction index)
  int64_t col0, col_end;
  int64_t zj1, zj2;
  int K, ldl;
  // Unstructured mode: while the new weights are at hand, the columns right of the block are
  // histogrammed for the NEXT block's selection (window around the current threshold, see
  // k_select); hist == nullptr switches this off.
  unsigned int* hist;         // 2048 bins, global
  unsigned int* below_part;   // keys below the window, one count per workgroup
  unsigned int* cand_n;       // per workgroup: keys inside the window ...
  uint2* cand;                // ... and the keys with their rows, kCandStage slots per workgroup
  SelState* st;
  const float* sx;
  const float* sc;            // scales of the columns ...
  const float* rsc;           // ... and of the rows' multipliers
  const uint8_t* pexp;        // scales of P for the product (rows pexp_n, stride b)
  int pexp_n;
  int gx, gy;                 // tile grid (set by launch_update)
  int cand_cap;               // entries of a list (k_update: kCandStage)
};

typedef unsigned short u16u __attribute__((aligned(1)));  // two mask bytes

// two slabs of the operands; after the product the staged tile and, behind it, the window counts and the
// reciprocal scales of the columns
constexpr size_t kUpdSmemBytes = kH2SmemBytes;
constexpr size_t kUpdInvOffset = kXSmemBytes + 2048 * sizeof(unsigned int) + 16 * sizeof(unsigned int) +
                                 kCandStage * sizeof(uint2);
static_assert(kUpdInvOffset + kTN * sizeof(float) <= kUpdSmemBytes, "both fit");

constexpr int kUpdXcdRows = 16;  // tile rows from which on k_update deals them out to the XCDs

// H2: two-way split of the operands.  Not for short reductions: of K products it loses the last bits once,
// the three-way split rounds its running sum twice as often.  Errors of this kernel's results against float64,
// solve included, two-way and three-way: K = 16 1.83 and 1.70e-7, 48 2.77 and 2.73, 64 3.13 and 3.14, 80 3.67 and
// 3.69, 128 4.68 and 4.74.  The scales come from the values of P (per column) and of the multipliers (per row):
// with the block size as the bound of P, whose values get smaller as b grows, updates of 1024 to 2048 products
// were off by 5.7e-7 at 8192 columns, B = 128, 8.2e-7 at B = 256, 2.1e-6 at 28672 columns; three-way 5.3, 6.6 and
// 6.0e-7; now 4.4, 5.0 and 4.8e-7.  Price: 0.6 % of 4096x11008 at 50 %.
template <bool H2>
__global__ __launch_bounds__(kXThreads, 4) void k_update(UpdateArgs a) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  if (threadIdx.x == 0) TL_MARK(0);
  unsigned int* hw = reinterpret_cast<unsigned int*>(sm + kXSmemBytes);  // window histogram
  unsigned int* nb_wave = hw + 2048;  // 8 counts per wavefront, then: staged keys, list offset
  uint2* stage = reinterpret_cast<uint2*>(nb_wave + 16);
  // Tile of this workgroup.  Consecutive workgroup ids go to the eight XCDs in turn, each with
  // an L2 of its own: XCD x takes the row tiles x*rp .. x*rp + rp - 1 and walks them column by
  // column, so that it reads one eighth of the multipliers and every tile of P_k once.
  // (With fewer than 16 row tiles the XCDs would not get equal shares: plain order.)
  int bx, by;
  if (a.gy >= kUpdXcdRows) {
    const int rp = (a.gy + 7) >> 3;
    const int slot = (int)blockIdx.x >> 3;
    bx = slot / rp;
    by = ((int)blockIdx.x & 7) * rp + (slot - bx * rp);
    if (by >= a.gy) return;
  } else {
    by = (int)blockIdx.x / a.gx;
    bx = (int)blockIdx.x - by * a.gx;
  }
  const int64_t m0 = (int64_t)by * kTM;
  const int64_t n0 = a.col0 + (int64_t)bx * kTN;
  const int m_ext = (int)min((int64_t)kTM, a.c - m0);
  const int n_ext = (int)min((int64_t)kTN, a.col_end - n0);
  const float* A = a.Lam + m0 * a.ldl;          // (m,k) at A[m*ldl + k]
  const float* Bm = a.P + a.prow0 * a.b + n0;   // (k,n) at B[k*b + n]
  // does this tile feed the next selection?  (uniform per workgroup)
  const bool win = a.hist != nullptr && !a.st->none && a.st->pred_try && n0 + n_ext > a.zj2;
  TileAcc acc;
  acc_zero(acc);
  const float* rsc = a.rsc + m0;
  // P is fetched 16 bytes at a time whatever its row stride: up to three columns past the last one, values of
  // the next row or of what lies behind P in the workspace, which end in columns that are not written
  const int n4 = (n_ext + 3) & ~3;
  float* const inv = reinterpret_cast<float*>(sm + kUpdInvOffset);
  if constexpr (H2)
    gemm_tile_h2<false, true, 2, true, true, true>(acc, sm, A, a.ldl, m_ext, 1.f, rsc, Bm, a.b, n4, 1.f,
                                                   {a.pexp + n0, a.b, a.pexp_n}, inv, 0, a.K);
  else
    gemm_tile_x3<false, true>(acc, sm, A, a.ldl, m_ext, Bm, a.b, n4, 0, a.K);
  if (threadIdx.x == 0) TL_MARK(1);
  if (win) {
    for (int e = threadIdx.x; e < 2048; e += kXThreads) hw[e] = 0u;  // a barrier follows in the staging
    if (threadIdx.x == 0) nb_wave[8] = 0u;                            // staged keys
  }
  const float* T = x3_stage_tile(acc, sm);
  if (threadIdx.x == 0) TL_MARK(2);
  // row pass: wavefront w takes rows w, w + 8, ..., lane l the columns 2l, 2l + 1
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c0 = 2 * lane;
  const int64_t cg = n0 + c0;
  const bool in_block = n0 < a.zj2 && n0 + kTN > a.zj1;  // tile overlaps the columns holding masks
  float* Wg = a.W + m0 * a.b + cg;
  const uint8_t* Mg = a.mask + m0 * a.b + cg;
  // the scales taken out of the product again, per column and per row
  float f0 = pow2_inv(a.sc[min(cg, a.b - 1)]), f1 = pow2_inv(a.sc[min(cg + 1, a.b - 1)]);
  if (H2) {
    f0 *= inv[c0];
    f1 *= inv[c0 + 1];
  }
  // window count of one new weight (columns right of the block only)
  const unsigned int wlo = win ? a.st->win_lo : 0u;
  const int wsh = win ? a.st->win_shift : kWinShiftMin;
  unsigned int nb = 0;
  auto count = [&](float w, float sxj, int row) {
    const unsigned int key = metric_key(w, sxj);
    const unsigned int p28 = key >> wsh;
    if (p28 < wlo) {
      ++nb;
    } else if (p28 - wlo < 2048u) {
      atomicAdd(&hw[p28 - wlo], 1u);
      const unsigned int k = atomicAdd(&nb_wave[8], 1u);
      if (k < (unsigned int)kCandStage) stage[k] = make_uint2(key, (unsigned int)(m0 + row));
    }
  };
  if (m_ext == kTM && n_ext == kTN) {  // whole tile: pairs of columns, of any alignment
    const bool z0 = in_block && cg >= a.zj1 && cg < a.zj2;
    const bool z1 = in_block && cg + 1 >= a.zj1 && cg + 1 < a.zj2;
    const bool h0 = win && cg >= a.zj2, h1 = win && cg + 1 >= a.zj2;
    const float sx0 = h0 ? a.sx[cg] : 0.f, sx1 = h1 ? a.sx[cg + 1] : 0.f;
    f32x2u old[16];
    unsigned short mk[16];
    float fr[16];  // the row is the wavefront's: scalar loads
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t off = (int64_t)(wave + 8 * i) * a.b;
      fr[i] = H2 ? pow2_inv(rsc[wave + 8 * i]) : 1.f;
      old[i] = *reinterpret_cast<const f32x2u*>(Wg + off);
      mk[i] = in_block ? *reinterpret_cast<const u16u*>(Mg + off) : (unsigned short)0;
    }
    TL_WAIT_LOADS();
    if (threadIdx.x == 0) TL_MARK(3);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = wave + 8 * i;
      const float2 t = *reinterpret_cast<const float2*>(T + row * kXCLd + c0);
      f32x2u o;
      o.x = (z0 && (mk[i] & 0xffu)) ? 0.f : fmaf(-t.x, fr[i] * f0, old[i].x);
      o.y = (z1 && (mk[i] >> 8)) ? 0.f : fmaf(-t.y, fr[i] * f1, old[i].y);
      *reinterpret_cast<f32x2u*>(Wg + (int64_t)row * a.b) = o;
      if (h0) count(o.x, sx0, row);
      if (h1) count(o.y, sx1, row);
    }
  } else {
    // all loads first, from clamped addresses: one at a time between the stores, rows of 1365 columns took 30
    // us per launch instead of 17
    const bool ok0 = c0 < n_ext, ok1 = c0 + 1 < n_ext;
    const bool z0 = in_block && cg >= a.zj1 && cg < a.zj2, z1 = in_block && cg + 1 >= a.zj1 && cg + 1 < a.zj2;
    const bool h0 = win && ok0 && cg >= a.zj2, h1 = win && ok1 && cg + 1 >= a.zj2;
    const float sx0 = h0 ? a.sx[cg] : 0.f, sx1 = h1 ? a.sx[cg + 1] : 0.f;
    const int64_t d0 = (ok0 ? 0 : n_ext - 1 - c0), d1 = (ok1 ? 1 : n_ext - 1 - c0);  // to a column that exists
#pragma clang loop unroll(disable)
    for (int r0 = wave; r0 < m_ext; r0 += 32) {  // four rows at a time
      float w0[4], w1[4], fr[4];
      uint8_t k0[4], k1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = min(r0 + 8 * i, m_ext - 1);
        const int64_t off = (int64_t)row * a.b;
        fr[i] = H2 ? pow2_inv(rsc[row]) : 1.f;
        w0[i] = Wg[off + d0];
        w1[i] = Wg[off + d1];
        k0[i] = in_block ? Mg[off + d0] : (uint8_t)0;
        k1[i] = in_block ? Mg[off + d1] : (uint8_t)0;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = r0 + 8 * i;
        if (row >= m_ext) break;
        const float2 t = *reinterpret_cast<const float2*>(T + row * kXCLd + c0);
        const float o0 = (z0 && k0[i]) ? 0.f : fmaf(-t.x, fr[i] * f0, w0[i]);
        const float o1 = (z1 && k1[i]) ? 0.f : fmaf(-t.y, fr[i] * f1, w1[i]);
        if (ok0) Wg[(int64_t)row * a.b] = o0;
        if (ok1) Wg[(int64_t)row * a.b + 1] = o1;
        if (h0) count(o0, sx0, row);
        if (h1) count(o1, sx1, row);
      }
    }
  }
  if (threadIdx.x == 0) TL_MARK(4);
  if (a.hist == nullptr) {
    if (threadIdx.x == 0) TL_MARK(5);
    return;
  }
  // one partial count of the keys below the window per workgroup (summed by k_select:
  // thousands of atomics on one address would cost more than the pass), window bins by atomics
  for (int off = 32; off > 0; off >>= 1) nb += __shfl_down(nb, off, 64);
  if (lane == 0) nb_wave[wave] = nb;
  __syncthreads();
  const int tile = by * a.gx + bx;
  if (threadIdx.x == 0) {
    unsigned int t = 0;
    for (int v = 0; v < kXThreads / 64; ++v) t += nb_wave[v];
    a.below_part[tile] = t;
    unsigned int n = win ? nb_wave[8] : 0u;
    if (n > (unsigned int)kCandStage) {  // more window keys than a list holds: no prediction
      a.st->cand_overflow = 1;
      n = 0u;
    }
    a.cand_n[tile] = n;
  }
  if (blockIdx.x == 0) {
    // between two launches of k_select: the histograms of its radix passes and its counters
    for (int e = threadIdx.x; e < 3 * 2048; e += kXThreads) a.hist[2048 + e] = 0u;
    if (threadIdx.x == 0) a.st->arrived = a.st->nbin = a.st->bar = 0u;
  }
  if (!win) {
    if (threadIdx.x == 0) TL_MARK(5);
    return;
  }
  const unsigned int n = min(nb_wave[8], (unsigned int)kCandStage);
  uint2* list = a.cand + (size_t)tile * kCandStage;
  for (unsigned int e = threadIdx.x; e < n; e += kXThreads) list[e] = stage[e];
  for (int e = threadIdx.x; e < 2048; e += kXThreads)
    if (hw[e]) atomicAdd(&a.hist[e], hw[e]);
  if (threadIdx.x == 0) TL_MARK(5);
}

// The same where few tiles are left (two-way split, reduction a multiple of 128).  The kernel above needs 12 us for one
// round of tiles, most of it the phases of a tile behind each other, while 16 of 256 compute units work at 512 x
// 512.  Here a wavefront owns 32 x 32 of W and requests all it reads at the start: its operands straight into
// the registers that the MFMAs read them from, as in k_gemm_direct (lane (lo, hi) holds k = 8 q + 4 hi + c
// of its row of multipliers and of its column of P), and the old values, which it changes where the sums are.
// All four partial products: the matrix pipes are idle.  A workgroup is a strip of 32 rows x 128 columns with a
// count and a list of window keys of its own.  Whole passes: 256 x 256 2:4 146.8 -> 143.0 us, 512 x 512 at 50 % 409 ->
// 395, 1111 x 1365 1324 -> 1277, three of 768 x 768 1057 -> 1037.
__global__ __launch_bounds__(256, 2) void k_update_direct(UpdateArgs a) {
  __shared__ unsigned int below[4], listed;
  const int lane = threadIdx.x & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int by = (int)blockIdx.x / a.gx, bx = (int)blockIdx.x - by * a.gx;
  const int64_t m0 = 32 * (int64_t)by, n0 = a.col0 + (int64_t)kTN * bx;
  const int64_t cg = n0 + 32 * wave + lo, cc = min(cg, a.col_end - 1);  // this lane's column, and one that exists
  const int rows = (int)min((int64_t)32, a.c - m0);
  const bool win = a.hist != nullptr && !a.st->none && a.st->pred_try && min(n0 + kTN, a.col_end) > a.zj2;
  const bool in_block = n0 < a.zj2 && n0 + kTN > a.zj1;
  if (threadIdx.x == 0) listed = 0u;
  const float* pa = a.Lam + (m0 + min(lo, rows - 1)) * a.ldl + 4 * hi;
  const float* pb = a.P + a.prow0 * a.b;  // uniform; the lane's offset has 32 bits
  const uint32_t ob = (uint32_t)(4 * hi) * (uint32_t)a.b + (uint32_t)cc;
  f32x4 x[2][8], y[2][8];
  auto load = [&](int buf, int k) {
    const float* pk = pb + k * a.b;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      x[buf][q] = *reinterpret_cast<const f32x4u*>(pa + k + 8 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e, pk += a.b) y[buf][q][e] = pk[ob];
      pk += 4 * a.b;
    }
  };
  // what is needed first is requested first (loads return in order)
  const float sa = a.rsc[m0 + min(lo, rows - 1)];
  uint32_t ex = 253u;  // a column takes the smallest of its exponents, one per block and 128 rows of it
  for (int t = 4; t < a.pexp_n; ++t) ex = min(ex, (uint32_t)a.pexp[t * a.b + cc]);
  uint32_t e4[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) e4[e] = a.pexp[min(e, a.pexp_n - 1) * a.b + cc];
  const float scol = a.sc[cc];
  const float sxj = win ? a.sx[cc] : 0.f;
  load(0, 0);
  load(1, 64);
  float old[16];
  uint8_t mk[16];
  auto row_of = [&](int r) { return 8 * (r >> 2) + 4 * hi + (r & 3); };
  float* const Wt = a.W + m0 * a.b;
  const uint8_t* const Mt = a.mask + m0 * a.b;
  uint32_t at[16];  // 32 rows of at most 65535 columns
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    at[r] = (uint32_t)min(row_of(r), rows - 1) * (uint32_t)a.b + (uint32_t)cc;
    old[r] = Wt[at[r]];
  }
  if (in_block) {
#pragma unroll
    for (int r = 0; r < 16; ++r) mk[r] = Mt[at[r]];
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) mk[r] = 0;
  }
  const float sb = exponent_scale(min(min(min(e4[0], e4[1]), min(e4[2], e4[3])), ex));
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
  for (int k = 128; k < a.K; k += 128) {
    multiply(0);
    load(0, k);
    multiply(1);
    load(1, k + 64);
  }
  multiply(0);
  multiply(1);
  const float f = pow2_inv(scol) * pow2_inv(sb);
  const bool there = cg < a.col_end;
  const bool z = in_block && cg >= a.zj1 && cg < a.zj2, h = win && there && cg >= a.zj2;
  const unsigned int wlo = win ? a.st->win_lo : 0u;
  const int wsh = win ? a.st->win_shift : kWinShiftMin;
  uint2* const list = a.cand + (size_t)blockIdx.x * a.cand_cap;
  unsigned int nb = 0;
  __syncthreads();  // listed == 0
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = row_of(r);
    const float fr = pow2_inv(__shfl(sa, row, 64));
    const float o = (z && mk[r]) ? 0.f : fmaf(-(acc[r] + acc2[r]), fr * f, old[r]);
    if (there && row < rows) {
      Wt[at[r]] = o;
      if (h) {
        const unsigned int key = metric_key(o, sxj), bin = key >> wsh;
        if (bin < wlo) {
          ++nb;
        } else if (bin - wlo < 2048u) {
          atomicAdd(&a.hist[bin - wlo], 1u);
          const unsigned int k = atomicAdd(&listed, 1u);
          if (k < (unsigned int)a.cand_cap) list[k] = make_uint2(key, (unsigned int)(m0 + row));
        }
      }
    }
  }
  if (a.hist == nullptr) return;
  for (int off = 32; off > 0; off >>= 1) nb += __shfl_down(nb, off, 64);
  if (lane == 0) below[wave] = nb;
  __syncthreads();
  if (threadIdx.x == 0) {
    a.below_part[blockIdx.x] = below[0] + below[1] + below[2] + below[3];
    unsigned int n = listed;
    if (n > (unsigned int)a.cand_cap) {  // no prediction
      a.st->cand_overflow = 1;
      n = 0u;
    }
    a.cand_n[blockIdx.x] = n;
  }
  if (blockIdx.x == 0) {  // as in k_update
    for (int e = threadIdx.x; e < 3 * 2048; e += 256) a.hist[2048 + e] = 0u;
    if (threadIdx.x == 0) a.st->arrived = a.st->nbin = a.st->bar = 0u;
  }
}
// Counts and lists of its workgroups, four for every tile of the array that k_update keeps its lists in (tiles of them).
// A list is a quarter as long and overflows no sooner on the data tried: rows of equal scale, or of scales over e^+-2 at
// random, sorted, by strips of 32 or in one strip of four, 512 x 512 to 2048 x 2048: the selections of a pass take what they
// take with lists of 384 (512 x 512 58 to 75 us, 2048 x 2048 193 to 222 of 196 to 225).
struct DirectLists {
  unsigned int *below_part, *cand_n;
  uint2* cand;
  static constexpr int cap = kCandStage / 4 - 1;
};
static inline DirectLists direct_lists(uint2* cand, int64_t tiles) {
  unsigned int* const n = reinterpret_cast<unsigned int*>(cand);
  return {n, n + 4 * tiles, cand + 4 * tiles};
}
static_assert(4 * (2 * sizeof(unsigned int) + DirectLists::cap * sizeof(uint2)) <= kCandStage * sizeof(uint2), "they fit");
// Every operand row is fetched once per tile of 32 columns instead of 128, which pays while the launch waits for its
// latency: up to one workgroup per compute unit, and up to two where the keys of the next selection are counted
// (window) and k_update has too few tile rows to deal them out to the XCDs.  us a launch of k_update -> of this one:
//   rows, reduction     512 workgroups (or)       256 (or)                128
//   1000, 128, window   18.6 -> 15.7              15.9 -> 11.1            15.8 -> 9.7
//   1536, 128, window   16.4 -> 16.1 (480)        14.4 -> 11.1 (240)
//   2048, 128, window   13.9 -> 14.8              13.6 -> 11.8            13.0 -> 9.8
//   3000, 128, window   14.3 -> 14.8 (470)        13.4 -> 10.8 (188)
//   1536, 128           11.3 -> 11.3 (384)        10.7 -> 10.1 (240)       9.7 -> 8.0 (96)
//   2048, 128           10.2 -> 13.4 (448)         9.7 -> 10.6             9.5 -> 8.6
//   3000, 128           11.6 -> 12.6 (376)        11.0 ->  8.8 (188)
//   2048, 256           15.3 -> 18.0              14.4 -> 13.7            14.4 -> 13.2
//   2048, 512           23.5 -> 27.8              22.4 -> 19.5
constexpr int64_t kUpdDirectWgs = 256, kUpdDirectWgsWindow = 512;
// Columns of the update from col0 on.
static inline bool update_direct_ok(int64_t c, int64_t cols, int K, bool window) {
  const int64_t most = window && ceil_div(c, kTM) < kUpdXcdRows ? kUpdDirectWgsWindow : kUpdDirectWgs;
  return K > kShortK && K % 128 == 0 && K <= 512 && ceil_div(c, 32) * ceil_div(cols, kTN) <= most;
}

// ------------------------------------------------------------------------------------------
// Outlier rows (App. G.4.4 / Sec. 4.7): h_i = ||W_i X||^2 = W_i H W_i^T; the ceil(alpha c) rows
// with the largest h are left untouched.
// W_i H W_i^T = 2 sum_n W_in sum_{k >= n} W_ik Hl_kn with Hl = the lower triangle of H with its
// diagonal halved and zeros above it: the product T = W Hl only needs the reduction range
// k >= n of every output column, i.e. half of the full product.
// Channels are scaled by powers of two d as in the factorisation, W' = W D^-1, H' = D H D with a diagonal in [1, 4):
// nothing changes in the losses, and the product's operands have a known range (gemm_tile_h2.h) whatever the scales
// of the channels are (undamped: a channel far below the damping keeps its bits; loss_scale for those without any
// activations).  A caller's own H need not be positive semidefinite before it is damped; larger elements of H' than a
// Gram matrix has are looked after where they overflow (k_gemm_topped, k_rowdot).  Where there is no factorisation to
// take d from, and too many columns for k_loss_prep to look at the diagonal itself:
__global__ __launch_bounds__(256) void k_loss_scales(const float* __restrict__ H, int64_t b, float* __restrict__ d) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < b) d[j] = loss_scale(H[j * b + j]);
}
constexpr int64_t kLossFewCols = 1024;  // a launch less: 4 of the 112 us of 64 x 128
// The first nt workgroups (tiles of kHalfRows x 256): Hl, scaled, in the tiles of 128 on and below the diagonal, which
// are all that the product reads; a thread takes kHalfRows rows of a column, all in flight (64 x 128: with 64 rows,
// eight at a time, 14.8 us).  The others: the largest magnitudes of the rows of W' (NaN counts as large), one wavefront
// per row.
constexpr int kHalfRows = 8;
static_assert(kTN % kHalfRows == 0, "the rows of a thread lie in one tile row");
// d_out: d is made from the diagonal of H, and left there.
__global__ __launch_bounds__(256) void k_loss_prep(const float* __restrict__ H, const float* __restrict__ W, int64_t c,
                                                   int64_t b, const float* __restrict__ d, float* __restrict__ Hl,
                                                   float* __restrict__ top, int nx, int nt, float* __restrict__ d_out) {
  auto raw = [&](int64_t j) { return d_out ? H[j * b + j] : d[j]; };
  auto scale = [&](float v) { return d_out ? loss_scale(v) : v; };
  if ((int)blockIdx.x < nt) {
    const int64_t i0 = (int64_t)(blockIdx.x / nx) * kHalfRows, i1 = min(b, i0 + kHalfRows);
    const int64_t j = (int64_t)(blockIdx.x % nx) * 256 + threadIdx.x;
    if (j >= b || j / kTN > i0 / kTN) return;
    const float dj = scale(raw(j));
    if (d_out && j >= i0 && j < i1) d_out[j] = dj;
    float v[kHalfRows], di[kHalfRows];
#pragma unroll
    for (int e = 0; e < kHalfRows; ++e) {
      v[e] = H[max(min(i0 + e, b - 1), j) * b + j];  // never above the diagonal
      di[e] = raw(min(i0 + e, b - 1));
    }
#pragma unroll
    for (int e = 0; e < kHalfRows; ++e) {
      const int64_t i = i0 + e;
      if (i < i1) Hl[i * b + j] = j > i ? 0.f : v[e] * (dj * scale(di[e])) * (j == i ? 0.5f : 1.f);
    }
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)((int)blockIdx.x - nt) * 4 + (threadIdx.x >> 6);
  if (i >= c) return;
  const float* row = W + i * b;
  uint32_t u = 0;
  for (int64_t j = lane; j < b; j += 8 * 64) {
    float v[8], g[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = row[min(j + 64 * e, b - 1)];
      g[e] = raw(min(j + 64 * e, b - 1));
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) u = max(u, __float_as_uint(fabsf(v[e] * pow2_inv(scale(g[e])))));
  }
  for (int off = 32; off > 0; off >>= 1) u = max(u, (uint32_t)__shfl_xor((int)u, off, 64));
  if (lane == 0) top[i] = __uint_as_float(u);
}

// h[i] = 2 sum_j T[i][j] * W[i][j] / d[j]; one wavefront per row, fp64 sum in a fixed order.
// A loss that fp32 does not hold in the scaled coordinates (a caller's own H with elements between channels whose diagonal
// is zero) is taken straight from H, lower triangle, where the weights of the row are finite: slow, and rare.
__global__ __launch_bounds__(256) void k_rowdot(const float* __restrict__ T, const float* __restrict__ W,
                                                const float* __restrict__ d, const float* __restrict__ H, int64_t c,
                                                int64_t b, float* __restrict__ h) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= c) return;
  const float* const row = W + i * b;
  double acc = 0.0;
  for (int64_t j = lane; j < b; j += 64) acc += (double)T[i * b + j] * (double)(row[j] * pow2_inv(d[j]));
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  acc *= 2.0;
  if (!(fabs(acc) < (double)INFINITY)) {
    bool finite = true;
    for (int64_t j = lane; j < b; j += 64) finite = finite && fabsf(row[j]) < INFINITY;
    if (__all(finite)) {
      acc = 0.0;
      for (int64_t k = 0; k < b && __all(fabs(acc) < (double)INFINITY); ++k) {
        double part = 0.0;
        for (int64_t n = lane; n <= k; n += 256) {
          float v[4], w[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int64_t m = min(n + 64 * e, k);
            v[e] = H[k * b + m];
            w[e] = n + 64 * e > k ? 0.f : row[m];
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) part += (n + 64 * e == k ? 1.0 : 2.0) * (double)v[e] * (double)w[e];
        }
        acc += part * (double)row[k];
      }
      for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    }
  }
  if (lane == 0) h[i] = (float)acc;
}

// skip[i] = 1 for the n_out rows with the largest (h, row) (ascending order, ties by row index).
__global__ __launch_bounds__(256) void k_row_rank(const float* __restrict__ h, int64_t c,
                                                  int64_t n_out, uint8_t* __restrict__ skip) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= c) return;
  const int64_t rank = wave_rank(h, c, i);
  if ((threadIdx.x & 63) == 0) skip[i] = rank >= c - n_out ? 1 : 0;
}

// skip[i] = 1 for the n_out rows of W (c x b fp32) with the largest loss W_i H W_i^T (H: lower
// triangle).  Hf (b x b, receives the scaled lower triangle with halved diagonal), T (c x b) and h (c) are
// scratch.  The product takes the two-way split: errors of the losses against float64, three-way -> two-way, 0.8 ->
// 0.75e-7 at 64 columns, 1.7 -> 1.4 at 512, 2.1 -> 1.6 at 1364, 2.7 -> 2.1e-7 at 4096; 4096 x 4096
// 390 -> 252 us, 5120 x 5120 4:8 beside the factorisation 930 -> 640, 4940 -> 4800 us for the whole call.
thanos_status row_outliers(hipStream_t s, const float* W, const float* H, int64_t c, int64_t b,
                           long long n_out, float* Hf, float* T, float* h, const float* d, float* d_room,
                           uint8_t* skip, bool beside) {
  float* d_out = nullptr;
  if (!d) {
    if (b <= kLossFewCols) {
      d_out = d_room;
    } else {
      hipLaunchKernelGGL(k_loss_scales, dim3((unsigned)ceil_div(b, 256)), dim3(256), 0, s, H, b, d_room);
      THANOS_LAUNCH_CHECK();
    }
    d = d_room;
  }
  const int nx = (int)ceil_div(b, 256), nt = nx * (int)ceil_div(b, kHalfRows);
  hipLaunchKernelGGL(k_loss_prep, dim3((unsigned)(nt + ceil_div(c, 4))), dim3(256), 0, s, H, W, c, b, d, Hf, h, nx, nt,
                     d_out);
  THANOS_LAUNCH_CHECK();
  THANOS_CHECK(gemm_topped(s, c, b, b, W, b, h, Hf, b, nullptr, kBoundA, T, b, kTriLower, d, nullptr, beside));
  hipLaunchKernelGGL(k_rowdot, dim3((unsigned)ceil_div(c, 4)), dim3(256), 0, s, T, W, d, H, c, b, h);
  THANOS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_row_rank, dim3((unsigned)ceil_div(c, 4)), dim3(256), 0, s, h, c,
                     (int64_t)n_out, skip);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

// ------------------------------------------------------------------------------------------
struct SweepWs {
  float* sx;
  float* sc;
  float* Lam;
  float* P;
  uint8_t* pexp;
  unsigned int* hist;
  SelState* st;
  int* row_cand;
  int* row_eq;
  unsigned int* below_part;  // one count per workgroup of the block update
  unsigned int* cand_n;      // per update workgroup: keys inside the selection window ...
  uint2* cand;               // ... and (key, row) of each, kCandStage slots per workgroup
  unsigned long long* binlist;  // k_select: the keys of the threshold's bin
  unsigned int* wgflag;      // k_select: one word per workgroup, a cache line each
  float* Hf;        // alpha > 0: symmetric copy of H, b x b
  float* T;         // alpha > 0: W * H, c x b
  float* h;         // alpha > 0: row losses, c
  uint8_t* row_skip;  // alpha > 0: c
  float* tile_scratch;  // large blocks: tile grids of the rows in flight
  float* Kc;            // inverse of every block's G (B x B per block), or nullptr
};

static char* carve(char*& p, size_t bytes) {
  char* q = p;
  p += align_up(bytes, 256);
  return q;
}

// Large blocks (more than 256 unknowns per row, or more than 512 columns): workgroups of
// k_solve_tiled<.., BIG> that run at once, each with a slot for the tile grid of its row.
constexpr int kBigSlots = 512;
static inline bool needs_big(int B, int smax) { return smax > kTlSmax || B > kTlBw; }
static inline int64_t big_slot_floats(int smax) {
  return (int64_t)tl_ntiles((std::min(smax, kBigSmax) + 31) / 32) * kTlSz;
}

constexpr int64_t kPickRows = 2560;

static void launch_update(hipStream_t s, UpdateArgs ua, dim3 tiles) {
  ua.gx = (int)tiles.x;
  if (update_direct_ok(ua.c, ua.col_end - ua.col0, ua.K, ua.hist != nullptr)) {
    hipLaunchKernelGGL(k_update_direct, dim3(tiles.x * (unsigned)ceil_div(ua.c, 32)), dim3(256), 0, s, ua);
    return;
  }
  ua.gy = (int)tiles.y;
  const unsigned rp = (tiles.y + 7) / 8;
  const unsigned n = tiles.y >= kUpdXcdRows ? 8 * rp * tiles.x : tiles.x * tiles.y;
  if (ua.K > kShortK) hipLaunchKernelGGL(k_update<true>, dim3(n), dim3(kXThreads), kUpdSmemBytes, s, ua);
  else hipLaunchKernelGGL(k_update<false>, dim3(n), dim3(kXThreads), kUpdSmemBytes, s, ua);
}

// Whether rows that lose more than half of a block are solved through K = G^{-1} (see
// comp_tile, k_solve_tiled): only the tiled solver does it (blocks wider than 128 columns),
// the blocks' K come from the factor of the same call (not available with a given factor), the
// matrix-vector products read K in aligned groups of four columns, and n:m patterns that remove
// at most half of every group never need it.
bool sweep_uses_complement(const thanos_prune_opts* o, int64_t b) {
  const int B = o->block_size;
  if (o->factor_in) return false;
  if (o->mode == THANOS_NM && !o->mask_in && 2 * o->n <= o->m) return false;
  // blocks of up to 128 columns: the one-wavefront solver holds 96 unknowns and takes the rare
  // rows with more through the complement (no alignment needed there); nothing to do when no
  // row can have more
  if (B <= 128) return B > 96 && (o->mode != THANOS_NM || o->mask_in);
  return B % 4 == 0 && b % 4 == 0;
}

// Four columns at a time are read from pexp.
static size_t pexp_bytes(int64_t b, int B) {
  return kSuper * B > kShortK ? (size_t)(ceil_div(b, B) * block_row_tiles(B) * b + 4) : 0;
}

size_t sweep_workspace_bytes(int64_t c, int64_t b, int B, bool outliers, int smax, bool comp) {
  size_t n = 0;
  if (comp) n += align_up((size_t)ceil_div(b, B) * B * B * 4, 256);  // K blocks
  if (needs_big(B, smax))
    n += align_up((size_t)std::min<int64_t>(c, kBigSlots) * big_slot_floats(smax) * 4, 256);
  n += 2 * align_up((size_t)b * 4, 256);        // sx, sc
  n += align_up((size_t)lam_buffer_floats(c, B) * 4, 256);  // Lam
  n += align_up((size_t)b * b * 4, 256);        // P
  n += align_up(pexp_bytes(b, B), 256);
  n += align_up(4 * 2048 * 4, 256);             // hist: window + three passes
  n += align_up(sizeof(SelState), 256);         // state
  n += 2 * align_up((size_t)c * 4, 256);        // row_cand, row_eq
  n += align_up((size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * 4, 256);  // below_part
  n += align_up((size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * 4, 256);  // cand_n
  n += align_up((size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * kCandStage * sizeof(uint2), 256);  // cand
  n += align_up((size_t)kBinCap * 8, 256);                              // binlist
  n += align_up((size_t)kSelMaxWgs * kFlagStride * 4, 256);                     // wgflag
  if (outliers) {
    n += align_up((size_t)b * b * 4, 256);      // Hf
    n += align_up((size_t)c * b * 4, 256);      // T
    n += align_up((size_t)c * 4, 256);          // h
    n += align_up((size_t)c, 256);              // row_skip
  }
  return n;
}

static SweepWs carve_ws(void* ws, int64_t c, int64_t b, int B, bool outliers, int smax,
                        bool comp) {
  char* p = reinterpret_cast<char*>(ws);
  SweepWs w;
  w.Kc = nullptr;
  if (comp) w.Kc = reinterpret_cast<float*>(carve(p, (size_t)ceil_div(b, B) * B * B * 4));
  w.tile_scratch = nullptr;
  if (needs_big(B, smax))
    w.tile_scratch = reinterpret_cast<float*>(
        carve(p, (size_t)std::min<int64_t>(c, kBigSlots) * big_slot_floats(smax) * 4));
  w.sx = reinterpret_cast<float*>(carve(p, (size_t)b * 4));
  w.sc = reinterpret_cast<float*>(carve(p, (size_t)b * 4));
  w.Lam = reinterpret_cast<float*>(carve(p, (size_t)lam_buffer_floats(c, B) * 4));
  w.P = reinterpret_cast<float*>(carve(p, (size_t)b * b * 4));
  w.pexp = reinterpret_cast<uint8_t*>(carve(p, pexp_bytes(b, B)));
  w.hist = reinterpret_cast<unsigned int*>(carve(p, 4 * 2048 * 4));  // window + three passes
  w.st = reinterpret_cast<SelState*>(carve(p, sizeof(SelState)));
  w.row_cand = reinterpret_cast<int*>(carve(p, (size_t)c * 4));
  w.row_eq = reinterpret_cast<int*>(carve(p, (size_t)c * 4));
  w.below_part = reinterpret_cast<unsigned int*>(
      carve(p, (size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * 4));
  w.cand_n = reinterpret_cast<unsigned int*>(
      carve(p, (size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * 4));
  w.cand = reinterpret_cast<uint2*>(
      carve(p, (size_t)ceil_div(b, kTN) * ceil_div(c, kTM) * kCandStage * sizeof(uint2)));
  w.binlist = reinterpret_cast<unsigned long long*>(carve(p, (size_t)kBinCap * 8));
  w.wgflag = reinterpret_cast<unsigned int*>(carve(p, (size_t)kSelMaxWgs * kFlagStride * 4));
  w.Hf = w.T = w.h = nullptr;
  w.row_skip = nullptr;
  if (outliers) {
    w.Hf = reinterpret_cast<float*>(carve(p, (size_t)b * b * 4));
    w.T = reinterpret_cast<float*>(carve(p, (size_t)c * b * 4));
    w.h = reinterpret_cast<float*>(carve(p, (size_t)c * 4));
    w.row_skip = reinterpret_cast<uint8_t*>(carve(p, (size_t)c));
  }
  return w;
}

// Compute units of the current device (k_select launches at most one workgroup per unit).
static int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
    return 32;
  return n;
}

// Everything a sweep starts from, in one launch (a launch that does next to nothing costs 4.5 us, and
// these were up to five of them): the first n_conv workgroups convert the weights, the rest take
// square roots of the channel norms and, in unstructured mode (st), clear the selection's state.
struct InitArgs {
  const void* W_in;  // n weights of the layer's type -> W; n_conv == 0: already converted
  float* W;
  int64_t n;
  int n_conv, vec;
  const float* xn2;
  float* sx;
  const float* umax;  // largest magnitudes of the columns of U -> sc, unless nullptr
  float* sc;
  int64_t b;
  SelState* st;
  long long r;
  unsigned int *hist, *wgflag;
  int32_t* info;  // cleared unless nullptr
};
constexpr int kInitWgs = 32;
template <typename I>
__global__ __launch_bounds__(256) void k_sweep_init(InitArgs a) {
  if ((int)blockIdx.x < a.n_conv) {
    convert_quad((const I*)a.W_in, a.W, 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x), a.n, a.vec);
    return;
  }
  const int64_t i0 = (int64_t)((int)blockIdx.x - a.n_conv) * 256 + threadIdx.x;
  if (a.info && i0 == 0) *a.info = 0;
  for (int64_t i = i0; i < a.b; i += kInitWgs * 256) {
    a.sx[i] = sqrtf(a.xn2[i]);
    if (a.umax) a.sc[i] = col_scale(a.umax[i]);
  }
  if (!a.st) return;
  for (int64_t i = i0; i < 4 * 2048; i += kInitWgs * 256) a.hist[i] = 0u;
  for (int64_t i = i0; i < kSelMaxWgs * kFlagStride; i += kInitWgs * 256) a.wgflag[i] = 0u;
  if (i0 == 0) {
    SelState* st = a.st;
    st->r_rem = a.r;
    st->need_eq = 0;
    st->ties_all = 0;
    st->deferred = 0;
    st->tau = 0u;
    st->none = (a.r <= 0) ? 1 : 0;
    st->win_lo = 0u;
    st->win_shift = kWinShiftMin;
    st->pred_try = 0;
    st->cand_overflow = 0;
    st->arrived = st->nbin = st->bar = 0u;
  }
}

// k_solve_tiled with the tiles in registers: systems of up to smax <= 256 unknowns.
template <int SEL>
static void launch_tiled(hipStream_t s, SolveArgs a, int smax) {
  // Four wavefronts per row hold systems of up to 128 unknowns, eight up to 256.  When s varies
  // from row to row and may be larger than 128, each size gets a launch and the rows pick theirs.
  const size_t smem4 = rs_smem_floats<4>() * sizeof(float), smem8 = rs_smem_floats<8>() * sizeof(float);
  const bool small = smax <= 128, varies = SEL != SEL_NM;
  a.nt_lo = 0;
  a.nt_max = 4;
  if (small || varies)
    hipLaunchKernelGGL((k_solve_tiled<SEL, 4>), dim3((unsigned)a.c), dim3(256), smem4, s, a);
  if (small) return;
  a.nt_lo = varies ? 5 : 0;
  a.nt_max = kTlSmax / 32;  // the launch that reports systems beyond the solver's limit
  hipLaunchKernelGGL((k_solve_tiled<SEL, 8>), dim3((unsigned)a.c), dim3(512), smem8, s, a);
}

// k_solve_mfma for up to 64 unknowns per row
template <int SEL, int WPB>
static void launch_mfma2(hipStream_t s, const SolveArgs& a, bool full) {
  auto* const kern = full ? k_solve_mfma<SEL, WPB, 2, SEL == SEL_NM> : k_solve_mfma<SEL, WPB, 2, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(a.c, WPB)), dim3(64 * WPB), WPB * sizeof(SolveMfmaSmem<2>), s, a);
}

template <int SEL>
static void launch_solve(hipStream_t s, SolveArgs a, int smax) {
  // rows that lose more than half of the block are solved through the complement
  // (up to 128 columns: where that lets all rows run at once.  The kernel for 96 unknowns has eight of them per compute
  // unit, 18 KB of LDS each, the one for 64 has sixteen or twenty, and a row of it that goes through the complement
  // waits longer: 512 x 512 at 50 % 347 us and 358, 1111 x 1365 1100 and 1115, 4096 x 4096 9.0 and 8.2 ms)
  if (a.Kc && (a.bw > 128 || a.c > kRowsOf96)) smax = SEL == SEL_NM ? std::min(smax, a.bw - smax) : a.bw / 2;
  if (a.bw <= 128 && smax <= 64) {
    a.defer_large = a.Kc ? 1 : 0;
    const bool full = SEL == SEL_NM && a.bw * a.n == 64 * a.m && a.bw % a.m == 0;  // 64 unknowns in every row, or none
    if (solve_rows_per_group(a.c, full && !a.row_skip) == 5) launch_mfma2<SEL, 5>(s, a, full);
    else launch_mfma2<SEL, 4>(s, a, full);
  } else if (a.bw <= 128) {
    // Up to 96 unknowns: one wavefront per row on the matrix cores.  When s varies from row to
    // row (and may exceed 96) the few larger rows get a launch of the 128-thread kernel.
    constexpr int kWpb = 2;
    const size_t smem = kWpb * sizeof(SolveMfmaSmem<3>);
    const bool varies = SEL != SEL_NM;
    if (varies || smax <= 96) {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_solve_mfma<SEL, kWpb, 3>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
      a.defer_large = (varies && a.bw > 96) ? 1 : 0;
      hipLaunchKernelGGL((k_solve_mfma<SEL, kWpb, 3>), dim3((unsigned)ceil_div(a.c, kWpb)),
                         dim3(64 * kWpb), smem, s, a);
      a.defer_large = 0;
      // rows with more than 96 unknowns: solved by that launch through the complement when the
      // blocks' K are at hand, else by the 128-thread kernel
      if (!(varies && a.bw > 96) || a.Kc) return;
      a.s_min = 97;
    }
    hipLaunchKernelGGL((k_solve_wide<SEL, 128>), dim3((unsigned)a.c), dim3(128), 0, s, a);
  } else if (smax > kTlSmax || a.bw > kTlBw) {
    // large blocks: tile grids in global memory, persistent workgroups (two per compute unit)
    constexpr int kNw = 8;
    a.nt_lo = 0;
    a.nt_max = kBigSmax / 32;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_solve_tiled<SEL, kNw, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)tl_big_smem_bytes());
    hipLaunchKernelGGL((k_solve_tiled<SEL, kNw, true>),
                       dim3((unsigned)std::min<int64_t>(a.c, kBigSlots)), dim3(64 * kNw),
                       tl_big_smem_bytes(), s, a);
  } else {
    launch_tiled<SEL>(s, a, smax);
  }
}

// The part of the sweep that needs neither the factor nor the diagonal of H: the fp32 working
// copy of the weights and, with outlier rows, the rows to leave alone.  The caller may run it on
// another stream while the factorisation is going (the two touch disjoint memory) and then
// passes prepared = true to sweep().
thanos_status sweep_prepare(hipStream_t s, const void* W_in, thanos_dtype wdt, int64_t c, int64_t b,
                            const float* H, const thanos_prune_opts* o, long long n_out, float* W,
                            void* ws, const float* d, bool beside) {
  const int B = o->block_size;
  const bool outliers = n_out > 0;
  const int smax_all = (o->mode == THANOS_NM && !o->mask_in) ? B / o->m * o->n : B;
  SweepWs w = carve_ws(ws, c, b, B, outliers, smax_all, sweep_uses_complement(o, b));
  THANOS_CHECK(convert_in(s, W_in, wdt, W, c * b));
  if (outliers) {
    thanos_status st = row_outliers(s, W, H, c, b, n_out, w.Hf, w.T, w.h, d, w.sx, w.row_skip, beside);
    if (st != THANOS_OK) return st;
  }
  return THANOS_OK;
}

thanos_status sweep(hipStream_t s, const void* W_in, thanos_dtype wdt, int64_t c, int64_t b,
                    const float* H, const float* U, const float* xnorm2,
                    const thanos_prune_opts* o, long long r_total, long long n_out, float* W,
                    void* W_cast, uint8_t* mask, void* ws, int32_t* info, bool single_stream,
                    PhaseTimer* pt, const float* Lfac, int64_t ldL, const float* Ldiag, const float* Hscale,
                    const float* umax,
                    bool prepared,
                    bool clear_info, int sharers) {
  const int B = o->block_size;
  const bool outliers = n_out > 0;
  const int smax_all = (o->mode == THANOS_NM && !o->mask_in) ? B / o->m * o->n : B;
  const bool comp = sweep_uses_complement(o, b) && Lfac != nullptr;
  SweepWs w = carve_ws(ws, c, b, B, outliers, smax_all, sweep_uses_complement(o, b));

  const bool unstructured = (o->mode == THANOS_UNSTRUCTURED) && o->mask_in == nullptr;
  if (!prepared && outliers)  // the row losses need the converted weights
    THANOS_CHECK(sweep_prepare(s, W_in, wdt, c, b, H, o, n_out, W, ws, Hscale, false));
  const bool conv = !prepared && !outliers;
  const InitArgs ia{W_in, W, c * b, conv ? (int)ceil_div(c * b, 1024) : 0,
                    conv ? convert_vec(W_in, wdt, W, THANOS_F32) : 0, xnorm2, w.sx, umax, w.sc, b,
                    unstructured ? w.st : nullptr, r_total, w.hist, w.wgflag,
                    clear_info ? info : nullptr};
  const dim3 igrid((unsigned)(ia.n_conv + kInitWgs));
  if (wdt == THANOS_F32) hipLaunchKernelGGL(k_sweep_init<float>, igrid, dim3(256), 0, s, ia);
  else if (wdt == THANOS_F16) hipLaunchKernelGGL(k_sweep_init<__half>, igrid, dim3(256), 0, s, ia);
  else hipLaunchKernelGGL(k_sweep_init<__hip_bfloat16>, igrid, dim3(256), 0, s, ia);
  THANOS_LAUNCH_CHECK();

  const int super = unstructured ? 1 : kSuper;  // the global residual mask needs current weights
  if (!umax) {
    hipLaunchKernelGGL(k_col_scales, dim3((unsigned)ceil_div(b, 64)), dim3(1024), 0, s, U, b, B, w.sc);
    THANOS_LAUNCH_CHECK();
  }

  {
    dim3 grid((unsigned)ceil_div(b, kTN), (unsigned)ceil_div(b, B), (unsigned)ceil_div(B, kTM));
    BlockRowsArgs a{U, w.P, w.sc, B * super > kShortK ? w.pexp : nullptr, b, B, {nullptr, 0, nullptr, nullptr, 0, 0}};
    if (comp) {
      const int nt = (int)ceil_div(B, 32);
      a.comp = {Lfac, ldL, Ldiag, w.Kc, nt, (int)grid.z};
      grid.z += (unsigned)ceil_div((int64_t)nt * nt, grid.x);
    }
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_block_rows),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)kBlockRowsSmem));
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_update<true>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kUpdSmemBytes));
    THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_update<false>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kUpdSmemBytes));
    hipLaunchKernelGGL(k_block_rows, grid, dim3(kXThreads), kBlockRowsSmem, s, a);
    THANOS_LAUNCH_CHECK();
  }

  const int ldl = B * super;
  // The update that reaches right of a super-block is split like the wide update of the
  // factorisation: the columns of the next super-block on the caller's stream, the rest on a
  // second stream next to the (latency-bound) blocks of the next super-block.  The multipliers
  // of consecutive super-blocks alternate between two buffers.
  const int n_super = (int)ceil_div(b, (int64_t)B * super);
  AuxStream aux(s, super > 1 ? 2 * n_super : 0, single_stream);
  if (!aux.ok) return THANOS_ERR_HIP;
  int pending_join = -1;
  const int64_t row_tiles = block_row_tiles(B);
  int win_parts = 0;  // workgroups of the previous block's update (partial counts to sum) ...
  DirectLists lists = {w.below_part, w.cand_n, w.cand};  // ... their counts and lists
  int cand_cap = kCandStage;
  for (int64_t j1 = 0; j1 < b; j1 += B) {
    const int bw = (int)std::min<int64_t>(B, b - j1);
    const int64_t blk = j1 / B;
    const int64_t sbi = blk / super;
    const int64_t sb_start = sbi * super * (int64_t)B;
    const int64_t sb_end = (super == 1) ? b : std::min<int64_t>(b, sb_start + (int64_t)super * B);
    const int64_t loff = (super == 1) ? 0 : (j1 - sb_start);
    const LamLayout at = lam_layout(c, ldl, sbi);
    float* lam_sb = w.Lam + at.lam;
    float* rsc = unstructured ? w.Lam + at.rsc : reinterpret_cast<float*>(sbi & 1 ? w.row_eq : w.row_cand);
    if (unstructured) {
      phase_mark(pt, THANOS_PHASE_MASK);
      // 16-byte loads need W + i*b + j1 and sx + j1 aligned (W, sx come 256-byte aligned)
      const int sel_vec = (b % 4 == 0 && j1 % 4 == 0 &&
                           reinterpret_cast<uintptr_t>(W) % 16 == 0) ? 1 : 0;
      // the previous block's update counted the window around its threshold, and listed the
      // keys inside it, while it wrote the new weights
      SelectArgs ga;
      ga.W = W;
      ga.sx = w.sx;
      ga.st = w.st;
      ga.hist = w.hist;
      ga.below_part = lists.below_part;
      ga.n_part = win_parts;
      ga.cand_n = lists.cand_n;
      ga.cand = lists.cand;
      ga.cand_cap = cand_cap;
      ga.binlist = w.binlist;
      ga.row_cnt = w.row_cand;
      ga.row_cand = w.row_cand;
      ga.row_eq = w.row_eq;
      ga.tau_out = o->threshold_out ? o->threshold_out + blk : nullptr;
      ga.info = info;
      ga.c = c;
      ga.b = b;
      ga.j1 = j1;
      ga.first = j1 == 0 ? 1 : 0;
      ga.vec = sel_vec;
      ga.seq = (unsigned int)(blk + 1);
      ga.wgflag = w.wgflag;
      const unsigned sel_wgs = (unsigned)select_workgroups(c, compute_units(), sharers);
      hipLaunchKernelGGL(k_select, dim3(sel_wgs), dim3(kSelThreads), 0, s, ga);
      THANOS_LAUNCH_CHECK();
    }
    phase_mark(pt, THANOS_PHASE_SOLVE);
    SolveArgs sa;
    sa.W = W;
    sa.P = w.P;
    sa.sx = w.sx;
    sa.sc = w.sc;
    sa.rsc = rsc;
    sa.rsc_first = j1 == sb_start ? 1 : 0;
    sa.mask_in = o->mask_in;
    sa.mask_out = mask;
    sa.Lam = lam_sb + loff;
    sa.st = w.st;
    sa.st_rw = w.st;
    sa.row_skip = w.row_skip;
    sa.row_eq = w.row_eq;
    sa.row_cnt = w.row_cand;  // free once k_select has read the candidate flags
    sa.info = info;
    sa.c = c;
    sa.b = b;
    sa.j1 = j1;
    sa.bw = bw;
    sa.ldl = ldl;
    sa.n = o->n;
    sa.m = o->m;
    sa.nt_lo = sa.nt_max = 0;
    sa.s_min = 0;
    sa.defer_large = 0;
    sa.tile_scratch = w.tile_scratch;
    sa.slot_floats = big_slot_floats(smax_all);
    sa.Kc = comp ? w.Kc + blk * (int64_t)B * B : nullptr;
    sa.ldk = B;
    sa.Z = nullptr;
    sa.WK = nullptr;
    sa.ldz = 0;
    if (o->mask_in) {
      launch_solve<SEL_GIVEN>(s, sa, bw);
    } else if (o->mode == THANOS_NM) {
      launch_solve<SEL_NM>(s, sa, bw / o->m * o->n);
    } else {
      // Four launches instead of one pay from two rounds of rows on (five rows per compute unit), where
      // half of the rows or more go the complement way.  Whole sweeps of 1024 columns at B = 256, one
      // launch against four: 50 %: 1536 rows 1006 and 1027 us, 2560 1172 and 1132, 8192 2079 and 1908;
      // 40 %: 2560 rows 1025 and 1100, 8192 1726 and 1818; 60 %: 1024 rows 897 and 926, 8192 2321 and
      // 1864.  B = 512: 50 %: 2560 rows 1573 and 1443; 40 %: 8192 rows 2531 and 2596.
      const bool many = comp && bw > 128 && !needs_big(bw, bw / 2) && c >= kPickRows && o->sparsity >= 0.5;
      if (many) {
        float* const wk = w.Lam + at.wk;
        sa.Z = w.Lam + at.z;
        sa.WK = wk;
        sa.ldz = ldl;
        hipLaunchKernelGGL(k_pick, dim3((unsigned)ceil_div(c, 4)), dim3(256), 0, s, sa);
        THANOS_LAUNCH_CHECK();
        THANOS_CHECK(gemm_f32(s, false, false, c, bw, bw, 1.f, sa.Z, ldl, sa.Kc, B, 0.f, wk, ldl, false));
        launch_tiled<SEL_PICKED>(s, sa, bw / 2);
        THANOS_LAUNCH_CHECK();
        THANOS_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_lam_rows),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)kXSmemBytes));
        hipLaunchKernelGGL(k_lam_rows, dim3((unsigned)ceil_div(bw, kTN), (unsigned)ceil_div(c, kTM)),
                           dim3(kXThreads), kXSmemBytes, s, sa);
      } else {
        launch_solve<SEL_THRESHOLD>(s, sa, bw);
      }
    }
    THANOS_LAUNCH_CHECK();

    phase_mark(pt, THANOS_PHASE_UPDATE);
    {  // this block's update, up to the end of its super-block
      dim3 grid((unsigned)ceil_div(sb_end - j1, kTN), (unsigned)ceil_div(c, kTM));
      const bool feed = unstructured && j1 + bw < b;  // a next block exists: count its window
      if (feed) {
        const bool direct = update_direct_ok(c, sb_end - j1, bw, true);
        win_parts = (int)(grid.x * (direct ? ceil_div(c, 32) : grid.y));
        lists = direct ? direct_lists(w.cand, ceil_div(b, kTN) * ceil_div(c, kTM))
                       : DirectLists{w.below_part, w.cand_n, w.cand};
        cand_cap = direct ? DirectLists::cap : kCandStage;
      }
      UpdateArgs ua{W, lam_sb + loff, w.P, mask, c, b, j1, j1, sb_end, j1, j1 + bw, bw, ldl,
                    feed ? w.hist : nullptr, lists.below_part, lists.cand_n, lists.cand, w.st, w.sx, w.sc, rsc,
                    w.pexp + blk * row_tiles * b, (int)ceil_div(bw, kTM), 0, 0, cand_cap};
      launch_update(s, ua, grid);
      THANOS_LAUNCH_CHECK();
    }
    if (super > 1 && j1 + bw == sb_end && sb_end < b) {  // all blocks of the super-block
      const int64_t next_end = std::min<int64_t>(b, sb_end + (int64_t)super * B);
      const int kk = (int)(sb_end - sb_start);
      // The strip (the columns of the next super-block) first: the next block's solve waits for
      // it, so it gets the chip before the much larger rest does.  It was last written by the
      // previous rest.
      if (pending_join >= 0) THANOS_CHECK(aux.join(pending_join));
      {
        UpdateArgs ua{W, lam_sb, w.P, mask, c, b, sb_start, sb_end, next_end, 0, 0, kk, ldl,
                      nullptr, nullptr, nullptr, nullptr,
                      nullptr, nullptr, w.sc, rsc, w.pexp + sbi * super * row_tiles * b,
                      (int)(super * row_tiles), 0, 0, 0};
        dim3 grid((unsigned)ceil_div(next_end - sb_end, kTN), (unsigned)ceil_div(c, kTM));
        launch_update(s, ua, grid);
        THANOS_LAUNCH_CHECK();
      }
      if (next_end < b) {  // rest: right of the next super-block, second stream
        THANOS_CHECK(aux.fork((int)(2 * sbi)));
        UpdateArgs ua{W, lam_sb, w.P, mask, c, b, sb_start, next_end, b, 0, 0, kk, ldl,
                      nullptr, nullptr, nullptr, nullptr,
                      nullptr, nullptr, w.sc, rsc, w.pexp + sbi * super * row_tiles * b,
                      (int)(super * row_tiles), 0, 0, 0};
        dim3 grid((unsigned)ceil_div(b - next_end, kTN), (unsigned)ceil_div(c, kTM));
        launch_update(aux.stream, ua, grid);
        THANOS_LAUNCH_CHECK();
        THANOS_CHECK(aux.record((int)(2 * sbi + 1)));
        pending_join = (int)(2 * sbi + 1);
      }
    }
  }
  if (pending_join >= 0) THANOS_CHECK(aux.join(pending_join));

  phase_mark(pt, THANOS_PHASE_FINALISE);
  if (W_cast) THANOS_CHECK(convert_out(s, W, W_cast, wdt, c * b));
  return THANOS_OK;
}

}  // namespace thanos

#ifdef THANOS_TIMELINE
// Diagnostic build only (see timeline.h): which launch to record, and the recorded timestamps.
extern "C" int thanos_timeline_select(int grid_workgroups) {
  return (int)hipMemcpyToSymbol(HIP_SYMBOL(thanos::g_timeline_grid), &grid_workgroups, sizeof(int));
}
extern "C" int thanos_timeline_read(unsigned long long* host, size_t bytes) {
  if (bytes > sizeof(unsigned long long) * thanos::kTlWgs * thanos::kTlSlots) return -1;
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(thanos::g_timeline), bytes);
}
extern "C" int thanos_timeline_clear(void) {
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(thanos::g_timeline)) != hipSuccess) return -1;
  return (int)hipMemset(p, 0, sizeof(unsigned long long) * thanos::kTlWgs * thanos::kTlSlots);
}
#endif

