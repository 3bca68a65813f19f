// Shared host/device helpers of libthanos (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/thanos.h"

#define THANOS_HIP_CHECK(expr)                      \
  do {                                              \
    hipError_t e_ = (expr);                         \
    if (e_ != hipSuccess) return THANOS_ERR_HIP;    \
  } while (0)

#define THANOS_LAUNCH_CHECK()                                   \
  do {                                                          \
    if (hipGetLastError() != hipSuccess) return THANOS_ERR_HIP; \
  } while (0)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// the same where only the elements are aligned (one load or store all the same)
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Helper streams and their events are host objects that cost tens of microseconds to create
// and whose destruction waits for the stream to drain (which would stall the host inside every
// call).  They are therefore kept: a call borrows a context (one stream of default priority and
// as many events as it needs) from a per-process pool and hands it back on return; contexts are
// created on demand, one set per device and per concurrently running call, and live until the
// process ends.  A context is handed back only after its work has been joined into the
// caller's stream, so the next borrower's work is merely queued behind it.
struct StreamCtx {
  int device = -1;
  int order = 0;  // of creation: the pool lends the oldest idle context of a device
  hipStream_t stream = nullptr;
  hipEvent_t* ev = nullptr;
  int nev = 0, cap = 0;
};
StreamCtx* stream_ctx_acquire(int n_events);  // nullptr on failure (api.hip)
void stream_ctx_release(StreamCtx* c);

// A helper stream (default priority) for the duration of one call, forked from and joined back
// into the caller's stream with events; it runs a long, throughput-bound update next to a chain
// of short, latency-bound kernels.
//   fork(i)    the helper waits for everything the caller's stream holds now (event i)
//   record(i)  event i <- everything the helper holds now; no launch on the helper may follow
//              a record without a new fork
//   join(i)    the caller's stream waits for event i
// If the object is destroyed while forked work has not been joined (an error return between a
// fork and its join), the destructor joins it first, so that the caller's stream never runs
// ahead of kernels that still use the caller's buffers.
// inline_mode: there is no helper: `stream` IS the caller's stream and fork / record / join do
// nothing (one in-order stream runs the kernels in the order the host enqueues them, and that
// order respects every dependency the events express).  Nothing is created or borrowed.
class AuxStream {
 public:
  hipStream_t stream = nullptr;
  bool ok = false;
  AuxStream(hipStream_t caller, int n_events, bool inline_mode)
      : caller_(caller), inline_(inline_mode || n_events <= 0) {
    if (inline_) {  // also when no fork will happen
      stream = caller;
      ok = true;
      return;
    }
    ctx_ = stream_ctx_acquire(n_events + 1);  // the last event serves the destructor
    if (!ctx_) return;
    stream = ctx_->stream;
    nev_ = n_events + 1;
    ok = true;
  }
  thanos_status fork(int i) {
    if (inline_) return THANOS_OK;
    if (i < 0 || i >= nev_ - 1) return THANOS_ERR_HIP;
    if (hipEventRecord(ctx_->ev[i], caller_) != hipSuccess) return THANOS_ERR_HIP;
    if (hipStreamWaitEvent(stream, ctx_->ev[i], 0) != hipSuccess) return THANOS_ERR_HIP;
    open_ = true;
    last_rec_ = -1;
    return THANOS_OK;
  }
  thanos_status record(int i) {
    if (inline_) return THANOS_OK;
    if (i < 0 || i >= nev_ - 1) return THANOS_ERR_HIP;
    if (hipEventRecord(ctx_->ev[i], stream) != hipSuccess) return THANOS_ERR_HIP;
    last_rec_ = i;
    return THANOS_OK;
  }
  thanos_status join(int i) {
    if (inline_) return THANOS_OK;
    if (i < 0 || i >= nev_ - 1) return THANOS_ERR_HIP;
    if (hipStreamWaitEvent(caller_, ctx_->ev[i], 0) != hipSuccess) return THANOS_ERR_HIP;
    if (i == last_rec_) open_ = false;
    return THANOS_OK;
  }
  ~AuxStream() {
    if (inline_ || !ctx_) return;
    if (open_ && hipEventRecord(ctx_->ev[nev_ - 1], stream) == hipSuccess)
      (void)hipStreamWaitEvent(caller_, ctx_->ev[nev_ - 1], 0);
    stream_ctx_release(ctx_);
  }
  AuxStream(const AuxStream&) = delete;
  AuxStream& operator=(const AuxStream&) = delete;

 private:
  hipStream_t caller_;
  StreamCtx* ctx_ = nullptr;
  int nev_ = 0;
  bool inline_;
  bool open_ = false;  // forked work that no join covers yet
  int last_rec_ = -1;  // event of the last record since the last fork
};
// Diagnostic phase timing of one call: mark(p) records a timing event on the stream and says
// "what follows belongs to phase p"; collect() waits for the stream and adds the time between
// consecutive marks to the phase of the earlier one.  A null pointer or a disabled timer costs
// nothing.  Only meaningful when all kernels of the call run on the one stream.
class PhaseTimer {
 public:
  explicit PhaseTimer(hipStream_t s) : s_(s) {}
  void mark(int phase) {
    if (n_ >= kMax - (phase < 0 ? 0 : 1)) return;  // the last slot is kept for the closing mark
    if (hipEventCreate(&ev_[n_]) != hipSuccess) return;
    (void)hipEventRecord(ev_[n_], s_);
    ph_[n_++] = phase;
  }
  thanos_status collect(float* out) {  // THANOS_N_PHASES floats
    mark(-1);
    thanos_status st = hipStreamSynchronize(s_) == hipSuccess ? THANOS_OK : THANOS_ERR_HIP;
    for (int p = 0; p < THANOS_N_PHASES; ++p) out[p] = 0.f;
    for (int i = 0; i + 1 < n_ && st == THANOS_OK; ++i) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, ev_[i], ev_[i + 1]) != hipSuccess) st = THANOS_ERR_HIP;
      else if (ph_[i] >= 0 && ph_[i] < THANOS_N_PHASES) out[ph_[i]] += ms;
    }
    return st;
  }
  ~PhaseTimer() {
    for (int i = 0; i < n_; ++i) (void)hipEventDestroy(ev_[i]);
  }
  PhaseTimer(const PhaseTimer&) = delete;
  PhaseTimer& operator=(const PhaseTimer&) = delete;

 private:
  static constexpr int kMax = 4096;
  hipStream_t s_;
  hipEvent_t ev_[kMax];
  int ph_[kMax];
  int n_ = 0;
};
static inline void phase_mark(PhaseTimer* t, int phase) {
  if (t) t->mark(phase);
}

// A key whose unsigned order is the order of the floats, with -0 = +0 and NaN after everything: ranks
// are then a permutation whatever the values are, so they can be used as addresses.
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
  return x != x ? 0xffffffffu : (u & 0x80000000u) ? ~u : u | 0x80000000u;
}

// Number of elements that come before v[i] in ascending (value, index) order, computed by one
// wavefront (every lane gets it).  All n^2 comparisons of a ranking are cheap when they are spread
// over the chip: one thread per element used to walk all n values (4096 rows on 16 workgroups 310 us,
// 5120 434 us); one wavefront per element reads them 64 at a time, four loads in flight (10 us, and 14 to
// 31 beside the factorisation).
__device__ __forceinline__ int64_t wave_rank(const float* __restrict__ v, int64_t n, int64_t i) {
  const int lane = threadIdx.x & 63;
  const uint32_t mine = order_key(v[i]);
  int cnt = 0;  // this lane looks at n / 64 elements
  auto before = [&](float x, int64_t k) {
    const uint32_t o = order_key(x);
    return (o < mine || (o == mine && k < i)) ? 1 : 0;
  };
  int64_t k = lane;
  for (; k + 192 < n; k += 256) {
    const float o0 = v[k], o1 = v[k + 64], o2 = v[k + 128], o3 = v[k + 192];
    cnt += before(o0, k) + before(o1, k + 64) + before(o2, k + 128) + before(o3, k + 192);
  }
  for (; k < n; k += 64) cnt += before(v[k], k);
  int64_t r = cnt;
  for (int off = 32; off > 0; off >>= 1) r += __shfl_xor(r, off, 64);
  return r;
}

// d[j], the power of two with d^2 h in [1, 4) for a diagonal element h (1 where h is not positive or
// not finite: the factorisation reports those).
__device__ __forceinline__ float diag_scale(float h) {
  if (!(h > 0.f) || !(h < INFINITY)) return 1.f;
  const int e = min(max(ilogbf(h), -124), 124);
  return ldexpf(1.f, -(e >> 1));
}

// The same for the row losses, which take H without damping.  Channels without activations add nothing to a loss
// whatever their weights are: divided by the largest of the scales, these do not set the scale of a row.
__device__ __forceinline__ float loss_scale(float h) { return h == 0.f ? 0x1p62f : diag_scale(h); }

#define THANOS_CHECK(expr)                 \
  do {                                     \
    thanos_status st_ = (expr);            \
    if (st_ != THANOS_OK) return st_;      \
  } while (0)
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- conversions between the layer's type and fp32 -----------------------------------------
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__half x) { return __half2float(x); }
__device__ __forceinline__ float to_f32(__hip_bfloat16 x) { return __bfloat162float(x); }
__device__ __forceinline__ void from_f32(float x, float& o) { o = x; }
__device__ __forceinline__ void from_f32(float x, __half& o) { o = __float2half_rn(x); }
__device__ __forceinline__ void from_f32(float x, __hip_bfloat16& o) { o = __float2bfloat16(x); }

template <typename T>
struct __attribute__((aligned(4 * sizeof(T)))) Quad {
  T v[4];
};

// Four elements per thread as one load and one store where both pointers allow it (vec), else one
// by one; one element per thread kept memory at 2.6 TB/s.
template <typename I, typename O>
__device__ __forceinline__ void convert_quad(const I* __restrict__ in, O* __restrict__ out, int64_t i,
                                             int64_t n, int vec) {
  if (i >= n) return;
  if (vec && i + 4 <= n) {
    const Quad<I> x = *reinterpret_cast<const Quad<I>*>(in + i);
    Quad<O> y;
#pragma unroll
    for (int e = 0; e < 4; ++e) from_f32(to_f32(x.v[e]), y.v[e]);
    *reinterpret_cast<Quad<O>*>(out + i) = y;
  } else {
    for (int e = 0; e < 4 && i + e < n; ++e) from_f32(to_f32(in[i + e]), out[i + e]);
  }
}
template <typename I, typename O>
__global__ __launch_bounds__(256) void k_convert(const I* __restrict__ in, O* __restrict__ out,
                                                 int64_t n, int vec) {
  convert_quad(in, out, 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x), n, vec);
}
static inline int convert_vec(const void* in, thanos_dtype it, const void* out, thanos_dtype ot) {
  const uintptr_t ia = it == THANOS_F32 ? 16 : 8, oa = ot == THANOS_F32 ? 16 : 8;
  return reinterpret_cast<uintptr_t>(in) % ia == 0 && reinterpret_cast<uintptr_t>(out) % oa == 0;
}
template <typename I, typename O>
static inline void launch_convert(hipStream_t s, const void* in, void* out, int64_t n, int vec) {
  hipLaunchKernelGGL((k_convert<I, O>), dim3((unsigned)ceil_div(n, 1024)), dim3(256), 0, s,
                     (const I*)in, (O*)out, n, vec);
}
// W (fp32) <- weights of the layer's type, and back
static inline thanos_status convert_in(hipStream_t s, const void* in, thanos_dtype dt, float* out,
                                       int64_t n) {
  const int vec = convert_vec(in, dt, out, THANOS_F32);
  if (dt == THANOS_F32) launch_convert<float, float>(s, in, out, n, vec);
  else if (dt == THANOS_F16) launch_convert<__half, float>(s, in, out, n, vec);
  else launch_convert<__hip_bfloat16, float>(s, in, out, n, vec);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}
static inline thanos_status convert_out(hipStream_t s, const float* in, void* out, thanos_dtype dt,
                                        int64_t n) {
  const int vec = convert_vec(in, THANOS_F32, out, dt);
  if (dt == THANOS_F32) launch_convert<float, float>(s, in, out, n, vec);
  else if (dt == THANOS_F16) launch_convert<float, __half>(s, in, out, n, vec);
  else launch_convert<float, __hip_bfloat16>(s, in, out, n, vec);
  THANOS_LAUNCH_CHECK();
  return THANOS_OK;
}

// ---- internal entry points shared between translation units -------------------------------
namespace thanos {

constexpr int kFactorNB = 128;  // block size of the blocked factorisation
// Bounds of a symmetric positive definite matrix scaled to a diagonal in [1, 4), of its Schur complements, and of its
// factor, with room for rounding.
constexpr float kBoundA = 7.f, kBoundL = 3.f;
constexpr int kShortK = 64;      // reductions up to here stay on the three-way split (gemm_tile_h2.h)

// C[M x N] (ldc) = beta*C + alpha * op(A) * op(B), fp32 on the matrix cores, 128x128 tiles.
//   a_kmajor: element (m,k) of op(A) is A[k*lda + m], else A[m*lda + k]
//   b_kmajor: element (k,n) of op(B) is B[k*ldb + n], else B[n*ldb + k]
//   lower_only: compute only tiles with tile_row >= tile_col (C square)
thanos_status gemm_f32(hipStream_t s, bool a_kmajor, bool b_kmajor, int64_t M, int64_t N,
                       int64_t K, float alpha, const float* A, int64_t lda, const float* B,
                       int64_t ldb, float beta, float* C, int64_t ldc, bool lower_only);

// C = beta*C + alpha * A B^T for operands whose magnitude is bounded (A[m*lda + k], B[n*ldb + k]; bound_b_dev:
// the bound of B is read from the device instead).  The same precision in half of the matrix instructions.
thanos_status gemm_bounded(hipStream_t s, int64_t M, int64_t N, int64_t K, float alpha, const float* A,
                           int64_t lda, float bound_a, const float* B, int64_t ldb, float bound_b,
                           const float* bound_b_dev, float beta, float* C, int64_t ldc, bool lower_only,
                           bool company = false);

// C[M x N] = A B (A[m*lda + k], B[k*ldb + n]) likewise, for an A whose largest magnitudes are known by row (a_top)
// and a B whose are known by column (b_top) or bounded (bound_b).
//   b_tri: B (K x N, K == N) is bounded and lower triangular (zero for k < n): the reduction of an output tile
//          starts at its first column; or upper triangular (zero for k > n): it ends at its last
//   kd: with kTriLower: A diag(kd)^-1 in the place of A, kd powers of two; a_top is its
//   row_top: the rows of C raise theirs there (zeroed before), unless nullptr
//   beside: runs next to a chain of short kernels on another stream: one workgroup per compute unit
enum TriB { kTriNone = 0, kTriLower = 1, kTriUpper = 2 };
thanos_status gemm_topped(hipStream_t s, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                          const float* a_top, const float* B, int64_t ldb, const float* b_top, float bound_b,
                          float* C, int64_t ldc, TriB b_tri, const float* kd, float* row_top, bool beside);

thanos_status syrk_accumulate(hipStream_t s, float* H, int64_t b, const void* Xc,
                              thanos_dtype xdt, int64_t n_tok, int64_t ldx, float alpha);

// Damped factorisation (factor.hip).  After it the lower triangle of the reversed, padded copy
// in the workspace holds the Cholesky factor L of J D H_d D J, D diagonal with powers of two
// (U = J L^{-1} J D): factor_L() returns it and its leading dimension, factor_scale() the diagonal of D.
size_t factor_workspace_bytes(int64_t b);
// company: a product with gemm_topped(.., beside) runs at the same time on another stream.
// single_stream: no helper streams, everything on `s` in enqueue order (nothing is created).
thanos_status factor(hipStream_t s, const float* H, int64_t b, float damping, float* U,
                     float* xnorm2, void* ws, int32_t* info, bool single_stream = false,
                     bool begun = false, bool company = false);
// Its first two launches (diagonal, damped copy), which is all of it that reads H; factor(..., begun =
// true) goes on from there.  losses: the scales of the row losses as well (0.4 of 5.4 us at 1024 columns, of
// a launch that all others wait for).
thanos_status factor_begin(hipStream_t s, const float* H, int64_t b, float damping, float* xnorm2,
                           void* ws, int32_t* info, bool losses);
const float* factor_L(const void* ws, int64_t b, int64_t* ld);
const float* factor_scale(const void* ws, int64_t b);
// loss_scale() of the diagonal of H (factor_begin(.., losses = true))
const float* factor_loss_scale(const void* ws, int64_t b);
// largest magnitude of each column of U
const float* factor_umax(const void* ws, int64_t b);

// skip[i] = 1 for the n_out rows of W (c x b fp32) with the largest loss W_i H W_i^T (sweep.hip).  d: the
// factorisation's scales of the row losses for this H; nullptr: they are worked out into d_room (b floats).
thanos_status row_outliers(hipStream_t s, const float* W, const float* H, int64_t c, int64_t b,
                           long long n_out, float* Hf, float* T, float* h, const float* d, float* d_room,
                           uint8_t* skip, bool beside = false);

}  // namespace thanos
