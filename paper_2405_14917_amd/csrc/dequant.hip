// The linear layer on the stored form (App. B.2, inference): Y = X dequant(W_int)^T straight from the packed
// integers, the group-width array and the start rows that slim_pack writes, with the scales and zeros of
// slim_gptq_quantize.  W^_ij = scale[i][g] (q_ij - zero[i][g]), g = j / beta (Eq. 1).
//
// Up to 64 tokens go to the kernel of dequant_few.hip, more to that of dequant_gemm.hip; both fetch the activations 16 bytes
// at a time.  Here are the entry points and the form for activations that are not aligned for that: a thread owns one
// output row i (one column of W_int, so that the 256 threads of a workgroup read 1 KiB of consecutive words per step),
// walks a range of groups and dequantises a group's bit stream 32 elements at a time; the group's activations sit in LDS
// and are read by all threads at once (broadcast).  Several workgroups share a block of output rows by splitting the
// groups among them; their partial sums are added in a fixed order by a second kernel, so the result does not depend
// on timing.
#include <algorithm>

#include <mutex>

#include "dequant_device.h"
#include "slim_device.h"
#include "slim_internal.h"

namespace {

using namespace slimdev;
using namespace slimdq;

constexpr int DQ_THREADS = 256;
constexpr int DQ_MAX_T = 16;
// rows per workgroup and padding of an activation row that the limit of the fixed buffer is stated with (dq_splits)
constexpr int DM_ROWS = 128, DM_PAD = 8;

__device__ __forceinline__ float widen16(uint16_t h, int bf16) {
  if (bf16) return __uint_as_float((unsigned)h << 16);
  return __half2float(__ushort_as_half(h));
}

// acc[t] += (q - z) x[t][r0 + e] for the 32 elements e of one chunk of a group's bit stream; `w` holds its B words.
template <int B, int T>
__device__ __forceinline__ void chunk_dot(const uint32_t (&w)[B], float z, const float* __restrict__ xs, int beta,
                                          int r0, float (&acc)[T]) {
  auto use = [&](int e, unsigned q) {
    const float d = (float)q - z;
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = fmaf(d, xs[t * beta + r0 + e], acc[t]);
  };
  if (B == 3) {
    // 96 bits: elements 0 .. 20 lie in the first 63, element 21 starts at bit 63
    const uint64_t lo = (uint64_t)w[0] | ((uint64_t)w[1 % B] << 32);
    const uint64_t hi = ((uint64_t)w[2 % B] << 1) | (w[1 % B] >> 31);
#pragma unroll
    for (int e = 0; e < 21; ++e) use(e, (unsigned)(lo >> (3 * e)) & 7u);
#pragma unroll
    for (int e = 21; e < 32; ++e) use(e, (unsigned)(hi >> (3 * (e - 21))) & 7u);
  } else if (32 % B != 0) {
    // any other width that does not divide 32 (5: 160 bits in 5 words): an element that straddles takes its upper
    // bits from the next word; every index and shift is a compile-time constant after unrolling
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const int wi = (e * B) / 32, sh = (e * B) % 32;
      unsigned v = w[wi] >> sh;
      if (sh + B > 32) v |= w[(wi + 1) % B] << (32 - sh);
      use(e, v & ((1u << B) - 1u));
    }
  } else {
    constexpr int PER = 32 / B;            // elements per word: no element straddles two words
#pragma unroll
    for (int wi = 0; wi < B; ++wi)
#pragma unroll
      for (int e = 0; e < PER; ++e) use(wi * PER + e, (w[wi] >> (B * e)) & ((1u << B) - 1u));
  }
}

template <int B, int T>
__device__ __forceinline__ void group_dot(const DqArgs& a, int i, int base, float z, const float* xs, float (&acc)[T]) {
  const uint32_t* p = a.packed + (int64_t)base * a.ldp + i;
  for (int c = 0; c < a.beta / 32; ++c) {
    uint32_t w[B];
#pragma unroll
    for (int wi = 0; wi < B; ++wi) w[wi] = p[(int64_t)(c * B + wi) * a.ldp];
    chunk_dot<B, T>(w, z, xs, a.beta, 32 * c, acc);
  }
}

template <int T>
__global__ __launch_bounds__(DQ_THREADS) void dequant_matmul(DqArgs a) {
  extern __shared__ float xs[];                    // [T][beta]: the current group's activations
  const int tid = threadIdx.x;
  const int i = blockIdx.x * DQ_THREADS + tid;     // output row
  const int g0 = blockIdx.y * a.gper, g1 = min(a.k, g0 + a.gper);
  float y[T];
#pragma unroll
  for (int t = 0; t < T; ++t) y[t] = 0.f;
  const uint16_t* X = static_cast<const uint16_t*>(a.X);
  for (int g = g0; g < g1; ++g) {
    __syncthreads();
    for (int idx = tid; idx < T * a.beta; idx += DQ_THREADS) {
      const int t = idx / a.beta, r = idx - t * a.beta;
      xs[idx] = (t < a.t_x) ? widen16(X[(int64_t)t * a.ldx + (int64_t)g * a.beta + r], a.x_bf16) : 0.f;
    }
    __syncthreads();
    if (i < a.n) {
      const int b = (int)((a.gbits[g >> 4] >> (2 * (g & 15))) & 3u) + a.bit_base;
      const int base = a.row_off[g];
      // a group whose start rows disagree with its width (a stored form read with the wrong bit_base, or a damaged
      // one) is skipped: its words are never touched, so no read leaves the rows the stored form itself declares
      if ((a.row_off[g + 1] - base) * 32 != a.beta * b) continue;
      const float s = (float)a.scale[(int64_t)i * a.k + g], z = (float)a.zero[(int64_t)i * a.k + g];
      float acc[T];
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = 0.f;
      switch (b) {                                 // the same for the whole workgroup
        case 1: group_dot<1, T>(a, i, base, z, xs, acc); break;
        case 2: group_dot<2, T>(a, i, base, z, xs, acc); break;
        case 3: group_dot<3, T>(a, i, base, z, xs, acc); break;
        case 4: group_dot<4, T>(a, i, base, z, xs, acc); break;
        default: group_dot<5, T>(a, i, base, z, xs, acc); break;
      }
#pragma unroll
      for (int t = 0; t < T; ++t) y[t] = fmaf(s, acc[t], y[t]);
    }
  }
  if (i < a.n) {
    float* o = a.out + (int64_t)blockIdx.y * a.split_stride;
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (t < a.t_x) o[(int64_t)t * a.ldo + i] = y[t];
  }
}

// Y[t][i] = sum over the splits, in split order
__global__ __launch_bounds__(256) void dequant_reduce(const float* __restrict__ part, int splits, int64_t split_stride,
                                                      int t_x, int n, float* __restrict__ Y, int64_t ldy) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)t_x * n) return;
  const int t = (int)(idx / n), i = (int)(idx - (int64_t)t * n);
  float s = 0.f;
  for (int p = 0; p < splits; ++p) s += part[p * split_stride + (int64_t)t * n + i];
  Y[(int64_t)t * ldy + i] = s;
}

template <int T>
slim_status launch(slim_ctx* ctx, const DqArgs& a, dim3 grid, size_t smem) {
  SLIM_LAUNCH(ctx, "dequant_matmul@dequant_matmul<T>", dequant_matmul<T>, grid, dim3(DQ_THREADS), smem, a);
  return SLIM_OK;
}

// Partial sums of the group ranges for callers that must not allocate: one array per GPU, held from the moment the
// library's code is loaded on that GPU until the process ends.  Host code never uses the array's name as an
// address; the device address is asked for once per device (slim_dq_scratch_resolve) and kept.
constexpr size_t DQ_SCRATCH_FLOATS = SLIM_DEQUANT_NOALLOC_MAX_FLOATS;      // 16 MiB
static __device__ __align__(256) float scratch[DQ_SCRATCH_FLOATS];

constexpr int DQ_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[DQ_MAX_DEVICES] = {};

// Group ranges the layer is split into (and groups per range): enough workgroups per CU to hide the latency of their loads
// behind one another; fewer for a small layer, where the reduction over the ranges would cost more than the ranges gain.
// mfma: the ranges in which the limit of the fixed buffer is stated for fp16 activations.
int dq_splits(int n, int m, int beta, int t_x, int cus, bool mfma, int& gper) {
  const int k = m / beta;
  const bool small = 2 * slim_cdiv(n, DM_ROWS) < cus;
  const int gx = slim_cdiv(n, mfma ? DM_ROWS : DQ_THREADS);
  const int per_cu = small ? 2 : 8;
  const int splits_wanted = std::max(1, std::min(k, (per_cu * cus + gx - 1) / gx));
  gper = slim_cdiv(k, splits_wanted);
  if (mfma) {
    // t_x + 1 rows of a range's activations and 10 bytes per row and group in 64 KiB
    const int fit = std::max(1, (int)((64 * 1024 - 2 * (t_x + 1) * DM_PAD) / (2 * (t_x + 1) * beta + 10 * DM_ROWS)));
    gper = std::min(gper, fit);
  }
  return slim_cdiv(k, gper);
}

// What both forms of the call are refused for; nothing has been launched then.
slim_status dq_check(slim_ctx* ctx, const char* fn, const DqArgs& a, slim_dtype x_dtype, int64_t t_x, int64_t ldy,
                     bool packed_zeros) {
  SLIM_REQUIRE(ctx, a.packed && a.gbits && a.row_off && a.scale && (a.zero || packed_zeros) && a.X && a.out, "%s: null pointer", fn);
  SLIM_REQUIRE(ctx, a.n > 0 && a.m > 0 && a.beta > 0 && a.m % a.beta == 0, "%s: need n, m > 0 and beta | m", fn);
  SLIM_REQUIRE(ctx, a.beta % 32 == 0, "%s: beta must be a multiple of 32 (got %d)", fn, a.beta);
  SLIM_REQUIRE(ctx, t_x >= 1, "%s: t_x must be at least 1 (got %lld)", fn, (long long)t_x);
  SLIM_REQUIRE(ctx, a.ldp >= a.n && a.ldx >= a.m && ldy >= a.n, "%s: leading dimension too small", fn);
  if (x_dtype != SLIM_F16 && x_dtype != SLIM_BF16)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "%s: X must be F16 or BF16", fn);
  if (a.bit_base != 1 && a.bit_base != 2)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "%s: bit_base must be 1 or 2 (widths up to 5), got %d", fn, a.bit_base);
  return SLIM_OK;
}

// Where the kernel writes: Y itself with one group range, else partial sums, which go to the context's workspace (grown
// if needed) or, if `fixed` is given, to `fixed`, which holds `fixed_floats` floats (nothing is allocated then).
slim_status dq_partials(slim_ctx* ctx, const char* fn, DqArgs& a, int splits, float* fixed, size_t fixed_floats) {
  if (splits <= 1) return SLIM_OK;
  const size_t part_floats = (size_t)splits * a.t_x * a.n;
  if (fixed) {
    if (part_floats > fixed_floats)
      return slim_fail(ctx, SLIM_ERR_UNSUPPORTED,
                       "%s: this layer needs %zu floats of partial sums (%d group ranges x %d tokens x %d rows), the "
                       "fixed buffer holds %zu: fewer tokens per call, or slim_dequant_matmul", fn, part_floats,
                       splits, a.t_x, a.n, fixed_floats);
    a.out = fixed;
  } else {
    slim_status st = slim_ws_reserve(ctx, slim_ws_need_dequant(a.n, a.m, a.beta, a.t_x, ctx->num_cus));
    if (st != SLIM_OK) return st;
    a.out = static_cast<float*>(slim_ws_alloc(ctx, sizeof(float) * part_floats));
  }
  a.ldo = a.n;
  a.split_stride = (int64_t)a.t_x * a.n;
  return SLIM_OK;
}

slim_status dq_reduce(slim_ctx* ctx, const DqArgs& a, int splits, float* Y, int64_t ldy) {
  if (splits > 1)
    SLIM_LAUNCH(ctx, "dequant_reduce", dequant_reduce, dim3(slim_cdiv((int64_t)a.t_x * a.n, 256)), dim3(256), 0, a.out,
                splits, a.split_stride, a.t_x, a.n, Y, ldy);
  return SLIM_OK;
}

// Up to DQ_MAX_T tokens whose activations the matrix-core kernels cannot fetch (arguments checked).
slim_status dequant_matmul_run(slim_ctx* ctx, const char* fn, DqArgs a, int64_t ldy, float* fixed, size_t fixed_floats) {
  float* const Y = a.out;
  int T = 1;
  while (T < a.t_x) T *= 2;
  const size_t smem = sizeof(float) * (size_t)T * a.beta;
  const int splits = dq_splits(a.n, a.m, a.beta, a.t_x, std::max(1, ctx->num_cus), false, a.gper);
  slim_status st = dq_partials(ctx, fn, a, splits, fixed, fixed_floats);
  if (st != SLIM_OK) return st;
  const dim3 grid(slim_cdiv(a.n, DQ_THREADS), splits);
  switch (T) {
    case 1: st = launch<1>(ctx, a, grid, smem); break;
    case 2: st = launch<2>(ctx, a, grid, smem); break;
    case 4: st = launch<4>(ctx, a, grid, smem); break;
    case 8: st = launch<8>(ctx, a, grid, smem); break;
    default: st = launch<16>(ctx, a, grid, smem); break;
  }
  if (st != SLIM_OK) return st;
  return dq_reduce(ctx, a, splits, Y, ldy);
}

// The limit of the fixed buffer is stated for the partial sums of slices of DQ_MAX_T tokens, whichever kernel runs: a layer
// is taken or refused by its sizes, not by the kernel that a release picks.
slim_status dq_fixed_limit(slim_ctx* ctx, const char* fn, DqArgs a, int64_t t_x, float* fixed, size_t fixed_floats) {
  if (!fixed) return SLIM_OK;
  const int cus = std::max(1, ctx->num_cus);
  a.t_x = (int)std::min<int64_t>(t_x, DQ_MAX_T);
  const bool small = 2 * slim_cdiv(a.n, DM_ROWS) < cus;
  const bool mfma = !a.x_bf16 && (a.beta == 32 || a.beta == 64 || a.beta % 128 == 0) && !(small && a.t_x <= 2);
  const int splits = dq_splits(a.n, a.m, a.beta, a.t_x, cus, mfma, a.gper);
  return dq_partials(ctx, fn, a, splits, fixed, fixed_floats);
}

// Any number of tokens: up to 64 in one launch of the kernel for few tokens, more in one of the kernel for many (or, where that
// one is not built for the layer, 64 at a time); activations that are not aligned to 16 bytes DQ_MAX_T tokens at a time, one
// after the other on the context's stream.  `zp` (zero points
// in their packed form) only where slim_dq_few_takes.  Nothing is launched if the call is refused.
slim_status dequant_matmul_tokens(slim_ctx* ctx, const char* fn, const uint32_t* packed, int64_t ldp,
                                  const uint32_t* gbits, const int32_t* row_off, const double* scale,
                                  const double* zero, int n, int m, int beta, int bit_base, const void* X,
                                  slim_dtype x_dtype, int64_t t_x, int64_t ldx, float* Y, int64_t ldy, float* fixed,
                                  size_t fixed_floats, const PackedZeros* zp = nullptr, __half* hand = nullptr, int64_t ldh = 0) {
  DqArgs a;
  a.packed = packed;
  a.ldp = ldp;
  a.gbits = gbits;
  a.row_off = row_off;
  a.scale = scale;
  a.zero = zero;
  a.n = n;
  a.m = m;
  a.beta = beta;
  a.bit_base = bit_base;
  a.X = X;
  a.x_bf16 = (x_dtype == SLIM_BF16);
  a.ldx = ldx;
  a.out = Y;
  a.ldo = ldy;
  a.split_stride = 0;
  slim_status st = dq_check(ctx, fn, a, x_dtype, t_x, ldy, zp != nullptr);
  if (st != SLIM_OK) return st;
  a.k = m / beta;
  a.gper = a.k;
  // `hand` where Y has been written (the product for many tokens with one range of groups writes it itself)
  auto handed = [&](slim_status done) {
    return done == SLIM_OK && hand ? slim_round_transpose(ctx, Y, (int)t_x, n, ldy, hand, ldh) : done;
  };
  if (slim_dq_few_takes(t_x, ldp, beta, X, ldx)) {
    st = dq_fixed_limit(ctx, fn, a, t_x, fixed, fixed_floats);
    if (st != SLIM_OK) return st;
    a.t_x = (int)t_x;
    return handed(slim_dq_few_launch(ctx, a, zp));
  }
  const int cus = std::max(1, ctx->num_cus);
  if (slim_dq_gemm_takes(t_x, m, beta, X, ldx)) {
    st = dq_fixed_limit(ctx, fn, a, t_x, fixed, fixed_floats);
    if (st != SLIM_OK) return st;
    a.t_x = (int)t_x;
    const int splits = slim_dq_gemm_splits(n, m, beta, t_x, cus, a.gper);
    if (hand && splits == 1) return slim_dq_gemm_launch(ctx, a, 1, hand, ldh);
    st = dq_partials(ctx, fn, a, splits, fixed, fixed_floats);
    if (st == SLIM_OK) st = slim_dq_gemm_launch(ctx, a, splits);
    if (st == SLIM_OK) st = dq_reduce(ctx, a, splits, Y, ldy);
    return handed(st);
  }
  if (slim_dq_few_takes(1, ldp, beta, X, ldx)) {
    st = dq_fixed_limit(ctx, fn, a, t_x, fixed, fixed_floats);
    for (int64_t t0 = 0; t0 < t_x && st == SLIM_OK; t0 += DQ_FEW_TOKENS) {
      a.t_x = (int)std::min<int64_t>(DQ_FEW_TOKENS, t_x - t0);
      a.X = static_cast<const uint16_t*>(X) + t0 * ldx;
      a.out = Y + t0 * ldy;
      st = slim_dq_few_launch(ctx, a, zp);
    }
    return handed(st);
  }
  for (int64_t t0 = 0; t0 < t_x; t0 += DQ_MAX_T) {
    a.t_x = (int)std::min<int64_t>(DQ_MAX_T, t_x - t0);
    a.X = static_cast<const uint16_t*>(X) + t0 * ldx;
    a.out = Y + t0 * ldy;
    st = dequant_matmul_run(ctx, fn, a, ldy, fixed, fixed_floats);
    if (st != SLIM_OK) return st;
  }
  return handed(SLIM_OK);
}

}  // namespace

// The requirement does not change from DQ_MAX_T tokens on: a workspace that serves one such call serves every number of tokens.
size_t slim_ws_need_dequant(int n, int m, int beta, int t_x, int ncu) {
  ncu = std::max(1, ncu);
  size_t need = t_x >= DQ_MAX_T ? slim_dq_gemm_partials(n, m, beta, ncu) : 0;
  t_x = std::min(t_x, DQ_MAX_T);
  for (int mfma = 0; mfma < 2; ++mfma) {       // whichever kernel the activations' type and alignment select
    int gper = 0;
    const int splits = dq_splits(n, m, beta, t_x, ncu, mfma != 0, gper);
    if (splits > 1) need = std::max(need, slim_ws_round(sizeof(float) * (size_t)splits * t_x * n));
  }
  return need;
}

// Device address of this GPU's copy of the fixed buffer: asked for once per device, with that device current
// (slim_create calls this on the context's device), and kept for the life of the process.
slim_status slim_dq_scratch_resolve(slim_ctx* ctx) {
  if (ctx->device < 0 || ctx->device >= DQ_MAX_DEVICES)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "device ordinal %d is beyond the %d this library keeps buffers for",
                     ctx->device, DQ_MAX_DEVICES);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[ctx->device]) {
    int cur = -1;
    SLIM_HIP_TRY(ctx, hipGetDevice(&cur));
    if (cur != ctx->device) return slim_fail(ctx, SLIM_ERR_INVALID_ARG, "the context's device is not the current one");
    float* ptr = nullptr;
    SLIM_HIP_TRY(ctx, hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch)));
    if (!ptr) return slim_fail(ctx, SLIM_ERR_HIP, "hipGetSymbolAddress returned a null address");
    g_scratch_ptr[ctx->device] = ptr;
  }
  ctx->dq_scratch = g_scratch_ptr[ctx->device];
  return SLIM_OK;
}

extern "C" slim_status slim_dequant_matmul(slim_ctx* ctx, const uint32_t* packed, int64_t ldp, const uint32_t* gbits,
                                           const int32_t* row_off, const double* scale, const double* zero, int n,
                                           int m, int beta, int bit_base, const void* X, slim_dtype x_dtype, int t_x,
                                           int64_t ldx, float* Y, int64_t ldy) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  return dequant_matmul_tokens(ctx, "slim_dequant_matmul", packed, ldp, gbits, row_off, scale, zero, n, m, beta,
                               bit_base, X, x_dtype, t_x, ldx, Y, ldy, nullptr, 0);
}

extern "C" slim_status slim_dequant_matmul_handover(slim_ctx* ctx, const uint32_t* packed, int64_t ldp, const uint32_t* gbits,
                                                    const int32_t* row_off, const double* scale, const double* zero, int n,
                                                    int m, int beta, int bit_base, const void* X, slim_dtype x_dtype, int t_x,
                                                    int64_t ldx, float* Y, int64_t ldy, void* Xn, int64_t ldn) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  SLIM_REQUIRE(ctx, Xn && (reinterpret_cast<uintptr_t>(Xn) & 1u) == 0, "slim_dequant_matmul_handover: Xn null or misaligned");
  SLIM_REQUIRE(ctx, ldn >= t_x, "slim_dequant_matmul_handover: ldn < t_x");
  return dequant_matmul_tokens(ctx, "slim_dequant_matmul_handover", packed, ldp, gbits, row_off, scale, zero, n, m, beta,
                               bit_base, X, x_dtype, t_x, ldx, Y, ldy, nullptr, 0, nullptr, static_cast<__half*>(Xn), ldn);
}

extern "C" slim_status slim_dequant_matmul_noalloc(slim_ctx* ctx, const uint32_t* packed, int64_t ldp,
                                                 const uint32_t* gbits, const int32_t* row_off, const double* scale,
                                                 const double* zero, int n, int m, int beta, int bit_base,
                                                 const void* X, slim_dtype x_dtype, int t_x, int64_t ldx, float* Y,
                                                 int64_t ldy) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  if (!ctx->dq_scratch) return slim_fail(ctx, SLIM_ERR_HIP, "slim_dequant_matmul_noalloc: the fixed buffer was not resolved");
  // per-kernel event timing creates events on demand, which allocates: it is off for the length of this call
  const bool prof = ctx->prof;
  ctx->prof = false;
  const slim_status st = dequant_matmul_tokens(ctx, "slim_dequant_matmul_noalloc", packed, ldp, gbits, row_off, scale,
                                               zero, n, m, beta, bit_base, X, x_dtype, t_x, ldx, Y, ldy,
                                               ctx->dq_scratch, DQ_SCRATCH_FLOATS);
  ctx->prof = prof;
  return st;
}

// The same layer with the zero points in their packed form (App. B.2: weights AND zeros are stored as packed integers
// and the kernel dequantises both).  The kernel for up to 64 tokens takes them apart itself; for the others they are unpacked
// into the context's workspace (n x k doubles, exact: stored value / 2).  The result is bit for bit that of
// slim_dequant_matmul on the unpacked zero points.
extern "C" slim_status slim_dequant_matmul_zp(slim_ctx* ctx, const uint32_t* packed, int64_t ldp, const uint32_t* gbits,
                                              const int32_t* row_off, const double* scale, const uint32_t* zpacked,
                                              int64_t ldzp, int zbits, int n, int m, int beta, int bit_base,
                                              const void* X, slim_dtype x_dtype, int t_x, int64_t ldx, float* Y,
                                              int64_t ldy) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  SLIM_REQUIRE(ctx, zpacked != nullptr, "slim_dequant_matmul_zp: null pointer");
  SLIM_REQUIRE(ctx, n > 0 && m > 0 && beta > 0 && m % beta == 0, "slim_dequant_matmul_zp: need n, m > 0 and beta | m");
  SLIM_REQUIRE(ctx, t_x >= 1, "slim_dequant_matmul_zp: t_x must be at least 1");
  const int k = m / beta;
  if (slim_dq_few_takes(t_x, ldp, beta, X, ldx)) {
    SLIM_REQUIRE(ctx, zbits >= 2 && zbits <= 16, "slim_dequant_matmul_zp: zbits must be in 2..16 (got %d)", zbits);
    SLIM_REQUIRE(ctx, ldzp >= slim_cdiv((int64_t)n * zbits, 32), "slim_dequant_matmul_zp: ldzp too small");
    const PackedZeros z{zpacked, ldzp, zbits};
    return dequant_matmul_tokens(ctx, "slim_dequant_matmul_zp", packed, ldp, gbits, row_off, scale, nullptr, n, m, beta,
                                 bit_base, X, x_dtype, t_x, ldx, Y, ldy, nullptr, 0, &z);
  }
  const size_t need_dq = slim_ws_need_dequant(n, m, beta, t_x, std::max(1, ctx->num_cus));
  const size_t need_z = slim_ws_round(sizeof(double) * (size_t)n * k);
  slim_status st = slim_ws_reserve(ctx, need_dq + need_z);
  if (st != SLIM_OK) return st;
  // the zero points live behind the partial sums, which the product below takes from the start of the workspace
  double* zero = reinterpret_cast<double*>(ctx->ws + need_dq);
  st = slim_unpack_zeros(ctx, zpacked, ldzp, n, k, zbits, zero, k);
  if (st != SLIM_OK) return st;
  return dequant_matmul_tokens(ctx, "slim_dequant_matmul_zp", packed, ldp, gbits, row_off, scale, zero, n, m, beta,
                               bit_base, X, x_dtype, t_x, ldx, Y, ldy, nullptr, 0);
}
