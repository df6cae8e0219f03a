// a4  Salience-Determined Bit Allocation (Eq. 4; Alg. 2 SBA; App. C, App. D).
//
// The search evaluates floor(k/2)+1 allocations that differ from one another in two groups only, so the layer outputs are
// carried incrementally.  Every product with the objective's tokens is EXACT integer arithmetic on the int8 matrix cores:
//   * X_s is one integer matrix times a power of two (fp16 values are multiples of 2^-24 below 2^16), cut into signed base-256
//     digits (balanced: -128 .. 127); of every chunk of channels only the digits in use are kept (`sba_meta`), three to five
//     for activations;
//   * a fake-quantised weight is scale * (q - z) with a small integer q - z: one int8 matrix, and one scale per (row, group);
//   * W itself is cut into digits the same way (two to four for 16-bit weights).
// A chunk's products of digits are summed exactly in int32 (128 channels of 127 * 128 * 257 < 2^31 for two digits chained by a
// shift) and enter the fp64 outputs with two roundings per (row, group): fewer than the fp64 matrix cores make, which round
// after every four channels.  What is lost: a bf16 or fp32 input that spans more than 53 binary digits (largest exponent
// of the matrix against the last digit of the element) is rounded there, 2^-54 of the largest element.
//
//   sba_rank        stable ascending rank of the k group saliences (one workgroup, counting sort by comparison; NaN
//                   ranks last) -> order[]
//   sba_*_stats, sba_meta, sba_x_digits     which digits there are, and the digits of X_s in MFMA operand order
//   sba_codes       per (row, group): Eq. 1 / Eq. 2 at width N and at the one other width the group can take, as integers
//                   in operand order with their scales; the digits of W
//   sba_outputs     Y^T = W X_s and Y_0^T = W_N X_s (n x t_s, fp64)
//   kl_ref_*        once: per token the maximum M_t and log-sum-exp of the reference outputs; Y is then overwritten
//                   by P = softmax(Y) and B_t = sum_i P_i log P_i is kept
//   sba_search      all candidates in one kernel: obj[p] = sum_t [ B_t - (sum_i P_i q_i - lse(q)) ] with the reference
//                   maximum M_t as the shift of the exponentials (Y_p differs from Y by quantisation noise), then
//                   Y_{p+1} = Y_p + D_lo(g_lo) X_s(g_lo) + D_hi(g_hi) X_s(g_hi) in registers
//   sba_finalize    first minimum of obj, bit vector of p*
//
// Measured on 28672 x 8192, 2048 tokens, beside the inverse where it runs there (fp64 matrix cores -> this): outputs 32 ->
// 10.6 ms (reference 7.8, width N 2.8), search 15.2 -> 6.4 ms, widening and fake quantisation 3.4 -> 1.0 ms; 4096 x 4096:
// 3.5 -> 0.8, 1.19 -> 0.47 ms.  The fp64 products ran at 76 to 81 % of their roof.
#include <algorithm>

#include "slim_device.h"
#include "slim_internal.h"

namespace {

using namespace slimdev;

constexpr int KL_TOK = 64;     // tokens per workgroup
constexpr int KL_PART = 3;     // planes of the reference side's partials: max y, sum exp y, sum P log P

__global__ __launch_bounds__(256) void sba_rank(const double* __restrict__ sal, int k, int* __restrict__ order,
                                                int* __restrict__ rank_of) {
  for (int g = threadIdx.x; g < k; g += 256) {
    double v = sal[g];
    if (v != v) v = INFINITY;
    int rank = 0;
    for (int h = 0; h < k; ++h) {
      double u = sal[h];
      if (u != u) u = INFINITY;
      rank += (u < v || (u == v && h < g)) ? 1 : 0;
    }
    order[rank] = g;
    rank_of[g] = rank;
  }
}

// default parameters of Eq. 1 / Eq. 2 of one (row, group)
struct RtnParams {
  double delta0, z, qmax, alpha;
  bool sign;
};

__device__ __forceinline__ RtnParams rtn_params(double mn, double mx, double mean_abs, int bits, int q1_mode) {
  RtnParams p;
  p.sign = (bits == 1 && q1_mode == SLIM_Q1_SIGN);
  p.alpha = mean_abs;
  p.qmax = (double)((1 << bits) - 1);
  p.delta0 = 1.0;
  p.z = 0.0;
  if (!p.sign) {
    if (mx == mn) {
      mn = fmin(mn, 0.0);
      mx = fmax(mx, 0.0);
    }
    if (mx != mn) {
      p.delta0 = (mx - mn) / p.qmax;
      p.z = -rint(mn / p.delta0);
    }
  }
  return p;
}

// ---- reference side, once per call ----------------------------------------------------------------
// grid (ceil(ts / 64), parts): 64 tokens x 4 row lanes per workgroup; part r owns rows [r*rpp, (r+1)*rpp).
// per (part, token): max y and sum exp(y - max)
__global__ __launch_bounds__(256) void kl_ref_partial(const double* __restrict__ Y, int n, int64_t ts, int rows_per_part,
                                                      double* __restrict__ partial) {
  __shared__ double red[2][4][KL_TOK];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * KL_TOK + tx;
  const int r0 = blockIdx.y * rows_per_part;
  const int r1 = min(n, r0 + rows_per_part);
  const bool live = t < ts;
  double my = -INFINITY;
  if (live)
    for (int r = r0 + ty; r < r1; r += 4) my = fmax(my, Y[(int64_t)r * ts + t]);
  red[0][ty][tx] = my;
  __syncthreads();
  my = fmax(fmax(red[0][0][tx], red[0][1][tx]), fmax(red[0][2][tx], red[0][3][tx]));
  double zy = 0.0;
  if (live && my > -INFINITY)
    for (int r = r0 + ty; r < r1; r += 4) zy += exp(Y[(int64_t)r * ts + t] - my);
  red[1][ty][tx] = zy;
  __syncthreads();
  if (ty == 0 && live) {
    double* o = partial + (int64_t)blockIdx.y * KL_PART * ts + t;
    o[0] = my;
    o[ts] = ((red[1][0][tx] + red[1][1][tx]) + red[1][2][tx]) + red[1][3][tx];
  }
}

// one thread per token: merges the parts into tok[t] = {M_t, lse_t}
__global__ __launch_bounds__(256) void kl_ref_merge(const double* __restrict__ partial, int parts, int64_t ts,
                                                    double* __restrict__ tok) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= ts) return;
  double M = -INFINITY;
  for (int p = 0; p < parts; ++p) M = fmax(M, partial[(int64_t)p * KL_PART * ts + t]);
  double Z = 0.0;
  for (int p = 0; p < parts; ++p) {
    const double* o = partial + (int64_t)p * KL_PART * ts + t;
    Z += o[ts] * exp(o[0] - M);
  }
  tok[2 * t] = M;
  tok[2 * t + 1] = M + log(Z);
}

// Y <- P = exp(Y - lse); per (part, token) the partial sum of P log P goes to slot 2
__global__ __launch_bounds__(256) void kl_ref_softmax(double* __restrict__ Y, int n, int64_t ts, int rows_per_part,
                                                      const double* __restrict__ tok, double* __restrict__ partial) {
  __shared__ double red[4][KL_TOK];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * KL_TOK + tx;
  const int r0 = blockIdx.y * rows_per_part;
  const int r1 = min(n, r0 + rows_per_part);
  double b = 0.0;
  if (t < ts) {
    const double lse = tok[2 * t + 1];
    for (int r = r0 + ty; r < r1; r += 4) {
      const double lp = Y[(int64_t)r * ts + t] - lse;
      const double pr = exp(lp);
      Y[(int64_t)r * ts + t] = pr;
      b = fma(pr, lp, b);
    }
  }
  red[ty][tx] = b;
  __syncthreads();
  if (ty == 0 && t < ts)
    partial[((int64_t)blockIdx.y * KL_PART + 2) * ts + t] = ((red[0][tx] + red[1][tx]) + red[2][tx]) + red[3][tx];
}

// one thread per token: B_t = sum_i P_i log P_i (fixed order over the parts) into tok2[t]
__global__ __launch_bounds__(256) void kl_ref_entropy(const double* __restrict__ partial, int parts, int64_t ts,
                                                      double* __restrict__ tokB) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= ts) return;
  double b = 0.0;
  for (int p = 0; p < parts; ++p) b += partial[((int64_t)p * KL_PART + 2) * ts + t];
  tokB[t] = b;
}

// obj[p] = sum of the token-block sums of step p (fixed order); then the first minimum and its bit vector
__global__ __launch_bounds__(256) void sba_finalize(const double* __restrict__ block_sums, int nblocks,
                                                    double* __restrict__ obj, int pmax, const int* __restrict__ order,
                                                    int k, int N, const int* __restrict__ nonfinite,
                                                    uint8_t* __restrict__ bits, int* __restrict__ p_star) {
  __shared__ int best_p;
  for (int p = threadIdx.x; p <= pmax; p += 256) {
    double s = 0.0;
    for (int w = 0; w < nblocks; ++w) s += block_sums[(int64_t)p * nblocks + w];
    // (a weight or an activation that is not a number makes every candidate's objective one that is none)
    obj[p] = *nonfinite ? NAN : s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int bp = 0;
    double bv = obj[0];
    for (int p = 1; p <= pmax; ++p) {
      if (obj[p] < bv) {
        bv = obj[p];
        bp = p;
      }
    }
    best_p = bp;
    *p_star = bp;
  }
  __syncthreads();
  const int ps = best_p;
  for (int r = threadIdx.x; r < k; r += 256) {
    int b = N;
    if (r < ps) b = N - 1;
    if (r >= k - ps) b = N + 1;
    bits[order[r]] = (uint8_t)b;
  }
}

// ---- integers ---------------------------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int SI_MAXD = 7;         // digits of a value
constexpr int SI_ROWS = 256, SI_TOK = 32;   // outputs and tokens per workgroup of the products
constexpr int SE_ROWS = 128;       // outputs per workgroup of the search
constexpr int SI_CHUNK = 128;      // most channels whose products are summed in int32

// Shapes of the operands.  A group is cut into chunks of `chk` channels (32, 64 or 128, the last ones padded with zeros); an
// operand fragment is 1 KiB: 32 rows (of W) or tokens x 32 channels as the 64 lanes of v_mfma_i32_32x32x32_i8 hold them
// (lane l: row l % 32, channels 16 (l / 32) .. + 15).
struct SbaShape {
  int n, m, beta, k;
  int64_t ts;
  int chk, ks, nchg, C;            // channels per chunk, fragments per chunk, chunks per group, chunks
  int npad, RB, RT;                // rows padded to SI_ROWS, blocks of 32 rows, tiles of SI_ROWS
  int tpad, TB;                    // tokens padded to SI_TOK, blocks of 32
};

// device-side description: per chunk {lowest digit in use, digits in use}
struct SbaMeta {
  int* x;                          // 2 C: digits of X_s
  int* w;                          // 2 C: digits of W
  int* unit;                       // unit[0], unit[1]: exponents of the units of X_s and W; unit[2]: non-finite inputs seen
  int* rest_n;                     // k: some row of the group has a zero outside int8 (width N)
  int* rest_o;                     // k: the same at the other width
  unsigned* xmax;                  // C largest |x| as float bits, C smallest exponent of a last digit (as int); then W's
  int* xlsb;
  unsigned* wmax;
  int* wlsb;
};

template <typename T>
__device__ __forceinline__ unsigned float_bits(T v);
template <>
__device__ __forceinline__ unsigned float_bits<__half>(__half v) { return __float_as_uint(__half2float(v)); }
template <>
__device__ __forceinline__ unsigned float_bits<__hip_bfloat16>(__hip_bfloat16 v) {
  return (unsigned)*reinterpret_cast<const unsigned short*>(&v) << 16;
}
template <>
__device__ __forceinline__ unsigned float_bits<float>(float v) { return __float_as_uint(v); }

// |v| = mant * 2^e0 of a finite float
__device__ __forceinline__ void split_float(unsigned bits, unsigned& mant, int& e0) {
  const int e = (int)((bits >> 23) & 255u);
  mant = (bits & 0x7fffffu) | (e ? 0x800000u : 0u);
  e0 = (e ? e : 1) - 150;
}
// v / 2^unit as an integer (rounded where v has digits below the unit); 0 for what is not finite
__device__ __forceinline__ int64_t fixed_point(unsigned bits, int unit) {
  unsigned mant;
  int e0;
  split_float(bits, mant, e0);
  if (((bits >> 23) & 255u) == 255u) mant = 0;
  const int sh = e0 - unit;
  uint64_t v;
  if (sh >= 0)
    v = (uint64_t)mant << min(sh, 40);
  else
    v = (sh > -32) ? ((uint64_t)mant + (1ull << (-sh - 1))) >> (-sh) : 0ull;
  return (bits >> 31) ? -(int64_t)v : (int64_t)v;
}
// the byte lanes of v + sum_i 128 * 256^i are the balanced digits plus 128
__device__ __forceinline__ uint64_t digit_bytes(int64_t v) { return ((uint64_t)v + 0x0080808080808080ull) ^ 0x8080808080808080ull; }

__device__ __forceinline__ void stat(unsigned bits, unsigned& mx, int& lsb, int& bad) {
  bits &= 0x7fffffffu;
  if (bits >= 0x7f800000u) {
    bad = 1;
    return;
  }
  if (bits == 0) return;
  unsigned mant;
  int e0;
  split_float(bits, mant, e0);
  mx = max(mx, bits);
  lsb = min(lsb, e0 + __builtin_ctz(mant));
}

__global__ __launch_bounds__(256) void sba_clear(SbaMeta mt, int C, int k) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < C) {
    mt.xmax[i] = mt.wmax[i] = 0u;
    mt.xlsb[i] = mt.wlsb[i] = INT_MAX;
  }
  if (i < k) mt.rest_n[i] = mt.rest_o[i] = 0;
  if (i == 0) mt.unit[2] = 0;
}

// first channel and number of channels of a chunk
__device__ __forceinline__ int chunk_begin(const SbaShape& s, int c, int& len) {
  const int g = c / s.nchg, j0 = (c - g * s.nchg) * s.chk;
  len = min(s.chk, s.beta - j0);
  return g * s.beta + j0;
}

// grid (C, splits): largest magnitude and last digit of the chunk's rows of X_s
template <typename T>
__global__ __launch_bounds__(256) void sba_x_stats(const T* __restrict__ X, int64_t ldx, SbaShape s, SbaMeta mt) {
  int len;
  const int ch0 = chunk_begin(s, blockIdx.x, len);
  unsigned mx = 0;
  int lsb = INT_MAX, bad = 0;
  const int64_t quads = s.ts / 4;
  for (int64_t q = (int64_t)blockIdx.y * 256 + threadIdx.x; q < quads; q += (int64_t)gridDim.y * 256)
    for (int r = 0; r < len; ++r) {
      const uint2 raw = *reinterpret_cast<const uint2*>(X + (int64_t)(ch0 + r) * ldx + 4 * q);
      const T* v = reinterpret_cast<const T*>(&raw);
#pragma unroll
      for (int i = 0; i < 4; ++i) stat(float_bits<T>(v[i]), mx, lsb, bad);
    }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    mx = max(mx, (unsigned)__shfl_xor((int)mx, d, WAVE));
    lsb = min(lsb, __shfl_xor(lsb, d, WAVE));
  }
  if (bad) atomicOr(&mt.unit[2], 1);
  if ((threadIdx.x & 63) == 0 && mx) {
    atomicMax(&mt.xmax[blockIdx.x], mx);
    atomicMin(&mt.xlsb[blockIdx.x], lsb);
  }
}

// grid (ceil(m / 1024), splits): the same for the chunk's columns of W; a thread owns four columns
template <typename T>
__global__ __launch_bounds__(256) void sba_w_stats(const T* __restrict__ W, int64_t ldw, SbaShape s, SbaMeta mt) {
  __shared__ unsigned lmax[264];
  __shared__ int llsb[264];
  for (int i = threadIdx.x; i < 264; i += 256) {
    lmax[i] = 0u;
    llsb[i] = INT_MAX;
  }
  __syncthreads();
  auto chunk_of = [&](int ch) { const int g = ch / s.beta; return g * s.nchg + (ch - g * s.beta) / s.chk; };
  const int c0 = chunk_of(blockIdx.x * 1024);
  const int ch = blockIdx.x * 1024 + threadIdx.x * 4;
  if (ch < s.m) {
    unsigned mx = 0;
    int lsb = INT_MAX, bad = 0;
    for (int r = blockIdx.y; r < s.n; r += gridDim.y) {
      T v[4];
      if constexpr (sizeof(T) == 2)
        *reinterpret_cast<uint2*>(v) = *reinterpret_cast<const uint2*>(W + (int64_t)r * ldw + ch);
      else
        *reinterpret_cast<uint4*>(v) = *reinterpret_cast<const uint4*>(W + (int64_t)r * ldw + ch);
#pragma unroll
      for (int i = 0; i < 4; ++i) stat(float_bits<T>(v[i]), mx, lsb, bad);
    }
    const int c = chunk_of(ch) - c0;
    atomicMax(&lmax[c], mx);
    atomicMin(&llsb[c], lsb);
    if (bad) atomicOr(&mt.unit[2], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 264; i += 256)
    if (lmax[i]) {
      atomicMax(&mt.wmax[c0 + i], lmax[i]);
      atomicMin(&mt.wlsb[c0 + i], llsb[i]);
    }
}

// Units and digits in use: block 0 for X_s, block 1 for W.  The unit is the last digit of all values, but no more than 53
// digits below the largest one; a chunk keeps the digits between its own last one and its own largest value.
__global__ __launch_bounds__(256) void sba_meta(SbaMeta mt, int C) {
  __shared__ unsigned smx[256];
  __shared__ int slsb[256];
  const unsigned* cmax = blockIdx.x ? mt.wmax : mt.xmax;
  const int* clsb = blockIdx.x ? mt.wlsb : mt.xlsb;
  int* out = blockIdx.x ? mt.w : mt.x;
  unsigned mx = 0;
  int lsb = INT_MAX;
  for (int c = threadIdx.x; c < C; c += 256) {
    mx = max(mx, cmax[c]);
    lsb = min(lsb, clsb[c]);
  }
  smx[threadIdx.x] = mx;
  slsb[threadIdx.x] = lsb;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      smx[threadIdx.x] = max(smx[threadIdx.x], smx[threadIdx.x + st]);
      slsb[threadIdx.x] = min(slsb[threadIdx.x], slsb[threadIdx.x + st]);
    }
    __syncthreads();
  }
  mx = smx[0];
  lsb = slsb[0];
  unsigned mant;
  int e0, unit = 0;
  if (mx) {
    split_float(mx, mant, e0);
    unit = max(lsb, e0 + (31 - __builtin_clz(mant)) - 53);
  }
  if (threadIdx.x == 0) mt.unit[blockIdx.x] = unit;
  for (int c = threadIdx.x; c < C; c += 256) {
    int lo = 0, hi = 0;
    if (cmax[c]) {
      const uint64_t v = (uint64_t)fixed_point(cmax[c], unit);
      lo = max(0, clsb[c] - unit) / 8;
      uint64_t lim = 0;                                  // largest value of hi balanced digits
      while (lim < v) {
        lim = lim * 256 + 127;
        ++hi;
      }
      hi = max(hi, lo);
    }
    out[2 * c] = lo;
    out[2 * c + 1] = hi - lo;
  }
}

// grid (ceil(TB / 4), k): a wavefront cuts 32 tokens of one group into digits and sums its channels per token
template <typename T>
__global__ __launch_bounds__(256) void sba_x_digits(const T* __restrict__ X, int64_t ldx, SbaShape s, SbaMeta mt,
                                                    char* __restrict__ Xd, double* __restrict__ SX) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int tb = blockIdx.x * 4 + (threadIdx.x >> 6), g = blockIdx.y;
  if (tb >= s.TB) return;
  const int unit = mt.unit[0];
  const int64_t t = (int64_t)tb * 32 + l32;
  int64_t sum = 0;
  for (int cc = 0; cc < s.nchg; ++cc) {
    const int c = g * s.nchg + cc, lo = mt.x[2 * c], nd = mt.x[2 * c + 1];
    char* dst = Xd + ((int64_t)c * s.TB + tb) * SI_MAXD * s.ks * 1024 + lane * 16;
    for (int f = 0; f < s.ks; ++f) {
      const int j0 = cc * s.chk + f * 32 + h * 16;
      uint64_t u[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        int64_t v = 0;
        if (j0 + i < s.beta && t < s.ts) v = fixed_point(float_bits<T>(X[(int64_t)(g * s.beta + j0 + i) * ldx + t]), unit);
        sum += v;
        u[i] = digit_bytes(v) >> (8 * lo);
      }
      for (int d = 0; d < nd; ++d) {
        unsigned w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          w[q] = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            w[q] |= ((unsigned)u[4 * q + i] & 255u) << (8 * i);
            u[4 * q + i] >>= 8;
          }
        }
        *reinterpret_cast<uint4*>(dst + ((int64_t)d * s.ks + f) * 1024) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  }
  // (a sum of up to 512 channels of 54 bits may not fit 53 bits: one rounding)
  const double other = __shfl_xor((double)sum, 32, WAVE);
  if (h == 0) SX[(int64_t)g * s.tpad + t] = (double)sum + other;
}

__device__ __forceinline__ double row_sum(double v) {
  v += dpp_f64<DPP_XOR1>(v);
  v += dpp_f64<DPP_XOR2>(v);
  v += dpp_f64<DPP_HALF_MIRROR>(v);
  return v + dpp_f64<DPP_MIRROR>(v);
}
template <typename OP>
__device__ __forceinline__ double row_reduce(double v) {
  v = OP::f(v, dpp_f64<DPP_XOR1>(v));
  v = OP::f(v, dpp_f64<DPP_XOR2>(v));
  v = OP::f(v, dpp_f64<DPP_HALF_MIRROR>(v));
  return OP::f(v, dpp_f64<DPP_MIRROR>(v));
}

// The integers of one quantiser: codes minus z0, the part of the zero point for which they fit int8, and what is left of it.
struct IntQuant {
  RtnParams p;
  double inv, z0;
};
__device__ __forceinline__ IntQuant int_quant(double mn, double mx, double mean_abs, int bits, int q1_mode) {
  IntQuant q;
  q.p = rtn_params(mn, mx, mean_abs, bits, q1_mode);
  q.inv = 1.0 / q.p.delta0;
  q.z0 = fmin(fmax(q.p.z, q.p.qmax - 127.0), 128.0);       // codes 0 .. qmax minus z0 lie in -128 .. 127
  return q;
}
__device__ __forceinline__ int int_code(const IntQuant& q, double w) {
  if (q.p.sign) return (w >= 0.0) ? 1 : -1;
  double r = w * q.inv;
  double c = rint(r);
  // the product and the quotient differ by less than 1e-15 of it: only next to a tie can they round apart
  if (fabs(fabs(r - c) - 0.5) <= 1e-9 * (1.0 + fabs(r))) c = rint(w / q.p.delta0);
  return (int)(fmin(fmax(c + q.p.z, 0.0), q.p.qmax) - q.z0);
}
__device__ __forceinline__ double int_scale(const IntQuant& q) { return q.p.sign ? q.p.alpha : q.p.delta0; }

struct CodesArgs {
  SbaShape s;
  SbaMeta mt;
  int64_t ldw;
  int N, q1_mode, pmax;
  const int* rank_of;              // (width other than N)
  char* Q;                         // codes in operand order
  double* S;                       // k x npad scales
  double* Rz;                      // k x npad: the part of the zero that the codes do not hold, times the scale
  int* rest;                       // k
  char* Wd;                        // digits of W, or nullptr
};

// grid (npad / 16, y): 16 lanes per row, 16 rows per workgroup, groups blockIdx.y, blockIdx.y + gridDim.y, ...
template <typename T, bool OTHER>
__global__ __launch_bounds__(256) void sba_codes(const T* __restrict__ W, CodesArgs a) {
  const SbaShape& s = a.s;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4);
  const int rb = row >> 5, r32 = row & 31;
  const bool live = row < s.n;
  const int64_t plane = (int64_t)s.npad * s.C * s.chk;
  const int wunit = OTHER ? 0 : a.mt.unit[1];
  for (int g = blockIdx.y; g < s.k; g += gridDim.y) {
    int bits = a.N;
    if (OTHER) {
      const int pos = a.rank_of[g];
      if (pos >= a.pmax && pos < s.k - a.pmax) continue;          // a middle group is never changed
      bits = pos < a.pmax ? a.N - 1 : a.N + 1;
    }
    const T* w = W + (int64_t)min(row, s.n - 1) * a.ldw + (int64_t)g * s.beta;
    double mn = INFINITY, mx = -INFINITY, sabs = 0.0;
    for (int j = l16 * 4; j < s.beta; j += 64) {
      double v[4];
      load4<T>(w + j, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mn = fmin(mn, v[i]);
        mx = fmax(mx, v[i]);
        sabs += fabs(v[i]);
      }
    }
    mn = row_reduce<OpMin>(mn);
    mx = row_reduce<OpMax>(mx);
    sabs = row_sum(sabs) / (double)s.beta;
    const IntQuant q = int_quant(mn, mx, sabs, bits, a.q1_mode);
    const double rest = q.p.sign ? 0.0 : q.p.z - q.z0;
    if (l16 == 0) {
      a.S[(int64_t)g * s.npad + row] = live ? int_scale(q) : 0.0;
      a.Rz[(int64_t)g * s.npad + row] = live ? int_scale(q) * rest : 0.0;
      if (live && rest != 0.0) atomicOr(&a.rest[g], 1);
    }
    for (int j = l16 * 4; j < s.nchg * s.chk; j += 64) {
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      const bool in = live && j < s.beta;
      if (in) load4<T>(w + j, v);
      const int cc = j / s.chk, jj = j - cc * s.chk, c = g * s.nchg + cc;
      const int64_t dst = (((int64_t)rb * s.C + c) * s.ks + (jj >> 5)) * 1024 + ((jj >> 4) & 1) * 512 + r32 * 16 + (jj & 15);
      unsigned word = 0;
      if (in) {
#pragma unroll
        for (int i = 0; i < 4; ++i) word |= ((unsigned)int_code(q, v[i]) & 255u) << (8 * i);
      }
      *reinterpret_cast<unsigned*>(a.Q + dst) = word;
      if (!OTHER) {
        const int lo = a.mt.w[2 * c], nd = a.mt.w[2 * c + 1];
        uint64_t u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = digit_bytes(fixed_point(__float_as_uint((float)v[i]), wunit)) >> (8 * lo);
        for (int d = 0; d < nd; ++d) {
          word = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            word |= ((unsigned)u[i] & 255u) << (8 * i);
            u[i] >>= 8;
          }
          *reinterpret_cast<unsigned*>(a.Wd + d * plane + dst) = word;
        }
      }
    }
  }
}

// ---- products with the digits of X_s ----------------------------------------------------------------------------
// A workgroup has 256 outputs x 32 tokens.  The tokens are the rows of the first MFMA operand, so a lane owns one output
// per 32 x 32 tile (its scale is a lane constant) and 16 tokens.  The digits of X_s go to LDS directly, up to four of one
// chunk at a time (a stage: two pairs of digits, each summed in int32), the next stage's while the current one is
// multiplied; the codes go from memory to registers, where they serve all digits of the stage, and are asked for again as
// soon as the last MFMA that needs the old ones has been issued.
//
// R MFMA tiles of 32 outputs per wavefront.  What bounds these kernels is the vector work behind the MFMAs (a shift, a
// conversion and an fma per output and pair of digits, and the exponentials of the search), and a wavefront by itself
// issues only every other slot: the products keep three wavefronts per SIMD (two tiles each, which share the operand
// reads from LDS), and so does the search (one tile each, because it also holds the reference, and two sets of codes: with
// one set, asked for half a stage ahead, and four wavefronts per SIMD, half of the time went by waiting for codes, 6.9
// against 6.4 ms on 28672 x 8192).
constexpr int SI_STAGE_D = 4;      // digits per stage
constexpr int SI_TAB = 1024;       // stages whose description is kept in LDS

template <int KS, int R>
struct Tile {
  static constexpr int STAGE = SI_STAGE_D * KS * 1024;
  v4i w[R][KS];
  double s[R];

  // q, S: the same for the wavefront; rstride: bytes between blocks of 32 rows
  __device__ __forceinline__ void load_codes(const char* q, int64_t rstride, unsigned lane16) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int f = 0; f < KS; ++f) w[r][f] = *reinterpret_cast<const v4i*>(q + (int64_t)r * rstride + f * 1024 + lane16);
  }
  __device__ __forceinline__ void load_scales(const double* S, unsigned l32) {
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = (S + 32 * r)[l32];
  }

  // acc (+)= sum over the chunk of digit d times the codes
  template <bool FIRST>
  __device__ __forceinline__ void digit(const char* x, int d, v16i (&acc)[R]) const {
    v4i f[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i) f[i] = *reinterpret_cast<const v4i*>(x + (d * KS + i) * 1024);
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v16i c = acc[r];
        if (FIRST && i == 0) {
#pragma unroll
          for (int v = 0; v < 16; ++v) c[v] = 0;
        }
        acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f[i], w[r][i], c, 0, 0, 0);
      }
  }
  // acc = sum over the chunk of (256 X_{2p+1} + X_{2p}) * codes; `two`: digit 2 p + 1 is in use
  __device__ __forceinline__ void pair(const char* x, int p, bool two, v16i (&acc)[R]) const {
    if (two) {
      digit<true>(x, 2 * p + 1, acc);
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] <<= 8;
      digit<false>(x, 2 * p, acc);
    } else {
      digit<true>(x, 2 * p, acc);
    }
  }
};

template <int R>
__device__ __forceinline__ void add_scaled(double (&y)[R][16], const v16i (&acc)[R], const double (&s)[R], int e) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const double f = ldexp(s[r], e);
#pragma unroll
    for (int v = 0; v < 16; ++v) y[r][v] = fma(f, (double)acc[r][v], y[r][v]);
  }
}

__device__ __forceinline__ void lds_load16(unsigned lds_addr, unsigned voff, const char* gbase) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(gbase) : "m0");
#else
  (void)lds_addr, (void)voff, (void)gbase;
#endif
}

// A stage in one word: chunk, lowest digit (absolute), digits (at most SI_STAGE_D), and whether it is the chunk's first.
__device__ __forceinline__ int stage_word(int c, int lo, int nd, int first) { return (c << 8) | (first << 7) | (nd << 4) | lo; }
__device__ __forceinline__ int stage_chunk(int w) { return w >> 8; }
__device__ __forceinline__ int stage_nd(int w) { return (w >> 4) & 7; }
__device__ __forceinline__ int stage_lo(int w) { return w & 15; }
__device__ __forceinline__ bool stage_first(int w) { return (w >> 7) & 1; }
// The digits of a stage for token block tb -> LDS (1 KiB per load, the loads dealt to the wavefronts)
template <int KS, int NW>
__device__ __forceinline__ void stage_digits(const char* Xd, const SbaShape& s, int word, int base_lo, int tb,
                                             unsigned lds, int wave, int lane) {
  const char* src = Xd + (((int64_t)stage_chunk(word) * s.TB + tb) * SI_MAXD + (stage_lo(word) - base_lo)) * KS * 1024;
  const int cnt = stage_nd(word) * KS;
  for (int i = wave; i < cnt; i += NW) lds_load16(lds + i * 1024, lane * 16, src + i * 1024);
}

// Output tiles in bands of eight row tiles, the rows of a band fastest; XCD x (id mod 8) has the x-th run of consecutive
// tiles: what it works on at a time is a patch of 8 x 8 tiles that shares codes and digits in its L2.
__device__ __forceinline__ void tile_of(int id, int RT, int TB, int& rt, int& tb) {
  const int total = RT * TB, per = total / 8, rest = total % 8, x = id % 8;
  const int i = x * per + min(x, rest) + id / 8;
  const int band = i / (8 * TB), in = i - band * 8 * TB, hb = min(8, RT - band * 8);
  rt = band * 8 + in % hb;
  tb = in / hb;
}

struct OutArgs {
  SbaShape s;
  SbaMeta mt;
  const char* Xd;
  const double* SX;
  const char* Q;                   // codes (width N), or digits of W with planes `plane` bytes apart
  int64_t plane;
  const double* S;
  const double* Rz;
  double* Y;                       // n x ts
};

// REF: Y = W X_s from the digits of W; else Y = W_N X_s
template <int KS, bool REF>
__global__ __launch_bounds__(256, 3) void sba_outputs(OutArgs a) {
  constexpr int R = 2, NW = 4;
  using TL = Tile<KS, R>;
  extern __shared__ __align__(16) char si_smem[];
  const SbaShape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  int rt, tb;
  tile_of(blockIdx.x, s.RT, s.TB, rt, tb);
  const int row0 = rt * SI_ROWS + wave * 64;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)si_smem));
  const int64_t rstride = (int64_t)s.C * KS * 1024;
  const char* q0 = a.Q + (int64_t)(row0 >> 5) * rstride;
  const unsigned lane16 = lane * 16;
  // the chunks' digits (X_s: bits 0 .. 7 lowest digit and count, W: bits 8 .. 15) in LDS
  int* tab = reinterpret_cast<int*>(si_smem + 2 * TL::STAGE);
  auto describe = [&](int c) { return a.mt.x[2 * c] | (a.mt.x[2 * c + 1] << 4) | (a.mt.w[2 * c] << 8) | (a.mt.w[2 * c + 1] << 12); };
  for (int c = tid; c < min(s.C, SI_TAB); c += 256) tab[c] = describe(c);
  const int unit = __builtin_amdgcn_readfirstlane(a.mt.unit[0] + (REF ? a.mt.unit[1] : 0));
  __syncthreads();
  auto chunk_info = [&](int c) { return __builtin_amdgcn_readfirstlane(c < SI_TAB ? tab[c] : describe(c)); };

  double y[R][16];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < 16; ++v) y[r][v] = 0.0;
  TL tl;
  auto load_first = [&](int c) {                // the first (or only) set of chunk c
    tl.load_codes(q0 + (int64_t)c * KS * 1024, rstride, lane16);
    if (!REF) {
      tl.load_scales(a.S + (int64_t)(c / s.nchg) * s.npad + row0, l32);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) tl.s[r] = 1.0;
    }
  };
  auto first_stage = [&](int c, int info) { return stage_word(c, info & 15, min(SI_STAGE_D, (info >> 4) & 15), 1); };
  int info = chunk_info(0), word = first_stage(0, info), buf = 0;
  stage_digits<KS, NW>(a.Xd, s, word, info & 15, tb, lds0, wave, lane);
  load_first(0);
  for (;;) {
    const int c = stage_chunk(word), lo = stage_lo(word), nd = stage_nd(word);
    const int left = (info & 15) + ((info >> 4) & 15) - lo - nd;            // digits of the chunk behind this stage
    const bool done = left <= 0 && c + 1 == s.C;
    const int next_info = left > 0 ? info : chunk_info(min(c + 1, s.C - 1));
    const int next = left > 0 ? stage_word(c, lo + nd, min(SI_STAGE_D, left), 0) : first_stage(min(c + 1, s.C - 1), next_info);
    const int sets = REF ? (info >> 12) & 15 : 1, wlo = (info >> 8) & 15;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!done) stage_digits<KS, NW>(a.Xd, s, next, next_info & 15, tb, lds0 + (buf ^ 1) * TL::STAGE, wave, lane);
    const char* x = si_smem + buf * TL::STAGE + lane * 16;
    double sc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sc[r] = tl.s[r];
    if (sets == 0 || nd == 0) load_first(stage_chunk(next));                // a chunk of zeros
    for (int j = 0; j < sets; ++j) {
      for (int p = (nd - 1) >> 1; p >= 0; --p) {
        v16i acc[R];
        tl.pair(x, p, 2 * p + 1 < nd, acc);
        if (p == 0) {
          if (j + 1 < sets)
            tl.load_codes(q0 + (j + 1) * a.plane + (int64_t)c * KS * 1024, rstride, lane16);
          else
            load_first(stage_chunk(next));
        }
        add_scaled<R>(y, acc, sc, unit + 8 * (lo + 2 * p) + (REF ? 8 * (wlo + j) : 0));
      }
    }
    const int g = c / s.nchg;
    if (!REF && stage_first(word) && c == g * s.nchg && a.mt.rest_n[g]) {
      // zeros outside int8: what the codes do not hold times the sum of the group's activations
      const double* Rz = a.Rz + (int64_t)g * s.npad + row0 + l32;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const double sx = ldexp(a.SX[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)], unit);
#pragma unroll
        for (int r = 0; r < R; ++r) y[r][v] = fma(-Rz[32 * r], sx, y[r][v]);
      }
    }
    if (done) break;
    word = next;
    info = next_info;
    buf ^= 1;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int row = row0 + 32 * r + l32;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t t = (int64_t)tb * 32 + 8 * q + 4 * h;
      if (row < s.n && t < s.ts) {
        double* o = a.Y + (int64_t)row * s.ts + t;
        *reinterpret_cast<double2*>(o) = make_double2(y[r][4 * q], y[r][4 * q + 1]);
        *reinterpret_cast<double2*>(o + 2) = make_double2(y[r][4 * q + 2], y[r][4 * q + 3]);
      }
    }
  }
}

// exp in fp64: Cody-Waite reduction to |r| <= ln 2 / 2, Taylor polynomial to r^13 (remainder below 4e-18), scaling.  The
// coefficients stay in scalar registers (an instruction takes one), which the library's form does not.
__device__ __forceinline__ double exp_f64(double x) {
  auto step = [](double p, double r, double c) {
#if defined(__HIP_DEVICE_COMPILE__)
    double o;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(o) : "v"(p), "v"(r), "s"(c));
    return o;
#else
    return fma(p, r, c);
#endif
  };
  const double k = rint(x * 1.4426950408889634074);
  double r = fma(k, -6.93147180369123816490e-01, x);
  r = fma(k, -1.90821492927058770002e-10, r);
  double p = 1.0 / 6227020800.0;
  p = step(p, r, 1.0 / 479001600.0);
  p = step(p, r, 1.0 / 39916800.0);
  p = step(p, r, 1.0 / 3628800.0);
  p = step(p, r, 1.0 / 362880.0);
  p = step(p, r, 1.0 / 40320.0);
  p = step(p, r, 1.0 / 5040.0);
  p = step(p, r, 1.0 / 720.0);
  p = step(p, r, 1.0 / 120.0);
  p = step(p, r, 1.0 / 24.0);
  p = step(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, (int)k);
}

// Sum of value(i), i = 0 .. 15, over the 32 lanes of a half wavefront: lane l (and its neighbour) is left with the sum for
// i = bits 4, 3, 2, 1 of l, most significant first.  A lane halves the list it is responsible for in every step, so 16 sums
// take 15 + 1 exchanges and not 16 x 5.
template <typename F>
__device__ __forceinline__ double sum_scatter16(F value, int lane) {
  double a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    // after the swap one register holds v[i] of both rows of 16 lanes for the even row, v[i + 8] of both for the odd row
    const double u = value(i), v = value(i + 8);
    auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(u), __double2loint(v), false, false);
    auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(u), __double2hiint(v), false, false);
    a[i] = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    __builtin_amdgcn_sched_barrier(0);         // (one pair at a time: the values of all of them at once would spill)
  }
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = b3 ? a[i + 4] : a[i], give = b3 ? a[i] : a[i + 4];
    a[i] = keep + dpp_f64<DPP_MIRROR>(give);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = b2 ? a[i + 2] : a[i], give = b2 ? a[i] : a[i + 2];
    a[i] = keep + dpp_f64<DPP_HALF_MIRROR>(give);
  }
  const double keep = b1 ? a[1] : a[0], give = b1 ? a[0] : a[1];
  const double r = keep + dpp_f64<DPP_XOR2>(give);
  return r + dpp_f64<DPP_XOR1>(r);
}

struct SearchArgs {
  SbaShape s;
  SbaMeta mt;
  const char* Xd;
  const double* SX;
  const char *Qn, *Qo;
  const double *Sn, *So, *Rn, *Ro;
  const double* Yc;                // n x ts outputs of the all-N-bit weights
  const double* R;                 // n x ts reference: P = softmax(Y) (KL) or Y (squared error)
  const double* tok;               // per token {max, log-sum-exp} of the reference (KL)
  const int* order;
  double* part;                    // [candidate][tile of SE_ROWS rows][tpad]: sums of exp(q - M)
  double* lin;                     // [candidate][tile of SE_ROWS rows][TB]: sums of P (q - M), or of squared errors
  int pmax;
};

// The whole search in one kernel: a wavefront keeps its 32 x 32 outputs of the current candidate and the reference in
// registers from the first candidate to the last; per candidate it adds its terms of the objective to the candidate's
// partials (sum exp(q - M) per token; sum P (q - M), or the squared error, over all its outputs) and applies the two changed
// groups (new integers times new scale minus old integers times old scale).  The next set of codes is on its way while
// one is multiplied.
template <int KS, int OBJ>
__global__ __launch_bounds__(256, 3) void sba_search(SearchArgs a) {
  constexpr int NW = 4;
  using TL = Tile<KS, 1>;
  extern __shared__ __align__(16) char si_smem[];
  const SbaShape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  int rt, tb;
  tile_of(blockIdx.x, s.npad / SE_ROWS, s.TB, rt, tb);
  const int row0 = rt * SE_ROWS + wave * 32;
  double* red = reinterpret_cast<double*>(si_smem + 2 * TL::STAGE);           // [4 wavefronts][33]
  int* tab = reinterpret_cast<int*>(red + NW * 34);                           // the changed groups' chunks in search order
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)si_smem));
  const int64_t rowq = (int64_t)(row0 >> 5) * s.C * KS * 1024;
  const unsigned lane16 = lane * 16;
  // chunk i of the search (of candidate i / per): (chunk << 8) | (digits << 4) | lowest digit
  const int per = 2 * s.nchg, chunks = a.pmax * per;
  auto describe = [&](int i) {
    const int p = i / per, j = i - p * per, hi = j >= s.nchg;
    const int c = a.order[hi ? s.k - 1 - p : p] * s.nchg + (j - hi * s.nchg);
    return (c << 8) | (a.mt.x[2 * c + 1] << 4) | a.mt.x[2 * c];
  };
  for (int i = tid; i < min(chunks, SI_TAB); i += 256) tab[i] = describe(i);
  const int unit = __builtin_amdgcn_readfirstlane(a.mt.unit[0]);
  __syncthreads();
  auto chunk_info = [&](int i) { return __builtin_amdgcn_readfirstlane(i < SI_TAB ? tab[i] : describe(i)); };

  double y[1][16], ref[16];
  {
    const int row = row0 + l32;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t t = (int64_t)tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
      const bool in = row < s.n && t < s.ts;
      // outside the matrix: exp(-1e4) = 0 with a reference of 0 (KL), 0 against 0 (squared error)
      y[0][v] = in ? a.Yc[(int64_t)row * s.ts + t] - (OBJ == SLIM_OBJ_KL ? a.tok[2 * t] : 0.0) : (OBJ == SLIM_OBJ_KL ? -1e4 : 0.0);
      ref[v] = in ? a.R[(int64_t)row * s.ts + t] : 0.0;
    }
  }
  TL tl[2];                                       // [0]: integers at the new width, [1]: at width N
  auto load_set = [&](TL& t, int chunk, bool old) {
    t.load_codes((old ? a.Qn : a.Qo) + rowq + (int64_t)chunk * KS * 1024, 0, lane16);
    t.load_scales((old ? a.Sn : a.So) + (int64_t)(chunk / s.nchg) * s.npad + row0, l32);
  };
  auto first_stage = [&](int info) { return stage_word(info >> 8, info & 15, min(SI_STAGE_D, (info >> 4) & 15), 1); };
  int i = 0, info = 0, word = 0, buf = 0;
  if (chunks > 0) {
    info = chunk_info(0);
    word = first_stage(info);
    stage_digits<KS, NW>(a.Xd, s, word, info & 15, tb, lds0, wave, lane);
    load_set(tl[0], stage_chunk(word), false);
  }
  for (int p = 0;; ++p) {
    {
      double q = 0.0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const double d = ref[v] - y[0][v];
        q = (OBJ == SLIM_OBJ_KL) ? fma(ref[v], y[0][v], q) : fma(d, d, q);
      }
      q = wave_sum(q);
      int ln = lane;
      asm volatile("" : "+v"(ln));                // (formed again for every candidate: kept, these would cost registers)
      if (ln == 0) red[wave * 34 + 32] = q;
      if (OBJ == SLIM_OBJ_KL) {
        const double z = sum_scatter16([&](int v) { return exp_f64(y[0][v]); }, ln);
        const int idx = ((ln >> 4) & 1) * 8 + ((ln >> 3) & 1) * 4 + ((ln >> 2) & 1) * 2 + ((ln >> 1) & 1);
        if (!(ln & 1)) red[wave * 34 + 8 * (idx >> 2) + 4 * (ln >> 5) + (idx & 3)] = z;
      }
    }
    __syncthreads();
    if (tid <= 32) {
      const double sum = (red[tid] + red[34 + tid]) + (red[68 + tid] + red[102 + tid]);
      const int64_t tile = (int64_t)p * (s.npad / SE_ROWS) + rt;
      if (tid == 32)
        a.lin[tile * s.TB + tb] = sum;
      else if (OBJ == SLIM_OBJ_KL)
        a.part[tile * s.tpad + tb * 32 + tid] = sum;
    }
    if (p == a.pmax) break;
    for (int j = 0; j < per;) {
      const int c = stage_chunk(word), lo = stage_lo(word), nd = stage_nd(word);
      const int left = (info & 15) + ((info >> 4) & 15) - lo - nd;
      const bool done = left <= 0 && i + 1 == chunks;
      const int next_info = left > 0 ? info : chunk_info(min(i + 1, chunks - 1));
      const int next = left > 0 ? stage_word(c, lo + nd, min(SI_STAGE_D, left), 0) : first_stage(next_info);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                             // (also: everybody has read `red`)
      if (!done) stage_digits<KS, NW>(a.Xd, s, next, next_info & 15, tb, lds0 + (buf ^ 1) * TL::STAGE, wave, lane);
      const char* x = si_smem + buf * TL::STAGE + lane16;
      const int g = c / s.nchg;
      const bool whole = stage_first(word) && c == g * s.nchg;
#pragma unroll
      for (int old = 0; old < 2; ++old) {
        load_set(tl[old ^ 1], old ? stage_chunk(next) : c, !old);
        const double sc[1] = {old ? -tl[old].s[0] : tl[old].s[0]};
        for (int pr = (nd - 1) >> 1; pr >= 0; --pr) {
          v16i acc[1];
          tl[old].pair(x, pr, 2 * pr + 1 < nd, acc);
          add_scaled<1>(y, acc, sc, unit + 8 * (lo + 2 * pr));
        }
        if (whole && (old ? a.mt.rest_n : a.mt.rest_o)[g]) {
          const double rz = (old ? a.Rn : a.Ro)[(int64_t)g * s.npad + row0 + l32];
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const double sx = ldexp(a.SX[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)], unit);
            y[0][v] = fma(old ? rz : -rz, sx, y[0][v]);
          }
        }
      }
      if (left <= 0) {
        ++i;
        ++j;
      }
      word = next;
      info = next_info;
      buf ^= 1;
    }
  }
}

// Per candidate (grid.y) and 256 tokens: KL: sum over the tokens of B_t + log sum exp(q - M), minus the tiles' sums of P (q - M);
// squared error: the tiles' sums.  Every workgroup writes its sum.
template <int OBJ>
__global__ __launch_bounds__(256) void sba_token_sums(const double* __restrict__ part, const double* __restrict__ lin, SbaShape s,
                                                      const double* __restrict__ tokB, double* __restrict__ block_sums_all,
                                                      int nblocks) {
  __shared__ double red[256];
  const int tiles = s.npad / SE_ROWS;
  double acc = 0.0;
  if (OBJ == SLIM_OBJ_KL) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t < s.ts) {
      double Z = 0.0;
      for (int r = 0; r < tiles; ++r) Z += part[((int64_t)blockIdx.y * tiles + r) * s.tpad + t];
      acc = tokB[t] + log(Z);
    }
  }
  double lsum = 0.0;
  const int tb0 = blockIdx.x * 8, nb = min(8, s.TB - tb0);
  for (int j = threadIdx.x; j < tiles * nb; j += 256) lsum += lin[((int64_t)blockIdx.y * tiles + j / nb) * s.TB + tb0 + j % nb];
  acc = (OBJ == SLIM_OBJ_KL) ? acc - lsum : lsum;
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) block_sums_all[(int64_t)blockIdx.y * nblocks + blockIdx.x] = red[0];
}

// ---- host side -------------------------------------------------------------------------------------------------
SbaShape sba_shape(int n, int m, int beta, int64_t t_s) {
  SbaShape s;
  s.n = n;
  s.m = m;
  s.beta = beta;
  s.k = m / beta;
  s.ts = t_s;
  s.chk = beta <= 32 ? 32 : beta <= 64 ? 64 : SI_CHUNK;
  s.ks = s.chk / 32;
  s.nchg = slim_cdiv(beta, s.chk);
  s.C = s.k * s.nchg;
  s.npad = slim_cdiv(n, SI_ROWS) * SI_ROWS;
  s.RB = s.npad / 32;
  s.RT = s.npad / SI_ROWS;
  s.tpad = slim_cdiv(t_s, SI_TOK) * SI_TOK;
  s.TB = s.tpad / SI_TOK;
  return s;
}

// The workspace of slim_sba_allocate; slim_sba_prepare fills the part of it that does not depend on the ranking.
struct SbaWorkspace {
  SbaShape s;
  SbaMeta mt;
  int pmax, parts, kl_blocks;
  int64_t plane;                   // bytes of one int8 matrix in operand order
  char *Xd, *Wd, *Qn, *Qo;
  double *Sn, *So, *Rn, *Ro, *SX, *Yt, *Yc, *ref_part, *part, *lin, *obj, *block_sums, *tok, *tokB;
  int *order, *rank_of, *pstar_dev;
};
constexpr int KL_RPP = 256;        // rows per part of the reference side's reductions

// Lays the workspace out from `base` (nullptr: only the size is wanted) and returns its size.
size_t sba_layout(int n, int m, int beta, int64_t t_s, char* base, SbaWorkspace& w) {
  const SbaShape s = w.s = sba_shape(n, m, beta, t_s);
  w.pmax = s.k / 2;
  w.parts = slim_cdiv(n, KL_RPP);
  w.kl_blocks = slim_cdiv(t_s, 256);
  w.plane = (int64_t)s.npad * s.C * s.chk;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += slim_ws_round(bytes);
    return p;
  };
  auto doubles = [&](size_t count) { return reinterpret_cast<double*>(take(sizeof(double) * count)); };
  w.Xd = take((size_t)s.C * s.TB * SI_MAXD * s.ks * 1024);
  w.Wd = take((size_t)SI_MAXD * w.plane);
  w.Qn = take((size_t)w.plane);
  w.Qo = take((size_t)w.plane);
  w.Sn = doubles((size_t)s.k * s.npad);
  w.So = doubles((size_t)s.k * s.npad);
  w.Rn = doubles((size_t)s.k * s.npad);
  w.Ro = doubles((size_t)s.k * s.npad);
  w.SX = doubles((size_t)s.k * s.tpad);
  w.Yt = doubles((size_t)n * t_s);
  w.Yc = doubles((size_t)n * t_s);
  w.ref_part = doubles((size_t)w.parts * KL_PART * t_s);
  w.part = doubles((size_t)(w.pmax + 1) * (s.npad / SE_ROWS) * s.tpad);
  w.lin = doubles((size_t)(w.pmax + 1) * (s.npad / SE_ROWS) * s.TB);
  w.obj = doubles((size_t)(w.pmax + 2) * (size_t)(w.kl_blocks + 1));
  w.block_sums = w.obj + (w.pmax + 2);
  w.order = reinterpret_cast<int*>(take(sizeof(int) * (size_t)(2 * s.k + 2)));
  w.rank_of = w.order + (s.k + 1);
  w.pstar_dev = reinterpret_cast<int*>(take(256));
  w.tok = doubles(3 * (size_t)t_s);      // per token {max, log-sum-exp} of the reference; sum P log P behind
  w.tokB = w.tok + 2 * t_s;
  int* mi = reinterpret_cast<int*>(take(sizeof(int) * (8 * (size_t)s.C + 2 * (size_t)s.k + 4)));
  w.mt.x = mi;
  w.mt.w = mi + 2 * s.C;
  w.mt.xmax = reinterpret_cast<unsigned*>(mi + 4 * s.C);
  w.mt.xlsb = mi + 5 * s.C;
  w.mt.wmax = reinterpret_cast<unsigned*>(mi + 6 * s.C);
  w.mt.wlsb = mi + 7 * s.C;
  w.mt.rest_n = mi + 8 * s.C;
  w.mt.rest_o = w.mt.rest_n + s.k;
  w.mt.unit = w.mt.rest_o + s.k;
  return off;
}

}  // namespace

// The stated size has a floor of three n x m and two n x t_s and m x t_s fp64 matrices, which callers may have provided for.
size_t slim_ws_need_sba(int n, int m, int beta, int64_t t_s) {
  SbaWorkspace w;
  const size_t floor_bytes = 3 * slim_ws_round(8 * (size_t)n * m) + 2 * slim_ws_round(8 * (size_t)m * t_s) + 2 * slim_ws_round(8 * (size_t)n * t_s);
  return std::max(sba_layout(n, m, beta, t_s, nullptr, w), floor_bytes);
}

namespace {

slim_status sba_workspace(slim_ctx* ctx, int n, int m, int beta, int64_t t_s, SbaWorkspace& w) {
  const slim_status st = slim_ws_reserve(ctx, slim_ws_need_sba(n, m, beta, t_s));
  if (st != SLIM_OK) return st;
  sba_layout(n, m, beta, t_s, ctx->ws, w);
  return SLIM_OK;
}

slim_status sba_check(slim_ctx* ctx, const char* fn, const void* W, slim_dtype w_dtype, int n, int m, int64_t ldw,
                      int beta, int N, int objective, const void* X_s, slim_dtype x_dtype, int64_t t_s, int64_t ldxs,
                      const slim_params& prm) {
  SLIM_REQUIRE(ctx, W && X_s, "%s: null pointer", fn);
  SLIM_REQUIRE(ctx, n > 0 && m > 0 && beta > 0 && m % beta == 0, "%s: need n, m > 0 and beta | m", fn);
  SLIM_REQUIRE(ctx, N >= 2 && N <= 7, "%s: N must be in 2..7 (got %d)", fn, N);
  SLIM_REQUIRE(ctx, beta % 4 == 0 && ldw >= m && ldw % 4 == 0, "%s: beta and ldw must be multiples of 4", fn);
  SLIM_REQUIRE(ctx, t_s > 0 && t_s % 4 == 0 && ldxs >= t_s && ldxs % 4 == 0,
               "%s: t_s and ldxs must be positive multiples of 4", fn);
  SLIM_REQUIRE(ctx, slim_aligned16(W) && slim_aligned16(X_s), "%s: misaligned pointer", fn);
  SLIM_REQUIRE(ctx, prm.q1_mode == 0 || prm.q1_mode == 1, "%s: unknown q1_mode", fn);
  SLIM_REQUIRE(ctx, objective == SLIM_OBJ_KL || objective == SLIM_OBJ_MSE, "%s: unknown objective %d", fn, objective);
  if (w_dtype == SLIM_F64 || x_dtype == SLIM_F64 || x_dtype == SLIM_F32)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "%s: W must be F16/BF16/F32 and X_s F16/BF16", fn);
  SLIM_REQUIRE(ctx, (size_t)(m / beta / 2 + 2) * sizeof(double) <= (size_t)SLIM_HPIN_BYTES, "%s: too many groups", fn);
  return SLIM_OK;
}

template <typename T>
slim_status sba_codes_launch(slim_ctx* ctx, const T* W, const CodesArgs& a) {
  const dim3 grid(a.s.npad / 16, std::min(a.s.k, 8));
  if (a.rank_of)
    SLIM_LAUNCH(ctx, "sba_codes", (sba_codes<T, true>), grid, dim3(256), 0, W, a);
  else
    SLIM_LAUNCH(ctx, "sba_codes", (sba_codes<T, false>), grid, dim3(256), 0, W, a);
  return SLIM_OK;
}
slim_status sba_codes_launch(slim_ctx* ctx, const void* W, slim_dtype dt, const CodesArgs& a) {
  switch (dt) {
    case SLIM_F16: return sba_codes_launch(ctx, static_cast<const __half*>(W), a);
    case SLIM_BF16: return sba_codes_launch(ctx, static_cast<const __hip_bfloat16*>(W), a);
    default: return sba_codes_launch(ctx, static_cast<const float*>(W), a);
  }
}

template <typename T>
slim_status sba_x_launch(slim_ctx* ctx, const SbaWorkspace& w, const T* X, int64_t ldx) {
  SLIM_LAUNCH(ctx, "sba_x_stats", sba_x_stats<T>, dim3(w.s.C, slim_cdiv(w.s.ts, 1024)), dim3(256), 0, X, ldx, w.s, w.mt);
  return SLIM_OK;
}
template <typename T>
slim_status sba_digits_launch(slim_ctx* ctx, const SbaWorkspace& w, const T* X, int64_t ldx) {
  SLIM_LAUNCH(ctx, "sba_x_digits", sba_x_digits<T>, dim3(slim_cdiv(w.s.TB, 4), w.s.k), dim3(256), 0, X, ldx, w.s, w.mt, w.Xd, w.SX);
  return SLIM_OK;
}
template <typename T>
slim_status sba_w_launch(slim_ctx* ctx, const SbaWorkspace& w, const T* W, int64_t ldw) {
  SLIM_LAUNCH(ctx, "sba_w_stats", sba_w_stats<T>, dim3(slim_cdiv(w.s.m, 1024), std::min(w.s.n, 128)), dim3(256), 0, W, ldw, w.s, w.mt);
  return SLIM_OK;
}

template <int KS>
slim_status sba_outputs_launch(slim_ctx* ctx, const SbaShape& s, OutArgs a, bool ref) {
  const dim3 grid(s.RT * s.TB);
  const size_t smem = 2 * Tile<KS, 2>::STAGE + sizeof(int) * std::min(s.C, SI_TAB);
  if (ref)
    SLIM_LAUNCH(ctx, "sba_reference_outputs", (sba_outputs<KS, true>), grid, dim3(256), smem, a);
  else
    SLIM_LAUNCH(ctx, "sba_outputs", (sba_outputs<KS, false>), grid, dim3(256), smem, a);
  return SLIM_OK;
}
slim_status sba_outputs_launch(slim_ctx* ctx, const SbaShape& s, const OutArgs& a, bool ref) {
  return s.ks == 1 ? sba_outputs_launch<1>(ctx, s, a, ref) : s.ks == 2 ? sba_outputs_launch<2>(ctx, s, a, ref) : sba_outputs_launch<4>(ctx, s, a, ref);
}

template <int KS>
slim_status sba_search_launch(slim_ctx* ctx, const SearchArgs& a, int objective) {
  const dim3 grid((a.s.npad / SE_ROWS) * a.s.TB);
  const size_t smem = 2 * Tile<KS, 1>::STAGE + sizeof(double) * 4 * 34 + sizeof(int) * std::min(a.s.C, SI_TAB);
  if (objective == SLIM_OBJ_KL)
    SLIM_LAUNCH(ctx, "sba_search", (sba_search<KS, SLIM_OBJ_KL>), grid, dim3(256), smem, a);
  else
    SLIM_LAUNCH(ctx, "sba_search", (sba_search<KS, SLIM_OBJ_MSE>), grid, dim3(256), smem, a);
  return SLIM_OK;
}

// The part of the objective that does not depend on the ranking (Eq. 4): the digits of X_s and W and the codes of the
// all-N-bit weights, the reference outputs Y^T = W X_s and the outputs of the all-N-bit weights, and for the KL objective
// the reference softmax with its per-token statistics.
slim_status sba_rank_independent(slim_ctx* ctx, const SbaWorkspace& w, const void* W, slim_dtype w_dtype, int n,
                                 int64_t ldw, int N, int objective, const void* X_s, slim_dtype x_dtype, int64_t t_s,
                                 int64_t ldxs, int q1_mode) {
  const SbaShape& s = w.s;
  slim_status st;
  SLIM_LAUNCH(ctx, "sba_clear", sba_clear, dim3(slim_cdiv(std::max(s.C, s.k), 256)), dim3(256), 0, w.mt, s.C, s.k);
  const bool xh = x_dtype == SLIM_F16;
  st = xh ? sba_x_launch(ctx, w, static_cast<const __half*>(X_s), ldxs) : sba_x_launch(ctx, w, static_cast<const __hip_bfloat16*>(X_s), ldxs);
  if (st != SLIM_OK) return st;
  st = w_dtype == SLIM_F16 ? sba_w_launch(ctx, w, static_cast<const __half*>(W), ldw)
       : w_dtype == SLIM_BF16 ? sba_w_launch(ctx, w, static_cast<const __hip_bfloat16*>(W), ldw)
                              : sba_w_launch(ctx, w, static_cast<const float*>(W), ldw);
  if (st != SLIM_OK) return st;
  SLIM_LAUNCH(ctx, "sba_meta", sba_meta, dim3(2), dim3(256), 0, w.mt, s.C);
  st = xh ? sba_digits_launch(ctx, w, static_cast<const __half*>(X_s), ldxs) : sba_digits_launch(ctx, w, static_cast<const __hip_bfloat16*>(X_s), ldxs);
  if (st != SLIM_OK) return st;
  CodesArgs ca;
  ca.s = s;
  ca.mt = w.mt;
  ca.ldw = ldw;
  ca.N = N;
  ca.q1_mode = q1_mode;
  ca.pmax = w.pmax;
  ca.rank_of = nullptr;
  ca.Q = w.Qn;
  ca.S = w.Sn;
  ca.Rz = w.Rn;
  ca.rest = w.mt.rest_n;
  ca.Wd = w.Wd;
  st = sba_codes_launch(ctx, W, w_dtype, ca);
  if (st != SLIM_OK) return st;
  OutArgs oa;
  oa.s = s;
  oa.mt = w.mt;
  oa.Xd = w.Xd;
  oa.SX = w.SX;
  oa.Q = w.Wd;
  oa.plane = w.plane;
  oa.S = w.Sn;
  oa.Rz = w.Rn;
  oa.Y = w.Yt;
  st = sba_outputs_launch(ctx, s, oa, true);
  if (st != SLIM_OK) return st;
  oa.Q = w.Qn;
  oa.Y = w.Yc;
  st = sba_outputs_launch(ctx, s, oa, false);
  if (st != SLIM_OK) return st;
  if (objective == SLIM_OBJ_KL) {
    // reference side once: per-token maximum and log-sum-exp, then Y^T becomes P = softmax over the outputs
    const dim3 kgrid(slim_cdiv(t_s, KL_TOK), w.parts);
    SLIM_LAUNCH(ctx, "sba_kl_ref", kl_ref_partial, kgrid, dim3(256), 0, w.Yt, n, t_s, KL_RPP, w.ref_part);
    SLIM_LAUNCH(ctx, "sba_kl_ref", kl_ref_merge, dim3(w.kl_blocks), dim3(256), 0, w.ref_part, w.parts, t_s, w.tok);
    SLIM_LAUNCH(ctx, "sba_kl_ref", kl_ref_softmax, kgrid, dim3(256), 0, w.Yt, n, t_s, KL_RPP, w.tok, w.ref_part);
    SLIM_LAUNCH(ctx, "sba_kl_ref", kl_ref_entropy, dim3(w.kl_blocks), dim3(256), 0, w.ref_part, w.parts, t_s, w.tokB);
  }
  return SLIM_OK;
}

}  // namespace

extern "C" slim_status slim_sba_prepare(slim_ctx* ctx, const void* W, slim_dtype w_dtype, int n, int m, int64_t ldw,
                                        int beta, int N, int objective, const void* X_s, slim_dtype x_dtype,
                                        int64_t t_s, int64_t ldxs, const slim_params* params) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  slim_params prm;
  slim_default_params(&prm);
  if (params) prm = *params;
  slim_status st = sba_check(ctx, "slim_sba_prepare", W, w_dtype, n, m, ldw, beta, N, objective, X_s, x_dtype, t_s, ldxs, prm);
  if (st != SLIM_OK) return st;
  SbaWorkspace w;
  st = sba_workspace(ctx, n, m, beta, t_s, w);
  if (st != SLIM_OK) return st;
  st = sba_rank_independent(ctx, w, W, w_dtype, n, ldw, N, objective, X_s, x_dtype, t_s, ldxs, prm.q1_mode);
  if (st != SLIM_OK) return st;
  slim_sba_prepared& r = ctx->sba_prep;
  r.W = W;
  r.X_s = X_s;
  r.ws = ctx->ws;
  r.w_dtype = w_dtype;
  r.x_dtype = x_dtype;
  r.n = n;
  r.m = m;
  r.beta = beta;
  r.N = N;
  r.objective = objective;
  r.q1_mode = prm.q1_mode;
  r.ldw = ldw;
  r.t_s = t_s;
  r.ldxs = ldxs;
  r.valid = true;
  return SLIM_OK;
}

extern "C" slim_status slim_sba_allocate(slim_ctx* ctx, const void* W, slim_dtype w_dtype, int n, int m, int64_t ldw,
                                         const double* group_sal, int beta, int N, int objective, const void* X_s,
                                         slim_dtype x_dtype, int64_t t_s, int64_t ldxs, const slim_params* params,
                                         uint8_t* bits, int* p_star, double* obj_curve) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  slim_params prm;
  slim_default_params(&prm);
  if (params) prm = *params;
  SLIM_REQUIRE(ctx, group_sal && bits, "slim_sba_allocate: null pointer");
  slim_status st = sba_check(ctx, "slim_sba_allocate", W, w_dtype, n, m, ldw, beta, N, objective, X_s, x_dtype, t_s, ldxs, prm);
  if (st != SLIM_OK) return st;
  // a preceding slim_sba_prepare with the same arguments has left the rank-independent part in the workspace
  const slim_sba_prepared r = ctx->sba_prep;
  const bool prepared = r.valid && r.W == W && r.X_s == X_s && r.w_dtype == (int)w_dtype && r.x_dtype == (int)x_dtype &&
                        r.n == n && r.m == m && r.beta == beta && r.N == N && r.objective == objective &&
                        r.q1_mode == prm.q1_mode && r.ldw == ldw && r.t_s == t_s && r.ldxs == ldxs;
  SbaWorkspace w;
  st = sba_workspace(ctx, n, m, beta, t_s, w);
  if (st != SLIM_OK) return st;
  const SbaShape& s = w.s;
  const int k = s.k, pmax = w.pmax, kl_blocks = w.kl_blocks;
  int* const pstar_dev = w.pstar_dev;
  double* const obj = w.obj;

  const bool reuse = prepared && r.ws == ctx->ws;       // (the workspace was not reallocated in between)
  if (!reuse) {
    st = sba_rank_independent(ctx, w, W, w_dtype, n, ldw, N, objective, X_s, x_dtype, t_s, ldxs, prm.q1_mode);
    if (st != SLIM_OK) return st;
  }
  SLIM_LAUNCH(ctx, "sba_rank", sba_rank, dim3(1), dim3(256), 0, group_sal, k, w.order, w.rank_of);
  if (pmax > 0) {
    CodesArgs ca;
    ca.s = s;
    ca.mt = w.mt;
    ca.ldw = ldw;
    ca.N = N;
    ca.q1_mode = prm.q1_mode;
    ca.pmax = pmax;
    ca.rank_of = w.rank_of;
    ca.Q = w.Qo;
    ca.S = w.So;
    ca.Rz = w.Ro;
    ca.rest = w.mt.rest_o;
    ca.Wd = nullptr;
    st = sba_codes_launch(ctx, W, w_dtype, ca);
    if (st != SLIM_OK) return st;
  }
  SearchArgs sa;
  sa.s = s;
  sa.mt = w.mt;
  sa.Xd = w.Xd;
  sa.SX = w.SX;
  sa.Qn = w.Qn;
  sa.Qo = w.Qo;
  sa.Sn = w.Sn;
  sa.So = w.So;
  sa.Rn = w.Rn;
  sa.Ro = w.Ro;
  sa.Yc = w.Yc;
  sa.R = w.Yt;
  sa.tok = w.tok;
  sa.order = w.order;
  sa.part = w.part;
  sa.lin = w.lin;
  sa.pmax = pmax;
  st = s.ks == 1 ? sba_search_launch<1>(ctx, sa, objective) : s.ks == 2 ? sba_search_launch<2>(ctx, sa, objective) : sba_search_launch<4>(ctx, sa, objective);
  if (st != SLIM_OK) return st;
  if (objective == SLIM_OBJ_KL)
    SLIM_LAUNCH(ctx, "sba_token_sums", sba_token_sums<SLIM_OBJ_KL>, dim3(kl_blocks, pmax + 1), dim3(256), 0, w.part, w.lin, s, w.tokB,
                w.block_sums, kl_blocks);
  else
    SLIM_LAUNCH(ctx, "sba_token_sums", sba_token_sums<SLIM_OBJ_MSE>, dim3(kl_blocks, pmax + 1), dim3(256), 0, w.part, w.lin, s, w.tokB,
                w.block_sums, kl_blocks);
  SLIM_LAUNCH(ctx, "sba_finalize", sba_finalize, dim3(1), dim3(256), 0, w.block_sums, kl_blocks, obj, pmax, w.order, k, N,
              w.mt.unit + 2, bits, pstar_dev);

  if (!p_star && !obj_curve) return SLIM_OK;       // nothing for the host: the call does not wait
  double* host_obj = reinterpret_cast<double*>(ctx->hpin);
  int* host_p = reinterpret_cast<int*>(ctx->hpin + sizeof(double) * (size_t)(pmax + 1));
  SLIM_HIP_TRY(ctx, hipMemcpyAsync(host_obj, obj, sizeof(double) * (pmax + 1), hipMemcpyDeviceToHost, ctx->stream));
  SLIM_HIP_TRY(ctx, hipMemcpyAsync(host_p, pstar_dev, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  SLIM_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  if (p_star) *p_star = *host_p;
  if (obj_curve) memcpy(obj_curve, host_obj, sizeof(double) * (pmax + 1));
  return SLIM_OK;
}
