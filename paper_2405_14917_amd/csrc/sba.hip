// a4  Salience-Determined Bit Allocation (Eq. 4; Alg. 2 SBA; App. C, App. D).
//
// The search evaluates floor(k/2)+1 allocations that differ from one another in two groups only, so the layer outputs are
// carried incrementally.  Every product with the objective's tokens is EXACT integer arithmetic on the int8 matrix cores:
//   * X_s is integers times a power of two per 32 tokens of a chunk of channels (fp16 values are multiples of 2^-24 below 2^16),
//     cut into signed base-256 digits (balanced: -128 .. 127); of every such block only the digits in use are kept, three to
//     five for activations;
//   * a fake-quantised weight is scale * (q - z) with a small integer q - z: one int8 matrix, and one scale per (row, group);
//   * W itself is cut into digits the same way, with a power of two per row and chunk (two to four digits for 16-bit weights).
// A chunk's products of digits are summed exactly in int32 (128 channels of 127 * 128 * 257 < 2^31 for two digits chained by a
// shift) and enter the fp64 outputs with a rounding per pair of digits; the fp64 matrix cores round after every four channels.
// What is lost: an element of a block (X_s: 32 tokens of up to 128 channels; W: up to 128 channels of a row)
// of bf16 or fp32 values whose last digit lies more than 53 binary digits below the block's largest element is rounded
// there, by 2^-54 of that element (the objective, a sum over tokens and outputs, holds no more of it).  Relative error of W X_s on 2048 channels with outlier channels (model of either form's
// roundings against exact sums, groups of 32 to 128): 16-bit weights none in either form; fp32 weights 5e-17 to 1e-16 in
// either form.
//
//   sba_rank        stable ascending rank of the k group saliences (one workgroup, counting sort by comparison; NaN
//                   ranks last) -> order[]
//   int_w_units, int_x_digits               which digits there are, and the digits of X_s in MFMA operand order
//   sba_codes       per (row, group): Eq. 1 / Eq. 2 at width N and at the one other width the group can take, as integers
//                   in operand order with their scales; the digits of W
//   int_outputs     Y^T = W X_s and Y_0^T = W_N X_s (n x t_s, fp64)
//   kl_ref_*        once: per token the maximum M_t and log-sum-exp of the reference outputs; Y is then overwritten
//                   by P = softmax(Y) and B_t = sum_i P_i log P_i is kept
//   sba_search      all candidates in one kernel: obj[p] = sum_t [ B_t - (sum_i P_i q_i - lse(q)) ] with the reference
//                   maximum M_t as the shift of the exponentials (Y_p differs from Y by quantisation noise), then
//                   Y_{p+1} = Y_p + D_lo(g_lo) X_s(g_lo) + D_hi(g_hi) X_s(g_hi) in registers
//   sba_finalize    first minimum of obj, bit vector of p*
//
// Measured on 28672 x 8192, 2048 tokens, beside the inverse where it runs there (fp64 matrix cores -> this): outputs 32 ->
// 8.9 ms (reference 6.1, width N 2.8), search 15.2 -> 6.0 ms, widening and fake quantisation 3.4 -> 1.6 ms; 4096 x 4096:
// 3.5 -> 0.7, 1.19 -> 0.43 ms.  The fp64 products ran at 76 to 81 % of their roof.
#include <algorithm>

#include "int8_products.h"

namespace {

using namespace slimint;

constexpr int KL_TOK = 64;     // tokens per workgroup
constexpr int KL_UR = 8;        // loads in flight per thread: on small layers few workgroups share the chip
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
    for (int r = r0 + ty; r < r1; r += 4 * KL_UR) {
      double v[KL_UR];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u) v[u] = Y[(int64_t)min(r + 4 * u, r1 - 1) * ts + t];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u)
        if (r + 4 * u < r1) my = fmax(my, v[u]);
    }
  red[0][ty][tx] = my;
  __syncthreads();
  my = fmax(fmax(red[0][0][tx], red[0][1][tx]), fmax(red[0][2][tx], red[0][3][tx]));
  double zy = 0.0;
  if (live && my > -INFINITY)
    for (int r = r0 + ty; r < r1; r += 4 * KL_UR) {
      double v[KL_UR];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u) v[u] = Y[(int64_t)min(r + 4 * u, r1 - 1) * ts + t];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u)
        if (r + 4 * u < r1) zy += exp(v[u] - my);
    }
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
    for (int r = r0 + ty; r < r1; r += 4 * KL_UR) {
      double v[KL_UR];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u) v[u] = Y[(int64_t)min(r + 4 * u, r1 - 1) * ts + t];
#pragma unroll
      for (int u = 0; u < KL_UR; ++u)
        if (r + 4 * u < r1) {
          const double lp = v[u] - lse;
          const double pr = exp(lp);
          Y[(int64_t)(r + 4 * u) * ts + t] = pr;
          b = fma(pr, lp, b);
        }
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

constexpr int SE_ROWS = 128;       // outputs per workgroup of the search

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
  IntShape s;
  IntMeta mt;
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
  const IntShape& s = a.s;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4);
  const bool live = row < s.n;
  const int64_t plane = (int64_t)s.npad * s.C * s.chk;
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
      int c;
      const int64_t dst = operand_offset(s, row, g, j, c);
      unsigned word = 0;
      if (in) {
#pragma unroll
        for (int i = 0; i < 4; ++i) word |= ((unsigned)int_code(q, v[i]) & 255u) << (8 * i);
      }
      *reinterpret_cast<unsigned*>(a.Q + dst) = word;
      if (!OTHER) {
        const unsigned bits4[4] = {__float_as_uint((float)v[0]), __float_as_uint((float)v[1]), __float_as_uint((float)v[2]),
                                   __float_as_uint((float)v[3])};
        store_digits(a.Wd, plane, dst, bits4, a.mt.wunit[(int64_t)c * s.npad + row], digits_of_rows(s, a.mt.w, c, row));
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
  IntShape s;
  IntMeta mt;
  const char* Xd;
  const double* SX;
  const char *Qn, *Qo;
  const double *Sn, *So, *Rn, *Ro;
  const double* Yc;                // n x ts outputs of the all-N-bit weights
  const double* R;                 // n x ts reference: P = softmax(Y) (KL) or Y (squared error)
  const double* tok;               // per token {max, log-sum-exp} of the reference (KL)
  const int *order, *rest_n, *rest_o;
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
  const IntShape& s = a.s;
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
  // chunk i of the search (of candidate i / per): (chunk << 12) | (exponent of the lowest digit + 160) << 3 | digits
  const int per = 2 * s.nchg, chunks = a.pmax * per;
  auto describe = [&](int i) {
    const int p = i / per, j = i - p * per, hi = j >= s.nchg;
    const int c = a.order[hi ? s.k - 1 - p : p] * s.nchg + (j - hi * s.nchg);
    const int* x = a.mt.x + 2 * (c * s.TB + tb);                // (C TB blocks of at least 7 KiB: far below 2^30)
    return (int)((unsigned)c << 12 | (unsigned)(x[0] + 160) << 3 | (unsigned)x[1]);
  };
  for (int i = tid; i < min(chunks, SI_TAB); i += 256) tab[i] = describe(i);
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
  auto first_stage = [&](int info) { return stage_word((int)((unsigned)info >> 12), 0, min(SI_STAGE_D, info & 7), 1); };
  int i = 0, info = 0, word = 0, buf = 0;
  if (chunks > 0) {
    info = chunk_info(0);
    word = first_stage(info);
    stage_digits<KS, NW>(a.Xd, s, word, tb, lds0, wave, lane);
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
      const int left = (info & 7) - lo - nd, unit = ((info >> 3) & 511) - 160;
      const bool done = left <= 0 && i + 1 == chunks;
      const int next_info = left > 0 ? info : chunk_info(min(i + 1, chunks - 1));
      const int next = left > 0 ? stage_word(c, lo + nd, min(SI_STAGE_D, left), 0) : first_stage(next_info);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                             // (also: everybody has read `red`)
      if (!done) stage_digits<KS, NW>(a.Xd, s, next, tb, lds0 + (buf ^ 1) * TL::STAGE, wave, lane);
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
        if (whole && (old ? a.rest_n : a.rest_o)[g]) {
          const double rz = (old ? a.Rn : a.Ro)[(int64_t)g * s.npad + row0 + l32];
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const double sx = a.SX[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
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
__global__ __launch_bounds__(256) void sba_token_sums(const double* __restrict__ part, const double* __restrict__ lin, IntShape s,
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
// The workspace of slim_sba_allocate; slim_sba_prepare fills the part of it that does not depend on the ranking.
struct SbaWorkspace {
  IntShape s;
  IntMeta mt;
  int pmax, parts, kl_blocks;
  int64_t plane;                   // bytes of one int8 matrix in operand order
  char *Xd, *Wd, *Qn, *Qo;
  double *Sn, *So, *Rn, *Ro, *SX, *Yt, *Yc, *ref_part, *part, *lin, *obj, *block_sums, *tok, *tokB;
  int *order, *rank_of, *pstar_dev, *rest_n, *rest_o;
};
constexpr int KL_RPP = 256;        // rows per part of the reference side's reductions

// Lays the workspace out from `base` (nullptr: only the size is wanted) and returns its size.
size_t sba_layout(int n, int m, int beta, int64_t t_s, char* base, SbaWorkspace& w) {
  const IntShape s = w.s = slim_int_shape(n, m, beta, t_s);
  w.pmax = s.k / 2;
  w.parts = slim_cdiv(n, KL_RPP);
  w.kl_blocks = slim_cdiv(t_s, 256);
  w.plane = slim_int_plane(s);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += slim_ws_round(bytes);
    return p;
  };
  auto doubles = [&](size_t count) { return reinterpret_cast<double*>(take(sizeof(double) * count)); };
  w.Xd = take(slim_int_digits_bytes(s));
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
  w.mt.wunit = doubles((size_t)s.C * s.npad);
  w.mt.w = reinterpret_cast<uint8_t*>(take((size_t)s.C * (s.npad / 16)));
  int* mi = reinterpret_cast<int*>(take(sizeof(int) * (2 * (size_t)s.C * s.TB + 2 * (size_t)s.k + 1)));
  w.mt.x = mi;
  mi += 2 * (size_t)s.C * s.TB;
  w.rest_n = mi;                         // per group: some row has a zero outside int8 (width N; the other width)
  w.rest_o = w.rest_n + s.k;
  w.mt.nonfinite = w.rest_o + s.k;
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
  const IntShape& s = w.s;
  slim_status st;
  st = slim_int_clear(ctx, w.mt, w.rest_n, 2 * s.k);
  if (st == SLIM_OK) st = slim_int_w_units(ctx, s, w.mt, W, w_dtype, ldw);
  if (st == SLIM_OK) st = slim_int_x_digits(ctx, s, w.mt, X_s, x_dtype, ldxs, w.Xd, w.SX);
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
  ca.rest = w.rest_n;
  ca.Wd = w.Wd;
  st = sba_codes_launch(ctx, W, w_dtype, ca);
  if (st != SLIM_OK) return st;
  OutArgs oa;
  oa.s = s;
  oa.mt = w.mt;
  oa.rest = w.rest_n;
  oa.rest_from = 1;
  oa.token_unit = nullptr;
  oa.row_exp = nullptr;
  oa.Ylo = nullptr;
  oa.sub = oa.sublo = nullptr;
  oa.Xd = w.Xd;
  oa.SX = w.SX;
  oa.SXlo = nullptr;
  oa.Q = w.Wd;
  oa.plane = w.plane;
  oa.S = w.Sn;
  oa.Rz = w.Rn;
  oa.Y = w.Yt;
  st = slim_int_outputs(ctx, "sba_reference_outputs", oa, true, slim_int_sums::plain);
  if (st != SLIM_OK) return st;
  oa.Q = w.Qn;
  oa.Y = w.Yc;
  st = slim_int_outputs(ctx, "sba_outputs", oa, false, slim_int_sums::plain);
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
  const IntShape& s = w.s;
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
    ca.rest = w.rest_o;
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
  sa.rest_n = w.rest_n;
  sa.rest_o = w.rest_o;
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
              w.mt.nonfinite, bits, pstar_dev);

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
