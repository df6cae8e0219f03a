// Digits of the operands and the output products on the int8 matrix cores; see int8_products.h.
#include <algorithm>
#include <type_traits>

#include "int8_products.h"

namespace {

using namespace slimint;

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

__global__ __launch_bounds__(256) void int_clear(IntMeta mt, int* rest, int nrest) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < nrest) rest[i] = 0;
  if (i == 0) *mt.nonfinite = 0;
}

// grid (npad / 16, y): a wavefront takes 16 rows of a group, 4 lanes each, groups 4 blockIdx.y + wavefront and so on: the unit of
// every row's chunks, and the digits that the 16 rows of a chunk need.  (With 16 lanes a row and atomics for the digits of
// a chunk 156 us on 4096 x 4096.)
template <typename T>
__global__ __launch_bounds__(256) void int_w_units(const T* __restrict__ W, int64_t ldw, IntShape s, IntMeta mt) {
  const int lane = threadIdx.x & 63, l4 = lane & 3;
  const int row = blockIdx.x * 16 + (lane >> 2);
  const bool live = row < s.n;
  unsigned top = 0;
  for (int g = blockIdx.y * 4 + (threadIdx.x >> 6); g < s.k; g += gridDim.y * 4) {
    const T* w = W + (int64_t)min(row, s.n - 1) * ldw + (int64_t)g * s.beta;
    for (int cc = 0; cc < s.nchg; ++cc) {
      const int c = g * s.nchg + cc;
      unsigned mx = 0;
      int lsb = INT_MAX;
#pragma unroll 8
      for (int j = cc * s.chk + l4 * 4; j < min(s.beta, (cc + 1) * s.chk); j += 16) {
        T v[4];
        if constexpr (sizeof(T) == 2)
          *reinterpret_cast<uint2*>(v) = *reinterpret_cast<const uint2*>(w + j);
        else
          *reinterpret_cast<uint4*>(v) = *reinterpret_cast<const uint4*>(w + j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned bits = float_bits<T>(v[i]) & 0x7fffffffu;
          unsigned mant;
          int e0;
          split_float(bits, mant, e0);
          mx = max(mx, bits);
          lsb = min(lsb, bits ? e0 + __builtin_ctz(mant | 0x80000000u) : INT_MAX);
        }
      }
      mx = max(mx, (unsigned)dpp_b32<DPP_XOR1>((int)mx));
      mx = max(mx, (unsigned)dpp_b32<DPP_XOR2>((int)mx));
      lsb = min(lsb, dpp_b32<DPP_XOR1>(lsb));
      lsb = min(lsb, dpp_b32<DPP_XOR2>(lsb));
      if (!live) mx = 0;
      top = max(top, mx);
      // (a row with elements that are not finite has no sums: any unit will do)
      const int unit = block_unit(mx, lsb);
      unsigned used = (1u << digits_for((uint64_t)fixed_point(mx, unit))) - 1u;
      if (l4 == 0) mt.wunit[(int64_t)c * s.npad + row] = ldexp(1.0, unit);
#pragma unroll
      for (int d = 4; d < 64; d <<= 1) used |= (unsigned)__shfl_xor((int)used, d, WAVE);
      if (lane == 0) mt.w[(int64_t)c * (s.npad / 16) + blockIdx.x] = (uint8_t)used;
    }
  }
  if (top >= 0x7f800000u) atomicOr(mt.nonfinite, 1);
}

// grid (ceil(TB / 4), k): a wavefront finds the unit and the digits in use of 32 tokens of every chunk of one group, cuts them
// into digits, and sums the group's channels per token
template <typename T>
__global__ __launch_bounds__(256) void int_x_digits(const T* __restrict__ X, int64_t ldx, IntShape s, IntMeta mt,
                                                    char* __restrict__ Xd, double* __restrict__ SX) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int tb = blockIdx.x * 4 + (threadIdx.x >> 6), g = blockIdx.y;
  if (tb >= s.TB) return;
  const int64_t t = (int64_t)tb * 32 + l32;
  // sixteen channels from j on, their loads issued together (as reads of one value after another behind the branches of `stat`
  // a layer of 256 channels and 512 tokens took 17 us)
  const int64_t tc = t < s.ts ? t : s.ts - 1;
  auto values = [&](int j, unsigned (&v)[16]) {
    T x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = X[(int64_t)(g * s.beta + min(j + i, s.beta - 1)) * ldx + tc];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = (j + i < s.beta && t < s.ts) ? float_bits<T>(x[i]) : 0u;
  };
  double sum = 0.0;
  for (int cc = 0; cc < s.nchg; ++cc) {
    const int c = g * s.nchg + cc;
    unsigned mx = 0;
    int lsb = INT_MAX, bad = 0;
    for (int f = 0; f < s.ks; ++f) {
      unsigned v[16];
      values(cc * s.chk + f * 32 + h * 16, v);
#pragma unroll
      for (int i = 0; i < 16; ++i) stat(v[i], mx, lsb, bad);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      mx = max(mx, (unsigned)__shfl_xor((int)mx, d, WAVE));
      lsb = min(lsb, __shfl_xor(lsb, d, WAVE));
    }
    if (bad) atomicOr(mt.nonfinite, 1);
    const int unit = block_unit(mx, lsb), nd = digits_for((uint64_t)fixed_point(mx, unit));
    if (lane == 0) {
      mt.x[2 * ((int64_t)c * s.TB + tb)] = unit;
      mt.x[2 * ((int64_t)c * s.TB + tb) + 1] = nd;
    }
    int64_t csum = 0;                      // of this chunk: at most 64 channels of 54 bits
    char* dst = Xd + ((int64_t)c * s.TB + tb) * SI_MAXD * s.ks * 1024 + lane * 16;
    for (int f = 0; f < s.ks; ++f) {
      uint64_t u[16];
      unsigned raw[16];
      values(cc * s.chk + f * 32 + h * 16, raw);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t v = fixed_point(raw[i], unit);
        csum += v;
        u[i] = digit_bytes(v);
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
    sum += ldexp((double)csum, unit);
  }
  const double other = __shfl_xor(sum, 32, WAVE);
  if (h == 0) SX[(int64_t)g * s.tpad + t] = sum + other;
}

// ---- a unit per token ----------------------------------------------------------------------------------------------
// grid (ceil(ts / 1024), splits): a thread owns four columns; largest magnitude (as float bits) and last digit of each
__global__ __launch_bounds__(256) void int_g_stats(const float* __restrict__ G, int64_t ldg, IntShape s, int* __restrict__ work) {
  const int64_t t = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  if (t >= s.ts) return;
  unsigned mx[4] = {0, 0, 0, 0};
  int lsb[4] = {INT_MAX, INT_MAX, INT_MAX, INT_MAX}, bad[4] = {0, 0, 0, 0};
  for (int r = blockIdx.y; r < s.m; r += gridDim.y) {
    const float4 v = *reinterpret_cast<const float4*>(G + (int64_t)r * ldg + t);
    stat(__float_as_uint(v.x), mx[0], lsb[0], bad[0]);
    stat(__float_as_uint(v.y), mx[1], lsb[1], bad[1]);
    stat(__float_as_uint(v.z), mx[2], lsb[2], bad[2]);
    stat(__float_as_uint(v.w), mx[3], lsb[3], bad[3]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    atomicMax(&work[t + i], bad[i] ? INT_MAX : (int)mx[i]);
    atomicMin(&work[s.ts + t + i], lsb[i]);
  }
}
__global__ __launch_bounds__(256) void int_g_clear(int64_t ts, int* __restrict__ work) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < ts) {
    work[i] = 0;
    work[ts + i] = INT_MAX;
  }
}
// the unit of a column: its last digit, but no more than 53 digits below its largest value
__global__ __launch_bounds__(256) void int_g_units(int64_t ts, const int* __restrict__ work, int* __restrict__ token_unit) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= ts) return;
  const int mx = work[i];
  token_unit[i] = mx == INT_MAX ? INT_MIN : block_unit((unsigned)mx, work[ts + i]);
}

// What int_outputs_twice takes of a chunk without looking: zeros where there are fewer.
constexpr int TWICE_DIGITS = 5;
// What a chunk costs there, and in int_outputs_by_pairs if it has digits and per pair of them (in about 1/20 us per product of 4096
// outputs x 4096 columns)
constexpr int TWICE_CHUNK = 26, PAIRS_CHUNK = 3, PAIRS_PAIR = 10;

// grid (ceil(TB / 4), k): a wavefront finds the digits in use of 32 columns of every chunk of one group, and cuts them
__global__ __launch_bounds__(256) void int_g_digits(const float* __restrict__ G, int64_t ldg, IntShape s, int* __restrict__ meta,
                                                    const int* __restrict__ token_unit, char* __restrict__ Xd, double* __restrict__ SX,
                                                    double* __restrict__ SXlo) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int tb = blockIdx.x * 4 + (threadIdx.x >> 6), g = blockIdx.y;
  if (tb >= s.TB) return;
  const int64_t t = (int64_t)tb * 32 + l32;
  const bool live = t < s.ts;
  const int unit = live ? token_unit[t] : INT_MIN;
  auto value = [&](int j) -> int64_t {
    if (j >= s.beta || unit == INT_MIN) return 0;
    return fixed_point(__float_as_uint(G[(int64_t)(g * s.beta + j) * ldg + t]), unit);
  };
  double sum = 0.0, sumlo = 0.0;
  for (int cc = 0; cc < s.nchg; ++cc) {
    const int c = g * s.nchg + cc;
    uint64_t mx = 0, any = 0;
    int64_t csum = 0;                      // of this chunk: at most 64 channels of 54 bits
    for (int f = 0; f < s.ks; ++f)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t v = value(cc * s.chk + f * 32 + h * 16 + i);
        const uint64_t av = (uint64_t)(v < 0 ? -v : v);
        mx = mx > av ? mx : av;
        any |= av;
      }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      const uint64_t om = ((uint64_t)(unsigned)__shfl_xor((int)(mx >> 32), d, WAVE) << 32) | (unsigned)__shfl_xor((int)mx, d, WAVE);
      mx = mx > om ? mx : om;
      any |= ((uint64_t)(unsigned)__shfl_xor((int)(any >> 32), d, WAVE) << 32) | (unsigned)__shfl_xor((int)any, d, WAVE);
    }
    const int lo = mx ? __builtin_ctzll(any) / 8 : 0, nd = max(digits_for(mx) - lo, 0);
    if (lane == 0) {
      meta[2 * ((int64_t)c * s.TB + tb)] = 8 * lo;
      meta[2 * ((int64_t)c * s.TB + tb) + 1] = nd;
    }
    char* dst = Xd + ((int64_t)c * s.TB + tb) * SI_MAXD * s.ks * 1024 + lane * 16;
    for (int f = 0; f < s.ks; ++f) {
      uint64_t u[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t v = value(cc * s.chk + f * 32 + h * 16 + i);
        csum += v;
        u[i] = digit_bytes(v) >> (8 * lo);
      }
      for (int d = 0; d < max(nd, TWICE_DIGITS); ++d) {
        unsigned w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          w[q] = 0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            w[q] |= (d < nd ? (unsigned)u[4 * q + i] & 255u : 0u) << (8 * i);
            u[4 * q + i] >>= 8;
          }
        }
        *reinterpret_cast<uint4*>(dst + ((int64_t)d * s.ks + f) * 1024) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
    // both halves of the wavefront's channels, as a double and what it leaves; then two-sum with the chunks before
    csum += (int64_t)(((uint64_t)(unsigned)__shfl_xor((int)(csum >> 32), 32, WAVE) << 32) | (unsigned)__shfl_xor((int)csum, 32, WAVE));
    const double c_hi = (double)csum, c_lo = (double)(csum - (int64_t)c_hi);
    const double both = sum + c_hi, part = both - sum;
    sumlo += ((sum - (both - part)) + (c_hi - part)) + c_lo;
    sum = both;
  }
  if (h == 0) {
    SX[(int64_t)g * s.tpad + t] = sum;
    SXlo[(int64_t)g * s.tpad + t] = sumlo;
  }
}

// One workgroup: cost = what int_outputs_by_pairs would take for these digits (see there)
__global__ __launch_bounds__(1024) void int_g_cost(const int* __restrict__ meta, int64_t chunks, int* __restrict__ cost) {
  __shared__ unsigned sum;
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  unsigned mine = 0;
  for (int64_t i = threadIdx.x; i < chunks; i += 1024) {
    const int nd = meta[2 * i + 1];
    mine += nd ? PAIRS_CHUNK + PAIRS_PAIR * ((nd + 1) >> 1) : 0;
  }
  atomicAdd(&sum, mine);
  __syncthreads();
  if (threadIdx.x == 0) *cost = (int)(sum / (unsigned)chunks);
}

// What a chunk's digits are; in the place of W's digits, where there are none, whether it is the first of its group and some zero of
// the group lies outside int8.
template <bool REF>
__device__ __forceinline__ int describe_chunk(const OutArgs& a, int c, int tb, int row0) {
  const int* x = a.mt.x + 2 * ((int64_t)c * a.s.TB + tb);
  if (REF) return digits_word(x, digits_of_rows(a.s, a.mt.w, c, row0));
  return digits_word(x, c % a.s.nchg == 0 && a.rest[c / a.s.nchg] >= a.rest_from);
}

// REF: Y = W X_s from the digits of W; else Y = W_N X_s.
template <int KS, bool REF>
__global__ __launch_bounds__(256, 3) void int_outputs(OutArgs a) {
  constexpr int R = 2, NW = 4, SD = SI_STAGE_D;
  using TL = Tile<KS, R>;
  extern __shared__ __align__(16) char si_smem[];
  const IntShape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  int rt, tb;
  tile_of(blockIdx.x, s.RT, s.TB, rt, tb);
  const int row0 = rt * SI_ROWS + wave * 32 * R;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)si_smem));
  const int64_t rstride = (int64_t)s.C * KS * 1024;
  const char* q0 = a.Q + (int64_t)(row0 >> 5) * rstride;
  const unsigned lane16 = lane * 16;
  int* tab = reinterpret_cast<int*>(si_smem + 2 * TL::STAGE);
  for (int c = tid; c < min(s.C, SI_TAB); c += 64 * NW) tab[c] = describe_chunk<REF>(a, c, tb, row0);
  __syncthreads();
  auto chunk_info = [&](int c) { return __builtin_amdgcn_readfirstlane(c < SI_TAB ? tab[c] : describe_chunk<REF>(a, c, tb, row0)); };

  double y[R][16];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < 16; ++v) y[r][v] = 0.0;
  TL tl;
  auto load_first = [&](int c) {                // the first (or only) set of chunk c
    tl.load_codes(q0 + (int64_t)c * KS * 1024, rstride, lane16);
    tl.load_scales(REF ? a.mt.wunit + (int64_t)c * s.npad + row0 : a.S + (int64_t)(c / s.nchg) * s.npad + row0, l32);
  };
  auto first_stage = [&](int c, int info) { return stage_word(c, 0, min(SD, digits_x(info)), 1); };
  int info = chunk_info(0), word = first_stage(0, info), buf = 0;
  stage_digits<KS, NW>(a.Xd, s, word, tb, lds0, wave, lane);
  load_first(0);
  for (;;) {
    const int c = stage_chunk(word), lo = stage_lo(word), nd = stage_nd(word);
    const int left = digits_x(info) - lo - nd;                              // digits of the chunk behind this stage
    const bool done = left <= 0 && c + 1 == s.C;
    const int next_info = left > 0 ? info : chunk_info(min(c + 1, s.C - 1));
    const int next = left > 0 ? stage_word(c, lo + nd, min(SD, left), 0) : first_stage(min(c + 1, s.C - 1), next_info);
    const int sets = REF ? digits_w(info) : 1, unit = exponent_x(info);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!done) stage_digits<KS, NW>(a.Xd, s, next, tb, lds0 + (buf ^ 1) * TL::STAGE, wave, lane);
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
        add_scaled<R>(y, acc, sc, unit + 8 * (lo + 2 * p) + (REF ? 8 * j : 0));
      }
    }
    if (!REF && stage_first(word) && digits_w(info)) {
      const int g = c / s.nchg;
      // zeros outside int8: what the codes do not hold times the sum of the group's activations
      const double* Rz = a.Rz + (int64_t)g * s.npad + row0 + l32;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const double sx = a.SX[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
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
  for (int q = 0; q < 4; ++q) {
    const int64_t t = (int64_t)tb * 32 + 8 * q + 4 * h;
    if (t >= s.ts) continue;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + 32 * r + l32;
      if (row >= s.n) continue;
      double* out = a.Y + (int64_t)row * s.ts + t;
      *reinterpret_cast<double2*>(out) = make_double2(y[r][4 * q], y[r][4 * q + 1]);
      *reinterpret_cast<double2*>(out + 2) = make_double2(y[r][4 * q + 2], y[r][4 * q + 3]);
    }
  }
}

// Zeros outside int8 in sums to twice the precision: what the codes do not hold times the sum of the group's activations.
__device__ __forceinline__ void add_zeros(const OutArgs& a, int c, int tb, int row0, int lane, double (&y)[16], double (&low)[16]) {
  const int g = c / a.s.nchg;
  const double rz = -a.Rz[(int64_t)g * a.s.npad + row0 + (lane & 31)];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t at = (int64_t)g * a.s.tpad + tb * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    add_compensated(y[v], low[v], rz, a.SX[at]);
    low[v] = fma(rz, a.SXlo[at], low[v]);
    asm volatile("" : "+v"(y[v]), "+v"(low[v]) : : "memory");       // (rare: not all loads at once)
  }
}
// A wavefront's sums to twice the precision -> Y and Ylo, or Y = sums - (sub, sublo)
template <bool REF>
__device__ __forceinline__ void store_twice(const OutArgs& a, int row0, int tb, int lane, double base, const double (&y)[16], const double (&low)[16]) {
  const IntShape& s = a.s;
  const int row = row0 + (lane & 31), h = lane >> 5;
  if (row >= s.n) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t t = (int64_t)tb * 32 + 8 * q + 4 * h;
    if (t >= s.ts) continue;
    double o[4], ol[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int tu = a.token_unit ? a.token_unit[t + v] : 0;
      const int64_t at = (int64_t)row * s.ts + t + v;
      o[v] = tu == INT_MIN ? NAN : ldexp(y[4 * q + v] - base, tu);
      ol[v] = ldexp(low[4 * q + v], tu == INT_MIN ? 0 : tu);
      if (!REF) o[v] = (o[v] - a.sub[at]) + (ol[v] - a.sublo[at]);
    }
    if constexpr (REF) {
      double* outlo = a.Ylo + (int64_t)row * s.ts + t;
      *reinterpret_cast<double2*>(outlo) = make_double2(ol[0], ol[1]);
      *reinterpret_cast<double2*>(outlo + 2) = make_double2(ol[2], ol[3]);
    }
    double* out = a.Y + (int64_t)row * s.ts + t;
    *reinterpret_cast<double2*>(out) = make_double2(o[0], o[1]);
    *reinterpret_cast<double2*>(out + 2) = make_double2(o[2], o[3]);
  }
}

// The same with sums to twice the precision, for W_hat X - W X (add_compensated), and a unit per token.
//
// The digits of a chunk are summed in three int32 accumulators of a pair each.  The two lower ones are put together exactly in fp64
// (below 2^48), so that a chunk takes two compensated additions, and these stand behind the MFMAs of the next chunk, four outputs
// at a time: a wavefront fills both pipes by itself.  Two sets of accumulators and of codes and the sums are 234 registers: two
// wavefronts per SIMD, in two workgroups, so that one computes while the other waits at a chunk's barrier (one workgroup of eight
// wavefronts: 735 us against 615 before the order of the loads).  For the same reason all that the next chunk needs is asked for
// beside this one's products, and nothing between two chunks' products waits for memory.
// (A loop with one way out, and no choice among several bodies: else the compiler keeps the sums in memory between them.  So a
// chunk has five digits at least, zeros if need be: five are what most chunks of a Gram matrix of 16-bit activations have, the
// others six.  A G of fewer is left to int_outputs_by_pairs.)
// 4096 x 4096 against 4096 columns: 600 -> 545 us (a compensated addition per pair of digits and the vector work behind each
// pair's own MFMAs, four wavefronts per SIMD); vector instructions 53 % of the time, the matrix cores 28 %.
template <int KS, bool REF>
__global__ __launch_bounds__(256, 2) void int_outputs_twice(OutArgs a) {
  constexpr int NW = 4;
  constexpr int STAGE = SI_MAXD * KS * 1024, ND = TWICE_DIGITS;
  extern __shared__ __align__(16) char si_smem[];
  const IntShape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  int rt, tb;
  tile_of(blockIdx.x, s.npad / (32 * NW), s.TB, rt, tb);
  const int row0 = (rt * NW + wave) * 32;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)si_smem));
  int* tab = reinterpret_cast<int*>(si_smem + 2 * STAGE);
  for (int c = tid; c < min(s.C, SI_TAB); c += 64 * NW) tab[c] = describe_chunk<REF>(a, c, tb, row0);
  __syncthreads();

  const double base = sum_base(s.m, a.row_exp[row0 + l32]);
  double y[16], low[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    y[v] = base;
    low[v] = 0.0;
  }
  v16i sums[2][3];                   // of a chunk: digits 0 and 1, 2 and 3, 4 and 5
  double f0[2];                      // what the lowest digit counts
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int v = 0; v < 16; ++v) sums[1][k][v] = 0;
  f0[1] = 0.0;
  // The additions of p, four outputs at a time in five steps: each step has four independent chains of two instructions (one
  // output after the other, eight instructions that wait for one another, took 735 us).  What a step leaves is pinned there, or
  // the compiler moves all of it behind the chunk's products.
  struct {
    double c[4], t[4], s[4], b[4];
  } ad;
  auto add_step = [&](const v16i (&p)[3], double g0, double g2, int step) {
    const int v0 = step / 5 * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = v0 + i;
      if (step % 5 == 0) {
        ad.c[i] = (double)p[2][v];
        ad.s[i] = fma(g2, ad.c[i], y[v]);
        asm volatile("" : "+v"(ad.c[i]), "+v"(ad.s[i]));
      } else if (step % 5 == 1) {
        ad.b[i] = fma(g2, ad.c[i], y[v] - ad.s[i]);
        ad.t[i] = (double)p[1][v];
        asm volatile("" : "+v"(ad.b[i]), "+v"(ad.t[i]));
      } else if (step % 5 == 2) {
        low[v] += ad.b[i];
        ad.t[i] = fma(ad.t[i], 65536.0, (double)p[0][v]);
        asm volatile("" : "+v"(low[v]), "+v"(ad.t[i]));
      } else if (step % 5 == 3) {
        y[v] = fma(g0, ad.t[i], ad.s[i]);
        ad.b[i] = ad.s[i] - y[v];
        asm volatile("" : "+v"(y[v]), "+v"(ad.b[i]));
      } else {
        low[v] += fma(g0, ad.t[i], ad.b[i]);
        asm volatile("" : "+v"(low[v]));
      }
    }
  };
  // A part: a chunk and a set of W's digits (the codes are one set).  What a part needs from memory is asked for during the one
  // before it: codes into w[its parity], its chunk's digits into the other stage.
  v4i w[2][KS];
  const char* q0 = a.Q + (int64_t)(row0 >> 5) * s.C * KS * 1024 + lane * 16;
  auto load_codes = [&](v4i (&to)[KS], int c, int j) {
#pragma unroll
    for (int i = 0; i < KS; ++i) to[i] = *reinterpret_cast<const v4i*>(q0 + j * a.plane + (int64_t)(c * KS + i) * 1024);
  };
  auto chunk_word = [&](int c) { return c < SI_TAB ? tab[c] : describe_chunk<REF>(a, c, tb, row0); };
  const double* scales = REF ? a.mt.wunit + row0 : a.S + row0;            // of the next chunk
  int in_group = 0;
  auto next_scale = [&]() {
    const double v = scales[l32];
    if (REF || ++in_group == s.nchg) {
      in_group = 0;
      scales += s.npad;
    }
    return v;
  };
  const char* digits = a.Xd + (int64_t)tb * SI_MAXD * KS * 1024;          // of the next chunk
  const int64_t digits_step = (int64_t)s.TB * SI_MAXD * KS * 1024;
  auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };   // (what the compiler does not see is the same in all lanes)
  auto load_digit = [&](int to, int i) {
    const uint64_t from = (uint64_t)(uintptr_t)(digits + i * 1024);
    const uint64_t base = (uint64_t)(unsigned)uniform((int)(from >> 32)) << 32 | (unsigned)uniform((int)from);
    lds_load16((unsigned)uniform((int)(lds0 + to * STAGE + i * 1024)), lane * 16, reinterpret_cast<const char*>(base));
  };
  int c = 0, j = 0, buf = 0, info = uniform(chunk_word(0)), after = 0, next_info = chunk_word(min(1, s.C - 1));
  for (int i = wave; i < max(digits_x(info), ND) * KS; i += NW) load_digit(0, i);
  digits += digits_step;
  load_codes(w[0], 0, 0);
  double sc = next_scale(), sc_next = 0.0;
  bool live = true;                  // behind the last part one more is taken with a count of zero, where the loop needs it
  auto shift = [&](v16i& c) {
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] <<= 8;
  };
  auto digit = [&](const v4i (&wc)[KS], const char* x, int d, v16i& to) {
#pragma unroll
    for (int i = 0; i < KS; ++i) to = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i*>(x + (d * KS + i) * 1024), wc[i], to, 0, 0, 0);
  };
  // the digits of a part into sums[CUR], beside the products of the lower five the additions of sums[1 - CUR]
  auto part = [&](auto cur) {
    constexpr int CUR = decltype(cur)::value;
    constexpr int AHEAD = 2, NM = ND * KS;           // operand reads in flight; MFMAs with additions beside them
    constexpr int ORDER[ND] = {4, 3, 1, 2, 0};       // the pairs in turn: while one is shifted, another's products run
    const bool fresh_chunk = !REF || j == 0;
    if (fresh_chunk) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    v16i(&p)[3] = sums[CUR];
    const char* x = si_smem + buf * STAGE + lane * 16;
    const int nd = digits_x(info), sets = REF ? digits_w(info) : 1;       // five to seven digits
    const double count = live && sets > 0 ? ldexp(sc, exponent_x(info) + (REF ? 8 * j : 0)) : 0.0;
    // the next part
    const bool more = REF && j + 1 < sets;
    const int cn = min(more ? c : c + 1, s.C - 1), jn = more ? j + 1 : 0;
    if (fresh_chunk) after = uniform(next_info);
    const int left = fresh_chunk && c + 1 < s.C ? max(digits_x(after), ND) * KS : 0;
    load_codes(w[1 - CUR], cn, jn);
    if (fresh_chunk) {
      if (c + 1 < s.C) sc_next = next_scale();
      next_info = chunk_word(min(c + 2, s.C - 1));
      if (!REF && digits_w(info) && live) add_zeros(a, c, tb, row0, lane, y, low);
    }
    v4i fr[AHEAD + 1];
    auto frag = [&](int n) { fr[n % (AHEAD + 1)] = *reinterpret_cast<const v4i*>(x + (ORDER[n / KS] * KS + n % KS) * 1024); };
    const double o0 = f0[1 - CUR], o2 = o0 * 4294967296.0;
#pragma unroll
    for (int v = 0; v < 16; ++v) p[2][v] = 0;
    if (nd > 5) {
      if (nd > 6) {                                  // (rare: added at once)
        digit(w[CUR], x, 6, p[2]);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          add_compensated(y[v], low[v], count * 0x1p48, (double)p[2][v]);
          asm volatile("" : "+v"(y[v]), "+v"(low[v]));
          p[2][v] = 0;
        }
      }
      digit(w[CUR], x, 5, p[2]);
      shift(p[2]);
    }
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) frag(n);
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int d = ORDER[n / KS];
      if (n + AHEAD < NM) frag(n + AHEAD);
      if (n % KS == 0 && d < 3 && d != 1) shift(p[d / 2]);
      __builtin_amdgcn_sched_barrier(0);
      v16i in = p[d / 2];
      if (n % KS == 0 && (d & 1)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) in[v] = 0;
      }
      p[d / 2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr[n % (AHEAD + 1)], w[CUR][n % KS], in, 0, 0, 0);
#pragma unroll
      for (int step = n * 20 / NM; step < (n + 1) * 20 / NM; ++step) add_step(sums[1 - CUR], o0, o2, step);
      // the next chunk's digits, one KiB at a time: every chunk has these, the sixth and seventh follow below
      if (n % 2 == 0 && n / 2 * NW < ND * KS) {
        const int i = n / 2 * NW + wave;
        if (i < min(left, ND * KS)) load_digit(buf ^ 1, i);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int i = ND * KS + wave; i < left; i += NW) load_digit(buf ^ 1, i);
    f0[CUR] = count;
    if (more) {
      ++j;
    } else {
      j = 0;
      if (++c < s.C) {
        buf ^= 1;
        info = after;
        sc = sc_next;
        digits += digits_step;
      } else {
        live = false;
      }
    }
  };
  while (live) {
    part(std::integral_constant<int, 0>{});
    part(std::integral_constant<int, 1>{});
  }
#pragma unroll
  for (int step = 0; step < 20; ++step) add_step(sums[1], f0[1], f0[1] * 4294967296.0, step);
  store_twice<REF>(a, row0, tb, lane, base, y, low);
}

// The same for a G of few digits (diagonal, block diagonal, small integers): every pair of digits enters the sums by itself, and
// chunks without digits are passed over.  Four wavefronts per SIMD, eight to a workgroup and its 256 outputs: with the 256 threads
// and two wavefronts of int_outputs_twice most of the time is a chunk's barrier.  slim_lwc_quantize of 4096 x 4096, 20 steps, us,
// int_outputs_twice / this: diagonal G 13660 / 5730, blocks of 512 13790 / 6640, two digits (activations to 3) 13930 / 10060, four
// (to 200 and 2000) 14160 / 13420 and 14590 / 13910, a quarter of the channels dead 14220 / 13340; five 15000 / 16100.
template <int KS, bool REF>
__global__ __launch_bounds__(512, 4) void int_outputs_by_pairs(OutArgs a) {
  constexpr int NW = 8, STAGE = SI_MAXD * KS * 1024;
  extern __shared__ __align__(16) char si_smem[];
  const IntShape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  int rt, tb;
  tile_of(blockIdx.x, s.RT, s.TB, rt, tb);
  const int row0 = rt * SI_ROWS + wave * 32;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)si_smem));
  int* tab = reinterpret_cast<int*>(si_smem + 2 * STAGE);
  int outside = s.C > SI_TAB;        // (a table that holds all says whether any group has zeros outside int8)
  for (int c = tid; c < min(s.C, SI_TAB); c += 64 * NW) {
    tab[c] = describe_chunk<REF>(a, c, tb, row0);
    outside |= digits_w(tab[c]);
  }
  outside = __syncthreads_or(outside);
  auto chunk_info = [&](int c) { return __builtin_amdgcn_readfirstlane(c < SI_TAB ? tab[c] : describe_chunk<REF>(a, c, tb, row0)); };
  auto from = [&](int c, int& info) {              // the first chunk from c on with digits
    for (; c < s.C; ++c) {
      info = chunk_info(c);
      if (digits_x(info) && (!REF || digits_w(info))) break;
    }
    return c;
  };
  const double base = sum_base(s.m, a.row_exp[row0 + l32]);
  double y[16], low[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    y[v] = base;
    low[v] = 0.0;
  }
  const char* q0 = a.Q + (int64_t)(row0 >> 5) * s.C * KS * 1024;
  Tile<KS, 1> tl;
  auto load_first = [&](int c) {
    tl.load_codes(q0 + (int64_t)c * KS * 1024, 0, lane * 16);
    tl.load_scales(REF ? a.mt.wunit + (int64_t)c * s.npad + row0 : a.S + (int64_t)(c / s.nchg) * s.npad + row0, l32);
  };
  auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };   // (what the compiler does not see is the same in all lanes)
  auto stage = [&](int c, int info, int to) {
    const char* src = a.Xd + ((int64_t)c * s.TB + tb) * SI_MAXD * KS * 1024;
    for (int i = wave; i < digits_x(info) * KS; i += NW) lds_load16((unsigned)uniform((int)(lds0 + to * STAGE + i * 1024)), lane * 16, src + i * 1024);
  };
  int info = 0, next_info = 0, buf = 0, c = from(0, info);
  if (c < s.C) {
    stage(c, info, 0);
    load_first(c);
  }
  while (c < s.C) {
    const int nd = digits_x(info), sets = REF ? digits_w(info) : 1, next = from(c + 1, next_info);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (next < s.C) stage(next, next_info, buf ^ 1);
    const char* x = si_smem + buf * STAGE + lane * 16;
    const double sc = tl.s[0];
    for (int j = 0; j < sets; ++j) {
      for (int p = (nd - 1) >> 1; p >= 0; --p) {
        v16i acc[1];
        __builtin_amdgcn_s_setprio(1);
        tl.pair(x, p, 2 * p + 1 < nd, acc);
        __builtin_amdgcn_s_setprio(0);
        if (p == 0) {
          if (j + 1 < sets)
            tl.load_codes(q0 + (j + 1) * a.plane + (int64_t)c * KS * 1024, 0, lane * 16);
          else if (next < s.C)
            load_first(next);
        }
        const double f = ldexp(sc, exponent_x(info) + 16 * p + (REF ? 8 * j : 0));
#pragma unroll
        for (int v = 0; v < 16; ++v) add_compensated(y[v], low[v], f, (double)acc[0][v]);
      }
    }
    c = next;
    info = next_info;
    buf ^= 1;
  }
  if (!REF && outside) {
    for (int c = 0; c < s.C; c += s.nchg)
      if (digits_w(chunk_info(c))) add_zeros(a, c, tb, row0, lane, y, low);
  }
  store_twice<REF>(a, row0, tb, lane, base, y, low);
}

template <int KS>
slim_status outputs_launch(slim_ctx* ctx, const char* name, const OutArgs& a, bool ref, slim_int_sums sums) {
  const dim3 grid(a.s.RT * a.s.TB);
  const size_t table = sizeof(int) * std::min(a.s.C, SI_TAB);
  if (sums == slim_int_sums::by_pairs) {
    const size_t smem = 2 * SI_MAXD * KS * 1024 + table;
    if (ref)
      SLIM_LAUNCH(ctx, slim_prof_name(name, "int_outputs_by_pairs"), (int_outputs_by_pairs<KS, true>), grid, dim3(512), smem, a);
    else
      SLIM_LAUNCH(ctx, slim_prof_name(name, "int_outputs_by_pairs"), (int_outputs_by_pairs<KS, false>), grid, dim3(512), smem, a);
  } else if (sums == slim_int_sums::twice) {
    const size_t smem = 2 * SI_MAXD * KS * 1024 + table;
    if (ref)
      SLIM_LAUNCH(ctx, name, (int_outputs_twice<KS, true>), dim3(2 * grid.x), dim3(256), smem, a);
    else
      SLIM_LAUNCH(ctx, name, (int_outputs_twice<KS, false>), dim3(2 * grid.x), dim3(256), smem, a);
  } else {
    const size_t smem = 2 * Tile<KS, 2>::STAGE + table;
    if (ref)
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, true>), grid, dim3(256), smem, a);
    else
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, false>), grid, dim3(256), smem, a);
  }
  return SLIM_OK;
}

template <typename T>
slim_status x_digits(slim_ctx* ctx, const IntShape& s, const IntMeta& mt, const T* X, int64_t ldx, char* Xd, double* SX) {
  SLIM_LAUNCH(ctx, "int_x_digits", int_x_digits<T>, dim3(slim_cdiv(s.TB, 4), s.k), dim3(256), 0, X, ldx, s, mt, Xd, SX);
  return SLIM_OK;
}
template <typename T>
slim_status w_units(slim_ctx* ctx, const IntShape& s, const IntMeta& mt, const T* W, int64_t ldw) {
  SLIM_LAUNCH(ctx, "int_w_units", int_w_units<T>, dim3(s.npad / 16, std::min(slim_cdiv(s.k, 4), 8)), dim3(256), 0, W, ldw, s, mt);
  return SLIM_OK;
}

}  // namespace

IntShape slim_int_shape(int n, int m, int beta, int64_t t_s) {
  IntShape s;
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
  s.RT = s.npad / SI_ROWS;
  s.tpad = slim_cdiv(t_s, SI_TOK) * SI_TOK;
  s.TB = s.tpad / SI_TOK;
  return s;
}

slim_status slim_int_clear(slim_ctx* ctx, const IntMeta& mt, int* rest, int nrest) {
  SLIM_LAUNCH(ctx, "int_clear", int_clear, dim3(slim_cdiv(nrest, 256)), dim3(256), 0, mt, rest, nrest);
  return SLIM_OK;
}
slim_status slim_int_w_units(slim_ctx* ctx, const IntShape& s, const IntMeta& mt, const void* W, slim_dtype dt, int64_t ldw) {
  return dt == SLIM_F16    ? w_units(ctx, s, mt, static_cast<const __half*>(W), ldw)
         : dt == SLIM_BF16 ? w_units(ctx, s, mt, static_cast<const __hip_bfloat16*>(W), ldw)
                           : w_units(ctx, s, mt, static_cast<const float*>(W), ldw);
}
slim_status slim_int_x_digits(slim_ctx* ctx, const IntShape& s, const IntMeta& mt, const void* X, slim_dtype dt, int64_t ldx, char* Xd, double* SX) {
  return dt == SLIM_F16 ? x_digits(ctx, s, mt, static_cast<const __half*>(X), ldx, Xd, SX)
                        : x_digits(ctx, s, mt, static_cast<const __hip_bfloat16*>(X), ldx, Xd, SX);
}
slim_status slim_int_g_digits(slim_ctx* ctx, const IntShape& s, const IntMeta& mt, const float* G, int64_t ldg, int* work, int* token_unit,
                              char* Xd, double* SX, double* SXlo) {
  const dim3 tgrid(slim_cdiv(s.ts, 256)), block(256);
  SLIM_LAUNCH(ctx, "int_g_clear", int_g_clear, tgrid, block, 0, s.ts, work);
  SLIM_LAUNCH(ctx, "int_g_stats", int_g_stats, dim3(slim_cdiv(s.ts, 1024), std::min(s.m, 128)), block, 0, G, ldg, s, work);
  SLIM_LAUNCH(ctx, "int_g_units", int_g_units, tgrid, block, 0, s.ts, work, token_unit);
  SLIM_LAUNCH(ctx, "int_g_digits", int_g_digits, dim3(slim_cdiv(s.TB, 4), s.k), block, 0, G, ldg, s, mt.x, token_unit, Xd, SX, SXlo);
  SLIM_LAUNCH(ctx, "int_g_cost", int_g_cost, dim3(1), dim3(1024), 0, mt.x, (int64_t)s.C * s.TB, work);
  return SLIM_OK;
}
bool slim_int_pairs_pay(int cost) { return cost < TWICE_CHUNK; }
slim_status slim_int_outputs(slim_ctx* ctx, const char* name, const OutArgs& a, bool ref, slim_int_sums sums) {
  return a.s.ks == 1   ? outputs_launch<1>(ctx, name, a, ref, sums)
         : a.s.ks == 2 ? outputs_launch<2>(ctx, name, a, ref, sums)
                       : outputs_launch<4>(ctx, name, a, ref, sums);
}
