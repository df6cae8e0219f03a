// Digits of the operands and the output products on the int8 matrix cores; see int8_products.h.
#include <algorithm>

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

// REF: Y = W X_s from the digits of W; else Y = W_N X_s.
// COMP: sums to twice the precision, for W_hat X - W X (add_compensated).  Four vector instructions per output and pair of
// digits in place of one, and twice the registers, so one tile per wavefront and four wavefronts per SIMD (two tiles and two
// wavefronts, or one and three, are slower).  Those four leave little to hide a barrier behind, so a stage holds all digits of a
// chunk, eight wavefronts share it, and a wavefront in its MFMAs goes before one in its sums: 4096 x 4096 against 4096 columns
// 690 -> 625 us.  What bounds it is the vector work: 491 us with one instruction in place of the four, 590 to 600 without the
// codes' or the digits' way from memory.
template <int KS, bool REF, bool COMP>
__global__ __launch_bounds__(COMP ? 512 : 256, COMP ? 4 : 3) void int_outputs(OutArgs a) {
  constexpr int R = COMP ? 1 : 2, NW = COMP ? 8 : 4;
  constexpr int SD = COMP ? SI_MAXD : SI_STAGE_D;
  using TL = Tile<KS, R, SD>;
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
  // what the chunks' digits are, in LDS
  int* tab = reinterpret_cast<int*>(si_smem + 2 * TL::STAGE);
  auto describe = [&](int c) {
    const int* x = a.mt.x + 2 * ((int64_t)c * s.TB + tb);
    return digits_word(x, REF ? digits_of_rows(s, a.mt.w, c, row0) : 0);
  };
  for (int c = tid; c < min(s.C, SI_TAB); c += 64 * NW) tab[c] = describe(c);
  __syncthreads();
  auto chunk_info = [&](int c) { return __builtin_amdgcn_readfirstlane(c < SI_TAB ? tab[c] : describe(c)); };

  auto base = [&](int r) { return COMP ? sum_base(s.m, a.row_exp[row0 + 32 * r + l32]) : 0.0; };
  double y[R][16], low[COMP ? R : 1][16];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      y[r][v] = base(r);
      low[COMP ? r : 0][v] = 0.0;
    }
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
        if constexpr (COMP) __builtin_amdgcn_s_setprio(1);
        tl.pair(x, p, 2 * p + 1 < nd, acc);
        if constexpr (COMP) __builtin_amdgcn_s_setprio(0);
        if (p == 0) {
          if (j + 1 < sets)
            tl.load_codes(q0 + (j + 1) * a.plane + (int64_t)c * KS * 1024, rstride, lane16);
          else
            load_first(stage_chunk(next));
        }
        const int e = unit + 8 * (lo + 2 * p) + (REF ? 8 * j : 0);
        if constexpr (COMP) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double f = ldexp(sc[r], e);
#pragma unroll
            for (int v = 0; v < 16; ++v) add_compensated(y[r][v], low[r][v], f, (double)acc[r][v]);
          }
        } else {
          add_scaled<R>(y, acc, sc, e);
        }
      }
    }
    const int g = c / s.nchg;
    if (!REF && stage_first(word) && c == g * s.nchg && a.rest[g] >= a.rest_from) {
      // zeros outside int8: what the codes do not hold times the sum of the group's activations
      const double* Rz = a.Rz + (int64_t)g * s.npad + row0 + l32;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const double sx = a.SX[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (COMP) {
            add_compensated(y[r][v], low[r][v], -Rz[32 * r], sx);
            low[r][v] = fma(-Rz[32 * r], a.SXlo[(int64_t)g * s.tpad + tb * 32 + 8 * (v >> 2) + 4 * h + (v & 3)], low[r][v]);
          } else {
            y[r][v] = fma(-Rz[32 * r], sx, y[r][v]);
          }
        }
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
    int tu[4] = {0, 0, 0, 0};
    if (a.token_unit) {
#pragma unroll
      for (int v = 0; v < 4; ++v) tu[v] = a.token_unit[t + v];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row0 + 32 * r + l32;
      if (row >= s.n) continue;
      double o[4], ol[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        o[v] = COMP ? y[r][4 * q + v] - base(r) : y[r][4 * q + v];
        if (a.token_unit) o[v] = tu[v] == INT_MIN ? NAN : ldexp(o[v], tu[v]);
        if constexpr (COMP) {
          const int64_t at = (int64_t)row * s.ts + t + v;
          ol[v] = ldexp(low[r][4 * q + v], tu[v] == INT_MIN ? 0 : tu[v]);
          if (!REF) o[v] = (o[v] - a.sub[at]) + (ol[v] - a.sublo[at]);
        }
      }
      if constexpr (COMP && REF) {
        double* outlo = a.Ylo + (int64_t)row * s.ts + t;
        *reinterpret_cast<double2*>(outlo) = make_double2(ol[0], ol[1]);
        *reinterpret_cast<double2*>(outlo + 2) = make_double2(ol[2], ol[3]);
      }
      double* out = a.Y + (int64_t)row * s.ts + t;
      *reinterpret_cast<double2*>(out) = make_double2(o[0], o[1]);
      *reinterpret_cast<double2*>(out + 2) = make_double2(o[2], o[3]);
    }
  }
}

template <int KS>
slim_status outputs_launch(slim_ctx* ctx, const char* name, const OutArgs& a, bool ref, bool compensated) {
  const dim3 grid(a.s.RT * a.s.TB), block(compensated ? 512 : 256);
  const size_t smem = 2 * (compensated ? Tile<KS, 1, SI_MAXD>::STAGE : Tile<KS, 2>::STAGE) + sizeof(int) * std::min(a.s.C, SI_TAB);
  if (compensated) {
    if (ref)
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, true, true>), grid, block, smem, a);
    else
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, false, true>), grid, block, smem, a);
  } else {
    if (ref)
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, true, false>), grid, block, smem, a);
    else
      SLIM_LAUNCH(ctx, name, (int_outputs<KS, false, false>), grid, block, smem, a);
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
  return SLIM_OK;
}
slim_status slim_int_outputs(slim_ctx* ctx, const char* name, const OutArgs& a, bool ref, bool compensated) {
  return a.s.ks == 1   ? outputs_launch<1>(ctx, name, a, ref, compensated)
         : a.s.ks == 2 ? outputs_launch<2>(ctx, name, a, ref, compensated)
                       : outputs_launch<4>(ctx, name, a, ref, compensated);
}
