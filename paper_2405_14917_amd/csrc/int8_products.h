// Products on the int8 matrix cores whose results are exact up to the rounding of the fp64 accumulation: a matrix of
// weights as small integers with one scale per (row, group), or as base-256 digits, times a matrix of tokens (activations, or
// the columns of a Gram matrix) as base-256 digits.
//   * The token side is integers times a power of two per 32 tokens of a chunk of channels (or per token), cut into signed
//     digits (balanced: -128 .. 127); of every such block only the digits in use are kept, one to seven.
//   * A fake-quantised weight is scale * (q - z) with a small integer q - z: one int8 matrix.  Weights as they are become
//     digits the same way, with a power of two per row and chunk (two to four digits for 16-bit weights).
//   * A chunk's products of digits are summed exactly in int32 (128 channels of 128 * 128 * 257 < 2^31 for two digits chained by
//     a shift) and enter the fp64 outputs with one rounding per pair of digits; the fp64 matrix cores round after every four
//     channels.
#ifndef SLIM_INT8_PRODUCTS_H
#define SLIM_INT8_PRODUCTS_H

#include <limits.h>

#include "slim_device.h"
#include "slim_internal.h"

namespace slimint {

using namespace slimdev;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int SI_MAXD = 7;         // digits of a value
constexpr int SI_ROWS = 256, SI_TOK = 32;   // outputs and tokens per workgroup of the products
constexpr int SI_CHUNK = 128;      // most channels whose products are summed in int32

// Shapes of the operands.  A group is cut into chunks of `chk` channels (32, 64 or 128, the last ones padded with zeros); an
// operand fragment is 1 KiB: 32 rows (of W) or tokens x 32 channels as the 64 lanes of v_mfma_i32_32x32x32_i8 hold them
// (lane l: row l % 32, channels 16 (l / 32) .. + 15).
struct IntShape {
  int n, m, beta, k;
  int64_t ts;
  int chk, ks, nchg, C;            // channels per chunk, fragments per chunk, chunks per group, chunks
  int npad, RB, RT;                // rows padded to SI_ROWS, blocks of 32 rows, tiles of SI_ROWS
  int tpad, TB;                    // tokens padded to SI_TOK, blocks of 32
};

// What the kernels have to know about the digits.
struct IntMeta {
  int* x;                          // 2 C TB: exponent of the lowest digit in use and digits in use, per chunk and token block
  uint8_t* w;                      // C x npad / 16: digits in use of 16 rows of a chunk of W, a bit for each
  double* wunit;                   // C x npad: 2^(exponent of the lowest digit) of a row's weights in a chunk
  int* nonfinite;                  // non-finite inputs seen
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
// The unit of a block of values: their last digit, but no more than 53 digits below the largest one, whose float bits are mx.
// (Rounding there is by 2^-54 of the block's largest value.)
__device__ __forceinline__ int block_unit(unsigned mx, int lsb) {
  unsigned mant;
  int e0;
  split_float(mx, mant, e0);
  return mx ? max(lsb, e0 + (31 - __builtin_clz(mant)) - 53) : 0;
}
// balanced digits that hold magnitudes up to v (of at most 55 bits): nd of them reach 0x7f..7f
__device__ __forceinline__ int digits_for(uint64_t v) {
  if (v == 0) return 0;
  const int nd = (64 - __builtin_clzll(v)) / 8 + 1;
  return nd + (v > 0x007f7f7f7f7f7f7full >> (56 - 8 * min(nd, 7)) ? 1 : 0);
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

// Byte offset of channel j (of group g) of row `row` in operand order, for four channels at a time
__device__ __forceinline__ int64_t operand_offset(const IntShape& s, int row, int g, int j, int& chunk) {
  const int cc = j / s.chk, jj = j - cc * s.chk;
  chunk = g * s.nchg + cc;
  return (((int64_t)(row >> 5) * s.C + chunk) * s.ks + (jj >> 5)) * 1024 + ((jj >> 4) & 1) * 512 + (row & 31) * 16 + (jj & 15);
}
// digits in use of the weights of the 256 rows around `row` in a chunk
__device__ __forceinline__ int digits_of_rows(const IntShape& s, const uint8_t* w, int c, int row) {
  const uint4 m = *reinterpret_cast<const uint4*>(w + (int64_t)c * (s.npad / 16) + (row / SI_ROWS) * (SI_ROWS / 16));
  unsigned u = (m.x | m.y) | (m.z | m.w);
  u |= u >> 16;
  return __popc((u | (u >> 8)) & 255u);
}
// the digits of four weights in units of `wunit`, plane by plane
__device__ __forceinline__ void store_digits(char* Wd, int64_t plane, int64_t dst, const unsigned (&bits)[4], double wunit, int nd) {
  const int unit = ((__double2hiint(wunit) >> 20) & 2047) - 1023;
  uint64_t u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = digit_bytes(fixed_point(bits[i], unit));
  for (int d = 0; d < nd; ++d) {
    unsigned word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      word |= ((unsigned)u[i] & 255u) << (8 * i);
      u[i] >>= 8;
    }
    *reinterpret_cast<unsigned*>(Wd + d * plane + dst) = word;
  }
}

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

// The same for sums of which the difference of two is wanted: what an addition rounds away is kept in lo.  y starts from a
// constant above every partial sum (sum_base), so y - y' is exact and lo holds f a - (y' - y) to its own last digits.
__device__ __forceinline__ void add_compensated(double& y, double& lo, double f, double a) {
  const double s = fma(f, a, y);
  lo += fma(f, a, y - s);
  y = s;
}

// 1.5 * 2^e, e two above any partial sum of a row's integers times scale (times a token's digits, below 2^54 units): with
// wexp - ROW_EXP_BIAS the exponent above the row's largest weight, and W_hat and the parts it is summed from within 2^9 of that.
// (About 2^24 above the sums themselves, which leaves them some 75 bits.)
constexpr int ROW_EXP_BIAS = 2048;        // (a row of zeros keeps 0)
__device__ __forceinline__ double sum_base(int m, int wexp) {
  return ldexp(1.5, 54 + (32 - __builtin_clz(m)) + 9 + 2 + (wexp ? wexp - ROW_EXP_BIAS : 0));
}

__device__ __forceinline__ void lds_load16(unsigned lds_addr, unsigned voff, const char* gbase) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(gbase) : "m0");
#else
  (void)lds_addr, (void)voff, (void)gbase;
#endif
}

// What a chunk's digits are, in one word: digits in use of X (3 bits) and of W (3 bits), exponent of X's lowest.
__device__ __forceinline__ int digits_word(const int* x, int w) { return x[1] | (w << 3) | (x[0] * 64); }
__device__ __forceinline__ int digits_x(int d) { return d & 7; }
__device__ __forceinline__ int digits_w(int d) { return (d >> 3) & 7; }
__device__ __forceinline__ int exponent_x(int d) { return d >> 6; }

// A stage in one word: chunk, its first digit, digits (all of a chunk's at most), and whether it is the chunk's first.
static_assert(SI_MAXD <= 7, "three bits hold a stage's digits");
__device__ __forceinline__ int stage_word(int c, int lo, int nd, int first) { return (c << 8) | (first << 7) | (nd << 4) | lo; }
__device__ __forceinline__ int stage_chunk(int w) { return w >> 8; }
__device__ __forceinline__ int stage_nd(int w) { return (w >> 4) & 7; }
__device__ __forceinline__ int stage_lo(int w) { return w & 15; }
__device__ __forceinline__ bool stage_first(int w) { return (w >> 7) & 1; }
// The digits of a stage for token block tb -> LDS (1 KiB per load, the loads dealt to the wavefronts)
template <int KS, int NW>
__device__ __forceinline__ void stage_digits(const char* Xd, const IntShape& s, int word, int tb, unsigned lds, int wave, int lane) {
  const char* src = Xd + (((int64_t)stage_chunk(word) * s.TB + tb) * SI_MAXD + stage_lo(word)) * KS * 1024;
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
  IntShape s;
  IntMeta mt;
  const char* Xd;
  const double* SX;                // k x tpad: sums of the group's channels of a token (with token_unit: in units)
  const double* SXlo;              // what their rounding leaves (compensated sums)
  const char* Q;                   // codes, or digits of W with planes `plane` bytes apart
  int64_t plane;
  const double* S;                 // k x npad scales of the codes
  const double* Rz;                // k x npad: the part of the zero the codes do not hold, times the scale
  const int* rest;                 // k: rest[g] >= rest_from: some row of the group has such a part
  int rest_from;
  const int* token_unit;           // exponent of each token's unit (INT_MIN: not finite), which mt.x counts from, or nullptr
  double* Y;                       // n x ts
  // compensated sums:
  const int* row_exp;              // npad: exponent above the row's largest weight (sum_base)
  double* Ylo;                     // n x ts: what Y's rounding leaves (REF)
  const double *sub, *sublo;       // n x ts: subtracted from the result
};

}  // namespace slimint

// Host side (int8_products.hip).
slimint::IntShape slim_int_shape(int n, int m, int beta, int64_t ts);
inline int64_t slim_int_plane(const slimint::IntShape& s) { return (int64_t)s.npad * s.C * s.chk; }     // bytes of one int8 matrix
inline size_t slim_int_digits_bytes(const slimint::IntShape& s) { return (size_t)s.C * s.TB * slimint::SI_MAXD * s.ks * 1024; }
slim_status slim_int_clear(slim_ctx* ctx, const slimint::IntMeta& mt, int* rest, int nrest);
// mt.w and mt.wunit
slim_status slim_int_w_units(slim_ctx* ctx, const slimint::IntShape& s, const slimint::IntMeta& mt, const void* W, slim_dtype dt, int64_t ldw);
slim_status slim_int_x_digits(slim_ctx* ctx, const slimint::IntShape& s, const slimint::IntMeta& mt, const void* X, slim_dtype dt, int64_t ldx,
                              char* Xd, double* SX);
// The digits of a fp32 matrix with a unit per token (column): token_unit[ts]; work: 2 ts ints, of which the first then holds what
// sums by pairs of digits would cost (slim_int_pairs_pay).
slim_status slim_int_g_digits(slim_ctx* ctx, const slimint::IntShape& s, const slimint::IntMeta& mt, const float* G, int64_t ldg,
                              int* work, int* token_unit, char* Xd, double* SX, double* SXlo);
bool slim_int_pairs_pay(int cost);
// Y = W X (ref: from the digits of W) or W_hat X (from codes and scales); `twice`, `by_pairs`: Y and Ylo = W X to twice the
// precision, or W_hat X minus (sub, sublo), by the kernel for most G or the one for a G of few digits
enum class slim_int_sums { plain, twice, by_pairs };
slim_status slim_int_outputs(slim_ctx* ctx, const char* name, const slimint::OutArgs& a, bool ref, slim_int_sums sums);

#endif
