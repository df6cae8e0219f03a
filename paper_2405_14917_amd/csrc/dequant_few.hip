// The linear layer on the stored form for up to 64 tokens (a decoding step, a batch of them, a short prompt), in one
// launch: Y = X dequant(W_int)^T on the fp16 / bf16 matrix cores.
//
//  * A workgroup owns 16 RT output rows over ALL input channels; its wavefronts share the channels among them (units of
//    32 UC channels inside a group) and their sums meet in LDS, in a fixed order.  Nothing goes to memory but Y: ranges of
//    groups in several workgroups cost a second launch (5 us of 12 us at 4096 x 4096, one token) and partial sums.
//  * v_mfma_f32_16x16x32 with the tokens as rows of the first operand and the layer's rows as columns of the second: a lane
//    owns one output row per MFMA tile (scale and zero are lane constants) and, with its quarter h of the wavefront,
//    channels 8 h .. 8 h + 7 of every chunk of 32.  So a lane reads its 16 bytes of X as they lie in memory, one dword of
//    the packed words (two where its 8 codes may straddle, widths 3 and 5), and there is nothing to stage or to permute.
//    Token slots past the last token read the last token's row and are not stored.
//  * The operand is q - z, formed exactly in packed fp16: a code OR-ed into the mantissa of 1024.0 minus 1024 + z (width 1,
//    whose zero is 1/2: the code doubled, minus 1024 + 2 z, and half the scale).  bf16 activations take the exact difference
//    on to bf16.  A zero point outside that form is split: the nearest one that has it goes this way, and the rest
//    times the sum of the unit's activations, from the matrix cores too, is subtracted (rare).
//  * Scale and zero are fp64 rows of k values: the workgroup stages those of its rows in LDS, already in the form the
//    lanes use, coalesced; a packed zero point is taken apart there.
//  * The loads of a wavefront's next unit are in flight while it decodes the present one.
//
// What bounds it: decoding (10 to 12 vector instructions per MFMA and 16 x 32 codes; about twice that over the whole kernel at 28672 x 8192,
// with addresses, parameters and scaled sums) and the latency of a few loads in a row; a small layer is bound by the launch.  Against the kernels with ranges of groups (and
// their reduction): 28672 x 8192 at 2 bits, fp16, 16 tokens: 55.0 -> 35.6, now 33.6 us (2.7 TB/s); 4096 x 11008 at 3 bits, bf16, packed
// zero points, 5 tokens, which ran without matrix cores and unpacked the zero points in a launch of its own: 47.2 -> 15.2 us;
// 4096 x 4096, one token: 12.9 -> 9.5 us, of which the way of the call through Python is 9.
#include <algorithm>
#include <type_traits>

#include "dequant_device.h"
#include "slim_device.h"

namespace {

using namespace slimdq;

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int FW_PARAM_BYTES = 40 * 1024;       // LDS for the parameters of one range of groups

struct FewArgs {
  DqArgs d;
  PackedZeros z;                                // words null: d.zero
  int kp;                                       // groups per range of parameters
};

template <bool BF16>
__device__ __forceinline__ float4v mfma(const uint4& a, const uint4& b, float4v c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8v*>(&a), *reinterpret_cast<const bf16x8v*>(&b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const half8v*>(&a), *reinterpret_cast<const half8v*>(&b), c, 0, 0, 0);
}

// The second operand of an MFMA: c_i - z of a lane's 8 B-bit codes, which start at byte s / 8 of (w1 : w0); width 1: 2 c_i - 2 z.
// Bytes go to where they are wanted by v_perm (even codes in the low half, odd ones in the high half), a code stays at its bit of
// the byte and is OR-ed into the mantissa of 1024.0 there, which makes it 1024 + w c with w up to 256, and one fma per
// pair, exact, takes that to c - z: (1024 + w c) / w - (1024 / w + z).  Width 2: 10 instructions per 8 codes in place of 14 with the codes
// shifted to bit 0, width 1: 10 for 13, width 3: 12 for 16, width 4: 12 for 15.  28672 x 8192 at 2 bits: 35.5 -> 33.7 us with 16 tokens.
// The codes are shifted (SHIFT) at width 5, whose codes reach beyond the mantissa, in groups of 32, where the pairs' zeros are formed
// anew for every chunk (4096 x 4096 11.2 -> 11.6 us), and where a wavefront has 64 rows x 32 tokens, whose registers they do not fit
// into (11008 x 4096, 64 tokens: 34 -> 39 us).
template <int B>
struct Pairs;                                    // of the places of a pair's codes, as they repeat
template <>
struct Pairs<1> {                                // (one bit up: the operand is 2 c - 2 z)
  static constexpr int CLASSES = 4;
  static constexpr unsigned MASK[4] = {0x00040002u, 0x00100008u, 0x00400020u, 0x01000080u};
  static constexpr int W[4][2] = {{2, 4}, {8, 16}, {32, 64}, {128, 256}};
};
template <>
struct Pairs<2> {
  static constexpr int CLASSES = 2;
  static constexpr unsigned MASK[2] = {0x000c0003u, 0x00c00030u};
  static constexpr int W[2][2] = {{1, 4}, {16, 64}};
};
template <>
struct Pairs<3> {
  static constexpr int CLASSES = 4;
  static constexpr unsigned MASK[4] = {0x00380007u, 0x000e01c0u, 0x03800070u, 0x00e0001cu};
  static constexpr int W[4][2] = {{1, 8}, {64, 2}, {16, 128}, {4, 32}};
};
template <>
struct Pairs<4> {
  static constexpr int CLASSES = 1;
  static constexpr unsigned MASK[1] = {0x00f0000fu};
  static constexpr int W[1][2] = {{1, 16}};
};
template <int B, bool SHIFT>
constexpr int classes() {
  if constexpr (SHIFT) return 1;
  else return Pairs<B>::CLASSES;
}

// What a lane needs to place the codes of a width: v_perm selectors.
template <int B>
struct Places {
  static constexpr int N = B == 3 || B == 4 ? 4 : 1;
  unsigned sel[N];
  __device__ __forceinline__ explicit Places(int s) {
    const unsigned at = (unsigned)(s >> 3) * 0x01010101u;
    if constexpr (B == 1) sel[0] = 0x0c000c00u + (at & 0x00ff00ffu);
    if constexpr (B == 2) sel[0] = 0x01000100u + at;
    if constexpr (B == 3) {
      sel[0] = 0x01000100u + at;
      sel[1] = 0x02010100u + at;
      sel[2] = 0x02010201u + at;
      sel[3] = 0x03020302u + at;
    }
    if constexpr (B == 4) {
#pragma unroll
      for (int j = 0; j < 4; ++j) sel[j] = 0x0c000c00u + 0x00010001u * j;
    }
  }
};

template <int B>
__device__ __forceinline__ half2v pair_weight(int c) {
  half2v m;
  m[0] = (_Float16)((B == 1 ? 2.0f : 1.0f) / Pairs<B>::W[c][0]);
  m[1] = (_Float16)((B == 1 ? 2.0f : 1.0f) / Pairs<B>::W[c][1]);
  return m;
}

// (1024 + w c) pairs, class by class; SHIFT: w = 1 (width 1: 2)
template <int B, bool SHIFT>
__device__ __forceinline__ void spread(unsigned w0, unsigned w1, const Places<B>& p, int s, unsigned one, unsigned (&t)[4]) {
  if constexpr (SHIFT && B == 1) {
    const unsigned v = w0 >> s, u = ((v << 1) & 0xffffu) | (v << 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = ((u >> (2 * j)) & 0x00020002u) | one;
  } else if constexpr (SHIFT && B == 2) {
    const unsigned v = w0 >> s, u = (v & 0xffffu) | ((v << 14) & 0xffff0000u);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = ((u >> (4 * j)) & 0x00030003u) | one;
  } else if constexpr (SHIFT) {
    constexpr unsigned M = ((1u << B) - 1u) * 0x10001u;
    unsigned x[2];
    if constexpr (B == 5) {
      const uint64_t two = ((uint64_t)w1 << 32) | w0;
      x[0] = (unsigned)(two >> s);
      x[1] = (unsigned)(two >> (s + 4 * B));
    } else {
      x[0] = B == 4 ? w0 : __builtin_amdgcn_alignbit(w1, w0, s);
      x[1] = x[0] >> (4 * B);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned u = (x[i] & 0xffffu) | ((x[i] << (16 - B)) & 0xffff0000u);
      t[2 * i] = (u & M) | one;
      t[2 * i + 1] = ((u >> (2 * B)) & M) | one;
    }
  } else if constexpr (B == 1) {
    const unsigned u = __builtin_amdgcn_perm(w1, w0, p.sel[0]) << 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = (u & Pairs<1>::MASK[j]) | one;
  } else if constexpr (B == 2) {
    const unsigned u = __builtin_amdgcn_perm(w1, w0, p.sel[0]), v = u >> 8;
    t[0] = (u & Pairs<2>::MASK[0]) | one;
    t[1] = (u & Pairs<2>::MASK[1]) | one;
    t[2] = (v & Pairs<2>::MASK[0]) | one;
    t[3] = (v & Pairs<2>::MASK[1]) | one;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      t[j] = (__builtin_amdgcn_perm(w1, w0, p.sel[j]) & Pairs<B>::MASK[j % Pairs<B>::CLASSES]) | one;
  }
}

// 1024 / w + z of the classes, from 1024 + z: integers of at most 2046, which fp16 holds
template <int B, bool SHIFT>
__device__ __forceinline__ void zeros_of(half2v zz, half2v (&z)[classes<B, SHIFT>()]) {
  if constexpr (SHIFT) {
    z[0] = zz;
  } else {
#pragma unroll
    for (int c = 0; c < Pairs<B>::CLASSES; ++c) {
      half2v d;
      d[0] = (_Float16)(1024.0f - 1024.0f * (float)pair_weight<B>(c)[0]);
      d[1] = (_Float16)(1024.0f - 1024.0f * (float)pair_weight<B>(c)[1]);
      z[c] = zz - d;
    }
  }
}

template <int B, bool SHIFT, bool BF16>
__device__ __forceinline__ uint4 minus_zero(const unsigned (&t)[4], const half2v (&z)[classes<B, SHIFT>()]) {
  unsigned o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const half2v v = *reinterpret_cast<const half2v*>(&t[j]);
    half2v d;
    if constexpr (SHIFT)
      d = v - z[0];
    else
      d = __builtin_elementwise_fma(v, pair_weight<B>(j % Pairs<B>::CLASSES), -z[j % Pairs<B>::CLASSES]);
    if constexpr (BF16) {
      // an integer of at most 256 (few_zmax), so the upper 16 bits of the float are the exact bf16 value
      const unsigned lo = __float_as_uint((float)d[0]), hi = __float_as_uint((float)d[1]);
      o[j] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    } else {
      o[j] = *reinterpret_cast<const unsigned*>(&d);
    }
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// Bounds of the zero (doubled at width 1) that the operand carries: 1024 + z0 has to be an integer fp16 holds, and with bf16
// activations c - z0 one that bf16 holds (c <= 31).
template <bool BF16>
constexpr double few_zmax() { return BF16 ? 190.0 : 1022.0; }

// 2 z of (row, group), exactly
template <bool PACKED>
__device__ __forceinline__ double zero_twice(const FewArgs& f, int row, int g) {
  if constexpr (!PACKED) return 2.0 * f.d.zero[(int64_t)row * f.d.k + g];
  const int64_t bit = (int64_t)row * f.z.bits;
  const int64_t w = bit >> 5;
  const int sh = (int)(bit & 31);
  const uint32_t* p = f.z.words + (int64_t)g * f.z.ld + w;
  const uint64_t two = p[0] | ((uint64_t)p[sh + f.z.bits > 32 ? 1 : 0] << 32);    // (the upper half is used only then)
  return (double)((two >> sh) & ((1u << f.z.bits) - 1u));
}

template <bool BF16>
__device__ __forceinline__ double operand_zero(double z2, int b) {
  const double z = b == 1 ? z2 : 0.5 * z2;
  return fmin(fmax(rint(z), -few_zmax<BF16>()), few_zmax<BF16>());
}

template <int UC, int RT, int TT>
struct Unit {
  uint32_t w0[UC][RT], w1[UC][RT];
  uint4 x[UC][TT];
};

template <int B, int UC, int RT, int TT, bool BF16>
__device__ __forceinline__ void multiply(const Unit<UC, RT, TT>& u, int s, unsigned one, const half2v (&zz)[RT],
                                         float4v (&acc)[RT][TT]) {
  const Places<B> p(s);
  constexpr bool SHIFT = B == 5 || UC == 1 || RT * TT == 8;
  half2v z[RT][classes<B, SHIFT>()];
#pragma unroll
  for (int r = 0; r < RT; ++r) zeros_of<B, SHIFT>(zz[r], z[r]);
#pragma unroll
  for (int c = 0; c < UC; ++c)
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      unsigned t[4];
      spread<B, SHIFT>(u.w0[c][r], u.w1[c][r], p, s, one, t);
      const uint4 bf = minus_zero<B, SHIFT, BF16>(t, z[r]);
#pragma unroll
      for (int q = 0; q < TT; ++q) acc[r][q] = mfma<BF16>(u.x[c][q], bf, acc[r][q]);
    }
}

template <int WAVES, int UC, int RT, int TT, bool BF16>
__global__ __launch_bounds__(64 * WAVES) void dequant_few(FewArgs f) {
  constexpr int R = 16 * RT, T = 16 * TT;
  extern __shared__ __align__(16) char smem_few[];
  const DqArgs& a = f.d;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok0 = blockIdx.y * T, tokens = min(T, a.t_x - tok0);
  const int l16 = lane & 15, h = lane >> 4;
  // XCD x (block id mod 8) takes the x-th run of consecutive tiles: neighbours share the lines of the packed words
  const int total = gridDim.x, per = total / 8, rest8 = total % 8, c8 = (int)(blockIdx.x % 8);
  const int row0 = (c8 * per + min(c8, rest8) + (int)(blockIdx.x / 8)) * R;
  const int ldk = f.kp | 1;
  float* sp = reinterpret_cast<float*>(smem_few);                         // [R][ldk] scale (half of it at width 1)
  int* meta = reinterpret_cast<int*>(sp + R * ldk);                        // [kp] 8 start row + width
  _Float16* zp = reinterpret_cast<_Float16*>(meta + f.kp);                 // [R][ldk] 1024 + z0; negative: a rest is left
  const int upg = a.beta / (32 * UC);                                     // units per group

  uint32_t vrow[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) vrow[r] = (uint32_t)min(row0 + 16 * r + l16, a.n - 1) * 4u;
  const char* xtok[TT];
#pragma unroll
  for (int q = 0; q < TT; ++q)
    xtok[q] = static_cast<const char*>(a.X) + ((int64_t)(tok0 + min(16 * q + l16, tokens - 1)) * a.ldx + 8 * h) * 2;

  unsigned one16;                                                         // in a register: an instruction takes one constant
  asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(one16));

  float4v y[RT][TT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int q = 0; q < TT; ++q) y[r][q] = (float4v){0.f, 0.f, 0.f, 0.f};

  auto fetch = [&](int gb, int gi, int sb, Unit<UC, RT, TT>& d) {
    const int mt = __builtin_amdgcn_readfirstlane(meta[gi]), b = mt & 7;
    // quarter h starts at bit 8 b h of a chunk; its codes reach the next word where the width is 3 or 5.  A skipped group
    // reads the start of X instead.
    const int wi = (8 * b * h) >> 5, in = (8 * b * h) & 31;
    const uint32_t on = b ? ~0u : 0u, ld4 = (uint32_t)a.ldp * 4u;
    const uint32_t v0 = (uint32_t)wi * ld4, v1 = v0 + (in + 8 * b > 32 ? ld4 : 0u);
    const char* base = b ? reinterpret_cast<const char*>(a.packed + ((int64_t)(mt >> 3) + (int64_t)sb * UC * b) * a.ldp)
                         : static_cast<const char*>(a.X);
    const int64_t step = (int64_t)b * a.ldp * 4;
#pragma unroll
    for (int c = 0; c < UC; ++c)
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        d.w0[c][r] = *reinterpret_cast<const uint32_t*>(base + c * step + ((v0 + vrow[r]) & on));
        d.w1[c][r] = *reinterpret_cast<const uint32_t*>(base + c * step + ((v1 + vrow[r]) & on));
      }
    const int64_t col = ((int64_t)(gb + gi) * a.beta + sb * UC * 32) * 2;
#pragma unroll
    for (int c = 0; c < UC; ++c)
#pragma unroll
      for (int q = 0; q < TT; ++q) d.x[c][q] = *reinterpret_cast<const uint4*>(xtok[q] + col + c * 64);
  };
  auto consume = [&](int gb, int gi, const Unit<UC, RT, TT>& d) {
    const int b = __builtin_amdgcn_readfirstlane(meta[gi]) & 7, s = (8 * b * h) & 31;
    half2v zz[RT];
    bool left[RT], any = false;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const _Float16 z = zp[(16 * r + l16) * ldk + gi];
      left[r] = z < (_Float16)0.f;
      any |= left[r];
      zz[r][0] = zz[r][1] = left[r] ? -z : z;
    }
    float4v acc[RT][TT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int q = 0; q < TT; ++q) acc[r][q] = (float4v){0.f, 0.f, 0.f, 0.f};
    switch (b) {                              // the same for the whole wavefront
      case 0: return;
      case 1: multiply<1, UC, RT, TT, BF16>(d, s, one16, zz, acc); break;
      case 2: multiply<2, UC, RT, TT, BF16>(d, s, one16, zz, acc); break;
      case 3: multiply<3, UC, RT, TT, BF16>(d, s, one16, zz, acc); break;
      case 4: multiply<4, UC, RT, TT, BF16>(d, s, one16, zz, acc); break;
      default: multiply<5, UC, RT, TT, BF16>(d, s, one16, zz, acc); break;
    }
    if (__builtin_amdgcn_ballot_w64(any) != 0) {
      const unsigned one = BF16 ? 0x3f803f80u : 0x3c003c00u;
      const uint4 ones = make_uint4(one, one, one, one);
#pragma unroll
      for (int q = 0; q < TT; ++q) {
        float4v sx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < UC; ++c) sx = mfma<BF16>(d.x[c][q], ones, sx);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (left[r]) {
            const int row = min(row0 + 16 * r + l16, a.n - 1);
            const double z2 = f.z.words ? zero_twice<true>(f, row, gb + gi) : zero_twice<false>(f, row, gb + gi);
            const float rest = (float)((b == 1 ? z2 : 0.5 * z2) - operand_zero<BF16>(z2, b));
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[r][q][v] = fmaf(-rest, sx[v], acc[r][q][v]);
          }
      }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const float sc = sp[(16 * r + l16) * ldk + gi];
#pragma unroll
      for (int q = 0; q < TT; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[r][q][v] = fmaf(sc, acc[r][q][v], y[r][q][v]);
    }
  };

  for (int gb = 0; gb < a.k; gb += f.kp) {
    const int gc = min(f.kp, a.k - gb);
    if (gb > 0) __syncthreads();
    for (int i = tid; i < gc; i += 64 * WAVES) meta[i] = a.row_off[gb + i] * 8 + checked_width(a, gb + i);
    __syncthreads();
    const int nu = gc * upg, u0 = (int)((int64_t)nu * wave / WAVES), u1 = (int)((int64_t)nu * (wave + 1) / WAVES);
    Unit<UC, RT, TT> p, n;
    int gi = u0 / upg, sb = u0 - gi * upg;                                // of the unit that is fetched next
    auto advance = [&]() {
      if (++sb == upg) {
        sb = 0;
        ++gi;
      }
    };
    if (u0 < u1) fetch(gb, gi, sb, p);
    // Parameters: a wavefront takes 64 / gw rows of gw groups at a time, the loads of PF such steps together
    const int lg = gc > 32 ? 6 : gc > 16 ? 5 : gc > 8 ? 4 : 3, gw = 1 << lg, rows = 64 >> lg;
    constexpr int PF = 4;
    auto parameters = [&](auto packed_zeros) {
      constexpr bool PACKED = decltype(packed_zeros)::value;
      for (int i0 = 0; i0 < gc; i0 += gw) {
        const int i = i0 + (lane & (gw - 1)), ic = min(i, gc - 1), g = gb + ic, b = meta[ic] & 7;
        for (int r0 = wave * rows + (lane >> lg); r0 < R; r0 += PF * WAVES * rows) {
          double sc[PF], z2[PF];
  #pragma unroll
          for (int j = 0; j < PF; ++j) {
            const int row = min(row0 + r0 + j * WAVES * rows, a.n - 1);
            sc[j] = a.scale[(int64_t)row * a.k + g];
            z2[j] = zero_twice<PACKED>(f, row, g);
          }
  #pragma unroll
          for (int j = 0; j < PF; ++j) {
            const int r = r0 + j * WAVES * rows;
            if (r >= R || i >= gc) continue;
            const double z0 = operand_zero<BF16>(z2[j], b);
            const float zc = (float)(1024.0 + z0);
            sp[r * ldk + i] = (float)((b == 1 ? 0.5 : 1.0) * sc[j]);
            zp[r * ldk + i] = (_Float16)((b == 1 ? z2[j] : 0.5 * z2[j]) != z0 ? -zc : zc);
          }
        }
      }
    };
    if (f.z.words) parameters(std::true_type{}); else parameters(std::false_type{});
    __syncthreads();

    for (int u = u0; u < u1; u += 2) {
      int g = gi;
      if (u + 1 < u1) advance();                // behind the last unit it is fetched once more
      fetch(gb, gi, sb, n);
      consume(gb, g, p);
      if (u + 1 == u1) break;
      g = gi;
      if (u + 2 < u1) advance();
      fetch(gb, gi, sb, p);
      consume(gb, g, n);
    }
  }

  // the wavefronts' sums, added in their order
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem_few);                         // [WAVES][T][R]
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int q = 0; q < TT; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[(wave * T + 16 * q + 4 * h + v) * R + 16 * r + l16] = y[r][q][v];
  __syncthreads();
  for (int idx = tid; idx < tokens * R; idx += 64 * WAVES) {
    const int t = idx / R, r = idx % R;
    if (row0 + r >= a.n) continue;
    float s = red[t * R + r];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[(w * T + t) * R + r];
    a.out[(int64_t)(tok0 + t) * a.ldo + row0 + r] = s;
  }
}

template <int WAVES, int UC, int RT, int TT, bool BF16>
slim_status launch(slim_ctx* ctx, FewArgs& f) {
  constexpr int R = 16 * RT;
  f.kp = std::min(f.d.k, FW_PARAM_BYTES / (R * 6) - 2);
  const size_t params = (size_t)R * (f.kp | 1) * 6 + sizeof(int) * f.kp, sums = (size_t)WAVES * 16 * TT * R * sizeof(float);
  const size_t smem = (std::max(params, sums) + 15) / 16 * 16;
  if (smem > 64 * 1024)
    SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(dequant_few<WAVES, UC, RT, TT, BF16>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  SLIM_LAUNCH(ctx, "dequant_matmul@dequant_few", (dequant_few<WAVES, UC, RT, TT, BF16>), dim3(slim_cdiv(f.d.n, R), slim_cdiv(f.d.t_x, 16 * TT)), dim3(64 * WAVES),
              smem, f);
  return SLIM_OK;
}

template <int WAVES, int RT, int TT>
slim_status launch(slim_ctx* ctx, FewArgs& f) {
  const bool bf = f.d.x_bf16 != 0;
  if (f.d.beta % 128 == 0) return bf ? launch<WAVES, 4, RT, TT, true>(ctx, f) : launch<WAVES, 4, RT, TT, false>(ctx, f);
  if (f.d.beta % 64 == 0) return bf ? launch<WAVES, 2, RT, TT, true>(ctx, f) : launch<WAVES, 2, RT, TT, false>(ctx, f);
  return bf ? launch<WAVES, 1, RT, TT, true>(ctx, f) : launch<WAVES, 1, RT, TT, false>(ctx, f);
}

}  // namespace

bool slim_dq_few_takes(int64_t t_x, int64_t ldp, int beta, const void* X, int64_t ldx) {
  return t_x <= DQ_FEW_TOKENS && slim_aligned16(X) && ldx % 8 == 0 && beta % 32 == 0 && ldp < (int64_t)1 << 27;
}

// The tile by the layer's rows, so that every CU has a workgroup and the activations are not read more often than needed
// (each workgroup reads all of X).  It does not depend on the tokens: the order of a row's sums follows from it, and a token's
// outputs are the same bytes whichever other tokens share its call.  Measured in us, rows per tile / wavefronts per workgroup:
//   n = 4096, m = 11008, 1 token:   16/16 13.6, 16/8 15.0, 32/8 21.3, 64/8 34.6;  16 tokens: 19.0, 17.3, 22.2, 35.6
//   n = 11008, m = 4096, 16 tokens: 16/8 17.5, 32/8 15.0, 64/8 14.6, 64/4 20.4;   32 tokens: 29.9, 25.3, 17.0, 22.6
//   n = 28672, m = 8192, 16 tokens: 16/8 68.8, 32/8 52.4, 64/8 38.9, 64/4 34.5;   32 tokens: 134, 84.5, 55.2, 57.6
slim_status slim_dq_few_launch(slim_ctx* ctx, const DqArgs& d, const PackedZeros* zp) {
  FewArgs f;
  f.d = d;
  f.z = zp ? *zp : PackedZeros{nullptr, 0, 0};
  f.kp = 0;
  const int cus = std::max(1, ctx->num_cus);
  const bool two = d.t_x > 16;
  if (d.n > 64 * cus) return two ? launch<4, 4, 2>(ctx, f) : launch<4, 4, 1>(ctx, f);
  if (d.n > 32 * cus) return two ? launch<8, 4, 2>(ctx, f) : launch<8, 4, 1>(ctx, f);
  if (d.n > 16 * cus) return two ? launch<8, 2, 2>(ctx, f) : launch<8, 2, 1>(ctx, f);
  return two ? launch<8, 1, 2>(ctx, f) : launch<8, 1, 1>(ctx, f);
}
