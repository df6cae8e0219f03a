// The linear layer on the stored form for many tokens (a prompt, or the calibration activations handed on to the next
// layer): Y = X dequant(W_int)^T on the fp16 / bf16 matrix cores, every packed word decoded once per 128 tokens.
//
//  * Workgroup tile: 128 (or 64) tokens x 128 output rows, 4 wavefronts, each all of the tile's tokens x 32
//    rows, with the tokens as rows of v_mfma_f32_32x32x16's first operand and the layer's rows as columns of the second:
//    a lane owns one output row, whose scale and zero are lane constants, and 16 tokens per MFMA tile.
//  * The weights never exist in memory in decoded form: a lane takes the words of its row from LDS and forms 2 (q - z)
//    exactly in packed fp16 (a code OR-ed into the mantissa of 1024.0 minus 1024 + 2 z), 17 instructions per eight codes,
//    which serve 4 MFMAs (128 tokens); bf16 activations need three more per pair to turn the exact difference into
//    bf16.  The width of a group is a run-time scalar in all of this: a branch per width around the MFMAs made the compiler
//    keep the sums twice and copy them.  The two halves of a wavefront take the two halves of a slab's channels (the contraction may run in any
//    order as long as both operands agree), so a lane reads only the words it decodes.
//  * Per group the fp32 sums of the matrix cores are multiplied by the scale (rounded to fp32) and added in fp32, as in the
//    kernel for few tokens.
//  * X, the words and the parameters go from memory to LDS directly, three stages of one slab (64 channels; 32 where 64
//    does not divide the group), two of them in flight; one wait and one barrier per slab.
//
// What bounds it: issue (counters: 9.5 vector instructions per MFMA, itself included, i.e. 152 per wavefront and slab, beside 97
// scalar ones) and the barrier per slab; the matrix cores are busy 39 % of the time.  4096 x 11008 at 2 bits, 2048 tokens: 212 us (870 TFLOP/s)
// against 2848 us for 128 slices of 16 tokens, each of which reads and decodes the whole layer.
#include <algorithm>

#include "dequant_device.h"

namespace {

using namespace slimdq;

constexpr int PG_ROWS = 128, PG_THREADS = 256, PG_STAGES = 3, PG_MAXB = 5;
constexpr int PG_BAND = 8;                       // token tiles per band of the tile order
constexpr int PG_MAXK = 16384;                   // groups: three stages (at most 69 KiB) and these in 160 KiB of LDS

struct PgArgs {
  DqArgs d;
  int tiles_r, tiles_t;                          // tiles along the layer's rows and along the tokens
  __half* hand;                                  // HAND: n x t_x (ldh), in place of d.out
  int64_t ldh;
};

__device__ __forceinline__ void load_lds16(unsigned lds_addr, unsigned voff, const char* gbase) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(gbase) : "m0");
#else
  (void)lds_addr, (void)voff, (void)gbase;
#endif
}
__device__ __forceinline__ void load_lds4(unsigned lds_addr, unsigned voff, const char* gbase) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(lds_addr), "v"(voff), "s"(gbase) : "m0");
#else
  (void)lds_addr, (void)voff, (void)gbase;
#endif
}

// Eight codes of b bits whose first one starts at bit 1 of the stream (hi : lo) -> packed fp16 pairs
// (1024 + 2 c_{2j}, 1024 + 2 c_{2j+1}); mask = (2^b - 1) * 0x20002.  Even codes go to the low half of u, odd ones to the
// high half, so that one shift serves both; two pairs fit (1 + 3 b <= 16).
__device__ __forceinline__ void spread_codes_rt(unsigned hi, unsigned lo, int b, unsigned mask, unsigned one, unsigned (&t)[4]) {
  const unsigned u0 = (lo & 0xffffu) | ((lo << (16 - b)) & 0xffff0000u);
  const unsigned x2 = __builtin_amdgcn_alignbit(hi, lo, 4 * b);
  const unsigned u1 = (x2 & 0xffffu) | ((x2 << (16 - b)) & 0xffff0000u);
  t[0] = (u0 & mask) | one;
  t[1] = ((u0 >> (2 * b)) & mask) | one;
  t[2] = (u1 & mask) | one;
  t[3] = ((u1 >> (2 * b)) & mask) | one;
}

template <bool BF16>
__device__ __forceinline__ float16v mfma(const uint4& a, const uint4& b, float16v c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8v*>(&a), *reinterpret_cast<const bf16x8v*>(&b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const half8v*>(&a), *reinterpret_cast<const half8v*>(&b), c, 0, 0, 0);
}

// Second operand of one MFMA step: 2 (q - z) of eight codes, from the spread codes and 1024 + 2 z.
template <bool BF16>
__device__ __forceinline__ uint4 decode(const unsigned (&t)[4], half2v zz) {
  unsigned o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const half2v d = *reinterpret_cast<const half2v*>(&t[j]) - zz;
    if constexpr (BF16) {
      // |2 (q - z)| <= 256 here (PG_ZMAX), so the upper 16 bits of the float are the exact bf16 value
      const unsigned lo = __float_as_uint((float)d[0]), hi = __float_as_uint((float)d[1]);
      o[j] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
    } else {
      o[j] = *reinterpret_cast<const unsigned*>(&d);
    }
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// Bounds of the part z0 of 2 z that the operand carries: 1024 + z0 has to be an integer fp16 holds (fp16 activations), and
// 2 q - z0 one that bf16 holds (bf16 activations; 2 q <= 62).
template <bool BF16>
constexpr double pg_zmax() { return BF16 ? 190.0 : 1022.0; }

// LDS of one stage, in bytes
template <int SLAB, int TOK>
struct Stage {
  static constexpr int ROWB = SLAB * 2;                       // bytes of a token's row of a slab
  static constexpr int XB = TOK * ROWB;
  static constexpr int WROWS = PG_MAXB * SLAB / 32;           // word rows of a slab at the widest width
  static constexpr int WB = WROWS * PG_ROWS * 4;
  static constexpr int PB = 2 * PG_ROWS * 8;                  // scale and zero of the rows, as stored
  static constexpr int BYTES = XB + WB + PB;
};

template <int SLAB, int TOK, bool BF16>
struct Wave {
  using S = Stage<SLAB, TOK>;
  static constexpr int TA = TOK / 32, STEPS = SLAB / 16, NCH = SLAB / 8;

  // position (16-byte units) of chunk c of token row r: 16 lanes that read one chunk of 16 consecutive rows hit
  // sixteen different groups of four banks (64 banks of 4 bytes)
  static __device__ __forceinline__ int swz(int r, int c) { return c ^ ((r / (256 / S::ROWB)) & (NCH - 1)); }

  // What a lane needs to decode a group of b-bit codes: where its words start in a stage and the bits of its units.
  struct Codes {
    int b;
    unsigned mask, one;                  // (one: in a vector register, an instruction takes one scalar operand)
    half2v zz;                           // 1024 + z0
  };

  // One slab: STEPS MFMA steps; FIRST: the sums of the group start here.
  template <bool WIDE, bool FIRST>
  static __device__ __forceinline__ void slab(const char* stage, int lane, int wave, const Codes& cd, float16v (&acc)[TA]) {
    const int l32 = lane & 31, h = lane >> 5;
    const char* xr = stage + l32 * S::ROWB;
    // SLAB 64: half h of the wavefront takes channels 32 h .. 32 h + 31, i.e. the words from h b on
    const unsigned* wl = reinterpret_cast<const unsigned*>(stage + S::XB) + wave * 32 + l32 + (SLAB == 64 ? h * cd.b * PG_ROWS : 0);
    uint4 af[2][TA];
    auto load_a = [&](int st) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
        af[st & 1][i] = *reinterpret_cast<const uint4*>(xr + i * 32 * S::ROWB + swz(l32, st + h * STEPS) * 16);
    };
    unsigned wd[2][3];
    int sh[2];
    // the words around unit st (SLAB 32: st + 2 h), whose codes start at bit 8 b unit: read from the bit before it on
    auto load_w = [&](int st) {
      const int p1 = 8 * cd.b * (SLAB == 64 ? st : st + h * STEPS) - 1;
      const unsigned* q = wl + (p1 >> 5) * PG_ROWS;
      sh[st & 1] = p1 & 31;
      wd[st & 1][0] = q[0];
      wd[st & 1][1] = q[PG_ROWS];
      wd[st & 1][2] = WIDE ? q[2 * PG_ROWS] : 0u;
    };
    auto second = [&](int st) {
      const unsigned* w = wd[st & 1];
      const unsigned lo = __builtin_amdgcn_alignbit(w[1], w[0], sh[st & 1]), hi = __builtin_amdgcn_alignbit(w[2], w[1], sh[st & 1]);
      unsigned t[4];
      spread_codes_rt(hi, lo, cd.b, cd.mask, cd.one, t);
      return decode<BF16>(t, cd.zz);
    };
    load_w(0);
    load_a(0);
    load_w(1);
    uint4 bf = second(0);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      // the next step's operands are read and decoded in the shadow of this step's MFMAs
      __builtin_amdgcn_sched_barrier(0);
      uint4 bn = bf;
      if (st + 1 < STEPS) {
        load_a(st + 1);
        bn = second(st + 1);
      }
      if (st + 2 < STEPS) load_w(st + 2);
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        float16v c = acc[i];
        if (FIRST && st == 0) {
#pragma unroll
          for (int q = 0; q < 16; ++q) c[q] = 0.f;
        }
        acc[i] = mfma<BF16>(af[st & 1][i], bf, c);
      }
      if (st + 1 < STEPS) {
#pragma unroll
        for (int i = 0; i < TA; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, (BF16 ? 32 : 20) / TA, 0);
        }
      }
      bf = bn;
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // A zero point outside the operand's form: the part it does not hold times the sum of the slab's activations (rare).
  static __device__ __forceinline__ void rest_of_zero(const char* stage, int lane, float rest, float16v (&acc)[TA]) {
    const int l32 = lane & 31, h = lane >> 5;
    const char* xr = stage + l32 * S::ROWB;
    const unsigned one = BF16 ? 0x3f803f80u : 0x3c003c00u;
    const uint4 ones = make_uint4(one, one, one, one);
#pragma unroll
    for (int i = 0; i < TA; ++i) {
      float16v sx;
#pragma unroll
      for (int q = 0; q < 16; ++q) sx[q] = 0.f;
#pragma unroll
      for (int st = 0; st < STEPS; ++st)
        sx = mfma<BF16>(*reinterpret_cast<const uint4*>(xr + i * 32 * S::ROWB + swz(l32, st + h * STEPS) * 16), ones, sx);
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][q] = fmaf(-rest, sx[q], acc[i][q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// HAND: the next layer's calibration activations in place of the outputs.  (A kernel of its own, its arguments behind the others': as a
// branch its stores, half as much code again, made the other form up to 1.5 % slower, 5000 x 11008 with 2000 tokens in groups of 32,
// bf16, 609 -> 618 us.)
template <int SLAB, int TOK, bool BF16, bool WIDE, bool HAND>
__global__ __launch_bounds__(PG_THREADS, 2) void dequant_gemm(PgArgs pa) {
  using S = Stage<SLAB, TOK>;
  using W = Wave<SLAB, TOK, BF16>;
  constexpr int TA = W::TA, NCH = W::NCH;
  constexpr int XI = S::XB / 1024 / 4;                        // direct loads of X per wavefront and slab
  extern __shared__ __align__(16) char smem_dq[];
  const DqArgs& a = pa.d;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Tile order: bands of PG_BAND token tiles, inside a band the rows slowest; XCD x (id mod 8) takes the x-th run of
  // consecutive tiles, so that what it works on at one time is a patch that shares token rows and words in its L2.
  const int total = pa.tiles_r * pa.tiles_t, per = total / 8, rest8 = total % 8, c8 = (int)(blockIdx.x % 8);
  const int id = c8 * per + min(c8, rest8) + (int)(blockIdx.x / 8);
  const int full = pa.tiles_r * PG_BAND, band = id / full, inband = id - band * full;
  const int bw = min(PG_BAND, pa.tiles_t - band * PG_BAND);
  const int row0 = (inband / bw) * PG_ROWS, tok0 = (band * PG_BAND + inband % bw) * TOK;
  const int g0 = blockIdx.y * a.gper, g1 = min(a.k, g0 + a.gper);
  const int ns = a.beta / SLAB, units = (g1 - g0) * ns;
  // start row and width of the groups (8 row + width): read from here, one slab ahead, and not from memory, whose loads
  // would have to be waited for behind those of the slabs
  int* meta = reinterpret_cast<int*>(smem_dq + PG_STAGES * S::BYTES);
  for (int i = tid; i < g1 - g0; i += PG_THREADS) meta[i] = a.row_off[g0 + i] * 8 + checked_width(a, g0 + i);
  __syncthreads();

  // X: load i of this wavefront fills 1 KiB of the stage, i.e. 1024 / ROWB token rows; the lane fetches the chunk that
  // belongs at its place
  unsigned xoff[XI];
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int pos = (wave * XI + i) * 64 + lane, r = pos / NCH, c = pos % NCH;
    xoff[i] = (unsigned)((int64_t)min(r, a.t_x - 1 - tok0) * a.ldx * 2 + (unsigned)W::swz(r, c) * 16u);
  }
  const char* xbase = static_cast<const char*>(a.X) + ((int64_t)tok0 * a.ldx + (int64_t)g0 * a.beta) * 2;
  // words: one load is 64 rows of one word row, the wavefronts with an even number take the first 64 rows; parameters: one
  // load is 32 rows of one array (a pair of lanes per value)
  const int rlast = a.n - 1 - row0;
  const unsigned woff = (unsigned)min((wave & 1) * 64 + lane, rlast) * 4u;
  const unsigned poff = (unsigned)((int64_t)min(wave * 32 + (lane >> 1), rlast) * a.k * 8 + (lane & 1) * 4);
  const char* pbase = reinterpret_cast<const char*>(a.scale + (int64_t)row0 * a.k + g0);
  const char* zbase = reinterpret_cast<const char*>(a.zero + (int64_t)row0 * a.k + g0);
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)smem_dq));
  const char* wbase = reinterpret_cast<const char*>(a.packed + (int64_t)(wave >> 1) * a.ldp + row0);
  const int64_t wstep = a.ldp * 8;                            // two word rows

  // The loads run two slabs ahead: slab isb of group igi (start row and width imeta) goes to the stage at ilds.
  int igi = 0, isb = 0, islot = 0, imeta = 0;
  auto meta_of = [&](int gi) { return __builtin_amdgcn_readfirstlane(meta[gi]); };
  auto issue = [&](int next_meta) {
    const int b = imeta & 7, rows = b * (SLAB / 32);
    const unsigned st = lds0 + (unsigned)islot * S::BYTES;
    if (isb == 0) {
      load_lds4(st + S::XB + S::WB + wave * 256, poff, pbase);
      load_lds4(st + S::XB + S::WB + PG_ROWS * 8 + wave * 256, poff, zbase);
      pbase += 8;
      zbase += 8;
    }
    const char* w = wbase + (int64_t)((imeta >> 3) + isb * rows) * a.ldp * 4;
    unsigned wl = st + S::XB + (unsigned)(wave >> 1) * (PG_ROWS * 4) + (unsigned)(wave & 1) * 256;
    for (int i = wave >> 1; i < rows; i += 2) {
      load_lds4(wl, woff, w);
      w += wstep;
      wl += 2 * PG_ROWS * 4;
    }
#pragma unroll
    for (int i = 0; i < XI; ++i) load_lds16(st + (unsigned)(wave * XI + i) * 1024, xoff[i], xbase);
    xbase += S::ROWB;
    islot = (islot == PG_STAGES - 1) ? 0 : islot + 1;
    if (++isb == ns) {
      isb = 0;
      ++igi;
      imeta = next_meta;
    }
  };

  // Sums of sixteen groups, and of those: with up to 344 groups a single running sum would round more often than the
  // kernel for few tokens, which adds ranges of groups.
  float16v y[TA], ysum[TA];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) y[i][q] = ysum[i][q] = 0.f;

  const int gcount = g1 - g0;
  imeta = meta_of(0);
  int cmeta = imeta;                                          // of the group that is multiplied
  issue(meta_of(min(1, gcount - 1)));
  if (units > 1) issue(meta_of(min(igi + 1, gcount - 1)));
  int left = units, gi = 0;
  const char* stage = smem_dq;
  auto arrive = [&]() {
    // Loads complete in order: with at most XI outstanding (the X of the next slab, the last loads issued) everything of
    // this slab has landed.  Behind the last slab nothing follows, so all has to be waited for.
    if (left > 1)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(XI) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                              // everybody's loads of this slab; everybody is done with the one before
    if (left > 2) issue(meta_of(min(igi + 1, gcount - 1)));
  };
  auto leave = [&]() {
    stage = (stage == smem_dq + (PG_STAGES - 1) * S::BYTES) ? smem_dq : stage + S::BYTES;
    --left;
  };
  typename W::Codes cd;
  asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(cd.one));
  while (left > 0) {                              // groups
    arrive();
    cd.b = cmeta & 7;
    cd.mask = ((1u << cd.b) - 1u) * 0x20002u;
    const double* par = reinterpret_cast<const double*>(stage + S::XB + S::WB) + wave * 32 + (lane & 31);
    const float s2 = (float)(0.5 * par[0]);
    const double z2 = 2.0 * par[PG_ROWS], z0 = fmin(fmax(rint(z2), -pg_zmax<BF16>()), pg_zmax<BF16>());
    // a group that is skipped (width 0): the operand is zero
    const _Float16 zc = (_Float16)(float)(1024 + (cd.b ? (int)z0 : 0));
    const float zrest = cd.b ? (float)(z2 - z0) : 0.f;
    cd.zz[0] = zc;
    cd.zz[1] = zc;
    const bool any_rest = __builtin_amdgcn_ballot_w64(zrest != 0.f) != 0;
    float16v acc[TA];
    W::template slab<WIDE, true>(stage, lane, wave, cd, acc);
    if (any_rest) W::rest_of_zero(stage, lane, zrest, acc);
    leave();
    for (int sb = 1; sb < ns; ++sb) {
      arrive();
      W::template slab<WIDE, false>(stage, lane, wave, cd, acc);
      if (any_rest) W::rest_of_zero(stage, lane, zrest, acc);
      leave();
    }
    ++gi;
    cmeta = meta_of(min(gi, gcount - 1));
    if (cd.b != 0) {                              // (a skipped group adds nothing, also where its activations are not finite)
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q) y[i][q] = fmaf(s2, acc[i][q], y[i][q]);
    }
    if ((gi & 15) == 0 || left == 0) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          ysum[i][q] += y[i][q];
          y[i][q] = 0.f;
        }
    }
  }

  const int l32 = lane & 31, h = lane >> 5, row = row0 + wave * 32 + l32;
  if (row >= a.n) return;
  if constexpr (HAND) {
    // a lane has four consecutive tokens of its row at a time (both halves of the wavefront 16 bytes of a line, which meet in the L2)
    __half* o = pa.hand + (int64_t)row * pa.ldh;
    const bool wide = (reinterpret_cast<uintptr_t>(pa.hand) & 7u) == 0 && pa.ldh % 4 == 0;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = tok0 + 32 * i + 8 * q + 4 * h;
        __half v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float f = ysum[i][4 * q + j];
          f = f > 65504.f ? 65504.f : f < -65504.f ? -65504.f : f;         // (a NaN stays one)
          v[j] = __float2half_rn(f);
        }
        if (wide && t + 4 <= a.t_x) {
          *reinterpret_cast<uint2*>(o + t) = *reinterpret_cast<const uint2*>(v);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (t + j < a.t_x) o[t + j] = v[j];
        }
      }
  } else {
    float* o = a.out + (int64_t)blockIdx.y * a.split_stride + row;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int t = tok0 + 32 * i + 8 * (q >> 2) + 4 * h + (q & 3);
        if (t < a.t_x) o[(int64_t)t * a.ldo] = ysum[i][q];
      }
  }
}

template <int SLAB, int TOK, bool BF16, bool WIDE, bool HAND>
slim_status launch(slim_ctx* ctx, const PgArgs& pa, dim3 grid) {
  const int smem = PG_STAGES * Stage<SLAB, TOK>::BYTES + (pa.d.gper * 4 + 15) / 16 * 16;
  SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(dequant_gemm<SLAB, TOK, BF16, WIDE, HAND>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  SLIM_LAUNCH(ctx, "dequant_matmul@dequant_gemm", (dequant_gemm<SLAB, TOK, BF16, WIDE, HAND>), grid, dim3(PG_THREADS), smem, pa);
  return SLIM_OK;
}

template <int SLAB, int TOK, bool BF16, bool WIDE>
slim_status launch(slim_ctx* ctx, const PgArgs& pa, dim3 grid) {
  return pa.hand ? launch<SLAB, TOK, BF16, WIDE, true>(ctx, pa, grid) : launch<SLAB, TOK, BF16, WIDE, false>(ctx, pa, grid);
}

template <int SLAB, int TOK>
slim_status launch(slim_ctx* ctx, const PgArgs& pa, dim3 grid) {
  const bool wide = pa.d.bit_base + 3 > 4;           // the layer may hold five-bit groups
  if (pa.d.x_bf16) return wide ? launch<SLAB, TOK, true, true>(ctx, pa, grid) : launch<SLAB, TOK, true, false>(ctx, pa, grid);
  return wide ? launch<SLAB, TOK, false, true>(ctx, pa, grid) : launch<SLAB, TOK, false, false>(ctx, pa, grid);
}

// token tile: 128, or 64 where that leaves fewer than two workgroups per CU
int token_tile(int n, int64_t t_x, int cus) {
  return (int64_t)slim_cdiv(n, PG_ROWS) * slim_cdiv(t_x, 128) < 2 * (int64_t)cus ? 64 : 128;
}

}  // namespace

// From 65 tokens on.  (From 33 it is the faster one on a layer of few rows, 28 against 47 us on 4096 x 11008, but there a token's
// outputs are promised to be the same bytes whichever other tokens share its call, and its sums run in another order.)
// Up to PG_MAXK groups: a workgroup holds a word for each of its range in LDS; lane offsets in 32 bits bound the leading
// dimension.  What lies beyond is taken 64 tokens at a time by the kernel for few tokens.
bool slim_dq_gemm_takes(int64_t t_x, int m, int beta, const void* X, int64_t ldx) {
  return t_x > DQ_FEW_TOKENS && t_x < (1 << 30) && slim_aligned16(X) && ldx % 8 == 0 && ldx < (1 << 23) && m % beta == 0 &&
         beta % 32 == 0 && m / beta <= PG_MAXK;
}

int slim_dq_gemm_splits(int n, int m, int beta, int64_t t_x, int cus, int& gper) {
  const int k = m / beta;
  const int64_t tiles = (int64_t)slim_cdiv(n, PG_ROWS) * slim_cdiv(t_x, token_tile(n, t_x, cus));
  int64_t want = std::min<int64_t>(k, std::max<int64_t>(1, 2 * (int64_t)cus / tiles));
  want = std::max<int64_t>(1, std::min<int64_t>(want, (int64_t)SLIM_DEQUANT_NOALLOC_MAX_FLOATS / (t_x * n)));
  gper = slim_cdiv(k, want);
  return slim_cdiv(k, gper);
}

// Bytes of partial sums that suffice for any number of tokens: none where even the fewest are not split.
size_t slim_dq_gemm_partials(int n, int m, int beta, int cus) {
  int gper = 0;
  return slim_dq_gemm_splits(n, m, beta, DQ_FEW_TOKENS + 1, cus, gper) > 1 ? sizeof(float) * SLIM_DEQUANT_NOALLOC_MAX_FLOATS : 0;
}

slim_status slim_dq_gemm_launch(slim_ctx* ctx, const DqArgs& d, int splits, __half* hand, int64_t ldh) {
  PgArgs pa;
  pa.d = d;
  pa.hand = hand;
  pa.ldh = ldh;
  const int tok = token_tile(d.n, d.t_x, std::max(1, ctx->num_cus));
  pa.tiles_r = slim_cdiv(d.n, PG_ROWS);
  pa.tiles_t = slim_cdiv(d.t_x, tok);
  const dim3 grid((unsigned)(pa.tiles_r * pa.tiles_t), (unsigned)splits);
  if (d.beta % 64 == 0) return tok == 128 ? launch<64, 128>(ctx, pa, grid) : launch<64, 64>(ctx, pa, grid);
  return tok == 128 ? launch<32, 128>(ctx, pa, grid) : launch<32, 64>(ctx, pa, grid);
}
