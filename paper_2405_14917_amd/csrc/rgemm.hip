// fp64 products of rank up to 512 on the int8 matrix cores, through residues (declared in slim_internal.h).
//
// C = A B with the K <= 512 terms of an element summed exactly: every row of A and every column of B is scaled to integers
// of Euclidean norm 2^54.5, so that |sum| <= 2^109, and the sums are taken modulo 14 pairwise coprime numbers up to 256 whose
// product M is 2^110.27.  Modulo one of them both operands are bytes: fourteen int8 products, each exact in int32 (512 * 128 *
// 128 = 2^23), in place of the 28 or more that splitting both operands into digits would take.
// The Chinese remainder theorem gives sum / M = frac(sum over the moduli of S_i c_i) with c_i = (inverse of M / m_i mod m_i)
// / m_i, so an element needs no more than that sum, mod 1: the first 24 binary places of c_i times S_i in an unsigned 32-bit integer
// (whose overflow is what mod 1 drops), the places behind them times S_i in fp64.  The method is Ozaki, Uchino and Imamura's
// (matrix products through the Chinese remainder theorem, 2025); kernels, scaling by norms and the sum mod 1 are this library's.
//
// Precision: what is lost is the rounding of the operands to integers, 2^-55.5 of the norm of a row or column per element, and
// the roundings of the fp64 part, about 2^-59 of M.  Errors are small beside the norms of a row of A and a column of B, as those of a
// factorisation are; an element that is small beside the rest of its row keeps fewer digits than fp64 has, so a product in which
// such an element counts alone is not for these kernels.  Against exact sums at K = 512, relative (2-norm): 4.2e-16 on normal
// values and 2.8e-16 to 4.3e-16 with channels of very different scale and outliers of sixty times the rest, where the fp64
// matrix cores give 7.5e-16 and 7.1e-16 to 1.0e-15.  (With 15 moduli 1.3e-16 and 7 % slower, with 13 it would be 1e-14.)
//
// What bounds it: no pipe alone.  A tile takes 29 k cycles of MFMA per SIMD, 1.8 MB from the L2 to LDS and 5.2 MiB from there to the
// wavefronts (1.5 KiB per MFMA), which overlap in part: over a pass of 4096 x 11008 the matrix cores are busy 30 % of the cycles, the
// vector issue 20 %, and the wavefronts wait 39 % of theirs, at some 1.7 GHz of 2.4 (power).  Where a launch has one tile per CU, the
// old values and the stores of C come on top.  us for the product / with both operands' residues / on the fp64 matrix cores:
//   4096 x 1024  45 / 81 / 84    4096 x 2048  84 / 122 / 151    4096 x 3584  147 / 188 / 276    4096 x 10496  437 / 488 / 708
//   28672 x 4096  1234 / 1342 / 1838
#include <algorithm>

#include "slim_internal.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int NP = SLIM_RG_PLANES;
constexpr int KMAX = SLIM_RG_K;              // channels of an operand, zeros behind the real ones
constexpr int FRAG = 1024;                   // 32 rows x 32 channels as the lanes of v_mfma_i32_32x32x32_i8 hold them
constexpr int RB_BYTES = KMAX * 32;          // 32 rows of a plane
// pairwise coprime, in threes with a product below 2^24; none of the odd ones above 253, so that a remainder taken in fp32
// (which may be 1 off the nearest) stays inside a signed byte
constexpr int MOD[NP] = {256, 253, 251, 247, 245, 243, 241, 239, 233, 229, 227, 223, 211, 199};

struct Crt {
  int hi[NP];          // c_i in units of 2^-24, rounded
  double lo[NP];       // c_i minus that
};
constexpr Crt crt_constants() {
  Crt t{};
  for (int i = 0; i < NP; ++i) {
    int rest = 1;                                       // M / m_i mod m_i
    for (int j = 0; j < NP; ++j)
      if (j != i) rest = rest * MOD[j] % MOD[i];
    int x = 1;
    while (rest * x % MOD[i] != 1) ++x;
    if (2 * x > MOD[i]) x -= MOD[i];                    // c_i = x / m_i in (-1/2, 1/2]
    const long long num = (long long)x * (1 << 24);
    long long q = num / MOD[i];
    long long r = num - q * MOD[i];
    if (2 * r > MOD[i]) ++q, r -= MOD[i];
    if (2 * r < -MOD[i]) --q, r += MOD[i];
    t.hi[i] = (int)q;
    t.lo[i] = (double)r / MOD[i] / (1 << 24);
  }
  return t;
}
constexpr Crt kCrt = crt_constants();
constexpr double modulus_product() {                    // M 2^-109
  unsigned __int128 p = 1;
  for (int i = 0; i < NP; ++i) p *= (unsigned)MOD[i];
  return (double)p / 18014398509481984.0 / 36028797018963968.0;
}
constexpr double kM = modulus_product();
static_assert(kM > 2.1 && kM < 4.0, "products of norms up to 2^54.5 stay below M / 2");
constexpr double kNorm = 18014398509481984.0 * 1.4142135623730951;      // 2^54.5
__constant__ Crt d_crt = crt_constants();

// ---- residues of an operand -------------------------------------------------------------------------------------
// A workgroup has 32 rows (or columns: `T`) of all KMAX channels, a wavefront 32 x 32 of them, one fragment per plane: the
// lane's row l % 32, channels 16 (l / 32) .. + 15.  8 bytes in and 14 out per element: 28672 x 512 in 84 us (3.8 TB/s); fewer
// than some 8000 rows leave CUs idle (4096 x 512 22 us).
// A row with a value that is not finite has no residues: its scale is NaN, and so is what it is multiplied into.  (A row whose norm
// is no normal number would lose digits of its scale; what comes from 32-bit weights and activations stays far above.)
template <bool T>
__global__ __launch_bounds__(1024) void rg_residues(const double* __restrict__ src, int64_t ld, int rows, int K, char* __restrict__ out,
                                                    int64_t plane, double* __restrict__ scale) {
  __shared__ int top[32];
  __shared__ double sq[16][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
  const int row = blockIdx.x * 32 + l32, k0 = wave * 32 + h * 16;
  if (tid < 32) top[tid] = 0;
  double x[16];
  const int rc = min(row, rows - 1);
  if constexpr (T) {
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = src[(int64_t)min(k0 + i, K - 1) * ld + rc];
  } else {
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const double2 v = *reinterpret_cast<const double2*>(src + (int64_t)rc * ld + min(k0 + i, K - 2));
      x[i] = v.x;
      x[i + 1] = v.y;
    }
  }
  int mx = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (k0 + i >= K || row >= rows) x[i] = 0.0;
    mx = max(mx, __double2hiint(x[i]) & 0x7fffffff);
    mx |= (__double2loint(x[i]) != 0);                 // (a subnormal number may have no bits in the upper half)
  }
  __syncthreads();
  mx = max(mx, __shfl_xor(mx, 32, 64));
  if (h == 0) atomicMax(&top[l32], mx);
  __syncthreads();
  mx = top[l32];
  const bool finite = mx < 0x7ff00000;
  const int e = max(mx >> 20, 1) - 1022;               // |x| < 2^e
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    x[i] = ldexp(x[i], -e);
    s = fma(x[i], x[i], s);
  }
  s += __shfl_xor(s, 32, 64);
  if (h == 0) sq[wave][l32] = s;
  __syncthreads();
  s = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) s += sq[w][l32];
  const double norm = sqrt(s) * (1.0 + 0x1p-40);       // of the row times 2^-e
  const double g = finite && mx ? kNorm / norm : 0.0;
  if (tid < 32) scale[row] = finite ? (mx ? ldexp(norm, e) : 0.0) : __longlong_as_double(0x7ff8000000000000ll);
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = finite ? rint(x[i] * g) : 0.0;
  char* dst = out + (int64_t)blockIdx.x * RB_BYTES + wave * FRAG + lane * 16;
#pragma unroll
  for (int t = 0; t < (NP + 2) / 3; ++t) {
    constexpr int LAST = NP - 1;
    const double P = (double)MOD[3 * t] * MOD[min(3 * t + 1, LAST)] * (3 * t + 2 <= LAST ? MOD[min(3 * t + 2, LAST)] : 1);
    unsigned w[3][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      unsigned b[3] = {0, 0, 0};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double v = x[4 * q + i];
        const float r = (float)fma(-P, rint(v * (1.0 / P)), v);      // exact, an integer of at most P / 2 and a few (v / P is rounded): a float
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if (3 * t + c > LAST) continue;
          const float m = (float)MOD[min(3 * t + c, LAST)];
          const int res = (int)fmaf(-m, rintf(r * (1.0f / m)), r);
          b[c] |= ((unsigned)res & 255u) << (8 * i);
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) w[c][q] = b[c];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (3 * t + c <= LAST) *reinterpret_cast<uint4*>(dst + (3 * t + c) * plane) = make_uint4(w[c][0], w[c][1], w[c][2], w[c][3]);
  }
}

// ---- the product ----------------------------------------------------------------------------------------------------
__device__ __forceinline__ void lds_load16(unsigned lds_addr, unsigned voff, const char* gbase) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(gbase) : "m0");
#else
  (void)lds_addr, (void)voff, (void)gbase;
#endif
}

struct RgArgs {
  const char *A, *B;
  int64_t planeA, planeB;
  const double *sa, *sb;
  double* C;
  int64_t ldc;
  int M, N;
  double alpha;
  int tiles_m, tiles_n, upper;
  int ncu;
};

// A workgroup of eight wavefronts has a tile of 128 x 128: a lane keeps the sums of 32 elements in 3 registers each beside two
// sets of int32 accumulators, 252 registers in all, which is what bounds the tile.  The accumulators of one modulus fill while
// those of the one before are added up, three vector instructions behind every MFMA, so that the matrix pipe never waits for
// the vector work.  Operands go from memory to a ring of five 32 KiB stages in LDS (128 channels of both operands), four
// stages ahead, from one tile into the next; one barrier per stage.
constexpr int BT = 128;                      // tile edge
constexpr int STAGE_K = 128;                 // channels of a stage: 4 fragments of 8 blocks of 32 rows, 32 KiB
constexpr int NS = KMAX / STAGE_K;           // stages per plane
constexpr int UNIT = 2 * BT * STAGE_K;       // bytes
constexpr int UNITS = 5;
constexpr size_t RG_LDS = size_t(UNITS) * UNIT;
constexpr int RG_BESIDE = 64;                // CUs left to kernels of other streams

// Tiles in bands of eight rows, column by column; rounds of `ncu` workgroups take consecutive tiles, XCD c (id mod 8) the c-th
// eighth of them: a patch of 8 x 4 tiles, whose operands of a plane its L2 holds.
__device__ __forceinline__ bool rg_tile(const RgArgs& a, int id, int& bi, int& bj) {
  const int total = a.upper ? a.tiles_n * (a.tiles_n + 1) / 2 : a.tiles_m * a.tiles_n;
  const int whole = total / a.ncu * a.ncu;
  int t = id < whole ? id / a.ncu * a.ncu + id % 8 * (a.ncu / 8) + id % a.ncu / 8 : id;
  if (!a.upper) {
    const int band = t / (8 * a.tiles_n), in = t - band * 8 * a.tiles_n, hb = min(8, a.tiles_m - band * 8);
    bi = band * 8 + in % hb;
    bj = in / hb;
    return true;
  }
  for (int r0 = 0; r0 < a.tiles_n; r0 += 8) {
    const int hb = min(8, a.tiles_n - r0), tri = hb * (hb - 1) / 2, cnt = hb * (a.tiles_n - r0) - tri;
    if (t < cnt) {
      if (t >= tri) {
        bi = r0 + (t - tri) % hb;
        bj = r0 + hb - 1 + (t - tri) / hb;
      } else {
        int c = 0;
        while ((c + 1) * (c + 2) / 2 <= t) ++c;
        bi = r0 + t - c * (c + 1) / 2;
        bj = r0 + c;
      }
      return true;
    }
    t -= cnt;
  }
  return false;
}

__global__ __launch_bounds__(512, 2) void rgemm_kernel(RgArgs a) {
  extern __shared__ __align__(16) char sm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int wr = wave >> 1, wc = wave & 1;
  const int total = a.upper ? a.tiles_n * (a.tiles_n + 1) / 2 : a.tiles_m * a.tiles_n;
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)((__attribute__((address_space(3))) char*)sm));
  const int64_t plane = wave < 4 ? a.planeA : a.planeB;
  const unsigned mine = lds0 + wave * (4 * FRAG);
  // what is loaded runs four stages ahead of what is multiplied, from one tile into the next
  int ld_tile = blockIdx.x, ld_kc = 0, ld_plane = 0, ld_unit = 0;
  const char* src;
  auto source = [&]() {
    int i, j;
    rg_tile(a, ld_tile, i, j);
    src = wave < 4 ? a.A + (int64_t)(i * 4 + wave) * RB_BYTES : a.B + (int64_t)(j * 4 + wave - 4) * RB_BYTES;
  };
  auto stage_load = [&]() {                    // the next stage in order -> the next unit of the ring
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_load16(mine + ld_unit * UNIT + i * FRAG, lane * 16, src + i * FRAG);
    ld_unit = ld_unit + 1 == UNITS ? 0 : ld_unit + 1;
    src += 4 * FRAG;
    if (++ld_kc == NS) {
      ld_kc = 0;
      src += plane - NS * (4 * FRAG);
      if (++ld_plane == NP) {                  // (behind the last tile its first stages are loaded again)
        ld_plane = 0;
        if (ld_tile + (int)gridDim.x < total) ld_tile += gridDim.x;
        source();
      }
    }
  };
  source();
#pragma unroll
  for (int i = 0; i < 4; ++i) stage_load();    // stages 0 .. 3
  const int offA = wr * (4 * FRAG) + lane * 16, offB = 4 * (4 * FRAG) + wc * (8 * FRAG) + lane * 16;
  int unit = 0;
  v16i acc[2][2];
  unsigned hi[2][16];                          // (modulo 2^32: the sums overflow on purpose)
  double lo[2][16];
  v4i fa[2], fb[2][2];
  auto frags = [&](int buf, const char* u, int ks) {
    fa[buf] = *reinterpret_cast<const v4i*>(u + offA + ks * FRAG);
#pragma unroll
    for (int j = 0; j < 2; ++j) fb[buf][j] = *reinterpret_cast<const v4i*>(u + offB + j * (4 * FRAG) + ks * FRAG);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  frags(0, sm, 0);
  // A whole tile's results stay in `lo` and are stored beside the first two planes of the next tile, one store per two MFMAs: a CU
  // gets rid of 18 bytes per ns, and as one burst at the end the stores held up 7 of a tile's 45 us.
  bool pending = false;
  char* crow = nullptr;                        // the wavefront's part of the tile, at the row that is stored next
  const unsigned clane = (unsigned)((4 * h * a.ldc + l32) * 8);
  auto store = [&](int j, int v, bool inside) {                // in order: all v of one j, then of the other
    if (inside) *reinterpret_cast<double*>(crow + 256 * j + clane) = lo[j][v];
    crow += a.ldc * 8 * (v == 15 ? -27 : (v & 3) == 3 ? 5 : 1);
  };
  for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
    int bi, bj;
    rg_tile(a, tile, bi, bj);
    const int row0 = bi * BT + wr * 32 + 4 * h, col0 = bj * BT + wc * 64 + l32;
    auto old_values = [&](int j, double (&old)[16]) {
      const int col = min(col0 + 32 * j, a.N - 1);
#pragma unroll
      for (int v = 0; v < 16; ++v) old[v] = a.C[(int64_t)min(row0 + 8 * (v >> 2) + (v & 3), a.M - 1) * a.ldc + col];
    };
    double old[2][16];
    // one plane: its products into acc[NTH % 2], the sums of the plane before it taken into hi and lo beside them.  NTH: 0, 1, 2, or 3
    // and 4 for the odd and the even ones behind them; LAST: the old values of C are asked for
    auto run_plane = [&](auto nth, auto last, int p) {
      constexpr int NTH = decltype(nth)::value, P = NTH % 2;
      constexpr bool LAST = decltype(last)::value;
      const int ch = NTH == 0 ? 0 : d_crt.hi[p - 1];
      const double cl = NTH == 0 ? 0.0 : d_crt.lo[p - 1];
#pragma unroll
      for (int kc = 0; kc < NS; ++kc) {
        // Stage s + 1 has landed in every wavefront, and every wavefront has read the last of stage s - 1.  A tile's stages 0 to
        // 3 have landed before its loop.  What may still be on its way is newer: the loads of two stages and, where the last
        // tile's results are being stored, up to twelve stores (four per stage, in the first eight).
        constexpr int s = 4 * NTH;
        if (NTH == 0 && kc < NS - 1)
          asm volatile("" ::: "memory");
        else if (s + kc > 10 || !pending)
          asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else if (s + kc == 10)
          asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
        else if (s + kc == 9)
          asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        else
          asm volatile("s_waitcnt vmcnt(20)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        stage_load();                          // stage s + 4, into the unit of stage s - 1
        if (LAST && kc == NS - 1) old_values(0, old[0]);
        const char* u = sm + unit * UNIT;
        unit = unit + 1 == UNITS ? 0 : unit + 1;
        const char* un = sm + unit * UNIT;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const int b = ks & 1;
          if (ks < 3)
            frags(b ^ 1, u, ks + 1);
          else
            frags(b ^ 1, un, 0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            v16i c = acc[P][j];
            if (kc == 0 && ks == 0) {
#pragma unroll
              for (int v = 0; v < 16; ++v) c[v] = 0;
            }
            acc[P][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[b], fb[b][j], c, 0, 0, 0);
            const int el = (kc * 4 + ks) * 2 + j, ej = el / 16, ev = el % 16;
            if (NTH < 2 && el % 2 == 0) {      // (an element is stored before its register takes the new tile's sums)
              const int se = 16 * NTH + el / 2;
              if (pending) store(se / 16, se % 16, true);
            }
            if constexpr (NTH > 0) {
              const int s32 = acc[1 - P][ej][ev];
              if constexpr (NTH == 1) {
                hi[ej][ev] = (unsigned)__mul24(s32, ch);
                lo[ej][ev] = (double)s32 * cl;
              } else {
                hi[ej][ev] += (unsigned)__mul24(s32, ch);
                lo[ej][ev] = fma((double)s32, cl, lo[ej][ev]);
              }
              asm volatile("" : "+v"(hi[ej][ev]), "+v"(lo[ej][ev]));   // (or the compiler moves all of them behind the plane's products)
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    };
    constexpr std::integral_constant<int, 3> odd{};
    constexpr std::integral_constant<int, 4> even{};
    static_assert(NP % 2 == 0 && NP > 4, "the last plane is an odd one");
    run_plane(std::integral_constant<int, 0>{}, std::false_type{}, 0);
    run_plane(std::integral_constant<int, 1>{}, std::false_type{}, 1);
    run_plane(std::integral_constant<int, 2>{}, std::false_type{}, 2);
    for (int p = 3; p + 2 < NP; p += 2) {
      run_plane(odd, std::false_type{}, p);
      run_plane(even, std::false_type{}, p + 1);
    }
    run_plane(odd, std::true_type{}, NP - 1);
    old_values(1, old[1]);
    const int rowu = bi * BT + wr * 32, colu = bj * BT + wc * 64;
    const double sa = a.sa[min(rowu + l32, a.M - 1)];          // of the lane's row of the wavefront's 32
    double sb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) sb[j] = a.sb[min(col0 + 32 * j, a.N - 1)] * a.alpha;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // (the next tile's first stages with them)
    crow = reinterpret_cast<char*>(a.C + (int64_t)rowu * a.ldc + colu);
    pending = bi * BT + BT <= a.M && bj * BT + BT <= a.N;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 8 * (v >> 2) + 4 * h + (v & 3);
      const double sr = __hiloint2double(__shfl(__double2hiint(sa), r, 64), __shfl(__double2loint(sa), r, 64));
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int s = acc[1][j][v];
        const unsigned t = hi[j][v] + (unsigned)__mul24(s, d_crt.hi[NP - 1]);
        const double l = fma((double)s, d_crt.lo[NP - 1], lo[j][v]);
        double f = fma((double)(int)(t << 8), 0x1p-32, l);
        f -= rint(f);
        lo[j][v] = fma(f * sr, sb[j], old[j][v]);
        asm volatile("" : "+v"(lo[j][v]));
      }
    }
    if (!pending) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          store(j, v, row0 + 8 * (v >> 2) + (v & 3) < a.M && col0 + 32 * j < a.N);
    }
  }
  if (pending) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) store(j, v, true);
  }
}

}  // namespace

// A product by itself, of rank 512, with operands converted for it alone, against the fp64 form.  us: the kernel takes 27 per round of
// 256 tiles and 12 per 256 tiles; converting takes 35 and 3 per 1000 rows of an operand beyond 4096; the fp64 form 0.27 to 0.33 per
// tile.  Both sides measured, fp64 / residues: 256 tiles 4096 x 1024 82 / 81, 1024 x 4096 80 / 81; 384 4096 x 1536 110 / 109; 512
// 4096 x 2048 152 / 121, 1024 x 8192 152 / 124, 8192 x 1024 157 / 121; but tall ones, whose rows' residues take their time:
// 28672 x 256 142 / 198, 28672 x 512 288 / 279, 16384 x 512 150 / 142, 28672 x 1024 507 / 420.
bool slim_rg_pays(int M, int N) {
  const int tiles = slim_cdiv(M, BT) * slim_cdiv(N, BT);
  const double convert = 35.0 + 3e-3 * (std::max(0, M - 4096) + std::max(0, N - 4096));
  return 27.0 * slim_cdiv(tiles, 256) + 12.0 * tiles / 256 + convert < 0.27 * tiles;
}

size_t slim_rg_operand_bytes(int rows) {
  const int rp = slim_cdiv(rows, BT) * BT;
  return slim_ws_round((size_t)rp * KMAX * NP) + slim_ws_round(sizeof(double) * rp);
}

slim_rg_operand slim_rg_carve(slim_ctx* ctx, int rows) {
  slim_rg_operand o;
  const int rp = slim_cdiv(rows, BT) * BT;
  o.planes = static_cast<char*>(slim_ws_alloc(ctx, (size_t)rp * KMAX * NP));
  o.scale = static_cast<double*>(slim_ws_alloc(ctx, sizeof(double) * rp));
  return o;
}

slim_status slim_rg_residues(slim_ctx* ctx, const char* name, const slim_rg_operand& o, const double* src, int64_t ld, int rows, int K,
                             bool columns) {
  SLIM_REQUIRE(ctx, rows > 0 && K >= 2 && K <= KMAX && K % 2 == 0, "rgemm: bad operand (%d x %d)", rows, K);
  SLIM_REQUIRE(ctx, columns || (ld % 2 == 0 && slim_aligned16(src)), "rgemm: misaligned operand");
  const int rb = slim_cdiv(rows, BT) * (BT / 32);
  const int64_t plane = (int64_t)rb * RB_BYTES;
  if (columns)
    SLIM_LAUNCH(ctx, name, rg_residues<true>, dim3(rb), dim3(1024), 0, src, ld, rows, K, o.planes, plane, o.scale);
  else
    SLIM_LAUNCH(ctx, name, rg_residues<false>, dim3(rb), dim3(1024), 0, src, ld, rows, K, o.planes, plane, o.scale);
  return SLIM_OK;
}

slim_status slim_rgemm(slim_ctx* ctx, const char* name, const slim_rg_desc& d) {
  if (d.M <= 0 || d.N <= 0) return SLIM_OK;
  RgArgs a;
  a.A = d.A.planes;
  a.B = d.B.planes;
  a.sa = d.A.scale;
  a.sb = d.B.scale;
  a.planeA = (int64_t)slim_cdiv(d.rowsA, BT) * BT * KMAX;
  a.planeB = (int64_t)slim_cdiv(d.rowsB, BT) * BT * KMAX;
  a.C = d.C;
  a.ldc = d.ldc;
  a.M = d.M;
  a.N = d.N;
  a.alpha = d.alpha * kM;
  a.upper = d.upper ? 1 : 0;
  a.tiles_m = slim_cdiv(d.M, BT);
  a.tiles_n = slim_cdiv(d.N, BT);
  a.ncu = std::max(8, ctx->num_cus / 8 * 8);
  const int total = d.upper ? a.tiles_n * (a.tiles_n + 1) / 2 : a.tiles_m * a.tiles_n;
  static bool done = false;
  if (!done) {
    SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(rgemm_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                          (int)RG_LDS));
    done = true;
  }
  // Beside other streams' work the products leave some CUs alone, or they hold the inverse's chain of links up; more than 64, and
  // they get long themselves.  Left alone 0 / 16 / 32 / 64 / 96 / 128, medians of three runs of one box, which scatter by 0.5 %:
  // inverse of 6144 columns 4000 / 3980 / 3950 / 3840 / 3800 / 3910 us, 8192 7490 / 7530 / 7450 / 7290 / 7310 / 7540, 11008 15540 / 15680
  // / 15350 / 15160 / 15670 / 16130; up to 4096 no difference; pass of 4096 x 11008 56.0 / 56.3 / 56.0 / 55.7 / 55.9 / 56.4 ms.
  const int wgs = d.beside ? std::max(8, a.ncu - RG_BESIDE) : a.ncu;
  SLIM_LAUNCH(ctx, slim_prof_name(name, "rgemm_kernel"), rgemm_kernel, dim3(std::min(total, wgs)), dim3(512), RG_LDS, a);
  return SLIM_OK;
}
