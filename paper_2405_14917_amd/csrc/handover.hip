// Layout changes around the linear layer when a quantised layer hands its outputs on as the calibration activations of the next
// one (Sec. 3.4): channels x tokens -> tokens x channels in 16 bits, and, where the product itself does not write it
// (dequant_gemm's handed-on form), fp32 tokens x rows -> fp16 rows x tokens.
//
// Bound by memory: a tile of 64 x 64 goes through LDS so that both sides move whole 128-byte lines, 16 bytes per lane.
// 4096 channels x 4096 tokens (67 MB read and written): 75 us as a strided copy, about 16 here.  8192 tokens through a
// 4096 x 4096 layer, handed on: 680 us with torch's copies, clamp and rounding around the product, 389 with these.
#include "dequant_device.h"

namespace {

constexpr int HO_T = 64;                    // tile edge
constexpr int HO_LD = HO_T + 2;             // 16-bit elements per LDS row: 33 words, odd, so a column is free of bank conflicts

__device__ __forceinline__ unsigned short to_half_clamped(float v) {
  v = v > 65504.f ? 65504.f : v < -65504.f ? -65504.f : v;       // (a NaN stays one)
  const __half h = __float2half_rn(v);
  return *reinterpret_cast<const unsigned short*>(&h);
}

// the tile of column block bx, row block by, of a rows x cols matrix whose element (r, c) load8 gives eight at a time, written
// transposed: cols x rows.  256 threads; a thread moves eight elements four times (two on each side).
template <typename LOAD>
__device__ __forceinline__ void transpose_tile(unsigned short (*tile)[HO_LD], LOAD load8, int rows, int64_t cols, unsigned short* out,
                                               int64_t ldo, bool wide_out) {
  const int tid = threadIdx.x;
  const int64_t c0 = (int64_t)blockIdx.x * HO_T;
  const int r0 = blockIdx.y * HO_T;
  const int e = (tid & 7) * 8;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = q * 32 + (tid >> 3);
    unsigned short v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (r0 + r < rows && c0 + e < cols) load8(r0 + r, c0 + e, (int)(cols - c0 - e < 8 ? cols - c0 - e : 8), v);
    unsigned* d = reinterpret_cast<unsigned*>(&tile[r][e]);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = (unsigned)v[2 * i] | ((unsigned)v[2 * i + 1] << 16);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = q * 32 + (tid >> 3);
    if (c0 + c >= cols || r0 + e >= rows) continue;
    unsigned w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (unsigned)tile[e + 2 * i][c] | ((unsigned)tile[e + 2 * i + 1][c] << 16);
    unsigned short* o = out + (c0 + c) * ldo + r0 + e;
    if (wide_out && r0 + e + 8 <= rows) {
      *reinterpret_cast<uint4*>(o) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (r0 + e + i < rows) o[i] = (unsigned short)(w[i >> 1] >> (16 * (i & 1)));
    }
  }
}

__global__ __launch_bounds__(256) void transpose_16(const unsigned short* __restrict__ X, int rows, int64_t cols, int64_t ldx,
                                                    unsigned short* __restrict__ out, int64_t ldo, bool wide_in, bool wide_out) {
  __shared__ unsigned short tile[HO_T][HO_LD];
  transpose_tile(
      tile,
      [&](int r, int64_t c, int cnt, unsigned short (&v)[8]) {
        const unsigned short* p = X + (int64_t)r * ldx + c;
        if (wide_in && cnt == 8) {
          *reinterpret_cast<uint4*>(v) = *reinterpret_cast<const uint4*>(p);
        } else {
          for (int i = 0; i < cnt; ++i) v[i] = p[i];
        }
      },
      rows, cols, out, ldo, wide_out);
}

__global__ __launch_bounds__(256) void round_transpose(const float* __restrict__ Y, int rows, int64_t cols, int64_t ldy,
                                                       unsigned short* __restrict__ out, int64_t ldo, bool wide_in, bool wide_out) {
  __shared__ unsigned short tile[HO_T][HO_LD];
  transpose_tile(
      tile,
      [&](int r, int64_t c, int cnt, unsigned short (&v)[8]) {
        const float* p = Y + (int64_t)r * ldy + c;
        if (wide_in && cnt == 8) {
          const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
          const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] = to_half_clamped(f[i]);
        } else {
          for (int i = 0; i < cnt; ++i) v[i] = to_half_clamped(p[i]);
        }
      },
      rows, cols, out, ldo, wide_out);
}

}  // namespace

slim_status slim_round_transpose(slim_ctx* ctx, const float* Y, int rows, int64_t cols, int64_t ldy, void* out, int64_t ldo) {
  const dim3 grid((unsigned)slim_cdiv(cols, HO_T), (unsigned)slim_cdiv(rows, HO_T));
  SLIM_LAUNCH(ctx, "handover_round", round_transpose, grid, dim3(256), 0, Y, rows, cols, ldy, static_cast<unsigned short*>(out), ldo,
              slim_aligned16(Y) && ldy % 4 == 0, slim_aligned16(out) && ldo % 8 == 0);
  return SLIM_OK;
}

extern "C" slim_status slim_transpose_16(slim_ctx* ctx, const void* X, int rows, int cols, int64_t ldx, void* out, int64_t ldo) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  SLIM_REQUIRE(ctx, X && out, "slim_transpose_16: null pointer");
  SLIM_REQUIRE(ctx, rows > 0 && cols > 0 && ldx >= cols && ldo >= rows, "slim_transpose_16: need rows, cols > 0, ldx >= cols, ldo >= rows");
  SLIM_REQUIRE(ctx, ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(out)) & 1u) == 0, "slim_transpose_16: misaligned pointer");
  if (rows > HO_T * 65535) return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "slim_transpose_16: too many rows");
  const dim3 grid((unsigned)slim_cdiv(cols, HO_T), (unsigned)slim_cdiv(rows, HO_T));
  SLIM_LAUNCH(ctx, "handover_transpose", transpose_16, grid, dim3(256), 0, static_cast<const unsigned short*>(X), rows, (int64_t)cols, ldx,
              static_cast<unsigned short*>(out), ldo, slim_aligned16(X) && ldx % 8 == 0, slim_aligned16(out) && ldo % 8 == 0);
  return SLIM_OK;
}
