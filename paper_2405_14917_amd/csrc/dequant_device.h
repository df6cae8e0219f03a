// Device-side pieces that the kernels of the linear layer on the stored form share.
#ifndef SLIM_DEQUANT_DEVICE_H
#define SLIM_DEQUANT_DEVICE_H

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "slim_internal.h"

namespace slimdq {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int DQ_FEW_TOKENS = 64;     // up to here the kernel for few tokens, above that for many

struct DqArgs {
  const uint32_t* packed;
  int64_t ldp;
  const uint32_t* gbits;
  const int32_t* row_off;
  const double* scale;   // n x k
  const double* zero;    // n x k
  int n, m, beta, k;
  int bit_base;          // the width that the 2-bit group value 0 stands for
  const void* X;         // t_x x m, 16-bit
  int x_bf16;
  int t_x;
  int64_t ldx;
  int gper;              // groups per workgroup along grid.y
  float* out;            // Y (one split) or the partial sums [split][T][n]
  int64_t ldo;           // leading dimension of `out` per token
  int64_t split_stride;  // elements between the partial sums of two splits (0 when writing Y)
};

// Width of group g, or 0 for a group whose start rows disagree with its width (a stored form read with the wrong
// bit_base, or a damaged one): such a group is skipped and none of its words is read.
__device__ __forceinline__ int checked_width(const DqArgs& a, int g) {
  const int b = (int)((a.gbits[g >> 4] >> (2 * (g & 15))) & 3u) + a.bit_base;
  return ((a.row_off[g + 1] - a.row_off[g]) * 32 == a.beta * b) ? b : 0;
}

// Zero points in the packed form of slim_pack_zeros: 2 z of row i of group g in zbits bits from bit i zbits on of row g.
struct PackedZeros {
  const uint32_t* words;
  int64_t ld;
  int bits;
};

}  // namespace slimdq

// The linear layer for up to 64 tokens (dequant_few.hip), with the zero points as doubles (a.zero) or packed (zp).
bool slim_dq_few_takes(int64_t t_x, int64_t ldp, int beta, const void* X, int64_t ldx);
slim_status slim_dq_few_launch(slim_ctx* ctx, const slimdq::DqArgs& a, const slimdq::PackedZeros* zp);

// The linear layer for many tokens (dequant_gemm.hip).  `dq_gemm_takes` tells whether it is built for the call;
// dq_gemm_splits gives the group ranges the layer is cut into (and groups per range in `gper`).
bool slim_dq_gemm_takes(int64_t t_x, int m, int beta, const void* X, int64_t ldx);
int slim_dq_gemm_splits(int n, int m, int beta, int64_t t_x, int cus, int& gper);
size_t slim_dq_gemm_partials(int n, int m, int beta, int cus);
// hand: instead of a.out, n x t_x (ldh): the results clamped and rounded to fp16 (one split)
slim_status slim_dq_gemm_launch(slim_ctx* ctx, const slimdq::DqArgs& a, int splits, __half* hand = nullptr, int64_t ldh = 0);
// out (cols x rows, fp16) = Y^T (fp32, rows x cols), clamped to fp16's range and rounded (handover.hip)
slim_status slim_round_transpose(slim_ctx* ctx, const float* Y, int rows, int64_t cols, int64_t ldy, void* out, int64_t ldo);

#endif
