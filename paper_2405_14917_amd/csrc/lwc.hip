// n4  SliM-LLM+ on one linear layer (Sec. 3.4; Sec. 4; App. B): the widths of SBA stay, SQC and the error compensation
// are left out, and every (row, group) gets a quantiser with learnable weight clipping whose two clipping strengths
// are trained with AdamW on the layer-output error.  The paper names the method it borrows (the learnable weight
// clipping of OmniQuant) and the optimiser; the forward pass built here is
//     hi = sigmoid(gamma) max_j w_j,  lo = sigmoid(beta) min_j w_j,  delta = (hi - lo) / (2^b - 1),
//     z = -round(lo / delta),  q_j = clamp(round(w_j / delta) + z, 0, 2^b - 1),  w_hat_j = delta (q_j - z)
// (Eq. 1 on the clipped range, every width in this affine form), the loss L = tr(dW G dW^T) / (n T), the mean
// squared error of the layer's outputs over the T calibration tokens (Eq. 3), taken full batch: it depends on X only
// through G = X X^T, so one step sees all tokens.  The backward pass takes the rounding as the identity and lets the
// clamp pass derivatives where it does not clip:
//     g = dL/dW_hat = 2 (W_hat - W) G / (n T)
//     dW_hat_j / d delta = (q_j - z) - w_j / delta   or, clipped,   (q_j - z) - lo / delta
//     dW_hat_j / d lo at fixed delta = 0   or, clipped,   1
// Everything is fp64.  D G = W_hat G - W G with W_hat = delta (q - z): the first product is one of small integers with G's
// digits (int8_products.h, a unit per column of G, which G's fp32 entries fit exactly unless they are 2^-30 of their column's
// largest: those are rounded by 2^-54 of it, as one addition to the fp64 sum would), the second one does not change and is
// taken once, from the digits of W.  Two kernels per step: the product, and one pass over W and D G that forms the
// derivatives, takes the AdamW step and writes the next step's integers, 16 lanes per (row, group), fixed-order reductions.
// The difference of the two products loses the digits that W_hat and W share, so both are summed to twice the precision.
// Relative error of D G on rows of 1024 channels with outlier channels (model of either form's roundings against exact sums):
// 5e-17 at every width and for weights of one sign, group sizes 32 to 256.  (W_hat - W) G on the fp64 matrix cores, which
// round after every four channels: 4e-16 at two bits, 1e-15 at four and five, 4e-15 at eight; the two products in plain fp64
// sums: 4e-16, 1.6e-15, 2.6e-15 and 1e-14.
// Group sizes that 4 does not divide multiply W_hat - W on the fp64 matrix cores: the integers' operand order has no place
// for them, and the passes over W then take one channel per lane in place of four (V), since four would reach into the next
// group.
// What bounds it: the vector work behind the MFMAs of the product (figures at lwc_step).
#include <cmath>

#include "int8_products.h"

namespace {

using namespace slimint;

struct LwcGroup {
  double M, m_, s_hi, s_lo, lo, delta, z, Q;
  bool live;
};

// parameters of one (row, group) from its extreme values and clipping strengths; the same in the lanes of a row
__device__ __forceinline__ LwcGroup lwc_group(double M, double m_, double gamma, double betap, int bits) {
  LwcGroup p;
  p.M = M;
  p.m_ = m_;
  p.Q = (double)((1 << bits) - 1);
  p.s_hi = 1.0 / (1.0 + exp(-gamma));
  p.s_lo = 1.0 / (1.0 + exp(-betap));
  const double hi = p.s_hi * M;
  p.lo = p.s_lo * m_;
  p.live = hi > p.lo;
  p.delta = p.live ? (hi - p.lo) / p.Q : 1.0;
  p.z = p.live ? -rint(p.lo / p.delta) : 0.0;
  return p;
}


struct LwcArgs {
  IntShape s;             // n x m weights against the m columns of G
  IntMeta mt;
  int64_t ldw;
  const uint8_t* bits;    // k
  double *M, *mn;         // k x npad each: extreme values, strengths, moments
  double *gamma, *betap, *m1g, *vg, *m1b, *vb;
  char* Q;                // integers of the next product, in operand order
  double *S, *Rz;         // k x npad: their scales, and the scale times what the zero has beyond the integers
  int* rest;              // k: last step at which some row of the group had such a part
  int* row_exp;           // npad: exponent above the row's largest weight, biased
  char* Wd;               // digits of W
  double* D;              // n x m: W_hat - W in place of the integers (group sizes that 4 does not divide), else nullptr
  const double* DG;       // n x m: D G
  double* lp;             // the workgroups' sums of D_j (D G)_j
  double gscale;          // 2 / (n T)
  double init, lr, b1, b2, eps, c1, c2;   // AdamW; c1 = 1 - b1^step, c2 = 1 - b2^step
  int step;               // of the integers that are written
  // final quantisation
  uint8_t* codes;         // n x m (ld = m)
  double* scale;          // n x k
  double* zero;
  void* What;
  int what_f64;
};

// rint(w / delta): the product with the reciprocal differs from the quotient by less than 1e-15 of it, so the two can round
// apart only next to a tie
__device__ __forceinline__ double rint_quotient(double w, const LwcGroup& p, double inv) {
  const double r = w * inv;
  double c = rint(r);
  if (fabs(fabs(r - c) - 0.5) <= 1e-9 * (1.0 + fabs(r))) c = rint(w / p.delta);
  return c;
}

// V consecutive weights
template <typename T, int V>
__device__ __forceinline__ void load_weights(const T* p, double (&v)[V]) {
  if constexpr (V == 4)
    load4<T>(p, v);
  else
    v[0] = (double)__uint_as_float(float_bits<T>(*p));
}

// the integers (with a.D: the differences W_hat - W), scale and zero's rest of one (row, group)
template <typename T, int V>
__device__ __forceinline__ void write_integers(const LwcArgs& a, const T* w, int row, int g, int l16, bool live, const LwcGroup& p) {
  const IntShape& s = a.s;
  const double inv = 1.0 / p.delta;
  if (a.D) {
    double* d = a.D + (int64_t)row * s.m + (int64_t)g * s.beta;
    for (int j = l16 * V; live && j < s.beta; j += 16 * V) {
      double v[V];
      load_weights<T, V>(w + j, v);
#pragma unroll
      for (int i = 0; i < V; ++i) v[i] = p.delta * (fmin(fmax(rint_quotient(v[i], p, inv) + p.z, 0.0), p.Q) - p.z) - v[i];
      if constexpr (V == 4) {
        *reinterpret_cast<double2*>(d + j) = make_double2(v[0], v[1]);
        *reinterpret_cast<double2*>(d + j + 2) = make_double2(v[2], v[3]);
      } else {
        d[j] = v[0];
      }
    }
    return;
  }
  if constexpr (V != 4) return;                    // (such groups have no integers: a.D is set)
  const double z0 = fmin(fmax(p.z, p.Q - 127.0), 128.0);
  if (l16 == 0) {
    a.S[(int64_t)g * s.npad + row] = live ? p.delta + (p.M - p.m_) * 0.0 : 0.0;      // (infinite weights: not a number)
    a.Rz[(int64_t)g * s.npad + row] = live ? p.delta * (p.z - z0) : 0.0;
    if (live && p.z != z0) atomicMax(&a.rest[g], a.step);
  }
  for (int j = l16 * 4; j < s.nchg * s.chk; j += 64) {
    int c;
    const int64_t dst = operand_offset(s, row, g, j, c);
    unsigned word = 0;
    if (live && j < s.beta) {
      double v[4];
      load4<T>(w + j, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double q = fmin(fmax(rint_quotient(v[i], p, inv) + p.z, 0.0), p.Q);
        word |= ((unsigned)(int)(q - z0) & 255u) << (8 * i);
      }
    }
    *reinterpret_cast<unsigned*>(a.Q + dst) = word;
  }
}

// grid (npad / 16, y): 16 lanes per row, groups blockIdx.y, + gridDim.y, ...: extremes, start values, the digits of W and the
// first integers
template <typename T, int V>
__global__ __launch_bounds__(256) void lwc_init(const T* __restrict__ W, LwcArgs a) {
  const IntShape& s = a.s;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4);
  const bool live = row < s.n;
  const int64_t plane = (int64_t)s.npad * s.C * s.chk;
  for (int g = blockIdx.y; g < s.k; g += gridDim.y) {
    const T* w = W + (int64_t)min(row, s.n - 1) * a.ldw + (int64_t)g * s.beta;
    double mx = -INFINITY, mn = INFINITY, none = 0.0;
    for (int j = l16 * V; j < s.beta; j += 16 * V) {
      double v[V];
      load_weights<T, V>(w + j, v);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        mx = fmax(mx, v[i]);
        mn = fmin(mn, v[i]);
        none += v[i] * 0.0;
      }
    }
    mx = row_reduce<OpMax>(mx);
    mn = row_reduce<OpMin>(mn);
    none = row_sum(none);
    const int64_t u = (int64_t)g * s.npad + row;
    if (l16 == 0) {
      a.M[u] = mx;
      a.mn[u] = mn;
      a.gamma[u] = a.betap[u] = a.init;
      a.m1g[u] = a.vg[u] = a.m1b[u] = a.vb[u] = 0.0;
      const double top = fmax(fabs(mx), fabs(mn));
      if (live && !a.D && top > 0.0 && top < INFINITY) {
        int e;
        (void)frexp(top, &e);
        atomicMax(&a.row_exp[row], e + ROW_EXP_BIAS);
      }
    }
    for (int j = l16 * 4; V == 4 && !a.D && j < s.nchg * s.chk; j += 64) {
      int c;
      const int64_t dst = operand_offset(s, row, g, j, c);
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      if (live && j < s.beta) load4<T>(w + j, v);
      const unsigned bits4[4] = {__float_as_uint((float)v[0]), __float_as_uint((float)v[1]), __float_as_uint((float)v[2]),
                                 __float_as_uint((float)v[3])};
      store_digits(a.Wd, plane, dst, bits4, a.mt.wunit[(int64_t)c * s.npad + row], digits_of_rows(s, a.mt.w, c, row));
    }
    const LwcGroup p = lwc_group(mx, mn, a.init, a.init, min(max((int)a.bits[g], 1), 8));
    write_integers<T, V>(a, w, row, g, l16, live, p);
    // a weight that is not a number: its integer is one, but (W_hat - W) G of its row is not (nor are the strengths from then on)
    if (l16 == 0 && live && !a.D && none != 0.0) a.S[u] = NAN;
  }
}

__device__ __forceinline__ double row_first(double v, int lane) {
  return __hiloint2double(__shfl(__double2hiint(v), lane & 48, WAVE), __shfl(__double2loint(v), lane & 48, WAVE));
}

// The (row, group)'s share of the loss and, with TRAIN, the derivatives of its two strengths, their AdamW step, and the
// integers of the next product.  4096 x 4096 (20 steps 14 instead of 42 ms): this pass 78 us, the product 620 us; on the fp64
// matrix cores the product took 1.9 ms, and the two passes over fp64 copies of W, W_hat - W and D G 0.2 ms.
template <typename T, bool TRAIN, int V>
__global__ __launch_bounds__(256) void lwc_step(const T* __restrict__ W, LwcArgs a) {
  __shared__ double red[16];
  const IntShape& s = a.s;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  const int slot = (threadIdx.x >> 6) * 4 + (lane >> 4), row = blockIdx.x * 16 + slot;
  const bool live = row < s.n;
  double loss = 0.0;
  for (int g = blockIdx.y; g < s.k; g += gridDim.y) {
    const int64_t u = (int64_t)g * s.npad + row;
    const T* w = W + (int64_t)min(row, s.n - 1) * a.ldw + (int64_t)g * s.beta;
    const double* dgp = a.DG + (int64_t)min(row, s.n - 1) * s.m + (int64_t)g * s.beta;
    const int bits = min(max((int)a.bits[g], 1), 8);
    double gamma = a.gamma[u], betap = a.betap[u];
    const double M = a.M[u], mn = a.mn[u];
    const LwcGroup p = lwc_group(M, mn, gamma, betap, bits);
    const double inv = 1.0 / p.delta, clipped = p.lo * inv;
    double s1 = 0.0, s2 = 0.0, lsum = 0.0;
    for (int j = l16 * V; j < s.beta; j += 16 * V) {
      double v[V], dg[V];
      load_weights<T, V>(w + j, v);
      if constexpr (V == 4) {
        const double2 d0 = *reinterpret_cast<const double2*>(dgp + j), d1 = *reinterpret_cast<const double2*>(dgp + j + 2);
        dg[0] = d0.x;
        dg[1] = d0.y;
        dg[2] = d1.x;
        dg[3] = d1.y;
      } else {
        dg[0] = dgp[j];
      }
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const double un = rint_quotient(v[i], p, inv) + p.z;
        const double q = fmin(fmax(un, 0.0), p.Q);
        const bool inside = (un >= 0.0) && (un <= p.Q);
        lsum += (p.delta * (q - p.z) - v[i]) * dg[i];
        if (TRAIN) {
          const double gj = a.gscale * dg[i];
          s1 += gj * ((q - p.z) - (inside ? v[i] * inv : clipped));
          s2 += inside ? 0.0 : gj;
        }
      }
    }
    lsum = row_sum(lsum);
    if (live) loss += lsum;
    if (TRAIN) {
      s1 = row_sum(s1);
      s2 = row_sum(s2);
      const double d_hi = p.live ? s1 / p.Q : 0.0;
      const double d_lo = p.live ? -s1 / p.Q + s2 : 0.0;
      const double gg = d_hi * M * p.s_hi * (1.0 - p.s_hi);
      const double gb = d_lo * mn * p.s_lo * (1.0 - p.s_lo);
      const double m1g = a.b1 * a.m1g[u] + (1.0 - a.b1) * gg, vg = a.b2 * a.vg[u] + (1.0 - a.b2) * gg * gg;
      const double m1b = a.b1 * a.m1b[u] + (1.0 - a.b1) * gb, vb = a.b2 * a.vb[u] + (1.0 - a.b2) * gb * gb;
      gamma -= a.lr * (m1g / a.c1) / (sqrt(vg / a.c2) + a.eps);
      betap -= a.lr * (m1b / a.c1) / (sqrt(vb / a.c2) + a.eps);
      if (l16 == 0) {
        a.m1g[u] = m1g;
        a.vg[u] = vg;
        a.m1b[u] = m1b;
        a.vb[u] = vb;
        a.gamma[u] = gamma;
        a.betap[u] = betap;
      }
      const LwcGroup pn = lwc_group(M, mn, row_first(gamma, lane), row_first(betap, lane), bits);
      write_integers<T, V>(a, w, row, g, l16, live, pn);
    }
  }
  if (l16 == 0) red[slot] = loss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i];
    a.lp[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
  }
}

// codes, scale, zero and W_hat with the final strengths
template <typename T, int V>
__global__ __launch_bounds__(256) void lwc_final(const T* __restrict__ W, LwcArgs a) {
  const IntShape& s = a.s;
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 6) * 4 + (lane >> 4);
  if (row >= s.n) return;
  for (int g = blockIdx.y; g < s.k; g += gridDim.y) {
    const int64_t u = (int64_t)g * s.npad + row, base = (int64_t)row * s.m + (int64_t)g * s.beta;
    const T* w = W + (int64_t)row * a.ldw + (int64_t)g * s.beta;
    const LwcGroup p = lwc_group(a.M[u], a.mn[u], a.gamma[u], a.betap[u], min(max((int)a.bits[g], 1), 8));
    const double inv = 1.0 / p.delta;
    for (int j = l16 * V; j < s.beta; j += 16 * V) {
      double v[V];
      load_weights<T, V>(w + j, v);
      unsigned word = 0;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const double q = fmin(fmax(rint_quotient(v[i], p, inv) + p.z, 0.0), p.Q);
        word |= (unsigned)q << (8 * i);
        v[i] = p.delta * (q - p.z);
      }
      if constexpr (V == 4)
        *reinterpret_cast<unsigned*>(a.codes + base + j) = word;
      else
        a.codes[base + j] = (uint8_t)word;
      if (a.What) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          if (a.what_f64)
            static_cast<double*>(a.What)[base + j + i] = v[i];
          else
            static_cast<float*>(a.What)[base + j + i] = (float)v[i];
        }
      }
    }
    if (l16 == 0) {
      a.scale[(int64_t)row * s.k + g] = p.delta;
      a.zero[(int64_t)row * s.k + g] = p.z;
    }
  }
}

struct LwcWorkspace {
  IntShape s;
  IntMeta mt;
  int64_t plane;
  int blocks_x, blocks_y;
  char *Xd, *Wd, *Q;
  double *SX, *SXlo, *WG, *WGlo, *DG, *lp, *loss;
  double* par[10];
  int *rest, *row_exp, *work, *token_unit;
};

size_t lwc_layout(int n, int m, int beta, int steps, char* base, LwcWorkspace& w) {
  const IntShape s = w.s = slim_int_shape(n, m, beta, m);
  w.plane = slim_int_plane(s);
  w.blocks_x = s.npad / 16;
  w.blocks_y = std::min(s.k, 8);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += slim_ws_round(bytes);
    return p;
  };
  auto doubles = [&](size_t count) { return reinterpret_cast<double*>(take(sizeof(double) * count)); };
  const bool ints = beta % 4 == 0;       // (else the fp64 form)
  w.Xd = take(std::max(ints ? slim_int_digits_bytes(s) : 0, sizeof(double) * (size_t)m * m));      // digits of G, or G in fp64
  w.Wd = take(ints ? (size_t)SI_MAXD * w.plane : 0);
  w.Q = take(ints ? (size_t)w.plane : 0);
  w.SX = doubles(ints ? (size_t)s.k * s.tpad : 0);
  w.SXlo = doubles(ints ? (size_t)s.k * s.tpad : 0);
  w.WG = doubles((size_t)n * m);
  w.WGlo = doubles(ints ? (size_t)n * m : 0);
  w.DG = doubles((size_t)n * m);
  w.lp = doubles((size_t)w.blocks_x * w.blocks_y);
  w.loss = doubles((size_t)steps + 1);
  for (double*& p : w.par) p = doubles((size_t)s.k * s.npad);
  w.mt.wunit = doubles(ints ? (size_t)s.C * s.npad : 0);
  w.mt.w = reinterpret_cast<uint8_t*>(take(ints ? (size_t)s.C * (s.npad / 16) : 0));
  int* mi = reinterpret_cast<int*>(take(sizeof(int) * (2 * (size_t)s.C * s.TB + (size_t)s.k + (size_t)s.npad + 1 + 3 * (size_t)m)));
  w.mt.x = mi;
  mi += 2 * (size_t)s.C * s.TB;
  w.rest = mi;
  w.row_exp = w.rest + s.k;
  w.mt.nonfinite = w.row_exp + s.npad;
  w.work = w.mt.nonfinite + 1;
  w.token_unit = w.work + 2 * m;
  return off;
}

template <typename T, int V>
slim_status lwc_run_v(slim_ctx* ctx, const LwcWorkspace& w, const T* W, LwcArgs& a, OutArgs& oa, slim_int_sums sums,
                      const slim_gemm_desc& wide, int steps, double beta1, double beta2) {
  const dim3 grid(w.blocks_x, w.blocks_y), block(256);
  SLIM_LAUNCH(ctx, "lwc_init", (lwc_init<T, V>), grid, block, 0, W, a);
  oa.Q = w.Wd;
  oa.Y = w.WG;
  oa.Ylo = w.WGlo;
  oa.sub = oa.sublo = nullptr;
  slim_status st = SLIM_OK;
  if (!a.D) st = slim_int_outputs(ctx, "lwc_wg_product", oa, true, sums);
  if (st != SLIM_OK) return st;
  oa.Q = w.Q;
  oa.Y = w.DG;
  oa.Ylo = nullptr;
  oa.sub = w.WG;
  oa.sublo = w.WGlo;
  for (int it = 1; it <= steps + 1; ++it) {
    oa.rest_from = it;
    st = a.D ? slim_dgemm(ctx, "lwc_grad_dgemm", 0, wide) : slim_int_outputs(ctx, "lwc_grad_product", oa, false, sums);
    if (st != SLIM_OK) return st;
    if (it <= steps) {
      a.c1 = 1.0 - std::pow(beta1, (double)it);
      a.c2 = 1.0 - std::pow(beta2, (double)it);
      a.step = it + 1;
      SLIM_LAUNCH(ctx, "lwc_step", (lwc_step<T, true, V>), grid, block, 0, W, a);
    } else {
      SLIM_LAUNCH(ctx, "lwc_loss", (lwc_step<T, false, V>), grid, block, 0, W, a);
    }
    st = slim_sum_f64(ctx, "lwc_loss_sum", w.lp, w.blocks_x * w.blocks_y, w.loss + (it - 1));
    if (st != SLIM_OK) return st;
  }
  SLIM_LAUNCH(ctx, "lwc_final", (lwc_final<T, V>), grid, block, 0, W, a);
  return SLIM_OK;
}
template <typename T>
slim_status lwc_run(slim_ctx* ctx, const LwcWorkspace& w, const T* W, LwcArgs& a, OutArgs& oa, slim_int_sums sums,
                    const slim_gemm_desc& wide, int steps, double beta1, double beta2) {
  return a.s.beta % 4 == 0 ? lwc_run_v<T, 4>(ctx, w, W, a, oa, sums, wide, steps, beta1, beta2)
                           : lwc_run_v<T, 1>(ctx, w, W, a, oa, sums, wide, steps, beta1, beta2);
}

}  // namespace

size_t slim_ws_need_lwc(int n, int m, int beta, int steps) {
  LwcWorkspace w;
  return lwc_layout(n, m, beta, steps, nullptr, w);
}

extern "C" slim_status slim_lwc_quantize(slim_ctx* ctx, const void* W, slim_dtype w_dtype, int n, int m, int64_t ldw,
                                         const float* G, int64_t ldg, int64_t n_tokens, const uint8_t* bits, int beta,
                                         int steps, double lr, double beta1, double beta2, double eps, double init,
                                         uint8_t* codes, double* scale, double* zero, void* What,
                                         slim_dtype what_dtype, double* loss_curve) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  SLIM_REQUIRE(ctx, W && G && bits && codes && scale && zero, "slim_lwc_quantize: null pointer");
  SLIM_REQUIRE(ctx, n > 0 && m > 0 && beta > 0 && m % beta == 0, "slim_lwc_quantize: need n, m > 0 and beta | m");
  SLIM_REQUIRE(ctx, m % 4 == 0 && ldw >= m && ldw % 4 == 0 && ldg >= m && ldg % 4 == 0,
               "slim_lwc_quantize: m, ldw and ldg must be multiples of 4");
  SLIM_REQUIRE(ctx, slim_aligned16(W) && slim_aligned16(G), "slim_lwc_quantize: misaligned pointer");
  SLIM_REQUIRE(ctx, n_tokens > 0 && steps >= 0 && steps <= 100000, "slim_lwc_quantize: need n_tokens > 0 and 0 <= steps <= 100000");
  SLIM_REQUIRE(ctx, lr > 0.0 && beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && eps > 0.0,
               "slim_lwc_quantize: need lr > 0, 0 <= beta1, beta2 < 1, eps > 0");
  if (w_dtype != SLIM_F16 && w_dtype != SLIM_BF16 && w_dtype != SLIM_F32)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "slim_lwc_quantize: W must be F16, BF16 or F32");
  if (What && what_dtype != SLIM_F32 && what_dtype != SLIM_F64)
    return slim_fail(ctx, SLIM_ERR_UNSUPPORTED, "slim_lwc_quantize: What must be F32 or F64");
  const int k = m / beta;
  SLIM_REQUIRE(ctx, (size_t)k <= (size_t)SLIM_HPIN_BYTES - sizeof(int) && sizeof(double) * (size_t)(steps + 1) <= (size_t)SLIM_HPIN_BYTES,
               "slim_lwc_quantize: too many groups or steps for the staging buffer");
  slim_status st = slim_ws_reserve(ctx, slim_ws_need_lwc(n, m, beta, steps));
  if (st != SLIM_OK) return st;
  LwcWorkspace w;
  lwc_layout(n, m, beta, steps, ctx->ws, w);
  const bool wide = beta % 4 != 0;
  slim_int_sums sums = slim_int_sums::twice;
  slim_gemm_desc d;
  d.A = w.WG;
  d.lda = m;
  d.B = reinterpret_cast<const double*>(w.Xd);
  d.ldb = m;
  d.C = w.DG;
  d.ldc = m;
  d.C2 = nullptr;
  d.ldc2 = 0;
  d.M = n;
  d.N = m;
  d.K = m;
  d.flags = 0;
  d.alpha = 1.0;
  d.beta = 0.0;
  if (wide) {
    st = slim_widen_f64(ctx, "lwc_widen_g", G, SLIM_F32, m, m, ldg, reinterpret_cast<double*>(w.Xd), (int64_t)m);
  } else {
    st = slim_int_clear(ctx, w.mt, w.rest, w.s.k + w.s.npad);
    if (st == SLIM_OK) st = slim_int_w_units(ctx, w.s, w.mt, W, w_dtype, ldw);
    if (st == SLIM_OK) st = slim_int_g_digits(ctx, w.s, w.mt, G, ldg, w.work, w.token_unit, w.Xd, w.SX, w.SXlo);
  }
  if (st != SLIM_OK) return st;
  // the widths are validated before anything but the workspace is written (not a hot path: the host waits for them); with them
  // comes which of the two products suits the digits of G
  constexpr int COST_AT = SLIM_HPIN_BYTES - (int)sizeof(int);
  const uint8_t* bits_h = reinterpret_cast<const uint8_t*>(ctx->hpin);
  SLIM_HIP_TRY(ctx, hipMemcpyAsync(ctx->hpin, bits, k, hipMemcpyDeviceToHost, ctx->stream));
  if (!wide) SLIM_HIP_TRY(ctx, hipMemcpyAsync(ctx->hpin + COST_AT, w.work, sizeof(int), hipMemcpyDeviceToHost, ctx->stream));
  SLIM_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  for (int g = 0; g < k; ++g)
    SLIM_REQUIRE(ctx, bits_h[g] >= 1 && bits_h[g] <= 8, "slim_lwc_quantize: bits[%d] = %d is outside 1..8", g, (int)bits_h[g]);
  if (!wide && slim_int_pairs_pay(*reinterpret_cast<const int*>(ctx->hpin + COST_AT))) sums = slim_int_sums::by_pairs;

  LwcArgs a;
  a.s = w.s;
  a.mt = w.mt;
  a.ldw = ldw;
  a.bits = bits;
  a.M = w.par[0];
  a.mn = w.par[1];
  a.gamma = w.par[2];
  a.betap = w.par[3];
  a.m1g = w.par[4];
  a.vg = w.par[5];
  a.m1b = w.par[6];
  a.vb = w.par[7];
  a.Q = w.Q;
  a.S = w.par[8];
  a.Rz = w.par[9];
  a.rest = w.rest;
  a.row_exp = w.row_exp;
  a.Wd = w.Wd;
  a.D = wide ? w.WG : nullptr;
  a.DG = w.DG;
  a.lp = w.lp;
  a.gscale = 2.0 / ((double)n * (double)n_tokens);
  a.init = init;
  a.lr = lr;
  a.b1 = beta1;
  a.b2 = beta2;
  a.eps = eps;
  a.c1 = a.c2 = 1.0;
  a.step = 1;
  a.codes = codes;
  a.scale = scale;
  a.zero = zero;
  a.What = What;
  a.what_f64 = (what_dtype == SLIM_F64);
  OutArgs oa;
  oa.s = w.s;
  oa.mt = w.mt;
  oa.Xd = w.Xd;
  oa.SX = w.SX;
  oa.SXlo = w.SXlo;
  oa.plane = w.plane;
  oa.S = a.S;
  oa.Rz = a.Rz;
  oa.rest = w.rest;
  oa.row_exp = w.row_exp;
  oa.rest_from = 1;
  oa.token_unit = w.token_unit;
  st = w_dtype == SLIM_F16    ? lwc_run(ctx, w, static_cast<const __half*>(W), a, oa, sums, d, steps, beta1, beta2)
       : w_dtype == SLIM_BF16 ? lwc_run(ctx, w, static_cast<const __hip_bfloat16*>(W), a, oa, sums, d, steps, beta1, beta2)
                              : lwc_run(ctx, w, static_cast<const float*>(W), a, oa, sums, d, steps, beta1, beta2);
  if (st != SLIM_OK) return st;
  if (!loss_curve) return SLIM_OK;                 // nothing for the host: the call does not wait
  double* host = reinterpret_cast<double*>(ctx->hpin);
  SLIM_HIP_TRY(ctx, hipMemcpyAsync(host, w.loss, sizeof(double) * (size_t)(steps + 1), hipMemcpyDeviceToHost, ctx->stream));
  SLIM_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  const double norm = (double)n * (double)n_tokens;
  for (int i = 0; i <= steps; ++i) loss_curve[i] = host[i] / norm;
  return SLIM_OK;
}
