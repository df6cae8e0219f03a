// a2  Damped inverse Hessian and its upper Cholesky factor (Def. 1; Alg. 1 line 2), all in fp64.
//
// Wanted: upper-triangular U with (H + lambda I)^-1 = U^T U.  Writing R = U^-1 (upper triangular) gives
// H + lambda I = R R^T, a Cholesky factorisation taken from the bottom-right corner upwards, so the
// textbook route (factor, invert, factor again) collapses to ONE factorisation and ONE triangular
// inverse, (2/3) m^3 flops instead of (4/3) m^3:
//
//   1. widen:   A = (2 / n_tokens) G + lambda I,  lambda = percdamp * mean(diag(2 / n_tokens G))
//   2. for the diagonal blocks J = last .. first (64 columns each; eight of them form a group), one launch each:
//        diagonal    one workgroup: applies the last pending rank-64 update to A_JJ itself, factors
//                    A_JJ = R_JJ R_JJ^T and inverts R_JJ (V_JJ, written into U)
//        panel       R[0:J+1, J+1] = A[0:J+1, J+1] V^T of the block to the right, beside it
//        update      rank-64 update with that panel of the columns from the start of block J's group on
//      and once per group rank-512 updates of everything further left; see the schedule at the call site.
//      (the large ones, and the large terms of step 3, from residues on the int8 matrix cores: rgemm.hip)
//   3. triangular inverse U = R^-1 group by group on a further stream, beside the factorisation: inside a group
//      strip by strip of 16 columns from the inverted diagonal blocks upwards, in one launch, the
//      rows right of the group from T = R[g, S] U[S, S], which is kept up to date for all rows above by one
//      rank-512 product per finished group (see the schedule at the call site).
//   4. hinv_diag_j = sum_i U_ij^2.
#include "slim_device.h"
#include "slim_internal.h"

namespace {

constexpr int NB = 64;          // diagonal block
// Diagonal blocks per group.  With 8 the far updates have rank 512 (64 flops per byte of A they move, against 32 with
// 4) and there are half as many of them; the windows of the chain get wider.  Inverse alone at m = 11008: 21.7 against
// 22.2 ms; whole pass: 0.5 ms less on the 4096 x 11008 and 28672 x 8192 layers, 0.2 ms less on 4096 x 4096.
constexpr int GRP = 8;

// mean of the diagonal of H = s * G, then lambda; single workgroup, fixed order
__global__ __launch_bounds__(1024) void damp_lambda(const float* __restrict__ G, int64_t ldg, int m, double s,
                                                    double percdamp, double* __restrict__ lam_out,
                                                    int* __restrict__ flag) {
  __shared__ double red[1024];
  if (threadIdx.x == 0) *flag = 0;
  double acc = 0.0;
  for (int i = threadIdx.x; i < m; i += 1024) acc += s * (double)G[(int64_t)i * ldg + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 512; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) *lam_out = percdamp * (red[0] / (double)m);
}

// A = s * G + lambda I on and above the diagonal; U = 0 below it.  V consecutive columns per thread.
// What lies below the diagonal of A is never read as a value that matters (the updates that sweep over it only
// add to it), and every element of U on or above the diagonal is written later (the inverted diagonal blocks,
// then the merged off-diagonal ones), so pieces entirely on one side are written to one matrix only.
template <int V>
__global__ __launch_bounds__(256) void widen_damp(const float* __restrict__ G, int64_t ldg, int m, double s,
                                                  const double* __restrict__ lam, double* __restrict__ A,
                                                  int64_t lda, double* __restrict__ U, int64_t ldu) {
  constexpr int ROWS = 8;                      // rows per thread: the loads of all of them are issued first
  const int c0 = (blockIdx.x * 256 + threadIdx.x) * V;
  const int r0 = blockIdx.y * ROWS;
  if (c0 >= m) return;
  float g[ROWS][V];
#pragma unroll
  for (int q = 0; q < ROWS; ++q) {
    const int r = r0 + q;
#pragma unroll
    for (int v = 0; v < V; ++v) g[q][v] = 0.0f;
    if (r < m && c0 + V - 1 >= r) {            // something of this piece lies on or above the diagonal
      const float* src = G + (int64_t)r * ldg + c0;
      if (V == 4) {
        const float4 t = *reinterpret_cast<const float4*>(src);
        g[q][0] = t.x, g[q][1] = t.y, g[q][2] = t.z, g[q][3] = t.w;
      } else if (V == 2) {
        const float2 t = *reinterpret_cast<const float2*>(src);
        g[q][0] = t.x, g[q][1] = t.y;
      } else {
        g[q][0] = src[0];
      }
    }
  }
  const double lambda = *lam;
#pragma unroll
  for (int q = 0; q < ROWS; ++q) {
    const int r = r0 + q;
    if (r >= m) break;
    double a[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int c = c0 + v;
      a[v] = c >= r ? s * (double)g[q][v] : 0.0;
      if (c == r) a[v] += lambda;
    }
    double* da = A + (int64_t)r * lda + c0;
    double* du = U + (int64_t)r * ldu + c0;
    const bool upper = c0 + V - 1 >= r;        // has an element on or above the diagonal
    const bool lower = c0 < r;                 // has an element below it
    if (V == 1) {
      if (upper) da[0] = a[0];
      if (lower) du[0] = 0.0;
    } else {
#pragma unroll
      for (int v = 0; v < V; v += 2) {
        if (upper) *reinterpret_cast<double2*>(da + v) = make_double2(a[v], a[v + 1]);
        if (lower) *reinterpret_cast<double2*>(du + v) = make_double2(0.0, 0.0);
      }
    }
  }
}

// 1 / x to full double precision for positive finite x: hardware estimate plus two Newton steps
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// ---- the diagonal block ----------------------------------------------------------------------------------------------
// One workgroup of eight wavefronts per diagonal block, with tiles of 16 x 16:
//   prologue  (nprev > 0)  Rn = A[J, J+1] V_{J+1}^T and A_JJ -= Rn Rn^T on the matrix cores: the update with the panel of block
//             J+1 restricted to this block, so that this kernel does not have to wait for the GEMMs of block J+1
//   factor    A_JJ = R R^T with R upper triangular, tile column by tile column from the last to the first: sixteen pivots in
//             registers, then the rank-16 update of the tiles left of them on the matrix cores
//   invert    V = R^-1, written to Vout
// A non-positive pivot is recorded in flag[0] (1-based global column); the outputs are then meaningless.
//
// The block is a chain of 64 pivots and what bounds it is latency.  A wavefront that owns a tile column eliminates it without
// LDS or barriers: lane = row, register = column, and the entries of the pivot column come to all lanes of a 16-lane row with
// the row_newbcast operand of v_fmac_f64_dpp (16 cycles behind the instruction that made them, a dependent fp64 fma 5, a
// reciprocal 25; an LDS write, barrier and read of eight wavefronts 170).  The diagonal tile lies in all four 16-lane rows.
// Wavefront 0 eliminates the tile column above it along with it (one lane a row of the block), wavefront 1 repeats the diagonal
// tile's elimination and turns the identity into the tile's inverse by the same row operations.  The reciprocal of the next
// pivot is formed between the updates of the columns that it does not need.  The other tiles of
// A stay in the accumulators of wavefronts 2, 3, 6 and 7, which also put V together while the next tile column is factored:
//   V_ik = -V_ii T_ik,  T_ik = sum over i < l <= k of R_il V_lk.
// Cycles (of 2.4 GHz) of the same block: loads 3500, prologue 5200, pivots and updates 24000, rest 1500, 15.9 us a launch back to
// back, against 4000, 10400, 32300 and 3500 (22.5 us) of a form that published four columns at a time through LDS.
constexpr int CB_LD = 66;       // rows of the staged 64 x 64 operands
constexpr int CB_PAN = 48;      // rows of a panel (a column of it after the other)
constexpr int CB_VLD = 18;      // rows of a tile of V

typedef double double4v __attribute__((ext_vector_type(4)));

struct CholArgs {
  const double* A;       // A[j0][j0]: the diagonal block (upper triangle valid)
  int64_t lda;
  int nbk;               // width of this block (64, less for a ragged last block)
  int nprev;             // width of block J+1 whose rank-64 update is still pending on this block (0: none)
  const double* Vprev;   // V of block J+1 (in U)
  double* Vout;          // V of this block (in U; its tiles below the diagonal ones are zero already)
  int64_t ldv;
  int* flag;
  int col_base;
};

template <int N>
__device__ __forceinline__ double newbcast(double x) {
  return __longlong_as_double(__builtin_amdgcn_update_dpp((long long)0, __double_as_longlong(x), 0x150 + N, 0xf, 0xf, true));
}
// Updates of columns with an entry of their 16-lane row, several to a statement: a DPP operand must have been written two
// instructions before it is read, and the compiler, which does not look into the statements, may put copies in front of one.
#define CB_FMAC(Y, X, S, N) "\n\tv_fmac_f64_dpp " Y ", " X ", " S " row_newbcast:" N " row_mask:0xf bank_mask:0xf"
// y[N .. N - M + 1] += (x of lane N, N - 1, ...) * s
template <int N, int M>
__device__ __forceinline__ void columns(double (&y)[16], double x, double s) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (M == 1)
    asm volatile("s_nop 1" CB_FMAC("%0", "%1", "%2", "%3") : "+v"(y[N]) : "v"(x), "v"(s), "n"(N));
  if constexpr (M == 2)
    asm volatile("s_nop 1" CB_FMAC("%0", "%2", "%3", "%4") CB_FMAC("%1", "%2", "%3", "%5")
                 : "+v"(y[N]), "+v"(y[N - 1]) : "v"(x), "v"(s), "n"(N), "n"(N - 1));
  if constexpr (M == 3)
    asm volatile("s_nop 1" CB_FMAC("%0", "%3", "%4", "%5") CB_FMAC("%1", "%3", "%4", "%6") CB_FMAC("%2", "%3", "%4", "%7")
                 : "+v"(y[N]), "+v"(y[N - 1]), "+v"(y[N - 2]) : "v"(x), "v"(s), "n"(N), "n"(N - 1), "n"(N - 2));
#endif
}
// both the tile's columns and those above it: d[N ..] += (x of lane N ..) * sd, o[N ..] += (x of lane N ..) * so
template <int N, int M>
__device__ __forceinline__ void columns(double (&d)[16], double (&o)[16], double x, double sd, double so) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (M == 1)
    asm volatile("s_nop 1" CB_FMAC("%0", "%2", "%3", "%5") CB_FMAC("%1", "%2", "%4", "%5")
                 : "+v"(d[N]), "+v"(o[N]) : "v"(x), "v"(sd), "v"(so), "n"(N));
  if constexpr (M == 2)
    asm volatile("s_nop 1" CB_FMAC("%0", "%4", "%5", "%7") CB_FMAC("%1", "%4", "%6", "%7") CB_FMAC("%2", "%4", "%5", "%8")
                     CB_FMAC("%3", "%4", "%6", "%8")
                 : "+v"(d[N]), "+v"(o[N]), "+v"(d[N - 1]), "+v"(o[N - 1]) : "v"(x), "v"(sd), "v"(so), "n"(N), "n"(N - 1));
#endif
}
// e[C .. C + M - 1] += (their own entry in lane N) * s
template <int N, int C, int M>
__device__ __forceinline__ void rows(double (&e)[16], double s) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (M == 1) asm volatile("s_nop 1" CB_FMAC("%0", "%0", "%1", "%2") : "+v"(e[C]) : "v"(s), "n"(N));
  if constexpr (M == 2)
    asm volatile("s_nop 1" CB_FMAC("%0", "%0", "%2", "%3") CB_FMAC("%1", "%1", "%2", "%3") : "+v"(e[C]), "+v"(e[C + 1]) : "v"(s), "n"(N));
  if constexpr (M == 3)
    asm volatile("s_nop 1" CB_FMAC("%0", "%0", "%3", "%4") CB_FMAC("%1", "%1", "%3", "%4") CB_FMAC("%2", "%2", "%3", "%4")
                 : "+v"(e[C]), "+v"(e[C + 1]), "+v"(e[C + 2]) : "v"(s), "n"(N));
#endif
}
#undef CB_FMAC
// holds its place among the updates above
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

// Pivot T of the diagonal tile d (lane = row, register = column): p and its reciprocal r.  The next pivot's are fetched and
// formed in five pieces between the updates of the columns left of it.
struct Pivot {
  double p, r, e;
  template <int S>
  __device__ __forceinline__ void piece() {
    if constexpr (S == 0) r = __builtin_amdgcn_rcp(p);
    if constexpr (S == 1 || S == 3) e = fma(-p, r, 1.0);
    if constexpr (S == 2 || S == 4) r = fma(e, r, r);
    pin(r);
    pin(e);
  }
  template <int N>
  __device__ __forceinline__ void fetch(double (&d)[16]) {
    asm volatile("s_nop 1" : "+v"(d[N]));
    p = newbcast<N>(d[N]);
    pin(p);
  }
};
// o: the tile column above the tile (lane = row of the block)
template <int T, int C, int S>
__device__ __forceinline__ void panel_columns(Pivot& pv, double (&d)[16], double (&o)[16], double sd, double so) {
  constexpr int M = C >= 1 ? 2 : (C == 0 ? 1 : 0);
  if constexpr (M > 0) columns<C, M>(d, o, d[T], sd, so);
  if constexpr (S < 5) pv.piece<S>();
  if constexpr (C - M >= 0 || S < 4) panel_columns<T, C - M, S + 1>(pv, d, o, sd, so);
}
template <int T>
__device__ __forceinline__ void panel_pivots(Pivot& pv, double (&d)[16], double (&o)[16], double* col, bool write) {
  const double sd = -d[T] * pv.r, so = -o[T] * pv.r;
  if (write) col[T * CB_PAN] = o[T];
  if constexpr (T > 0) {
    columns<T - 1, 1>(d, o, d[T], sd, so);
    pv.fetch<T - 1>(d);
    panel_columns<T, T - 2, 0>(pv, d, o, sd, so);
    panel_pivots<T - 1>(pv, d, o, col, write);
  }
}
// e: the tile's inverse, but for the scale of its rows.  C: the next column of d; E: the next one of e
template <int T, int C, int E, int S>
__device__ __forceinline__ void inverse_columns(Pivot& pv, double (&d)[16], double (&e)[16], double sd, double se) {
  constexpr int M = C >= 2 ? 3 : C + 1, K = M > 0 ? 0 : (E <= 12 ? 3 : 15 - E);
  if constexpr (M > 0) columns<C, M>(d, d[T], sd);
  if constexpr (K > 0) rows<T, E, K>(e, se);
  if constexpr (S < 5) pv.piece<S>();
  if constexpr (C - M >= 0 || E + K < 15 || S < 4) inverse_columns<T, C - M, E + K, S + 1>(pv, d, e, sd, se);
}
template <int T, int END>
__device__ __forceinline__ void inverse_pivots(Pivot& pv, double (&d)[16], double (&e)[16], double& own_p, double& own_r, int l16) {
  const double sd = -d[T] * pv.r;
  const double se = l16 < T ? sd : 0.0;          // rows at and below the pivot take no part in the row operations
  own_p = l16 == T ? pv.p : own_p;
  own_r = l16 == T ? pv.r : own_r;
  if constexpr (T > 0) {
    columns<T - 1, 1>(d, d[T], sd);
    rows<T, 15, 1>(e, se);
    pv.fetch<T - 1>(d);
    inverse_columns<T, T - 2, T, 0>(pv, d, e, sd, se);
    if constexpr (T > END) inverse_pivots<T - 1, END>(pv, d, e, own_p, own_r, l16);
  }
}
// 1 / sqrt(x) for positive finite x, within one unit of its last place: hardware estimate plus two Newton steps
__device__ __forceinline__ double fast_rsq(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// acc += A B^T of two staged operands (row = output row / column), columns 8 s0 .. 63
__device__ __forceinline__ double4v staged_product(const double* a, const double* b, int s0, double4v acc) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    if (s < s0) continue;                        // the same for the wavefront
    const double2 x = *reinterpret_cast<const double2*>(a + 8 * s), y = *reinterpret_cast<const double2*>(b + 8 * s);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, acc, 0, 0, 0);
  }
  return acc;
}

__device__ __forceinline__ void chol_block(const CholArgs& g, double* sm) {
  double* Ps = sm;                           // [64][CB_LD]: A[J, J+1], then Rn, then the tiles of V and 1 / sqrt(pivot)
  double* Vs = sm + NB * CB_LD;              // [64][CB_LD]: V_{J+1}, then the tile column in hand, panels and reciprocals
  double* Dn = Vs;                           // [16][CB_LD]: the next tile column, one column after the other
  double* rcps = Vs + 16 * CB_LD;            // [64]: reciprocals of the pivots
  double* pan = rcps + NB;                   // [3][16][CB_PAN]: panels of tile columns 1 to 3 (before their scale 1 / sqrt(pivot))
  double* rsq = Ps;                          // [64]
  double* Vt = Ps + NB;                      // [10][16][CB_VLD]: tiles (i, k) of V at vt(i, k)
  auto vt = [&](int i, int k) { return Vt + (i * 4 - i * (i - 1) / 2 + (k - i)) * 16 * CB_VLD; };
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int nbk = g.nbk, np = g.nprev;
  const int prior_flag = g.flag[0];
  // Tiles of A and of V, by wavefront: two of each for 2 and 3, one for 6 and 7.  The wavefronts that share a SIMD with the
  // pivots (0 and 4, 1 and 5) have none: fp64 MFMAs take the units that fp64 vector instructions need.
  const bool tiles = (w & 2) != 0;
  const int owned = w < 4 ? 2 : 1;
  const int ai[2] = {w == 2 ? 0 : (w == 3 ? 1 : (w == 6 ? 2 : 0)), w == 2 ? 0 : 1};
  const int ak[2] = {w == 7 ? 0 : 2, 1};
  const int vi[2] = {w == 7 ? 1 : 0, w == 2 ? 2 : 1};
  const int vk[2] = {w == 2 ? 1 : (w == 6 ? 3 : 2), 3};
  // result register v of a lane is row 4 v + lk, column l16 of a tile; identity padding of a ragged block
  auto load_tile = [&](int i, int k) {
    double4v t;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * i + 4 * v + lk, c = 16 * k + l16;
      t[v] = r == c ? 1.0 : 0.0;
      if (r < nbk && c < nbk) t[v] = c >= r ? g.A[(int64_t)r * g.lda + c] : 0.0;
    }
    return t;
  };
  double4v first = {0.0, 0.0, 0.0, 0.0}, at[2] = {first, first}, vtile[2] = {first, first};
  double2 ldp[4], ldv[4];
  if (np > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (tid >> 5) + 16 * i, c = 2 * (tid & 31);
      ldp[i] = ldv[i] = make_double2(0.0, 0.0);
      if (c < np) ldp[i] = *reinterpret_cast<const double2*>(g.A + (int64_t)r * g.lda + NB + c);
      if (c < np && r < np && c + 1 >= r) ldv[i] = *reinterpret_cast<const double2*>(g.Vprev + (int64_t)r * g.ldv + c);
    }
  }
  if (w < 4) first = load_tile(w, 3);
  if (tiles) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (j < owned) at[j] = load_tile(ai[j], ak[j]);
  }
  if (np > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at_ = ((tid >> 5) + 16 * i) * CB_LD + 2 * (tid & 31);
      *reinterpret_cast<double2*>(Ps + at_) = ldp[i];
      *reinterpret_cast<double2*>(Vs + at_) = ldv[i];
    }
    __syncthreads();
    // Rn: tile column tj needs k >= 16 tj only; every wavefront has 20 MFMAs
    const int ti = w & 3, tj0 = w < 4 ? 0 : 1, tj1 = w < 4 ? 3 : 2;
    const double4v zero = {0.0, 0.0, 0.0, 0.0};
    const double* ap = Ps + (16 * ti + l16) * CB_LD + 2 * lk;
    const double4v r0 = staged_product(ap, Vs + (16 * tj0 + l16) * CB_LD + 2 * lk, 2 * tj0, zero);
    const double4v r1 = staged_product(ap, Vs + (16 * tj1 + l16) * CB_LD + 2 * lk, 2 * tj1, zero);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double* row = Ps + (16 * ti + 4 * v + lk) * CB_LD + l16;
      row[16 * tj0] = r0[v];
      row[16 * tj1] = r1[v];
    }
    __syncthreads();
    if (w < 4)
      first -= staged_product(Ps + (16 * w + l16) * CB_LD + 2 * lk, Ps + (48 + l16) * CB_LD + 2 * lk, 0, zero);
  }
  auto store_column = [&](int i, const double4v& t) {     // tile (i, .) of the tile column that is next
#pragma unroll
    for (int v = 0; v < 4; ++v) Dn[l16 * CB_LD + 16 * i + 4 * v + lk] = t[v];
  };
  if (w < 4) store_column(w, first);
  __syncthreads();
  if (tiles && np > 0) {                         // beside the pivots of the last tile column
    const double4v zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (j < owned)
        at[j] -= staged_product(Ps + (16 * ai[j] + l16) * CB_LD + 2 * lk, Ps + (16 * ak[j] + l16) * CB_LD + 2 * lk, 0, zero);
  }
  // A operand of step s: row l16, column 4 s + lk
  auto panel_scaled = [&](int i, int b, int s) {          // R_ib
    return pan[((b - 1) * 16 + 4 * s + lk) * CB_PAN + 16 * i + l16] * rsq[16 * b + 4 * s + lk];
  };
  auto times_tile = [&](double4v acc, int i, int b, const double* B) {   // acc += R_ib B
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(panel_scaled(i, b, s), B[(4 * s + lk) * CB_VLD + l16], acc, 0, 0, 0);
    return acc;
  };
  auto finish_tile = [&](int i, int k, double4v T) {      // V_ik = -V_ii T_ik
    double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-vt(i, i)[l16 * CB_VLD + 4 * s + lk], T[s], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * i + 4 * v + lk, c = 16 * k + l16;
      vt(i, k)[(4 * v + lk) * CB_VLD + l16] = acc[v];
      if (r < nbk && c < nbk) g.Vout[(int64_t)r * g.ldv + c] = acc[v];
    }
  };
  auto store_diagonal = [&](int b) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * b + 4 * v + lk, c = 16 * b + l16;
      if (r < nbk && c < nbk) g.Vout[(int64_t)r * g.ldv + c] = vt(b, b)[(4 * v + lk) * CB_VLD + l16];
    }
  };
  int bad = 0;
#pragma unroll 1
  for (int b = 3; b >= 0; --b) {
    double own_p = 1.0, own_r = 1.0;
    double e[16];
    if (w == 0 && b > 0) {
      __builtin_amdgcn_s_setprio(3);
      double d[16], o[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        d[c] = Dn[c * CB_LD + 16 * b + l16];
        o[c] = Dn[c * CB_LD + lane];
      }
      Pivot pv;
      pv.e = 0.0;
      pv.fetch<15>(d);
      pv.r = fast_rcp(pv.p);
      panel_pivots<15>(pv, d, o, pan + (b - 1) * 16 * CB_PAN + lane, lane < 16 * b);
      __builtin_amdgcn_s_setprio(0);
    } else if (w == 1) {
      __builtin_amdgcn_s_setprio(3);
      double d[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        d[c] = Dn[c * CB_LD + 16 * b + l16];
        e[c] = l16 == c ? 1.0 : 0.0;
      }
      Pivot pv;
      pv.e = 0.0;
      pv.fetch<15>(d);
      pv.r = fast_rcp(pv.p);
      inverse_pivots<15, 8>(pv, d, e, own_p, own_r, l16);
      if (b == 0) __syncthreads();               // the tiles that the first tile row still needs
      inverse_pivots<7, 0>(pv, d, e, own_p, own_r, l16);
      if (lane < 16) rcps[16 * b + lane] = own_r;
      __builtin_amdgcn_s_setprio(0);
    } else if (tiles) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j >= owned) continue;
        // T_ik and V_ik as far as the tiles and panels of the tile rows below allow
        if (b == 2 && vk[j] == 3) vtile[j] = times_tile(vtile[j], vi[j], 3, vt(3, 3));
        if (b == 1 && vk[j] == 2) vtile[j] = times_tile(vtile[j], vi[j], 2, vt(2, 2));
        if (b == 1 && vi[j] == 2) finish_tile(2, 3, vtile[j]);
        if (b == 0) {
          if (vk[j] == 3 && vi[j] < 2) vtile[j] = times_tile(vtile[j], vi[j], 2, vt(2, 3));
          if (vk[j] == 1) vtile[j] = times_tile(vtile[j], 0, 1, vt(1, 1));
          if (vi[j] == 1) finish_tile(1, vk[j], vtile[j]);
        }
      }
      if (b < 3 && w == 7) store_diagonal(b + 1);
    }
    if (b == 0) {
      if (w != 1) __syncthreads();
      if (tiles && vi[0] == 0 && vk[0] > 1) vtile[0] = times_tile(vtile[0], 0, 1, vt(1, vk[0]));
    }
    __syncthreads();
    if (tiles) {
      // rank-16 update, with the panel's columns divided by their pivots on one side
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (j >= owned || ak[j] >= b) continue;
        const double* p = pan + ((b - 1) * 16 + lk) * CB_PAN + l16;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          at[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[4 * s * CB_PAN + 16 * ai[j]],
                                                       -p[4 * s * CB_PAN + 16 * ak[j]] * rcps[16 * b + 4 * s + lk], at[j], 0, 0, 0);
        if (ak[j] == b - 1) store_column(ai[j], at[j]);
      }
    }
    if (w == 1) {
      const double rs = fast_rsq(own_p);
      if (!(own_p > 0.0) && 16 * b + l16 < nbk) bad = max(bad, 16 * b + l16 + 1);
      if (lane < 16) {
        rsq[16 * b + lane] = rs;
#pragma unroll
        for (int c = 0; c < 16; c += 2)
          *reinterpret_cast<double2*>(vt(b, b) + lane * CB_VLD + c) = make_double2(e[c] * rs, e[c + 1] * rs);
      }
    }
    __syncthreads();
  }
  if (tiles && vi[0] == 0) finish_tile(0, vk[0], vtile[0]);
  if (w == 7) store_diagonal(0);
  // the first failure in elimination order is kept: the highest column of the first block that fails
  if (bad && prior_flag == 0) atomicMax(g.flag, g.col_base + bad);
}

constexpr size_t CHOL_LDS = sizeof(double) * 2 * NB * CB_LD;

__global__ __launch_bounds__(512) void chol_step(CholArgs g) {
  extern __shared__ __align__(16) double sm[];
  chol_block(g, sm);
}

struct LinkArgs {
  CholArgs next;         // the diagonal block left of J
  double* A;
  double* R;
  int64_t lda;
  const double* V;       // of block J
  int64_t ldv;
  int J, nbk;            // block J and its width
  int wt;                // first block of the window
};

// One link of the factorisation's chain in one launch: workgroup 0 factors the diagonal block left of J (which needs the panel
// of J restricted to its own rows only, see chol_block), the others share out the rest of what block J gives:
//   panel   R[0:j0, J] = A[0:j0, J] V_JJ^T
//   window  A[r, c] -= R[r, J] R[c, J]^T for the blocks r < J - 1 and wt <= c < J, r <= c
// A workgroup has one 64 x 64 block (r, c) and forms the two pieces of the panel that it needs itself (their product with the
// triangular V is 5/8 of a full one), so that nothing in the launch waits for anything else in it; the one with c = J - 1 writes
// the panel.  With the panel and the window as launches of their own on a second stream, whose events the diagonal steps waited
// for, a link was five calls of the host, which took 35 us, and 37 us on the chip.  The whole inverse alone on the chip, that
// form and this one: m = 256 260 and 133 us, 1504 980 and 622, 4096 2760 and 1960, 8192 9650 and 9010.
__global__ __launch_bounds__(512) void chol_link(LinkArgs g) {
  extern __shared__ __align__(16) double sm[];
  if (blockIdx.x == 0) {
    chol_block(g.next, sm);
    return;
  }
  const int nc = g.J - g.wt;
  int id = blockIdx.x - 1, r, c;
  if (id < g.wt * nc) {
    r = id / nc;
    c = g.wt + id % nc;
  } else {
    id -= g.wt * nc;
    r = g.wt;
    while (id >= g.J - r) id -= g.J - r++;       // (at most eight rows)
    c = r + id;
  }
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int ti = w & 3, tj0 = w < 4 ? 0 : 1, tj1 = w < 4 ? 3 : 2;
  const bool same = r == c, update = r < g.J - 1;
  double* bufr = sm;
  double* bufc = same ? sm : sm + NB * CB_LD;
  const int64_t j0 = (int64_t)g.J * NB;
  double2 ar[4], ac[4], v0[8], v1[8];
  double4v c0 = {0.0, 0.0, 0.0, 0.0}, c1 = c0;
  const double4v zero = c0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = (tid >> 5) + 16 * i, col = 2 * (tid & 31);
    ar[i] = ac[i] = make_double2(0.0, 0.0);
    if (col < g.nbk) {
      ar[i] = *reinterpret_cast<const double2*>(g.A + ((int64_t)r * NB + row) * g.lda + j0 + col);
      if (!same) ac[i] = *reinterpret_cast<const double2*>(g.A + ((int64_t)c * NB + row) * g.lda + j0 + col);
    }
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int k = 8 * s + 2 * lk, n0 = 16 * tj0 + l16, n1 = 16 * tj1 + l16;
    v0[s] = v1[s] = make_double2(0.0, 0.0);
    if (s >= 2 * tj0 && k < g.nbk && n0 < g.nbk) v0[s] = *reinterpret_cast<const double2*>(g.V + (int64_t)n0 * g.ldv + k);
    if (s >= 2 * tj1 && k < g.nbk && n1 < g.nbk) v1[s] = *reinterpret_cast<const double2*>(g.V + (int64_t)n1 * g.ldv + k);
  }
  double* C = g.A + ((int64_t)r * NB + 16 * ti + lk) * g.lda + (int64_t)c * NB + l16;
  if (update) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      c0[v] = C[4 * v * g.lda + 16 * tj0];
      c1[v] = C[4 * v * g.lda + 16 * tj1];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int at = ((tid >> 5) + 16 * i) * CB_LD + 2 * (tid & 31);
    *reinterpret_cast<double2*>(bufr + at) = ar[i];
    if (!same) *reinterpret_cast<double2*>(bufc + at) = ac[i];
  }
  __syncthreads();
  auto times_v = [&](const double* buf, const double2 (&v)[8], int tj) {       // rows 16 ti of the buffer times V^T
    const double* a = buf + (16 * ti + l16) * CB_LD + 2 * lk;
    double4v acc = zero;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (s < 2 * tj) continue;
      const double2 x = *reinterpret_cast<const double2*>(a + 8 * s);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v[s].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, v[s].y, acc, 0, 0, 0);
    }
    return acc;
  };
  const double4v r0 = times_v(bufr, v0, tj0), r1 = times_v(bufr, v1, tj1);
  double4v q0 = zero, q1 = zero;
  if (!same) {
    q0 = times_v(bufc, v0, tj0);
    q1 = times_v(bufc, v1, tj1);
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int at = (16 * ti + 4 * v + lk) * CB_LD + l16;
    bufr[at + 16 * tj0] = r0[v];
    bufr[at + 16 * tj1] = r1[v];
    if (!same) {
      bufc[at + 16 * tj0] = q0[v];
      bufc[at + 16 * tj1] = q1[v];
    }
  }
  if (c == g.J - 1) {
    double* R = g.R + ((int64_t)r * NB + 16 * ti + lk) * g.lda + j0 + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (16 * tj0 + l16 < g.nbk) R[4 * v * g.lda + 16 * tj0] = r0[v];
      if (16 * tj1 + l16 < g.nbk) R[4 * v * g.lda + 16 * tj1] = r1[v];
    }
  }
  if (!update) return;
  __syncthreads();
  const double* a = bufr + (16 * ti + l16) * CB_LD + 2 * lk;
  c0 -= staged_product(a, bufc + (16 * tj0 + l16) * CB_LD + 2 * lk, 0, zero);
  c1 -= staged_product(a, bufc + (16 * tj1 + l16) * CB_LD + 2 * lk, 0, zero);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    C[4 * v * g.lda + 16 * tj0] = c0[v];
    C[4 * v * g.lda + 16 * tj1] = c1[v];
  }
}

// ---- the triangular inverse inside a group -----------------------------------------------------------------------
// U[i, j] = -U[i, i] sum over k = i + 1 .. j of R[i, k] U[k, j] for the blocks of a group, i upwards from j - 1: a workgroup takes 16
// columns of a block column j and keeps them in LDS, so that the whole group is one launch.  grid: 4 strips of each block column from
// the second on, the longest chains first; 4 wavefronts, each 16 rows of the block in hand.
//
// What bounds it is the chain of a strip, on 28 CUs: 28 * 16 + 7 * 16 MFMAs per wavefront at most, 15 us by themselves, and the trips
// to memory and barriers between them.  512 columns: 40 us on an otherwise idle chip, 76 on average in a pass of 4096 x 11008, under
// the bulk products.  Merging inverted ranges pairwise does the same work in six launches, each a row of load latencies: 65 us
// alone, six times 17 in that pass and the gaps between them.
// The rows of R and U come 16 bytes per lane, a block of 64 x 64 ahead of the MFMAs: lane l has row l % 16 and four
// consecutive k from 4 (l / 16), which are the k of four MFMAs (the contraction may run in any order as long as both operands agree).
constexpr int GI_XS = 20;        // doubles per LDS row of 16 columns: the four rows that a wavefront reads lie in different banks
constexpr size_t GI_LDS = sizeof(double) * GI_XS * (GRP * NB + NB);

struct GroupInvArgs {
  const double* R;               // at (g0, g0)
  int64_t ldr;
  double* U;
  int64_t ldu;
  int w;                         // columns of the group
};

__global__ __launch_bounds__(256) void group_inverse_cols(GroupInvArgs a) {
  extern __shared__ __align__(16) double gi_sm[];
  double* X = gi_sm;                                 // [64 nb][GI_XS] the strip's columns of U
  double* T = X + GRP * NB * GI_XS;                  // [64][GI_XS]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lk = lane >> 4;
  const int nb = (a.w + NB - 1) / NB, j = nb - 1 - (int)blockIdx.x / 4, c0 = j * NB + ((int)blockIdx.x & 3) * 16;
  if (c0 >= a.w) return;                             // (the last block may be narrower)
  const bool live = c0 + l16 < a.w;
  for (int e = tid; e < NB * 16; e += 256) {
    const int r = e >> 4, c = e & 15;
    X[(j * NB + r) * GI_XS + c] = j * NB + r < a.w && c0 + c < a.w ? a.U[(int64_t)(j * NB + r) * a.ldu + c0 + c] : 0.0;
  }
  // this wavefront's 16 rows of the 64 x 64 block at p (row 0 of the block), `lim` columns of it valid: behind them X is zero
  auto load = [&](const double* p, int64_t ld, int lim, double2 (&f)[8]) {
    p += (int64_t)(16 * wave + l16) * ld;
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = *reinterpret_cast<const double2*>(p + min(16 * (q >> 1) + 4 * lk + 2 * (q & 1), lim - 2));
  };
  auto multiply = [&](const double2 (&f)[8], const double* x, int from, double4v acc) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (q < 2 * from) continue;
      const double* xq = x + (16 * (q >> 1) + 4 * lk + 2 * (q & 1)) * GI_XS + l16;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[q].x, xq[0], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[q].y, xq[GI_XS], acc, 0, 0, 0);
    }
    return acc;
  };
  auto block_r = [&](int i, int k) { return a.R + (int64_t)i * NB * a.ldr + k * NB; };
  auto width = [&](int k) { return min(NB, a.w - k * NB); };
  double2 f[8], fn[8], fu[8];
  load(block_r(j - 1, j), a.ldr, width(j), f);
  __syncthreads();
  for (int i = j - 1; i >= 0; --i) {
    load(a.U + (int64_t)i * NB * (a.ldu + 1), a.ldu, NB, fu);
    double4v acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = j; k > i; --k) {                    // (the block column that the last step has finished comes last)
      if (k > i + 1)
        load(block_r(i, k - 1), a.ldr, NB, fn);
      else if (i > 0)
        load(block_r(i - 1, j), a.ldr, width(j), fn);
      acc = multiply(f, X + k * NB * GI_XS, 0, acc);
#pragma unroll
      for (int q = 0; q < 8; ++q) f[q] = fn[q];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) T[(16 * wave + 4 * v + lk) * GI_XS + l16] = acc[v];
    __syncthreads();
    acc = double4v{0.0, 0.0, 0.0, 0.0};
    acc = multiply(fu, T, wave, acc);                // (U[i, i] is upper triangular: its columns left of the wavefront's rows are zero)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = i * NB + 16 * wave + 4 * v + lk;
      X[r * GI_XS + l16] = -acc[v];
      if (live) a.U[(int64_t)r * a.ldu + c0 + l16] = -acc[v];
    }
    __syncthreads();
  }
}

// partial column sums of squares of the upper triangle of U: grid (ceil(m/64), parts); part p owns 256 rows.  A thread has 64 of
// them and sixteen loads in flight (one load after the other took 20 us at 1504 columns, where few workgroups share the chip).
__global__ __launch_bounds__(256) void colsumsq_upper(const double* __restrict__ U, int64_t ldu, int m,
                                                      double* __restrict__ partial) {
  __shared__ double red[4][64];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + tx;
  const int r0 = blockIdx.y * 256;
  double acc = 0.0;
  if (c < m) {
    const int r1 = min(min(m, r0 + 256), c + 1);
    constexpr int UR = 16;
    for (int r = r0 + ty; r < r1; r += 4 * UR) {
      double v[UR];
#pragma unroll
      for (int u = 0; u < UR; ++u) v[u] = U[(int64_t)min(r + 4 * u, r1 - 1) * ldu + c];
#pragma unroll
      for (int u = 0; u < UR; ++u)
        if (r + 4 * u < r1) acc += v[u] * v[u];
    }
  }
  red[ty][tx] = acc;
  __syncthreads();
  if (ty == 0 && c < m) partial[(int64_t)blockIdx.y * m + c] = ((red[0][tx] + red[1][tx]) + red[2][tx]) + red[3][tx];
}

__global__ __launch_bounds__(256) void colsum_finalize(const double* __restrict__ partial, int parts, int m,
                                                       double* __restrict__ out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= m) return;
  double s = 0.0;
  const int pmax = min(parts, c / 256 + 1);   // parts whose rows lie above the diagonal entry of column c
  for (int p = 0; p < pmax; ++p) s += partial[(int64_t)p * m + c];
  out[c] = s;
}

}  // namespace

static size_t inverse_base_bytes(int m) {
  const int parts = slim_cdiv(m, 256);
  return 2 * slim_ws_round(sizeof(double) * (size_t)m * m) + slim_ws_round(sizeof(double) * (size_t)parts * m) + 256;
}
// The panels of a group and its rows of U as residues, where the rank-512 products of any group are taken that way: from 2^21 results
// on, and not for a narrow last group, whose fp64 product gets cheaper with its rank.  A product by itself gains from twice that on;
// beside the chain of links it counts that the residue product leaves 64 CUs alone, and the panels are converted once for both
// kinds of products.  The whole inverse, us, with all products in fp64 / from 2^22 / from 2^21 / from 2^20 (terms) results on: 3072
// 1218 / 1217 / 1203 / 1210, 3584 1547 / 1548 / 1466 / 1479, 4096 1918 / 1898 / 1769 / 1779, 5120 3003 / 2673 / 2638 / 2635, 8192 8850 /
// 7073 / 7110 / 7105.
constexpr int64_t RESIDUE_RESULTS = (int64_t)1 << 21;
constexpr int RESIDUE_RANK = 384;
static bool far_pays(int gp, int K) { return K > RESIDUE_RANK && (int64_t)gp * gp / 2 >= RESIDUE_RESULTS; }
static bool terms_pay(int g0, int right, int K) { return K > RESIDUE_RANK && (int64_t)g0 * right >= RESIDUE_RESULTS; }
static size_t inverse_residue_bytes(int m) {
  const int g = GRP * NB;
  for (int g0 = g; g0 < m; g0 += g) {
    const int right = std::max(0, m - g0 - g), K = std::min(g, m - g0);
    if (far_pays(g0 - g, K) || terms_pay(g0, right, K)) return 3 * slim_rg_operand_bytes(m);
  }
  return 0;
}
size_t slim_ws_need_inverse(int m) { return inverse_base_bytes(m) + inverse_residue_bytes(m); }

extern "C" slim_status slim_hessian_inverse(slim_ctx* ctx, const float* G, int64_t ldg, int m, int64_t n_tokens,
                                            double percdamp, double* U, int64_t ldu, double* hinv_diag, int* info) {
  if (!ctx) return SLIM_ERR_INVALID_ARG;
  SLIM_REQUIRE(ctx, G && U && hinv_diag && info, "slim_hessian_inverse: null pointer");
  SLIM_REQUIRE(ctx, m > 0 && m % 2 == 0, "slim_hessian_inverse: m must be positive and even (got %d)", m);
  SLIM_REQUIRE(ctx, ldg >= m && ldu >= m && ldu % 2 == 0, "slim_hessian_inverse: bad leading dimension");
  SLIM_REQUIRE(ctx, n_tokens > 0, "slim_hessian_inverse: n_tokens must be positive");
  SLIM_REQUIRE(ctx, percdamp >= 0.0, "slim_hessian_inverse: percdamp must be >= 0");
  SLIM_REQUIRE(ctx, slim_aligned16(U), "slim_hessian_inverse: U must be 16-byte aligned");
  *info = 0;

  const int nblk = slim_cdiv(m, NB);
  const int64_t lda = m;
  const int parts = slim_cdiv(m, 256);
  // A: the matrix being factored (upper triangle), later the scratch of the triangular inverse.
  // R: the factor, panel by panel (only the blocks above the diagonal are ever written or read).
  const size_t bytes_A = slim_ws_round(sizeof(double) * (size_t)m * m);
  const size_t bytes_part = slim_ws_round(sizeof(double) * (size_t)parts * m);
  bool residues = false;
  slim_status st = slim_ws_reserve_either(ctx, slim_ws_need_inverse(m), inverse_base_bytes(m), residues);
  if (st != SLIM_OK) return st;
  double* A = static_cast<double*>(slim_ws_alloc(ctx, bytes_A));
  double* R = static_cast<double*>(slim_ws_alloc(ctx, bytes_A));
  double* partial = static_cast<double*>(slim_ws_alloc(ctx, bytes_part));
  double* lam = static_cast<double*>(slim_ws_alloc(ctx, 256));
  slim_rg_operand panels[2] = {}, urows = {};
  if (residues) {
    for (slim_rg_operand& o : panels) o = slim_rg_carve(ctx, m);
    urows = slim_rg_carve(ctx, m);
  }
  int* flag = ctx->dflags + 1;

  const double s = 2.0 / (double)n_tokens;
  SLIM_LAUNCH(ctx, "inv_lambda", damp_lambda, dim3(1), dim3(1024), 0, G, ldg, m, s, percdamp, lam, flag);
  // one pass writes A (widened, damped) and clears U; 4 / 2 / 1 columns per thread as alignment allows
  const bool g16 = (reinterpret_cast<uintptr_t>(G) & 15u) == 0, g8 = (reinterpret_cast<uintptr_t>(G) & 7u) == 0;
  if (m % 4 == 0 && ldg % 4 == 0 && ldu % 4 == 0 && g16)
    SLIM_LAUNCH(ctx, "inv_widen", widen_damp<4>, dim3(slim_cdiv(m, 1024), slim_cdiv(m, 8)), dim3(256), 0, G, ldg, m, s, lam, A, lda, U, ldu);
  else if (ldg % 2 == 0 && g8)
    SLIM_LAUNCH(ctx, "inv_widen", widen_damp<2>, dim3(slim_cdiv(m, 512), slim_cdiv(m, 8)), dim3(256), 0, G, ldg, m, s, lam, A, lda, U, ldu);
  else
    SLIM_LAUNCH(ctx, "inv_widen", widen_damp<1>, dim3(slim_cdiv(m, 256), slim_cdiv(m, 8)), dim3(256), 0, G, ldg, m, s, lam, A, lda, U, ldu);

  // ---- factorisation from the bottom-right corner upwards.  Blocks of 64 columns, groups of GRP blocks;
  //      "the window of block K" = the columns from the start of the group of block K-1 up to block K.
  //   s0 (caller's stream)  step of the last block, then for K = last .. 1
  //        link(K)   the diagonal block K-1 (it applies the update with panel K to itself), panel K and the window of K
  //        next(G)   when K is the second block of its group G (all other panels of G are done):
  //                  A[0:G, columns of group G-1] -= the panels of G except the first block's
  //   s1  far(G):    A[left of group G-1]^2 -= all panels of G, upper tiles only            (rank 512)
  // Every element of A thus receives each panel's contribution exactly once: from far() if it lies two or more
  // groups to the left, from next() if one group to the left (the first block's panel comes through that block's
  // window), from a window update inside the group, and from the diagonal kernel for the neighbouring diagonal block.
  st = slim_ensure_side(ctx);
  if (st != SLIM_OK) return st;
  {
    static bool done = false;
    if (!done) {
      SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(chol_step),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)CHOL_LDS));
      SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(chol_link),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)CHOL_LDS));
      SLIM_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(group_inverse_cols),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)GI_LDS));
      done = true;
    }
  }
  hipStream_t s0 = ctx->stream, s1 = ctx->side, s2 = ctx->side2;
  hipEvent_t* ev_group = &ctx->ev[0];  // ring of 2: the links of a group are done
  hipEvent_t* ev_far = &ctx->ev[9];    // ring of 2
  hipEvent_t* ev_terms = &ctx->ev[3];  // ring of 2: the terms that read a set of panels' residues are done
  hipEvent_t ev_panels = ctx->ev[5];
  struct StreamSwap {
    slim_ctx* c;
    hipStream_t keep;
    StreamSwap(slim_ctx* cc, hipStream_t s) : c(cc), keep(cc->stream) {
      c->stream = s;
      c->on_side = true;
    }
    ~StreamSwap() {
      c->stream = keep;
      c->on_side = false;
    }
  };
  struct AttachGuard {  // no event stays offered to a later call's launch when this one returns early
    slim_ctx* c;
    ~AttachGuard() { c->attach_event = nullptr; }
  } attach_guard{ctx};
  // ---- s2: the triangular inverse U = R^-1, group by group behind the factorisation.  With S the columns right of
  //      group g, U[g, S] = -U[g, g] T[g, S] where T[g, S] = R[g, S] U[S, S] = sum over the groups h in S of
  //      R[g, h] U[h, S]: the term of group h exists as soon as the rows U[h, :] do, for all rows above h at once
  //      (a rank-512 product with a large result, like the far updates of the factorisation), so that the whole
  //      inverse runs beside the factorisation, whose second half is a chain of small kernels on a nearly idle chip,
  //      and only the last group's share is left when the last diagonal block is done.  Per group, in this order:
  //        inside   U[g, g] column strip by column strip, in one launch (group_inverse_cols)
  //        rows     U[g, S] = -U[g, g] T[g, S]
  //        terms    T[0:g0, g0:m] (+)= R[0:g0, g] U[g, g0:m]   (first term of the columns of g itself, added to the
  //                 columns right of it)
  //      T lives in A right of the group, where the panels' inputs lay: the last reader of those columns of A is the
  //      diagonal kernel of the block left of the group (its pending rank-64 update), which the caller waits for.
  // `pr`: the panels of the group as residues (inv_panel_residues), or nullptr
  auto group_inverse = [&](int Gi, const slim_rg_operand* pr) -> slim_status {
    const int64_t g0 = (int64_t)Gi * GRP * NB, g1 = std::min<int64_t>(m, g0 + GRP * NB);
    const int gw = (int)(g1 - g0);
    slim_status rs;
    if (gw > NB) {
      const GroupInvArgs ga{R + g0 * lda + g0, lda, U + g0 * ldu + g0, ldu, gw};
      SLIM_LAUNCH(ctx, slim_prof_name("inv_trtri_dgemm", "group_inverse_cols"), group_inverse_cols, dim3(4 * (slim_cdiv(gw, NB) - 1)),
                  dim3(256), GI_LDS, ga);
    }
    slim_gemm_desc d;
    d.C2 = nullptr;
    d.ldc2 = 0;
    if (g1 < m) {
      d.A = U + g0 * ldu + g0;
      d.lda = ldu;
      d.B = A + g0 * lda + g1;
      d.ldb = lda;
      d.C = U + g0 * ldu + g1;
      d.ldc = ldu;
      d.M = gw;
      d.N = (int)(m - g1);
      d.K = gw;
      d.flags = SLIM_GEMM_A_UPPER;
      d.alpha = -1.0;
      d.beta = 0.0;
      rs = slim_dgemm(ctx, "inv_trtri_rows_dgemm", 0, d);
      if (rs != SLIM_OK) return rs;
    }
    if (g0 > 0) {
      // The columns of the group itself in fp64 always: column j has terms of the channels up to j alone, and residues, which keep
      // 2^-55.5 of the norm over all of the group's channels, would lose digits of a small one beside a large later channel.
      d.A = R + g0;
      d.lda = lda;
      d.B = U + g0 * ldu + g0;
      d.ldb = ldu;
      d.C = A + g0;
      d.ldc = lda;
      d.M = (int)g0;
      d.N = gw;
      d.K = gw;
      d.flags = SLIM_GEMM_B_UPPER;
      d.alpha = 1.0;
      d.beta = 0.0;
      rs = slim_dgemm(ctx, "inv_trtri_terms_dgemm", 0, d);
      if (rs != SLIM_OK) return rs;
    }
    if (g0 > 0 && g1 < m) {
      const int cols = (int)(m - g1);
      if (pr) {
        rs = slim_rg_residues(ctx, "inv_trtri_residues", urows, U + g0 * ldu + g1, ldu, cols, gw, true);
        if (rs != SLIM_OK) return rs;
        rs = slim_rgemm(ctx, "inv_trtri_terms_dgemm", {*pr, urows, (int)g0, cols, A + g1, lda, (int)g0, cols, 1.0, false, true});
      } else {
        d.B = U + g0 * ldu + g1;
        d.C = A + g1;
        d.N = cols;
        d.flags = 0;
        d.beta = 1.0;
        rs = slim_dgemm(ctx, "inv_trtri_terms_dgemm", 0, d);
      }
      if (rs != SLIM_OK) return rs;
    }
    return SLIM_OK;
  };
  auto block = [&](int J) {              // the diagonal block J
    CholArgs ca;
    const int64_t j0 = (int64_t)J * NB;
    ca.A = A + j0 * lda + j0;
    ca.lda = lda;
    ca.nbk = std::min<int>(NB, m - (int)j0);
    ca.nprev = (J < nblk - 1) ? std::min<int>(NB, m - (int)j0 - NB) : 0;
    ca.Vprev = U + (j0 + NB) * ldu + (j0 + NB);
    ca.Vout = U + j0 * ldu + j0;
    ca.ldv = ldu;
    ca.flag = flag;
    ca.col_base = (int)j0;
    return ca;
  };
  bool far_issued = false, tri_issued = false, terms_issued[2] = {false, false};
  int panel_slot = 0;
  int last_far_slot = 0, group_slot = 0;
  SLIM_LAUNCH(ctx, "inv_chol_diag", chol_step, dim3(1), dim3(512), CHOL_LDS, block(nblk - 1));
  for (int J = nblk - 1; J > 0; --J) {
    const int j0 = J * NB;
    const int G = J / GRP;                          // group of block J
    const int g0 = G * GRP * NB;                    // first column of the group
    const int g1 = std::min(m, g0 + GRP * NB);      // one past its last column
    const bool first = J == G * GRP;                // the group's panels are complete with this link
    // the window of the first block of a group lies in the group to the left, which far() of the group before this one
    // also writes
    if (first && far_issued) SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s0, ev_far[last_far_slot], 0));
    LinkArgs la;
    la.next = block(J - 1);
    la.A = A;
    la.R = R;
    la.lda = lda;
    la.V = U + (int64_t)j0 * ldu + j0;
    la.ldv = ldu;
    la.J = J;
    la.nbk = std::min(NB, m - j0);
    la.wt = ((J - 1) / GRP) * GRP;
    const int nc = J - la.wt;
    if (first) {
      group_slot ^= 1;
      ctx->attach_event = ev_group[group_slot];     // (rides on the kernel's own completion signal)
    }
    SLIM_LAUNCH(ctx, "inv_chol_diag@chol_link", chol_link, dim3(1 + la.wt * nc + nc * (nc + 1) / 2), dim3(512), CHOL_LDS, la);
    SLIM_HIP_TRY(ctx, slim_attach_flush(ctx));
    if (J == G * GRP + 1 && g0 > 0) {
      // every panel of the group except the first block's is complete: bring the group to the left up to date
      if (far_issued) SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s0, ev_far[last_far_slot], 0));
      const int gp = g0 - GRP * NB;               // first column of the group to the left
      slim_gemm_desc d;
      d.A = R + j0;                               // R[0:g0, j0:g1]
      d.lda = lda;
      d.B = R + (int64_t)gp * lda + j0;
      d.ldb = lda;
      d.C = A + gp;
      d.ldc = lda;
      d.C2 = nullptr;
      d.ldc2 = 0;
      d.M = g0;
      d.N = g0 - gp;
      d.K = g1 - j0;
      d.flags = 0;
      d.alpha = -1.0;
      d.beta = 1.0;
      st = slim_dgemm(ctx, "inv_group_next_dgemm", 1, d);
      if (st != SLIM_OK) return st;
    }
    if (!first) continue;
    // ---- s1: everything two or more groups to the left
    const int gp = g0 - GRP * NB;
    const bool far_r = residues && gp > 0 && far_pays(gp, g1 - g0), terms_r = residues && terms_pay(g0, m - g1, g1 - g0);
    if (far_r || terms_r) {
      // the group's panels as residues, for the far update (both operands) and for the terms of the inverse, which may still
      // be reading the other set
      StreamSwap swap(ctx, s1);
      SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s1, ev_group[group_slot], 0));
      panel_slot ^= 1;
      if (terms_issued[panel_slot]) SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s1, ev_terms[panel_slot], 0));
      ctx->attach_event = ev_panels;
      st = slim_rg_residues(ctx, "inv_panel_residues", panels[panel_slot], R + g0, lda, g0, g1 - g0, false);
      if (st != SLIM_OK) return st;
      SLIM_HIP_TRY(ctx, slim_attach_flush(ctx));
    }
    if (gp > 0) {
      StreamSwap swap(ctx, s1);
      SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s1, ev_group[group_slot], 0));
      slim_gemm_desc d;
      d.A = R + g0;                                 // R[0:gp, g0:g1]
      d.lda = lda;
      d.B = R + g0;
      d.ldb = lda;
      d.C = A;
      d.ldc = lda;
      d.C2 = nullptr;
      d.ldc2 = 0;
      d.M = gp;
      d.N = gp;
      d.K = g1 - g0;
      // While this update is short next to the links it runs beside, it runs as a persistent kernel that leaves some CUs
      // to them; a large one is throughput-bound and takes the whole chip.
      d.flags = SLIM_GEMM_UPPER_ONLY | (gp <= 4096 ? SLIM_GEMM_ONE_PER_CU : 0);
      d.alpha = -1.0;
      d.beta = 1.0;
      last_far_slot ^= 1;
      ctx->attach_event = ev_far[last_far_slot];
      if (far_r)
        st = slim_rgemm(ctx, "inv_syrk_dgemm", {panels[panel_slot], panels[panel_slot], g0, g0, A, lda, gp, gp, -1.0, true, true});
      else
        st = slim_dgemm(ctx, "inv_syrk_dgemm", 1, d);
      if (st != SLIM_OK) return st;
      SLIM_HIP_TRY(ctx, slim_attach_flush(ctx));
      far_issued = true;
    }
    // ---- s2: the triangular inverse of the group, whose last reader of A right of its first block was this link
    {
      StreamSwap swap(ctx, s2);
      SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s2, ev_group[group_slot], 0));
      if (terms_r) SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s2, ev_panels, 0));
      st = group_inverse(G, terms_r ? &panels[panel_slot] : nullptr);
      if (st != SLIM_OK) return st;
      if (terms_r) {
        SLIM_HIP_TRY(ctx, hipEventRecord(ev_terms[panel_slot], s2));
        terms_issued[panel_slot] = true;
      }
      tri_issued = true;
    }
  }
  // The pivots are all known once the last diagonal block is done: the flag travels to the host from here, and the
  // call returns when it has arrived, with the triangular inverse still in flight on the stream.
  int* host = reinterpret_cast<int*>(ctx->hpin);
  hipEvent_t ev_info = ctx->ev[11];
  SLIM_HIP_TRY(ctx, hipMemcpyAsync(host, flag, sizeof(int), hipMemcpyDeviceToHost, s0));
  SLIM_HIP_TRY(ctx, hipEventRecord(ev_info, s0));
  // every side stream has joined the caller's before the leftmost group's share of the triangular inverse (whose rows need
  // the other groups' terms), and so before the workspace is reused
  if (far_issued) SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s0, ev_far[last_far_slot], 0));
  if (tri_issued) {
    hipEvent_t ev_tri = ctx->ev[14];
    SLIM_HIP_TRY(ctx, hipEventRecord(ev_tri, s2));
    SLIM_HIP_TRY(ctx, hipStreamWaitEvent(s0, ev_tri, 0));
  }
  st = group_inverse(0, nullptr);
  if (st != SLIM_OK) return st;

  SLIM_LAUNCH(ctx, "inv_diag_colsumsq", colsumsq_upper, dim3(slim_cdiv(m, 64), parts), dim3(256), 0, U, ldu, m, partial);
  SLIM_LAUNCH(ctx, "inv_diag_finalize", colsum_finalize, dim3(slim_cdiv(m, 256)), dim3(256), 0, partial, parts, m, hinv_diag);

  SLIM_HIP_TRY(ctx, hipEventSynchronize(ev_info));
  *info = host[0];
  if (host[0] != 0)
    return slim_fail(ctx, SLIM_ERR_NOT_PD, "slim_hessian_inverse: H + lambda I is not positive definite (pivot at column %d)", host[0]);
  return SLIM_OK;
}
