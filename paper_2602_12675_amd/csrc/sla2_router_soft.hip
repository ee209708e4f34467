// SoftTop-k router (Sec. 6 of the paper): the differentiable stand-in for the hard block selection that
// the first training stage uses,
//      M[i][j] = sigmoid(P_c[i][j] / tau + lambda_i),   P_c = row softmax of the router scores,
// with lambda_i such that row i sums to k.  fp64 throughout (the row sum decides lambda_i), fixed summation order.
//
// One workgroup of 16 waves handles 16 query blocks of one head: the scores come from the matrix cores as in the hard
// selection (router_scores.h), one wave then holds a complete row in registers and finds its lambda there, with no
// barrier and no LDS.  lambda is the root of a monotone function: Newton steps inside a bracket (a step that leaves the
// bracket is replaced by its midpoint), 5 to 7 evaluations of the row where a bisection to the last bit takes 55.  An
// evaluation costs a reciprocal per entry instead of an exponential and a division:
//      sigmoid(x + lambda) = 1 / (1 + exp(xmax - x) exp(-(lambda + xmax))),
// with exp(xmax - x) formed once per entry.  Measured on 12 heads of 256 x 512 blocks: 33 us, against 252 us
// for one workgroup per row that read all pooled keys itself and bisected through LDS reductions; what is left is the
// scoring (24 us, bound by the chain of fp64 products of a workgroup) and 9 us of exponentials and root search.
#include "router_scores.h"

namespace sla2 {

__device__ __forceinline__ double sigmoid_f64(double x) {
  const double e = exp(-fabs(x));
  return x >= 0.0 ? 1.0 / (1.0 + e) : e / (1.0 + e);
}

// all lanes get the same bits
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}
// 1 / x for x in [1, 1e300]: the hardware estimate and three Newton steps r <- r + r (1 - x r), each of which doubles
// the number of correct bits
__device__ __forceinline__ double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int i = 0; i < 3; i++) r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return r;
}

template <int D, int SLOTS>
__global__ __launch_bounds__(1024) void router_soft_kernel(const double* __restrict__ q_sum,
                                                           const double* __restrict__ k_frag,
                                                           const double* __restrict__ router_m,
                                                           float* __restrict__ mask, int H, int N, int bq, int bk,
                                                           int Tm, int Tn, int k, double tau, int w_per_head) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int row_tiles = (Tm + kRouterRows - 1) / kRouterRows;
  const int job = router_tile(blockIdx.x, gridDim.x), bh = job / row_tiles, row0 = job % row_tiles * kRouterRows;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int row = row0 + wave;
  float* out = mask + ((size_t)bh * Tm + row) * Tn;
  if (k <= 0 || k >= Tn) {                                // the limits lambda -> -inf / +inf
    if (row < Tm)
      for (int j = lane; j < Tn; j += kWave) out[j] = k <= 0 ? 0.f : 1.f;
    return;
  }
  double x[SLOTS];
  router_scores<D, SLOTS>(x, q_sum, k_frag, router_m + (w_per_head ? (size_t)(bh % H) * D * D : 0), lds, bh, row0, N, bq, bk,
                          Tm, Tn);
  if (row >= Tm) return;
  const int slots = (Tn + kColsPerRound - 1) / kColsPerRound * 4;
  auto column = [&](int s) { return (s / 4) * kColsPerRound + (s % 4) * kWave + lane; };

  // row softmax over tau; slots past T_n hold -infinity and come out as 0
  double mx = -INFINITY;
#pragma unroll
  for (int s = 0; s < SLOTS; s++) mx = fmax(mx, x[s]);
  mx = wave_max(mx);
  double se = 0.0;
#pragma unroll
  for (int s = 0; s < SLOTS; s++)
    if (s < slots) {
      x[s] = exp(x[s] - mx);
      se += x[s];
    }
  se = wave_sum(se);
  const double scale = 1.0 / (se * tau);
  double xmin = INFINITY;
#pragma unroll
  for (int s = 0; s < SLOTS; s++)
    if (s < slots) {
      x[s] *= scale;
      if (column(s) < Tn) xmin = fmin(xmin, x[s]);
    }
  const double xmax = scale;                              // the largest entry is exp(0) times the scale
  xmin = -wave_max(-xmin);

  // The root in y = lambda + xmax: sigmoid(x + lambda) = sigmoid(y - (xmax - x)).  With every x at xmax (xmin) the row
  // sums to k at y = logit (logit + xmax - xmin): the bracket.
  const double spread = xmax - xmin;
  const double logit = log((double)k / (double)(Tn - k));
  double lo = logit - 1e-9, hi = logit + spread + 1e-9;
  const bool fast = spread < 600.0;                       // the products of exponentials below stay finite
  if (fast) {
#pragma unroll
    for (int s = 0; s < SLOTS; s++)
      if (s < slots) x[s] = column(s) < Tn ? exp(xmax - x[s]) : INFINITY;
  } else {
#pragma unroll
    for (int s = 0; s < SLOTS; s++)
      if (s < slots) x[s] = column(s) < Tn ? xmax - x[s] : INFINITY;
  }
  // first guess: the row at its mean (the x sum to 1 / tau)
  double y = fmin(fmax(logit + (xmax - 1.0 / (tau * (double)Tn)), lo), hi);
  for (int it = 0; it < 200; it++) {
    double f = 0.0, df = 0.0;
    if (fast) {
      const double u = exp(-y);
#pragma unroll
      for (int s = 0; s < SLOTS; s++)
        if (s < slots) {
          const double p = column(s) < Tn ? reciprocal(__builtin_fma(x[s], u, 1.0)) : 0.0;
          f += p;
          df += p - p * p;
        }
    } else {
      for (int s = 0; s < slots; s++) {                   // a rare shape (tau below 1/600): plain, not unrolled
        double xs = INFINITY;
#pragma unroll
        for (int t = 0; t < SLOTS; t++) xs = t == s ? x[t] : xs;
        const double p = column(s) < Tn ? sigmoid_f64(y - xs) : 0.0;
        f += p;
        df += p - p * p;
      }
    }
    f = wave_sum(f) - (double)k;
    df = wave_sum(df);
    if (f < 0.0) lo = y;
    else hi = y;
    // A Newton step at rounding level ends the search (it is looked at before the bracket: there the sign of f is noise).
    // A row on which Newton does not settle, a function that is flat almost everywhere, falls back to halving the
    // bracket, which ends when the bracket stops shrinking.
    const double step = f / df;
    double next = y - step;
    if (fabs(step) <= 4e-15 * fmax(1.0, fabs(y))) break;
    if (!(next > lo && next < hi) || it >= 24) next = 0.5 * (lo + hi);
    y = next;
    if (next <= lo || next >= hi) break;
  }
  const double u = exp(-y);
#pragma unroll
  for (int s = 0; s < SLOTS; s++)
    if (s < slots && column(s) < Tn)
      out[column(s)] = (float)(fast ? reciprocal(__builtin_fma(x[s], u, 1.0)) : sigmoid_f64(y - x[s]));
}

hipError_t launch_router_soft(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                              float* mask, double tau, hipStream_t stream) {
  const dim3 grid((unsigned)(s.BH * ((s.Tm + kRouterRows - 1) / kRouterRows)));
  // The register classes of the hard selection (sla2_router.hip).  Measured on the same shapes, 20 slots against 32 at 1,182
  // key blocks: 117 against 131 us (d = 128), 216 against 245 (d = 64); against 16 with reads 8 at a time at 640 and 1,024:
  // 40.6 against 41.1 and 98.9 against 100.2 us (d = 128), 84.9 against 81.0 and 149.8 against 142.0 (d = 64).
  const int rounds = (s.Tn + kColsPerRound - 1) / kColsPerRound;
#define SLA2_SOFT(DD, SS)                                                                                            \
  {                                                                                                                  \
    static OncePerDevice once;                                                                                       \
    if (hipError_t e = allow_dynamic_lds(once, (const void*)router_soft_kernel<DD, SS>, (int)router_lds_bytes<DD>()); \
        e != hipSuccess)                                                                                             \
      return e;                                                                                                      \
    router_soft_kernel<DD, SS><<<grid, 1024, router_lds_bytes<DD>(), stream>>>(q_sum, k_frag, router_m, mask, s.H, s.N, \
                                                                               s.bq, s.bk, s.Tm, s.Tn, s.k, tau,      \
                                                                               s.w_per_head ? 1 : 0);                 \
  }
  if (s.d == 128) {
    if (rounds <= 2) SLA2_SOFT(128, 8) else if (rounds <= 5) SLA2_SOFT(128, 20) else SLA2_SOFT(128, 32)
  } else {
    if (rounds <= 2) SLA2_SOFT(64, 8) else if (rounds <= 5) SLA2_SOFT(64, 20) else SLA2_SOFT(64, 32)
  }
#undef SLA2_SOFT
  return hipGetLastError();
}

}  // namespace sla2
