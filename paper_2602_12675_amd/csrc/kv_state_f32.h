// States of the key blocks for fp32 tensors:
//   k' = k - colmean(K);  stats[token] = lnZ = log sum_c exp(k'_c);
//   K^phi = softmax_d(k');  h_j = (K^phi_j)^T V_j,  z_j = colsum(K^phi_j)
// (Alg. 2: K^phi, h, z).  Nothing here needs the selection, only the block sums of K, so that few of them run in the
// selection's launch (sla2_router.hip), on CUs that it leaves idle: 2 heads of 1,024 tokens (d = 64) 8.6 + 5.8 -> 8.7 us.
// Where there are more than CUs they have a launch of their own (sla2_f32.hip): in workgroups of 1,024 threads beside the
// selection, four blocks each, 768 of them (d = 128) took 47 us for 14 + 28.
#pragma once
#include "f32_tiles.h"

namespace sla2 {

// A block's state: h_j [d (c)][d (e)], then z_j [d].
__host__ __device__ constexpr int f32_state(int d) { return d * d + d; }

struct KvStateArgs {
  const float *k, *v;
  float *k_stats, *states;
  Strides sin;
  int first;                              // block whose state is the first of `states`
};
template <int D> constexpr int kKvStateFloats = kF32Tokens * kF32Ld<D> + D;   // LDS

// Key block block % Tn of head block / Tn, 256 threads.  OWN_MEAN: `sums` are the block sums as the router's fragments, and
// colmean(K) is formed of them here; otherwise it is `sums`.  Tokens past N contribute nothing.  A token's channels sit on
// neighbouring lanes, 4 each, so the softmax is taken in registers on the way into LDS; V goes from memory to its products.
// h_j is as large as the block's K and V together at d = 128: 12 heads of 4,096 tokens take 28 us for 100 MB (37 with V through
// LDS as well).
template <int D, bool OWN_MEAN>
__device__ __forceinline__ void kv_state_f32_job(const KvStateArgs& a, const double* __restrict__ sums, float* smem, int block, int tid, int H,
                                                 int N, int Tn, int smooth) {
  constexpr int LD = kF32Ld<D>;
  typedef ChunkMap<D, 256, kF32Tokens> CM;
  typedef StateSplit<D, 4> SS;
  float* kp = smem;                       // [64][LD]  K^phi tile
  float* mus = smem + kF32Tokens * LD;    // [D] colmean(K)
  const int bh = block / Tn, j = block % Tn;
  const int lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
  f32x4 kr[CM::kLoads];
  CM::load(kr, a.k + head_offset(a.sin, bh, H) + (size_t)t0 * a.sin.n, a.sin.n, valid, tid);
  typedef StateProduct<D> SP;
  SP sp;
  sp.begin(a.v + head_offset(a.sin, bh, H) + (size_t)t0 * a.sin.n, a.sin.n, valid, w, lane);
  if constexpr (!OWN_MEAN) {
    if (tid < D) mus[tid] = (float)sums[(size_t)bh * D + tid];
  } else {  // colmean(K) from the block sums, in their order as fragments (k_frag_offset): 16 lanes have 16 blocks of two channels
    typedef __attribute__((ext_vector_type(2))) double f64x2;
    constexpr int kPairs = D / 2 / 16;    // channel pairs per lane
    f64x2 sum[kPairs];
#pragma unroll
    for (int x = 0; x < kPairs; x++) sum[x] = f64x2{0.0, 0.0};
    const int b = lane % 16, pair = 4 * w + lane / 16;
    if (smooth)
      for (int first = 0; first < Tn; first += 16) {
        const int n = min(16, Tn - first);
        const double* src = sums + ((size_t)bh * Tn + first) * D + 2 * min(b, n - 1);
#pragma unroll
        for (int x = 0; x < kPairs; x++) {
          const f64x2 y = *reinterpret_cast<const f64x2*>(src + 2 * n * (pair + 16 * x));
          sum[x] += b < n ? y : f64x2{0.0, 0.0};
        }
      }
#pragma unroll
    for (int x = 0; x < kPairs; x++) {
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        sum[x][0] += __shfl_xor(sum[x][0], o);
        sum[x][1] += __shfl_xor(sum[x][1], o);
      }
      if (b < 2) mus[2 * (pair + 16 * x) + b] = (float)((b ? sum[x][1] : sum[x][0]) / (double)N);
    }
  }
  __syncthreads();
  const f32x4 mu = *reinterpret_cast<const f32x4*>(mus + 4 * ch);
  f32x4 zacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < CM::kLoads; i++) {
    const int t = trow + i * CM::kRows;
    const bool ok = t < valid;
    const f32x4 x = kr[i] - mu;
    const float m = CM::row_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
    f32x4 e;
#pragma unroll
    for (int c = 0; c < 4; c++) e[c] = exp2_f32((x[c] - m) * kLog2e);
    const float sum = CM::row_sum((e[0] + e[1]) + (e[2] + e[3]));
    const float inv = ok ? 1.f / sum : 0.f;
    e *= inv;
    zacc += e;
    *reinterpret_cast<f32x4*>(kp + t * LD + 4 * ch) = e;
    if (ok && ch == 0) a.k_stats[(size_t)bh * N + t0 + t] = m + __log2f(sum) * kLn2;
  }
  __syncthreads();
  f32x16 hacc[SS::kTiles];
#pragma unroll
  for (int x = 0; x < SS::kTiles; x++) hacc[x] = zero16();
  sp.add(hacc, kp, w, lane);
  float* ph = a.states + (size_t)(block - a.first) * f32_state(D);
  SP::store(hacc, 1.f, ph, w, lane);
  __syncthreads();                        // the tile fully consumed: its place takes the column sums
  *reinterpret_cast<f32x4*>(kp + trow * D + 4 * ch) = zacc;
  __syncthreads();
  if (tid < D) {
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < CM::kRows; r++) z += kp[r * D + tid];
    ph[D * D + tid] = z;
  }
}

}  // namespace sla2
