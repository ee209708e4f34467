// Backward pass of SLA2 (Alg. 3 of the paper's appendix, with the steps it leaves to automatic
// differentiation written out: phi = softmax over d, the smoothing of K, the mix of Eq. 13).
// High precision throughout, from the original Q, K, V (Sec. 5: the backward pass is never quantised).
//
// This file holds the launch sequence and the small kernels every tensor type shares (deterministic: no float atomics,
// fixed summation orders); the two heavy steps are in sla2_bwd_mfma.hip (bf16 tensors) and sla2_bwd_f32.hip.
//
//   bwd_mask_bits, bwd_col_count / _scan / _fill
//                  M_c as bits, then for every key block j the ascending list of query blocks i with
//                  M_c[i, j] = 1
//   (bwd_q)        per query block: D^s, D^l, d alpha parts, dQ, dH_i, dZ_i
//   bwd_sum        dH_total = sum_i dH_i, dZ_total = sum_i dZ_i
//   (bwd_kv)       per key block: dK', dV, column sums of dK'
//   bwd_colmean, bwd_unsmooth, bwd_dalpha
//                  dK = dK' - colmean(dK') (gradient of the smoothing), d alpha summed over its parts
#include "common.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// M_c as bits: row (bh, i) -> ceil(T_n / 32) words, bit j % 32 of word j / 32 set iff block j is selected
__global__ __launch_bounds__(64) void bwd_mask_bits_kernel(const int32_t* __restrict__ block_idx,
                                                           uint32_t* __restrict__ bits, int Tn, int ksel) {
  __shared__ uint32_t words[kMaxKeyBlocks / 32];
  const int W = (Tn + 31) / 32, tid = threadIdx.x;
  for (int x = tid; x < W; x += 64) words[x] = 0u;
  __syncthreads();
  const int32_t* row = block_idx + (size_t)blockIdx.x * ksel;
  for (int s = tid; s < ksel; s += 64) {
    const int j = row[s];
    atomicOr(&words[j >> 5], 1u << (j & 31));         // OR: the result does not depend on the order
  }
  __syncthreads();
  for (int x = tid; x < W; x += 64) bits[(size_t)blockIdx.x * W + x] = words[x];
}

// For every key block j of head bh: the ascending list of query blocks i with M_c[i, j] = 1, as
// offsets col_ptr[bh][0..T_n] into col_idx[bh][.].  Three small kernels: column counts, their
// exclusive scan, and the fill.  Counts and fill run one wave per (head, 32-column word): the wave
// walks the bit rows 64 at a time, one ballot per column; the rank of a set bit inside the ballot
// plus the running count of the column is its place in the (ascending) list.
__global__ __launch_bounds__(64) void bwd_col_count_kernel(const uint32_t* __restrict__ bits, int32_t* __restrict__ counts,
                                                           int Tm, int Tn) {
  const int W = (Tn + 31) / 32, x = blockIdx.x, bh = blockIdx.y, lane = threadIdx.x;
  const uint32_t* rows = bits + (size_t)bh * Tm * W + x;
  int run[32];
#pragma unroll
  for (int b = 0; b < 32; b++) run[b] = 0;
  for (int i0 = 0; i0 < Tm; i0 += 64) {
    const int i = i0 + lane;
    const uint32_t word = i < Tm ? rows[(size_t)i * W] : 0u;
#pragma unroll
    for (int b = 0; b < 32; b++) run[b] += __popcll(__ballot((word >> b) & 1u));
  }
  int mine = 0;
#pragma unroll
  for (int b = 0; b < 32; b++) mine = lane == b ? run[b] : mine;
  const int j = 32 * x + lane;
  if (lane < 32 && j < Tn) counts[(size_t)bh * Tn + j] = mine;
}

__global__ __launch_bounds__(256) void bwd_col_scan_kernel(const int32_t* __restrict__ counts, int32_t* __restrict__ col_ptr,
                                                           int Tn) {
  constexpr int PER = kMaxKeyBlocks / 256;
  __shared__ int part[256];
  const int bh = blockIdx.x, tid = threadIdx.x;
  int v[PER], sum = 0;
#pragma unroll
  for (int y = 0; y < PER; y++) {
    const int j = tid * PER + y;
    v[y] = j < Tn ? counts[(size_t)bh * Tn + j] : 0;
    sum += v[y];
  }
  part[tid] = sum;
  __syncthreads();
  if (tid == 0) {                                     // exclusive scan of the 256 partial sums, in place
    int run = 0;
    for (int t = 0; t < 256; t++) {
      const int c = part[t];
      part[t] = run;
      run += c;
    }
  }
  __syncthreads();
  int run = part[tid];
#pragma unroll
  for (int y = 0; y < PER; y++) {
    const int j = tid * PER + y;
    if (j < Tn) col_ptr[(size_t)bh * (Tn + 1) + j] = run;
    run += v[y];
    if (j == Tn - 1) col_ptr[(size_t)bh * (Tn + 1) + Tn] = run;
  }
}

__global__ __launch_bounds__(64) void bwd_col_fill_kernel(const uint32_t* __restrict__ bits, const int32_t* __restrict__ col_ptr,
                                                          int32_t* __restrict__ col_idx, int Tm, int Tn, int ksel) {
  const int W = (Tn + 31) / 32, x = blockIdx.x, bh = blockIdx.y, lane = threadIdx.x;
  const uint32_t* rows = bits + (size_t)bh * Tm * W + x;
  int32_t* out = col_idx + (size_t)bh * Tm * ksel;
  int run[32];
#pragma unroll
  for (int b = 0; b < 32; b++) run[b] = 32 * x + b < Tn ? col_ptr[(size_t)bh * (Tn + 1) + 32 * x + b] : 0;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int i0 = 0; i0 < Tm; i0 += 64) {
    const int i = i0 + lane;
    const uint32_t word = i < Tm ? rows[(size_t)i * W] : 0u;
#pragma unroll
    for (int b = 0; b < 32; b++) {
      const unsigned long long m = __ballot((word >> b) & 1u);
      if ((word >> b) & 1u) out[run[b] + __popcll(m & below)] = i;
      run[b] += __popcll(m);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// dst[bh][e] = sum over b < count of src[bh][b][e].  A workgroup covers 256 consecutive e: 32 threads
// of 8 elements each, times 8 interleaved subsets of b that are combined in a fixed order.
template <typename S>
__global__ __launch_bounds__(256) void bwd_sum_kernel(const S* __restrict__ src, float* __restrict__ dst, int count,
                                                      int len) {
  __shared__ float part[8][256];
  const int bh = blockIdx.y, tid = threadIdx.x, col = tid % 32, sub = tid / 32;
  const int e0 = blockIdx.x * 256 + 8 * col;
  float acc[8];
#pragma unroll
  for (int x = 0; x < 8; x++) acc[x] = 0.f;
  if (e0 < len) {
    const S* p = src + (size_t)bh * count * len + e0;
#pragma unroll 4
    for (int b = sub; b < count; b += 8) {
      float v[8];
      if constexpr (sizeof(S) == 2) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(p + (size_t)b * len);
#pragma unroll
        for (int y = 0; y < 8; y++) v[y] = (float)x[y];
      } else {
        const f32x4 x0 = *reinterpret_cast<const f32x4*>(p + (size_t)b * len), x1 = *reinterpret_cast<const f32x4*>(p + (size_t)b * len + 4);
#pragma unroll
        for (int y = 0; y < 4; y++) { v[y] = x0[y]; v[4 + y] = x1[y]; }
      }
#pragma unroll
      for (int y = 0; y < 8; y++) acc[y] += v[y];
    }
  }
#pragma unroll
  for (int x = 0; x < 8; x++) part[sub][8 * col + x] = acc[x];
  __syncthreads();
  const int e = blockIdx.x * 256 + tid;
  if (e < len) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 8; g++) t += part[g][tid];
    dst[(size_t)bh * len + e] = t;
  }
}

// ---------------------------------------------------------------------------------------------
// mean[bh][c] = sum_j colsum[bh][j][c] / N: 1024 / d interleaved subsets of j, combined in a fixed order
__global__ __launch_bounds__(1024) void bwd_colmean_kernel(const float* __restrict__ colsum, float* __restrict__ mean,
                                                           int Tn, int N, int d) {
  __shared__ float part[1024];
  const int bh = blockIdx.x, tid = threadIdx.x, c = tid % d, sub = tid / d, subs = 1024 / d;
  float s = 0.f;
#pragma unroll 4
  for (int j = sub; j < Tn; j += subs) s += colsum[((size_t)bh * Tn + j) * d + c];
  part[tid] = s;
  __syncthreads();
  if (tid < d) {
    float t = 0.f;
    for (int g = 0; g < subs; g++) t += part[g * d + tid];
    mean[(size_t)bh * d + tid] = t / (float)N;
  }
}

// dK = dK' - colmean(dK'): the gradient of K' = K - colmean(K); 8 elements (of one row) per thread
template <typename T>
__global__ __launch_bounds__(256) void bwd_unsmooth_kernel(T* __restrict__ dk, const float* __restrict__ mean, Strides sin,
                                                           int H, int N, int d) {
  const int bh = blockIdx.y;
  const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (e >= (size_t)N * d) return;
  const int t = (int)(e / d), c = (int)(e % d);
  T* p = dk + head_offset(sin, bh, H) + (size_t)t * sin.n + c;
  const float* m = mean + (size_t)bh * d + c;
  if constexpr (sizeof(T) == 2) {
    bf16x8 x = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int y = 0; y < 8; y++) x[y] = (__bf16)((float)x[y] - m[y]);
    *reinterpret_cast<bf16x8*>(p) = x;
  } else {
#pragma unroll
    for (int y = 0; y < 8; y++) p[y] -= m[y];
  }
}

// d alpha: per head [H] (sum over batch and query blocks) or per query block [H, T_m] (over batch).  One workgroup per output; thread t adds the parts t, t + 256, .. and thread 0 the 256 sums.
__global__ __launch_bounds__(256) void bwd_dalpha_kernel(const float* __restrict__ part, float* __restrict__ dalpha, int B,
                                                         int H, int Tm, int alpha_per_block) {
  __shared__ float red[256];
  const int x = blockIdx.x, tid = threadIdx.x;
  const int h = alpha_per_block ? x / Tm : x;
  const int per_b = alpha_per_block ? 1 : Tm;                      // consecutive parts of one batch entry
  float s = 0.f;
  for (int y = tid; y < B * per_b; y += 256) {
    const int b = y / per_b, z = y % per_b;
    const size_t first = (size_t)(b * H + h) * Tm + (alpha_per_block ? x % Tm : 0);
    s += part[first + z];
  }
  red[tid] = s;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
    for (int y = 0; y < 256; y++) t += red[y];
    dalpha[x] = t;
  }
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_bwd_lists(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  // k = 0: every list is empty (the bit rows are all zero)
  bwd_mask_bits_kernel<<<dim3((unsigned)(s.BH * s.Tm)), 64, 0, stream>>>(a.block_idx, a.mask_bits, s.Tn, s.k);
  const dim3 words((unsigned)((s.Tn + 31) / 32), (unsigned)s.BH);
  bwd_col_count_kernel<<<words, 64, 0, stream>>>(a.mask_bits, a.col_cnt, s.Tm, s.Tn);
  bwd_col_scan_kernel<<<dim3((unsigned)s.BH), 256, 0, stream>>>(a.col_cnt, a.col_ptr, s.Tn);
  bwd_col_fill_kernel<<<words, 64, 0, stream>>>(a.mask_bits, a.col_ptr, a.col_idx, s.Tm, s.Tn, s.k);
  return hipGetLastError();
}

hipError_t launch_bwd_q(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_q_bf16(s, a, stream) : launch_bwd_q_f32(s, a, stream);
}

hipError_t launch_bwd_totals(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  const int D = s.d, count = s.Tm;
  const dim3 grid_h((unsigned)((D * D + 255) / 256), (unsigned)s.BH), grid_z((unsigned)((D + 255) / 256), (unsigned)s.BH);
  if (s.bf16) bwd_sum_kernel<uint16_t><<<grid_h, 256, 0, stream>>>((const uint16_t*)a.dh, a.dh_total, count, D * D);
  else bwd_sum_kernel<float><<<grid_h, 256, 0, stream>>>((const float*)a.dh, a.dh_total, count, D * D);
  bwd_sum_kernel<float><<<grid_z, 256, 0, stream>>>(a.dz, a.dz_total, count, D);
  return hipGetLastError();
}

hipError_t launch_bwd_kv(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_kv_bf16(s, a, stream) : launch_bwd_kv_f32(s, a, stream);
}

hipError_t launch_bwd_finish(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  const int D = s.d;
  if (s.smooth) {
    bwd_colmean_kernel<<<dim3((unsigned)s.BH), 1024, 0, stream>>>(a.colsum, a.dk_mean, s.Tn, s.N, D);
    const dim3 grid((unsigned)(((size_t)s.N * D / 8 + 255) / 256), (unsigned)s.BH);
    if (s.bf16) bwd_unsmooth_kernel<uint16_t><<<grid, 256, 0, stream>>>((uint16_t*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
    else bwd_unsmooth_kernel<float><<<grid, 256, 0, stream>>>((float*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
  }
  const int n_alpha = s.alpha_per_block ? s.H * s.Tm : s.H;
  bwd_dalpha_kernel<<<dim3((unsigned)n_alpha), 256, 0, stream>>>(a.dalpha_part, a.dalpha, s.B, s.H, s.Tm,
                                                                 s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

}  // namespace sla2
