// Backward pass of SLA2 (Alg. 3 of the paper's appendix, with the steps it leaves to automatic
// differentiation written out: phi = softmax over d, the smoothing of K, the mix of Eq. 13).
// High precision throughout, from the original Q, K, V (Sec. 5: the backward pass is never quantised).
//
// This file holds the launch sequence and the small kernels every tensor type shares (deterministic: no float atomics,
// fixed summation orders; only the order of work on key blocks of equally long lists is open); the two heavy steps are in sla2_bwd_mfma.hip (bf16 tensors) and sla2_bwd_f32.hip.
//
//   (bwd_q)        per query block: D^s, D^l, d alpha parts, dQ, dH_i, dZ_i; its first workgroups make, for every key block j,
//                  the ascending list of query blocks i with M_c[i, j] = 1 (bwd_columns.h)
//   bwd_totals     per key block the sum of dH_i over the query blocks that did not select it, dZ_total = sum_i dZ_i; the order
//                  in which bwd_kv takes the key blocks (fp32 tensors: kernels of their own in sla2_bwd_f32.hip)
//   (bwd_kv)       per key block: dK', dV, column sums of dK'
//   bwd_finish     colmean(dK'); d alpha summed over its parts
//   bwd_unsmooth   dK = dK' - colmean(dK') (gradient of the smoothing)
//
// A launch costs 4.6 us however little it does, so what does not depend on each other shares one: this took eleven
// launches before, 45 us of the 210 us of the pass on 32 heads of 4,096 tokens (d = 64).
#include "masked_sums.h"
#include "work_order.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// dst[e] = sum over b < count of src[b][e] for the 256 entries from e0 on.  32 threads of 8 elements each, times 8
// interleaved subsets of b that are combined in a fixed order.
__device__ void sum_slots(const float* __restrict__ src, float* __restrict__ dst, int count, int len, int first, float (*part)[256]) {
  const int tid = threadIdx.x, col = tid % 32, sub = tid / 32;
  const int e0 = first + 8 * col;
  float acc[8];
#pragma unroll
  for (int x = 0; x < 8; x++) acc[x] = 0.f;
  if (e0 < len) {
    const float* p = src + e0;
#pragma unroll 8
    for (int b = sub; b < count; b += 8) {
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(p + (size_t)b * len), x1 = *reinterpret_cast<const f32x4*>(p + (size_t)b * len + 4);
#pragma unroll
      for (int y = 0; y < 4; y++) { acc[y] += x0[y]; acc[4 + y] += x1[y]; }
    }
  }
#pragma unroll
  for (int x = 0; x < 8; x++) part[sub][8 * col + x] = acc[x];
  __syncthreads();
  if (first + tid < len) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 8; g++) t += part[g][tid];
    dst[first + tid] = t;
  }
}

// workgroups: the jobs of the work order, per head one for dZ_total, then the tiles of dH_j, the sums of dH_i
// (masked_sums.h).  The tiles of one set of columns, which read the same dH_i, run next to each other on one XCD.
struct TotalsArgs {
  WorkOrder order;
  const uint16_t* dh;
  const float* dz;
  const uint32_t* bits;
  uint16_t* dh_sum;
  float* dz_total;
  int Tm, d;
};
__global__ __launch_bounds__(256, 2) void bwd_totals_kernel(const TotalsArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ int at[2 * kXcds];
  const int BH = a.order.BH, Tn = a.order.Tn;
  int id = blockIdx.x;
  if (id <= a.order.groups) return order_job(a.order, id, reinterpret_cast<int*>(smem), at);
  id -= a.order.groups + 1;
  if (id < BH)
    return sum_slots(a.dz + (size_t)id * a.Tm * a.d, a.dz_total + (size_t)id * a.d, a.Tm, a.d, 0, reinterpret_cast<float (*)[256]>(smem));
  id -= BH;
  const int len = a.d * a.d;
  const int x = blockIdx.x % kXcds, tiles = (Tn + kMaskedRows - 1) / kMaskedRows, sets = len / kMaskedCols;
  const int y = id / kXcds, set = y / tiles * kXcds + x, bh = set / sets;
  masked_sums_tile(a.dh + (size_t)bh * a.Tm * len, a.bits + (size_t)bh * masked_words(a.Tm) * masked_pitch(Tn),
                   a.dh_sum + (size_t)bh * Tn * len, a.Tm, Tn, len, y % tiles * kMaskedRows, set % sets * kMaskedCols, smem);
}

// ---------------------------------------------------------------------------------------------
// workgroups: per head d / 32 for mean[bh][c] = sum_j colsum[bh][j][c] / N, 32 channels and 32 interleaved subsets of j
// each; then d alpha, per head [H] (one workgroup per head: sum over batch and query blocks) or per query block [H, T_m]
// (1,024 outputs per workgroup: sum over batch).  `cols` column sums a head, `parts` of d alpha a query block.  Sums are
// combined in a fixed order.
__global__ __launch_bounds__(1024) void bwd_finish_kernel(const float* __restrict__ colsum, float* __restrict__ mean,
                                                          const float* __restrict__ part, float* __restrict__ dalpha,
                                                          int mean_blocks, int B, int H, int N, int Tm, int parts,
                                                          int cols, int d, int alpha_per_block) {
  __shared__ float red[1024];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < mean_blocks) {
    const int per_head = d / 32, bh = blockIdx.x / per_head, c = 32 * (blockIdx.x % per_head) + tid % 32, sub = tid / 32;
    float s = 0.f;
#pragma unroll 8
    for (int j = sub; j < cols; j += 32) s += colsum[((size_t)bh * cols + j) * d + c];
    red[tid] = s;
    __syncthreads();
    if (tid < 32) {
      float t = 0.f;
#pragma unroll
      for (int g = 0; g < 32; g++) t += red[g * 32 + tid];
      mean[(size_t)bh * d + c] = t / (float)N;
    }
    return;
  }
  const int x = blockIdx.x - mean_blocks;
  if (alpha_per_block) {
    const int o = x * 1024 + tid;                     // output h T_m + i
    if (o < H * Tm) {
      float s = 0.f;
      for (int b = 0; b < B; b++)
        for (int y = 0; y < parts; y++) s += part[((size_t)b * H * Tm + o) * parts + y];
      dalpha[o] = s;
    }
    return;
  }
  float s = 0.f;
  for (int y = tid, per_head = Tm * parts; y < B * per_head; y += 1024) s += part[((size_t)(y / per_head) * H + x) * per_head + y % per_head];
  red[tid] = s;
  __syncthreads();
#pragma unroll
  for (int o = 512; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) dalpha[x] = red[0];
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
    store_streamed(reinterpret_cast<bf16x8*>(p), x);
  } else {
#pragma unroll
    for (int y = 0; y < 8; y++) p[y] -= m[y];
  }
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_bwd_q(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_q_bf16(s, a, stream) : launch_bwd_q_f32(s, a, stream);
}

hipError_t launch_bwd_totals(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (!s.bf16) return launch_bwd_totals_f32(s, a, stream);
  const TotalsArgs t{make_order(s, a), (const uint16_t*)a.dh, a.dz, a.col_bits, (uint16_t*)a.dh_sum, a.dz_total, s.Tm, s.d};
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_totals_kernel, kMaskedLds); e != hipSuccess) return e;
  const int tiles = (s.Tn + kMaskedRows - 1) / kMaskedRows;           // sets of columns: a multiple of 8
  bwd_totals_kernel<<<dim3((unsigned)(1 + t.order.groups + s.BH + s.BH * (s.d * s.d / kMaskedCols) * tiles)), 256, kMaskedLds, stream>>>(t);
  return hipGetLastError();
}

hipError_t launch_bwd_kv(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_kv_bf16(s, a, stream) : launch_bwd_kv_f32(s, a, stream);
}

hipError_t launch_bwd_finish(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  const int D = s.d, mean_blocks = s.smooth ? s.BH * (D / 32) : 0;
  const int alpha_blocks = s.alpha_per_block ? (s.H * s.Tm + 1023) / 1024 : s.H;
  bwd_finish_kernel<<<dim3((unsigned)(mean_blocks + alpha_blocks)), 1024, 0, stream>>>(
      a.colsum, a.dk_mean, a.dalpha_part, a.dalpha, mean_blocks, s.B, s.H, s.N, s.Tm, bwd_alpha_parts(s), bwd_colsums(s), D,
      s.alpha_per_block ? 1 : 0);
  if (s.smooth) {
    const dim3 grid((unsigned)(((size_t)s.N * D / 8 + 255) / 256), (unsigned)s.BH);
    if (s.bf16) bwd_unsmooth_kernel<uint16_t><<<grid, 256, 0, stream>>>((uint16_t*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
    else bwd_unsmooth_kernel<float><<<grid, 256, 0, stream>>>((float*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
  }
  return hipGetLastError();
}

}  // namespace sla2
