// Backward pass of SLA2 (Alg. 3 of the paper's appendix, with the steps it leaves to automatic
// differentiation written out: phi = softmax over d, the smoothing of K, the mix of Eq. 13).
// High precision throughout, from the original Q, K, V (Sec. 5: the backward pass is never quantised).
//
// This file holds the launch sequence and the small kernels every tensor type shares (deterministic: no float atomics,
// fixed summation orders; only the order of work on key blocks of equally long lists is open); the two heavy steps are in sla2_bwd_mfma.hip (bf16 tensors) and sla2_bwd_f32.hip.
//
//   bwd_columns    for every key block j the ascending list of query blocks i with M_c[i, j] = 1
//   (bwd_q)        per query block: D^s, D^l, d alpha parts, dQ, dH_i, dZ_i
//   bwd_totals     dZ_total = sum_i dZ_i; bf16 tensors: per key block the sum of dH_i over the query blocks that did not select
//                  it, fp32: dH_total = sum_i dH_i; the order in which bwd_kv takes the key blocks
//   (bwd_kv)       per key block: dK', dV, column sums of dK'
//   bwd_finish     colmean(dK'); d alpha summed over its parts
//   bwd_unsmooth   dK = dK' - colmean(dK') (gradient of the smoothing)
//
// A launch costs 4.6 us however little it does, so what does not depend on each other shares one: this took eleven
// launches before, 45 us of the 210 us of the pass on 32 heads of 4,096 tokens (d = 64).
#include "masked_sums.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// For every key block j of head bh: the ascending list of query blocks i with M_c[i, j] = 1, as offsets
// col_ptr[bh][0..T_n] into col_idx[bh][.], and its length.  One workgroup per 64 columns of a head reads all index lists
// of the head: entries of its own columns become bits (column x, bit i), those of earlier columns are counted - the
// offset of its first list.  Then every thread writes out the bits of a few 32-row words at their places, and the complement
// of the words (bits from T_m on: 0) as rows of the bit matrix, if there is one.
__global__ __launch_bounds__(256) void bwd_columns_kernel(const int32_t* __restrict__ block_idx, int32_t* __restrict__ col_ptr,
                                                          int32_t* __restrict__ col_idx, int32_t* __restrict__ counts,
                                                          uint32_t* __restrict__ bits, int Tm, int Tn, int ksel) {
  extern __shared__ uint32_t words[];                 // [64][LW] bits, LW = W | 1 (odd: no bank conflicts down a column)
  const int W = (Tm + 31) / 32, LW = W | 1;           // W <= 64
  uint16_t* place = reinterpret_cast<uint16_t*>(words + 64 * LW);   // [64][LW] set bits of the column before the word
  __shared__ int before[4], first[64];
  const int j0 = blockIdx.x * 64, bh = blockIdx.y, tid = threadIdx.x, cols = min(64, Tn - j0);
  const int lane = tid % kWave, wave = tid / kWave;
  for (int x = tid; x < 64 * LW; x += 256) words[x] = 0u;
  __syncthreads();
  const int32_t* idx = block_idx + (size_t)bh * Tm * ksel;
  const unsigned entries = (unsigned)Tm * (unsigned)ksel;
  int earlier = 0;
#pragma unroll 8
  for (unsigned e = tid; e < entries; e += 256) {
    const int j = idx[e] - j0;
    earlier += j < 0;
    if (j >= 0 && j < 64) {
      const unsigned i = e / (unsigned)ksel;
      atomicOr(&words[j * LW + (i >> 5)], 1u << (i & 31));   // OR: the result does not depend on the order
    }
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) earlier += __shfl_xor(earlier, o);
  if (lane == 0) before[wave] = earlier;
  __syncthreads();
  if (wave == 0) {                                    // one lane per column: places of its words, list length and offset
    int n = 0;
    for (int x = 0; x < W; x++) {
      place[lane * LW + x] = (uint16_t)n;
      n += __popc(words[lane * LW + x]);
    }
    int at = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(at, o);
      if (lane >= o) at += y;
    }
    at += before[0] + before[1] + before[2] + before[3];
    first[lane] = at - n;
    if (lane < cols) {
      counts[(size_t)bh * Tn + j0 + lane] = n;
      col_ptr[(size_t)bh * (Tn + 1) + j0 + lane + 1] = at;
    }
    if (j0 == 0 && lane == 0) col_ptr[(size_t)bh * (Tn + 1)] = 0;
  }
  __syncthreads();
  int32_t* out = col_idx + (size_t)bh * Tm * ksel;
  for (int x = tid; x < 64 * W; x += 256) {
    const int c = x % 64, y = x / 64;
    uint32_t word = words[c * LW + y];
    int at = first[c] + place[c * LW + y];
    while (word) {
      out[at++] = 32 * y + __ffs(word) - 1;
      word &= word - 1u;
    }
  }
  if (bits != nullptr) {
    const int pitch = masked_pitch(Tn), rows = masked_words(Tm);
    for (int x = tid; x < 64 * rows; x += 256) {
      const int c = x % 64, y = x / 64, left = Tm - 32 * y;
      const uint32_t open = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
      bits[((size_t)bh * rows + y) * pitch + j0 + c] = y < W ? ~words[c * LW + y] & open : 0u;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The order in which bwd_kv takes the key blocks.  Its work on a key block is proportional to the length of the block's
// list, which varies a lot (mean 7.5, a tenth above 15, longest 91 on 12 heads of 512 key blocks): a long list that starts
// late runs on alone.  So the long ones go first, longest first over all heads.  The others follow head by head, in groups
// of heads whose gathered rows fit the caches, again longest first: neighbouring key blocks are selected by the same query
// blocks, whose rows they gather.  Every head is cut into 8 runs of consecutive key blocks, one per XCD (workgroup p runs
// on XCD p % 8).  With the groups alone the long lists of the last one kept a fifth of the CUs waiting (in a model of the
// 64 places of each XCD the last one ended at 1.54 times the mean, with the long lists first at 1.12): training step on
// such lists 1,747 -> 1,691 us, on 20 heads of 75,600 tokens 11.86 -> 11.60 ms.
// The order decides when a block is worked on, never what is summed.
//
// One call writes the places of one group: the long lists of all heads (h0 = 0, h1 = BH, LONG) or the others of heads
// [h0, h1).  Place 8 r + x is the r-th of XCD x; a counting sort on the length, cut off at 255.
constexpr int kNoLongList = 1 << 30;                  // every list is shorter
template <bool LONG>
__device__ void order_group(const int32_t* __restrict__ counts, int32_t* __restrict__ order, int BH, int h0, int h1, int Tn,
                            int long_list, int* hist /* LDS [8 x 256] */, int* at /* LDS [16] */) {
  const int tid = threadIdx.x, per_head = (Tn + kXcds - 1) / kXcds;
  auto each = [&](int first, int end, auto f) {       // f(key block bh T_n + j, its count), eight loads in flight
    for (int e0 = first + tid; e0 < end; e0 += 8 * 256) {
      int c[8];
#pragma unroll
      for (int y = 0; y < 8; y++) c[y] = e0 + 256 * y < end ? counts[e0 + 256 * y] : 0;
#pragma unroll
      for (int y = 0; y < 8; y++)
        if (e0 + 256 * y < end) f(e0 + 256 * y, c[y]);
    }
  };
  for (int x = tid; x < kXcds * 256; x += 256) hist[x] = 0;
  if (tid < 2 * kXcds) at[tid] = 0;                   // long lists per XCD: of all heads, of those before h0
  __syncthreads();
  if constexpr (LONG) {
    // places that a short last run of every head leaves empty: behind all others of their XCD
    for (int e = tid; e < BH * kXcds * per_head; e += 256) {
      const int x = e % kXcds, run = max(0, min(per_head, Tn - x * per_head));
      if (e / kXcds >= BH * run) order[e] = -1;
    }
  } else if (long_list != kNoLongList) {
    each(0, BH * Tn, [&](int e, int c) {
      if (c > long_list) {
        const int x = (e % Tn) / per_head;
        atomicAdd(&at[x], 1);
        if (e < h0 * Tn) atomicAdd(&at[kXcds + x], 1);
      }
    });
  }
  auto mine = [&](int c) { return (c > long_list) == LONG; };
  auto bin = [&](int e, int c) { return (e % Tn) / per_head * 256 + 255 - min(c, 255); };
  if (LONG && long_list == kNoLongList) return;
  each(h0 * Tn, h1 * Tn, [&](int e, int c) {
    if (mine(c)) atomicAdd(&hist[bin(e, c)], 1);
  });
  __syncthreads();
  for (int x = tid / kWave; x < kXcds; x += 4) {      // per XCD an exclusive scan of its 256 bins, 4 per lane
    const int lane = tid % kWave, run_len = max(0, min(per_head, Tn - x * per_head));
    int c[4], sum = 0;
#pragma unroll
    for (int y = 0; y < 4; y++) { c[y] = hist[256 * x + 4 * lane + y]; sum += c[y]; }
    int run = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(run, o);
      if (lane >= o) run += y;
    }
    run -= sum;
    if constexpr (!LONG) run += at[x] + h0 * run_len - at[kXcds + x];   // behind the long ones and the groups before
#pragma unroll
    for (int y = 0; y < 4; y++) { hist[256 * x + 4 * lane + y] = run; run += c[y]; }
  }
  __syncthreads();
  each(h0 * Tn, h1 * Tn, [&](int e, int c) {
    if (mine(c)) {
      const int b = bin(e, c);
      order[kXcds * atomicAdd(&hist[b], 1) + b / 256] = e / Tn * kMaxKeyBlocks + e % Tn;
    }
  });
}

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

// workgroups: one of order_group for the long lists and `groups` for the others, then per head one for dZ_total, then the
// sums of dH_i: fp32 tensors: per head the 256-entry slices of dH_total; bf16 tensors: the tiles of dH_j (masked_sums.h).
// The tiles of one set of columns, which read the same dH_i, run next to each other on one XCD.
struct TotalsArgs {
  const void* dh;
  const float* dz;
  const uint32_t* bits;
  void* dh_sum;                              // dH_total as fp32 or dH_j as bf16
  float* dz_total;
  const int32_t* counts;
  int32_t* order;
  int groups, heads_per_group, long_list, BH, Tm, Tn, d;
};
template <bool BF16>
__global__ __launch_bounds__(256, 2) void bwd_totals_kernel(const TotalsArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ int at[2 * kXcds];
  float (*part)[256] = reinterpret_cast<float (*)[256]>(smem);
  int id = blockIdx.x;
  if (id <= a.groups) {
    int* hist = reinterpret_cast<int*>(smem);
    const int h0 = (id - 1) * a.heads_per_group, h1 = min(a.BH, h0 + a.heads_per_group);
    if (id == 0) order_group<true>(a.counts, a.order, a.BH, 0, a.BH, a.Tn, a.long_list, hist, at);
    else order_group<false>(a.counts, a.order, a.BH, h0, h1, a.Tn, a.long_list, hist, at);
    return;
  }
  id -= a.groups + 1;
  if (id < a.BH) {
    sum_slots(a.dz + (size_t)id * a.Tm * a.d, a.dz_total + (size_t)id * a.d, a.Tm, a.d, 0, part);
    return;
  }
  id -= a.BH;
  const int len = a.d * a.d;
  if constexpr (BF16) {
    const int x = blockIdx.x % kXcds, tiles = (a.Tn + kMaskedRows - 1) / kMaskedRows, sets = len / kMaskedCols;
    const int y = id / kXcds, set = y / tiles * kXcds + x, bh = set / sets;
    masked_sums_tile((const uint16_t*)a.dh + (size_t)bh * a.Tm * len, a.bits + (size_t)bh * masked_words(a.Tm) * masked_pitch(a.Tn),
                     (uint16_t*)a.dh_sum + (size_t)bh * a.Tn * len, a.Tm, a.Tn, len, y % tiles * kMaskedRows,
                     set % sets * kMaskedCols, smem);
  } else {
    const int slices = len / 256, bh = id / slices;
    sum_slots((const float*)a.dh + (size_t)bh * a.Tm * len, (float*)a.dh_sum + (size_t)bh * len, a.Tm, len, 256 * (id % slices), part);
  }
}

// ---------------------------------------------------------------------------------------------
// workgroups: per head d / 32 for mean[bh][c] = sum_j colsum[bh][j][c] / N, 32 channels and 32 interleaved subsets of j
// each; then d alpha, per head [H] (one workgroup per head: sum over batch and query blocks) or per query block [H, T_m]
// (1,024 outputs per workgroup: sum over batch).  Sums are combined in a fixed order.
__global__ __launch_bounds__(1024) void bwd_finish_kernel(const float* __restrict__ colsum, float* __restrict__ mean,
                                                          const float* __restrict__ part, float* __restrict__ dalpha,
                                                          int mean_blocks, int B, int H, int N, int Tm, int Tn, int d,
                                                          int alpha_per_block) {
  __shared__ float red[1024];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < mean_blocks) {
    const int per_head = d / 32, bh = blockIdx.x / per_head, c = 32 * (blockIdx.x % per_head) + tid % 32, sub = tid / 32;
    float s = 0.f;
#pragma unroll 8
    for (int j = sub; j < Tn; j += 32) s += colsum[((size_t)bh * Tn + j) * d + c];
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
      for (int b = 0; b < B; b++) s += part[(size_t)b * H * Tm + o];
      dalpha[o] = s;
    }
    return;
  }
  float s = 0.f;
  for (int y = tid; y < B * Tm; y += 1024) s += part[((size_t)(y / Tm) * H + x) * Tm + y % Tm];
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
    *reinterpret_cast<bf16x8*>(p) = x;
  } else {
#pragma unroll
    for (int y = 0; y < 8; y++) p[y] -= m[y];
  }
}

// ---------------------------------------------------------------------------------------------
hipError_t launch_bwd_lists(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  // k = 0: every column is empty
  const size_t smem = (size_t)64 * (((s.Tm + 31) / 32) | 1) * (sizeof(uint32_t) + sizeof(uint16_t));   // at most 25 KB (T_m <= 2048)
  bwd_columns_kernel<<<dim3((unsigned)((s.Tn + 63) / 64), (unsigned)s.BH), 256, smem, stream>>>(a.block_idx, a.col_ptr, a.col_idx,
                                                                                               a.col_cnt, s.bf16 ? a.col_bits : nullptr, s.Tm, s.Tn,
                                                                                               s.k);
  return hipGetLastError();
}

hipError_t launch_bwd_q(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_q_bf16(s, a, stream) : launch_bwd_q_f32(s, a, stream);
}

hipError_t launch_bwd_totals(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  // Heads per order group.  What a head's key blocks gather: the Q and dO rows and the dH_i slots.  A group of more heads
  // ends in fewer stragglers, one of fewer keeps what is in flight closer to the caches; the sum of both is flat around
  // 48 MB a group (two heads of 32,760 tokens, d = 128: training step 1,801 us against 1,827 with one and 1,863 with four;
  // one head of 75,600: bwd_kv 11.9 ms against 12.8 with eight; 32 heads of 4,096, d = 64: 246 us against 263 with one).
  // fp32 products take long enough that only the stragglers count.
  const size_t head_bytes = ((size_t)2 * s.N * s.d + (size_t)s.Tm * s.d * s.d) * (s.bf16 ? 2 : 4);
  const size_t fit = ((size_t)(s.bf16 ? 48 : 192) << 20) / head_bytes;
  const int heads = fit < 1 ? 1 : fit > (size_t)s.BH ? s.BH : (int)fit;
  const int groups = (s.BH + heads - 1) / heads;
  // Length from which a list counts as long, see order_group: thrice the mean, and a sixth of what each of about 512
  // workgroups at a time has to do in all.  One group is sorted as a whole: none.
  const int64_t entries = (int64_t)s.Tm * s.k, share = entries * s.BH / (512 * 6);
  const int long_list = groups == 1 ? kNoLongList : (int)(3 * entries / s.Tn > share ? 3 * entries / s.Tn : share);
  const TotalsArgs t{a.dh, a.dz, a.col_bits, s.bf16 ? a.dh_sum : (void*)a.dh_total, a.dz_total, a.col_cnt, a.order,
                     groups, heads, long_list, s.BH, s.Tm, s.Tn, s.d};
  const int first = 1 + groups + s.BH, len = s.d * s.d;
  if (s.bf16) {
    static OncePerDevice once;
    if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_totals_kernel<true>, kMaskedLds); e != hipSuccess) return e;
    const int tiles = (s.Tn + kMaskedRows - 1) / kMaskedRows;           // sets of columns: a multiple of 8
    bwd_totals_kernel<true><<<dim3((unsigned)(first + s.BH * (len / kMaskedCols) * tiles)), 256, kMaskedLds, stream>>>(t);
  } else {
    bwd_totals_kernel<false><<<dim3((unsigned)(first + s.BH * (len / 256))), 256, 8 * 256 * sizeof(float), stream>>>(t);
  }
  return hipGetLastError();
}

hipError_t launch_bwd_kv(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.bf16 ? launch_bwd_kv_bf16(s, a, stream) : launch_bwd_kv_f32(s, a, stream);
}

hipError_t launch_bwd_finish(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  const int D = s.d, mean_blocks = s.smooth ? s.BH * (D / 32) : 0;
  const int alpha_blocks = s.alpha_per_block ? (s.H * s.Tm + 1023) / 1024 : s.H;
  bwd_finish_kernel<<<dim3((unsigned)(mean_blocks + alpha_blocks)), 1024, 0, stream>>>(
      a.colsum, a.dk_mean, a.dalpha_part, a.dalpha, mean_blocks, s.B, s.H, s.N, s.Tm, s.Tn, D, s.alpha_per_block ? 1 : 0);
  if (s.smooth) {
    const dim3 grid((unsigned)(((size_t)s.N * D / 8 + 255) / 256), (unsigned)s.BH);
    if (s.bf16) bwd_unsmooth_kernel<uint16_t><<<grid, 256, 0, stream>>>((uint16_t*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
    else bwd_unsmooth_kernel<float><<<grid, 256, 0, stream>>>((float*)a.dk, a.dk_mean, s.sin, s.H, s.N, D);
  }
  return hipGetLastError();
}

}  // namespace sla2
