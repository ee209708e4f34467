// The order in which the key side of the backward pass takes the key blocks, formed by spare workgroups of the launch
// before it.
#pragma once
#include "common.h"

namespace sla2 {

// The order in which bwd_kv takes the key blocks.  Its work on a key block is proportional to the length of the block's
// list, which varies a lot (mean 7.5, a tenth above 15, longest 91 on 12 heads of 512 key blocks): a long list that starts
// late runs on alone.  So the long ones go first, longest first over all heads.  The others follow head by head, in groups
// of heads whose gathered rows fit the caches, again longest first: neighbouring key blocks are selected by the same query
// blocks, whose rows they gather.  Every head is cut into 8 runs of consecutive key blocks, one per XCD (workgroup p runs
// on XCD p % 8), run y of head h on XCD (y + h) % 8: how often a key block is selected goes with its place in the sequence, and
// with the same run of every head on one XCD the fullest had 5 % more to do than the mean.  The last group takes at least four
// rounds of the 64 places of an XCD: what it ends in is the length of its shortest lists.  12 heads of 512 key blocks, the
// workgroups' times replayed: the last one ends at 1.035 instead of 1.10 times the mean; training step 1,474.6 -> 1,465.6 us, on 24
// heads of 4,096 tokens 279.8 -> 276.0, on 20 of 75,600 10.41 -> 10.24 ms.  (Where one group takes all heads, as on 32 heads of 64 key
// blocks, runs that stay on their XCD serve better: 199.4 against 200.7 us.)  With the groups alone the long lists of the last one
// kept a fifth of the CUs waiting (in a model of the 64 places of each XCD the last one ended at 1.54 times the mean, with the long
// lists first at 1.12): training step on such lists 1,747 -> 1,691 us, on 20 heads of 75,600 tokens 11.86 -> 11.60 ms.
// The order decides when a block is worked on, never what is summed.
//
// One call writes the places of one group: the long lists of all heads (h0 = 0, h1 = BH, LONG) or the others of heads
// [h0, h1).  Place 8 r + x is the r-th of XCD x; a counting sort on the length, cut off at 255.
constexpr int kNoLongList = 1 << 30;                  // every list is shorter
__device__ __forceinline__ int order_xcd(int head, int j, int per_head, bool turn) { return turn ? (j / per_head + head) % kXcds : j / per_head; }
// key blocks of heads [0, heads) on XCD x
__device__ __forceinline__ int order_before(int x, int heads, int per_head, int Tn, bool turn) {
  if (!turn) return heads * max(0, min(per_head, Tn - x * per_head));
  int n = heads / kXcds * Tn;
  for (int h = heads / kXcds * kXcds; h < heads; h++) n += max(0, min(per_head, Tn - (x + kXcds - h % kXcds) % kXcds * per_head));
  return n;
}
template <bool LONG>
__device__ void order_group(const int32_t* __restrict__ counts, int32_t* __restrict__ order, int BH, int h0, int h1, int Tn,
                            int long_list, bool turn, int* hist /* LDS [8 x 256] */, int* at /* LDS [16] */) {
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
      if (e / kXcds >= order_before(e % kXcds, BH, per_head, Tn, turn)) order[e] = -1;
    }
  } else if (long_list != kNoLongList) {
    each(0, BH * Tn, [&](int e, int c) {
      if (c > long_list) {
        const int x = order_xcd(e / Tn, e % Tn, per_head, turn);
        atomicAdd(&at[x], 1);
        if (e < h0 * Tn) atomicAdd(&at[kXcds + x], 1);
      }
    });
  }
  auto mine = [&](int c) { return (c > long_list) == LONG; };
  auto bin = [&](int e, int c) { return order_xcd(e / Tn, e % Tn, per_head, turn) * 256 + 255 - min(c, 255); };
  if (LONG && long_list == kNoLongList) return;
  each(h0 * Tn, h1 * Tn, [&](int e, int c) {
    if (mine(c)) atomicAdd(&hist[bin(e, c)], 1);
  });
  __syncthreads();
  for (int x = tid / kWave; x < kXcds; x += 4) {      // per XCD an exclusive scan of its 256 bins, 4 per lane
    const int lane = tid % kWave;
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
    if constexpr (!LONG) run += at[x] + order_before(x, h0, per_head, Tn, turn) - at[kXcds + x];   // behind the long ones and the groups before
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

// The groups of a call, and group `id` (0: the long lists, 1 .. groups: the others) by a workgroup of 256 threads
struct WorkOrder {
  const int32_t* counts;
  int32_t* order;
  int groups, heads_per_group, long_list, BH, Tn;
};
__device__ inline void order_job(const WorkOrder& o, int id, int* hist /* LDS [8 x 256] */, int* at /* LDS [16] */) {
  const int h0 = (id - 1) * o.heads_per_group, h1 = id == o.groups ? o.BH : h0 + o.heads_per_group;
  if (id == 0) order_group<true>(o.counts, o.order, o.BH, 0, o.BH, o.Tn, o.long_list, o.groups > 1, hist, at);
  else order_group<false>(o.counts, o.order, o.BH, h0, h1, o.Tn, o.long_list, o.groups > 1, hist, at);
}
inline WorkOrder make_order(const Shape& s, const BwdArgs& a) {
  // Heads per order group.  What a head's key blocks gather: the Q and dO rows and the dH_i slots.  A group of more heads
  // ends in fewer stragglers, one of fewer keeps what is in flight closer to the caches; the sum of both is flat around
  // 48 MB a group (two heads of 32,760 tokens, d = 128: training step 1,801 us against 1,827 with one and 1,863 with four;
  // one head of 75,600: bwd_kv 11.9 ms against 12.8 with eight; 32 heads of 4,096, d = 64: 246 us against 263 with one).
  // fp32 products take long enough that only the stragglers count.
  const size_t head_bytes = ((size_t)2 * s.N * s.d + (size_t)s.Tm * s.d * s.d) * (s.bf16 ? 2 : 4);
  const size_t fit = ((size_t)(s.bf16 ? 48 : 192) << 20) / head_bytes;
  const int heads = fit < 1 ? 1 : fit > (size_t)s.BH ? s.BH : (int)fit;
  const int per_head = (s.Tn + kXcds - 1) / kXcds, tail = (4 * 64 + per_head - 1) / per_head;   // heads of the last group, at least
  const int groups = (s.BH > tail ? (s.BH - tail) / heads : 0) + 1;
  // Length from which a list counts as long, see order_group: thrice the mean, and a sixth of what each of about 512
  // workgroups at a time has to do in all.  One group is sorted as a whole: none.
  const int64_t entries = (int64_t)s.Tm * s.k, share = entries * s.BH / (512 * 6);
  const int long_list = groups == 1 ? kNoLongList : (int)(3 * entries / s.Tn > share ? 3 * entries / s.Tn : share);
  return WorkOrder{a.col_cnt, a.order, groups, heads, long_list, s.BH, s.Tn};
}

}  // namespace sla2
