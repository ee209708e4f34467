// Learnable router: projections, scores and row-wise top-k (Sec. 4, Eq. 16 of the paper; router step of
// Alg. 2), all in fp64 so that the selection agrees with an fp64 reference up to summation order.
//
//   row i keeps its k largest R[i][j] (router_scores.h); equal scores go to the lower j; indices come out ascending.
//
// One workgroup of 16 waves handles 16 query blocks of one head; each wave ends up with one complete score row in
// registers.  The selection is a most-significant-bit-first search for the k-th largest key on
// order-preserving integer images of the scores (32-bit first, 64-bit where those do not decide): counting is a compare plus a scalar popcount
// of the lane mask, there is no sorting and no atomics, and the result does not depend on timing.
//
// Measured on 12 heads of 256 x 512 blocks 28.7 -> 26 us, on 40 heads of 591 x 1182 361 -> 315 us, with the pooled keys
// read as operand fragments and the search on 32-bit images.  At 309 us about 90 of the latter went with the search (220 us
// with a list that is not searched for), 40 with each round of 256 key blocks, 50 with the projection of the rows and the
// start of a workgroup; 275 to 290 now, with 64-bit keys only where the 32-bit images do not decide.
#include "kv_state_f32.h"
#include "router_scores.h"

namespace sla2 {

// monotone map double -> uint64: a < b  <=>  key(a) < key(b); every real score maps above 0
__device__ __forceinline__ uint64_t order_key(double x) {
  uint64_t u = __builtin_bit_cast(uint64_t, x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ __forceinline__ int wave_count(bool pred) { return __builtin_popcountll(__ballot(pred)); }

// KV: the states of the key blocks too, one by each workgroup from topk_blocks + mean_blocks on (kv_state_f32.h)
template <int D, int SLOTS, bool KV>
__global__ __launch_bounds__(1024) void router_topk_kernel(const double* __restrict__ q_sum,
                                                           const double* __restrict__ k_frag,
                                                           const double* __restrict__ router_m,
                                                           int32_t* __restrict__ block_idx,
                                                           double* __restrict__ k_mean, int H, int N, int bq, int bk,
                                                           int Tm, int Tn, int k, int w_per_head, int topk_blocks,
                                                           int mean_blocks, int smooth, const KvStateArgs kv) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  if constexpr (KV) {
    if ((int)blockIdx.x >= topk_blocks + mean_blocks) {
      if (threadIdx.x >= 256) return;                    // (a barrier counts the waves that are left)
      kv_state_f32_job<D, true>(kv, k_frag, reinterpret_cast<float*>(lds), (int)blockIdx.x - topk_blocks - mean_blocks, threadIdx.x, H, N, Tn,
                                smooth);
      return;
    }
  }
  if ((int)blockIdx.x >= topk_blocks) {
    // Spare workgroups of this launch form colmean(K) (K-smoothing step of Alg. 2) from the block sums
    // for the kernels that follow; the router itself does not need it.  16 channels per workgroup,
    // 64 row groups, fixed summation order.  With smoothing disabled the mean is written as zero.
    double* red = lds;
    const int job = blockIdx.x - topk_blocks, bh = job / (D / 16), c = 16 * (job % (D / 16)) + threadIdx.x % 16;
    const int g = threadIdx.x / 16;
    double s = 0.0;
    if (smooth)
      for (int j = g; j < Tn; j += 64) s += k_frag[k_frag_offset(bh, j, c, Tn, D)];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x < 16) {
      double tot = 0.0;
      for (int gi = 0; gi < 64; gi++) tot += red[gi * 16 + threadIdx.x];
      k_mean[(size_t)bh * D + c] = tot / (double)N;
    }
    return;
  }
  const int row_tiles = (Tm + kRouterRows - 1) / kRouterRows;
  const int job = router_tile(blockIdx.x, topk_blocks), bh = job / row_tiles, row0 = job % row_tiles * kRouterRows;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const double* M = router_m + (w_per_head ? (size_t)(bh % H) * D * D : 0);

  double score[SLOTS];
  router_scores<D, SLOTS>(score, q_sum, k_frag, M, lds, bh, row0, N, bq, bk, Tm, Tn);
  const int rounds = (Tn + kColsPerRound - 1) / kColsPerRound;
  auto used = [&](int s) { return lane < Tn - ((s / 4) * kColsPerRound + (s % 4) * kWave); };   // slots past T_n hold -infinity

  const int row = row0 + wave;
  if (row >= Tm || k <= 0) return;
  const int slots = rounds * 4;
  int32_t* out = block_idx + ((size_t)bh * Tm + row) * k;

  const uint64_t lane_lt = (1ull << lane) - 1ull;
  int written = 0;
  // The selection as a search on a linear 32-bit image of the row, its largest score at the top and its smallest at the
  // bottom: about log2(T_n) bits decide it, where the bits of the scores themselves spend a dozen on the exponent
  // first.  The image keeps the order but may merge neighbours: it serves if some threshold on it selects exactly k;
  // if not (equal or nearly equal scores at the edge, or not finite ones), the search below decides.
  {
    float top = -INFINITY, bottom = -INFINITY;           // maximum of the scores, and of their negatives
    bool finite = true;
#pragma unroll
    for (int s = 0; s < SLOTS; s++) {
      const float x = (float)score[s];                   // (a finite score that is none in fp32 makes the span too large)
      finite = finite && (!used(s) || __builtin_isfinite(score[s]));
      top = fmaxf(top, x);
      bottom = fmaxf(bottom, used(s) ? -x : -INFINITY);
    }
    top = wave_max(top);
    bottom = -wave_max(bottom);
    const double base = bottom, span = (double)top - base;
    if (__all(finite) && span > 0.0 && span < 1e38) {
      const double scale = 4294967040.0 / span;
      uint32_t lin[SLOTS], thr = 0;
#pragma unroll
      for (int s = 0; s < SLOTS; s++)
        lin[s] = used(s) ? 1u + (uint32_t)fmin(fmax((score[s] - base) * scale, 0.0), 4294967040.0) : 0u;
      for (int bit = 31; bit >= 0; bit--) {
        const uint32_t cand = thr | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; s++) cnt += wave_count(lin[s] >= cand);
        if (cnt < k) continue;
        thr = cand;
        if (cnt > k) continue;
#pragma unroll
        for (int s = 0; s < SLOTS; s++)
          if (s < slots) {
            const bool keep = lin[s] >= thr;
            const uint64_t m = __ballot(keep);
            if (keep) out[written + __builtin_popcountll(m & lane_lt)] = s * kWave + lane;
            written += __builtin_popcountll(m);
          }
        return;
      }
    }
  }

  uint64_t key[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; s++) key[s] = used(s) ? order_key(score[s] + 0.0) : 0ull;   // 0: below every real score; -0 -> +0: zeros tie
  // k-th largest key thr, most significant bit first, on 32-bit halves (32-bit compares run at full
  // rate).  Invariant of either search: at least `need` candidates are >= the current threshold.
  // `exact` is set as soon as {key >= thr} has exactly k members - no ties to resolve then.
  uint32_t hi[SLOTS], lo[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; s++) { hi[s] = (uint32_t)(key[s] >> 32); lo[s] = (uint32_t)key[s]; }
  uint32_t thr_hi = 0;
  bool exact = false;
  for (int bit = 31; bit >= 0; bit--) {
    const uint32_t cand = thr_hi | (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int s = 0; s < SLOTS; s++) cnt += wave_count(hi[s] >= cand);      // unused slots hold 0 < cand
    if (cnt >= k) {
      thr_hi = cand;
      if (cnt == k) { exact = true; break; }
    }
  }
  uint32_t thr_lo = 0;
  if (!exact) {
    // thr_hi is the high word of the k-th largest key; the keys above it in the high word are in,
    // `need` more come from those that share it, ranked by their low words
    int gt = 0, eq = 0;
#pragma unroll
    for (int s = 0; s < SLOTS; s++) { gt += wave_count(hi[s] > thr_hi); eq += wave_count(hi[s] == thr_hi); }
    const int need = k - gt;
    if (eq == need) {
      exact = true;                                    // all of them: {key >= (thr_hi, 0)} is the answer
    } else {
      for (int bit = 31; bit >= 0; bit--) {
        const uint32_t cand = thr_lo | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; s++) cnt += wave_count(hi[s] == thr_hi && lo[s] >= cand);
        if (cnt >= need) {
          thr_lo = cand;
          if (cnt == need) { exact = true; break; }
        }
      }
    }
  }
  const uint64_t thr = ((uint64_t)thr_hi << 32) | thr_lo;
  // not exact: thr is the k-th largest key itself and several keys equal it; those above it
  // are all kept, the equal ones are kept in ascending column order until k are taken.
  int need_eq = 0;
  if (!exact) {
    int gt = 0;
#pragma unroll
    for (int s = 0; s < SLOTS; s++) gt += wave_count(key[s] > thr);
    need_eq = k - gt;
  }
#pragma unroll
  for (int s = 0; s < SLOTS; s++) {
    if (s < slots) {
      bool keep;
      if (exact) {
        keep = key[s] >= thr;
      } else {
        const bool eq = key[s] == thr;
        const uint64_t eq_mask = __ballot(eq);
        const int my_rank = __builtin_popcountll(eq_mask & lane_lt);
        keep = key[s] > thr || (eq && my_rank < need_eq);
        const int taken = __builtin_popcountll(eq_mask);
        need_eq -= taken < need_eq ? taken : need_eq;
      }
      const uint64_t m = __ballot(keep);
      if (keep) out[written + __builtin_popcountll(m & lane_lt)] = s * kWave + lane;
      written += __builtin_popcountll(m);
    }
  }
}

template <int D, int SLOTS, bool KV>
static hipError_t launch_topk(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m, int32_t* block_idx,
                              double* k_mean, const KvStateArgs& kv, hipStream_t stream) {
  constexpr size_t job = KV ? kKvStateFloats<D> * sizeof(float) : 0, lds = job > router_lds_bytes<D>() ? job : router_lds_bytes<D>();
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)router_topk_kernel<D, SLOTS, KV>, (int)lds); e != hipSuccess) return e;
  const int row_tiles = (s.Tm + kRouterRows - 1) / kRouterRows;
  const int topk_blocks = s.k > 0 ? s.BH * row_tiles : 0;        // k = 0: only the colmean workgroups run
  const int mean_blocks = s.BH * (D / 16), kv_blocks = KV ? s.BH * s.Tn : 0;
  router_topk_kernel<D, SLOTS, KV><<<dim3((unsigned)(topk_blocks + mean_blocks + kv_blocks)), 1024, lds, stream>>>(
      q_sum, k_frag, router_m, block_idx, k_mean, s.H, s.N, s.bq, s.bk, s.Tm, s.Tn, s.k, s.w_per_head ? 1 : 0, topk_blocks, mean_blocks,
      s.smooth ? 1 : 0, kv);
  return hipGetLastError();
}
template <bool KV>
static hipError_t launch_topk_class(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m, int32_t* block_idx,
                                    double* k_mean, const KvStateArgs& kv, hipStream_t stream) {
  // Three register classes by rounds of 256 key blocks: up to 2 (8 slots a lane), up to 5 (20), up to 8 (32; kMaxKeyBlocks).
  // Up to 8 slots the operands are read 8 at a time, else 4 (router_scores.h): the slots take the registers.  The middle
  // class ends at 5 rounds for the 1,025 to 1,280 key blocks that 20 slots serve better than 32: 12 heads, d = 128, 128-row
  // blocks: 1,182 key blocks 112 -> 86 us; 16 heads, d = 64, 64-row blocks: 200 -> 140 us.  The price is paid by 513 to 1,024
  // key blocks, which 16 slots with reads 8 at a time serve in 3 to 6 % less (d = 128: 640 key blocks 34.2 against 35.4 us,
  // 1,024 75.0 against 78.0; 40 heads 198 against 207) to 10 % less (d = 64: 57.4 against 63.7, 96.2 against 105.5).
  const int rounds = (s.Tn + kColsPerRound - 1) / kColsPerRound;
#define SLA2_TOPK(DD, SS) return launch_topk<DD, SS, KV>(s, q_sum, k_frag, router_m, block_idx, k_mean, kv, stream)
  if (s.d == 128) {
    if (rounds <= 2) SLA2_TOPK(128, 8);
    if (rounds <= 5) SLA2_TOPK(128, 20);
    SLA2_TOPK(128, 32);
  }
  if (rounds <= 2) SLA2_TOPK(64, 8);
  if (rounds <= 5) SLA2_TOPK(64, 20);
  SLA2_TOPK(64, 32);
#undef SLA2_TOPK
}
hipError_t launch_router_topk(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                              int32_t* block_idx, double* k_mean, hipStream_t stream) {
  return launch_topk_class<false>(s, q_sum, k_frag, router_m, block_idx, k_mean, KvStateArgs{}, stream);
}
bool router_has_room(const Shape& s) {
  return !s.bf16 && (size_t)s.BH * ((s.Tm + kRouterRows - 1) / kRouterRows + s.d / 16 + s.Tn) <= 256;
}
hipError_t launch_router_topk_f32(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                                  int32_t* block_idx, double* k_mean, const float* k, const float* v, float* k_stats, float* states,
                                  hipStream_t stream) {
  return launch_topk_class<true>(s, q_sum, k_frag, router_m, block_idx, k_mean, KvStateArgs{k, v, k_stats, states, s.sin, 0}, stream);
}

}  // namespace sla2
