// For every key block j of a head: the ascending list of query blocks i with M_c[i, j] = 1, as offsets col_ptr[bh][0..T_n]
// into col_idx[bh][.], its length, and (bf16 tensors) the complement of the mask as the rows of a bit matrix.
//
// The job of one workgroup is 64 columns of a head.  It reads all index lists of the head: entries of its own columns become
// bits (column x, bit i), those of earlier columns are counted - the offset of its first list.  Then every thread writes
// out the bits of a few 32-row words at their places, and their complement (bits from T_m on: 0) as rows of the bit matrix.
//
// Nothing on the query side of the backward pass reads the lists, so these are the first workgroups of its launch; in one of
// their own their latency had the GPU to itself.  Training step, 32 heads of 4,096 tokens (d = 64) 222.5 -> 216.6 us, 12 heads
// of 4,096 in fp32 638.7 -> 633.9, 12 heads of 32,760 tokens 1,554 -> 1,546.
#pragma once
#include "common.h"
#include "masked_sums.h"

namespace sla2 {

struct BwdColumns {
  const int32_t* block_idx;
  int32_t *col_ptr, *col_idx, *counts;
  uint32_t* bits;                                     // null: no bit matrix
  int Tm, Tn, ksel, blocks, jobs;                     // blocks: workgroups, the jobs filled up to whole rounds of the XCDs
};
inline BwdColumns bwd_columns(const Shape& s, const BwdArgs& a) {
  const int jobs = s.BH * ((s.Tn + 63) / 64);
  return {a.block_idx, a.col_ptr, a.col_idx, a.col_cnt, s.bf16 ? a.col_bits : nullptr, s.Tm, s.Tn, s.k,
          (jobs + kXcds - 1) / kXcds * kXcds, jobs};
}
constexpr int kBwdColumnsLds = 64 * 65 * (int)(sizeof(uint32_t) + sizeof(uint16_t)) + (8 + 64) * (int)sizeof(int);   // T_m <= 2048

// THREADS of a workgroup; k = 0: every column is empty
template <int THREADS>
__device__ void bwd_columns_job(const BwdColumns& b, int job, unsigned char* lds) {
  if (job >= b.jobs) return;
  const int Tm = b.Tm, Tn = b.Tn, ksel = b.ksel, W = (Tm + 31) / 32, LW = W | 1;    // LW odd: no bank conflicts down a column
  int* before = reinterpret_cast<int*>(lds);                                       // [waves], then [64] offsets
  int* first = before + 8;
  uint32_t* words = reinterpret_cast<uint32_t*>(first + 64);                        // [64][LW] bits
  uint16_t* place = reinterpret_cast<uint16_t*>(words + 64 * LW);                   // [64][LW] set bits of the column before the word
  const int groups = (Tn + 63) / 64, bh = job / groups, j0 = job % groups * 64, tid = threadIdx.x, cols = min(64, Tn - j0);
  const int lane = tid % kWave, wave = tid / kWave;
  for (int x = tid; x < 64 * LW; x += THREADS) words[x] = 0u;
  __syncthreads();
  const int32_t* idx = b.block_idx + (size_t)bh * Tm * ksel;
  const unsigned entries = (unsigned)Tm * (unsigned)ksel;
  int earlier = 0;
#pragma unroll 8
  for (unsigned e = tid; e < entries; e += THREADS) {
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
#pragma unroll
    for (int x = 0; x < THREADS / kWave; x++) at += before[x];
    first[lane] = at - n;
    if (lane < cols) {
      b.counts[(size_t)bh * Tn + j0 + lane] = n;
      b.col_ptr[(size_t)bh * (Tn + 1) + j0 + lane + 1] = at;
    }
    if (j0 == 0 && lane == 0) b.col_ptr[(size_t)bh * (Tn + 1)] = 0;
  }
  __syncthreads();
  int32_t* out = b.col_idx + (size_t)bh * Tm * ksel;
  for (int x = tid; x < 64 * W; x += THREADS) {
    const int c = x % 64, y = x / 64;
    uint32_t word = words[c * LW + y];
    int at = first[c] + place[c * LW + y];
    while (word) {
      out[at++] = 32 * y + __ffs(word) - 1;
      word &= word - 1u;
    }
  }
  if (b.bits != nullptr) {
    const int pitch = masked_pitch(Tn), rows = masked_words(Tm);
    for (int x = tid; x < 64 * rows; x += THREADS) {
      const int c = x % 64, y = x / 64, left = Tm - 32 * y;
      const uint32_t open = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
      b.bits[((size_t)bh * rows + y) * pitch + j0 + c] = y < W ? ~words[c * LW + y] & open : 0u;
    }
  }
}

}  // namespace sla2
