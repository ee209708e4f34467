// Sums over the blocks a bit matrix names, as a matrix product: C[r][n] = sum over s with bit (r, s) of B[s][n], a
// block's d x d state being a row of B.  The linear branch needs such sums for every block of one side over the blocks of
// the other that are NOT selected together with it.  One by one they would cost a gather of one state per list entry;
// as a product of the 0/1 matrix with all states every state is read once per 128 rows, and the matrix cores have the
// rest: bits as operand are exact, products with them too, sums are fp32.
// Key side of the backward pass, dH_j of 12 heads of 256 query blocks by 512 key blocks (d = 128, 7.5 blocks a list): the
// gathers took 135 us of the key-side kernel and the sum of all dH_i 18 us, this product takes 84 us: 0.1 GB read, 0.2 GB
// written, 52 GFLOP.  A gather grows with the kept fraction, this does not.  At d = 64 (32 heads of 64 by 64, 6 blocks a list):
// 7 us of the key-side kernel against 6 us here.
// Query side of the forward pass with long lists: launch_kv_states_bf16.
#pragma once
#include "mfma_tiles.h"

namespace sla2 {

// Bit matrices: [head][words_of(S)][pitch_of(R)] 32-bit words, bit s % 32 of word s / 32 of row r; bits from S on are 0.
__host__ __device__ __forceinline__ int masked_words(int S) { return 2 * ((S + 63) / 64); }
__host__ __device__ __forceinline__ int masked_pitch(int R) { return (R + 63) & ~63; }

constexpr int kMaskedRows = 128, kMaskedCols = 256;   // of C, per workgroup of four waves; a wave has 64 of the columns
constexpr int kMaskedTile = 64 * kMaskedCols * 2;     // 64 rows of B
constexpr int kMaskedLds = 2 * kMaskedTile;           // two buffers: two workgroups a CU

// B rows are moved to LDS 512 bytes at a time; the eight 64-byte units of a row (32 columns: one operand tile) are
// permuted by the row bits in which the four rows of a transposing read differ (below), which then meet different banks.
__device__ __forceinline__ unsigned masked_unit(unsigned row) { return (row & 1) | (row >> 3 & 2); }

// The 128 x 256 tile of C from (row0, col0).  b: [S][cols] bf16, halves of what is summed, c: [R][cols] bf16, bits: words of this head.
//
// One step is 64 rows of B.  Operand order: contraction index k = 2 q + x (+ 8 g for the upper half of the wave) of
// 16-row product ks is row 32 g + 16 x + 4 ks + q of the step, so that the two bits of a register of the mask operand
// are 16 apart in the row's word and all of them come out of it with a shift and an AND: 0x4000 is 2.0 in bf16, so B holds
// halves (halving C at the end instead would lose what the sums hold above half of the largest number).
// Bound by the matrix cores: 8 products (256 cycles) a wave and ks against 128 cycles for the mask operands, 2 KB of LDS
// reads; B arrives one step ahead.  A wave with products before it is served ahead of one that requests or waits (H_i of 80 heads of
// 75,601 tokens: the call 42.07 -> 41.54 ms, training step on 12 heads of 32,760 1,409.6 -> 1,407.3 us).
__device__ __forceinline__ void masked_sums_tile(const uint16_t* __restrict__ b, const uint32_t* __restrict__ bits,
                                                 uint16_t* __restrict__ c, int S, int R, int cols, int row0, int col0,
                                                 unsigned char* smem) {
  constexpr int RT = kMaskedRows / 32, CT = kMaskedCols / 4 / 32;
  const int lane = threadIdx.x % kWave, g = lane / 32;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const unsigned lds0 = lds_address(smem);
  const int steps = (S + 63) / 64, pitch = masked_pitch(R);
  // transfer n of wave w: rows 16 w + 2 n, + 1 of the step
  auto request = [&](int step, int buf) {
    const char* base = reinterpret_cast<const char*>(b) + (size_t)step * 64 * cols * 2 + (size_t)col0 * 2;
    const unsigned rows = min(64, S - 64 * step);      // rows past the end repeat the last one (cleared below)
#pragma unroll
    for (int n = 0; n < 8; n++) {
      const unsigned row = 16 * w + 2 * n + lane / 32;
      const unsigned chunk = (lane % 32) ^ (4 * masked_unit(row));
      dma_lane16(base, min(row, rows - 1) * (unsigned)(cols * 2) + 16 * chunk, lds0 + buf * kMaskedTile + (16 * w + 2 * n) * 512);
    }
  };
  unsigned word[RT];
  auto request_words = [&](int step, unsigned (&to)[RT]) {
    const uint32_t* base = bits + (size_t)(2 * step) * pitch;
#pragma unroll
    for (int t = 0; t < RT; t++) {
      const unsigned r = (unsigned)min(row0 + 32 * t + lane % 32, R - 1);
      to[t] = __builtin_bit_cast(unsigned, load_untracked_at(reinterpret_cast<const float*>(base), 4 * (g * (unsigned)pitch + r)));
    }
  };
  auto landed = [&](unsigned (&x)[RT], int step) {
    wait_vmcnt<0>();
    // rows past the end: their bits are 0, but 0 times an infinite entry is NaN.  Of this wave's rows 16 w to 16 w + 15
    for (int row = max(S - 64 * step, 16 * w); row < 16 * w + 16; row++)
      *reinterpret_cast<u32x2*>(smem + (step & 1) * kMaskedTile + row * 512 + 8 * lane) = u32x2{0u, 0u};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int t = 0; t < RT; t++) settle(x[t]);
  };
  request_words(0, word);
  request(0, 0);
  f32x16 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; t++)
#pragma unroll
    for (int u = 0; u < CT; u++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[t][u][e] = 0.f;
  // transposing read (cf. read_tr4): lane l supplies row 32 g + 4 ks + 2 hi + r / 2 + 16 (r % 2), r = l % 16 / 4, and 4
  // columns from 16 (l / 16 % 2) + 4 (l % 4) on of unit CT w + u
  const unsigned quad = lane % 16 / 4, tr_row = 32 * g + quad / 2 + 16 * (quad % 2);
  unsigned at[CT];
#pragma unroll
  for (int u = 0; u < CT; u++)
    at[u] = lds0 + tr_row * 512 + 64 * ((unsigned)(CT * w + u) ^ masked_unit(tr_row)) + 32 * (lane / 16 % 2) + 8 * (lane % 4);
  landed(word, 0);
  phase_barrier();
  for (int step = 0; step < steps; step++) {
    const unsigned buf = (step & 1) * kMaskedTile;
    const bool more = step + 1 < steps;
    unsigned next[RT];
    request_words(more ? step + 1 : step, next);
    if (more) request(step + 1, (step + 1) & 1);
    u32x2 rb[2][CT][2];
    auto read = [&](int ks) {
#pragma unroll
      for (int u = 0; u < CT; u++)
#pragma unroll
        for (int hi = 0; hi < 2; hi++) rb[ks % 2][u][hi] = lds_read_tr_untracked_at<1024>(at[u] + buf, 2 * ks + hi);
    };
    read(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      if (ks < 3) read(ks + 1);
      u32x4 a[RT];
#pragma unroll
      for (int t = 0; t < RT; t++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int p = 4 * ks + q;
          a[t][q] = (p < 15 ? word[t] << (14 - p) : word[t] >> 1) & 0x40004000u;
        }
      wait_lgkmcnt(ks < 3 ? 2 * CT : 0);
#pragma unroll
      for (int u = 0; u < CT; u++) {
        settle(rb[ks % 2][u][0]);
        settle(rb[ks % 2][u][1]);
        const u32x4 v4 = {rb[ks % 2][u][0][0], rb[ks % 2][u][0][1], rb[ks % 2][u][1][0], rb[ks % 2][u][1][1]};
#pragma unroll
        for (int t = 0; t < RT; t++)
          acc[t][u] = mfma_bf16(__builtin_bit_cast(bf16x8, a[t]), __builtin_bit_cast(bf16x8, v4), acc[t][u]);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    landed(next, more ? step + 1 : step);              // the next step is there ...
#pragma unroll
    for (int t = 0; t < RT; t++) word[t] = next[t];
    phase_barrier();                                   // ... for everyone, and this one's tile is free
  }
  // Rows 8 (v / 4) + 4 g + v % 4 of a lane's column -> 16 bytes of a row, through LDS.  Two rows are packed into a
  // register and exchanged with the neighbouring lane, so that a lane writes two columns of one row.
  constexpr unsigned kPitch = kMaskedCols / 4 * 2 + 16;
  unsigned char* mine = smem + w * (64 * kPitch);
  static_assert(4 * 64 * kPitch <= kMaskedLds, "64 rows of every wave at a time");
  const unsigned odd = lane & 1, pick = odd ? 0x07060302u : 0x01000504u;   // v_perm_b32(own, other)
#pragma unroll
  for (int part = 0; part < 2; part++) {
    if (part) wave_lds_fence();
#pragma unroll
    for (int t = 0; t < RT / 2; t++)
#pragma unroll
      for (int u = 0; u < CT; u++)
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
          const f32x16& x = acc[part * (RT / 2) + t][u];
          const bf16x2 two = {(__bf16)x[v], (__bf16)x[v + 1]};
          const unsigned own = __builtin_bit_cast(unsigned, two);
          const unsigned other = (unsigned)__builtin_amdgcn_update_dpp((int)own, (int)own, 0xB1, 0xf, 0xf, false);   // lane ^ 1
          const unsigned row = 32 * t + 8 * (v / 4) + 4 * g + v % 4 + odd;
          *reinterpret_cast<unsigned*>(mine + row * kPitch + 64 * u + 4 * (lane % 32 / 2)) = __builtin_amdgcn_perm(own, other, pick);
        }
    wave_lds_fence();
#pragma unroll
    for (int n = 0; n < 8; n++) {
      const int row = 8 * n + lane / 8, r = row0 + 64 * part + row;
      if (r < R)
        *reinterpret_cast<u32x4*>(c + (size_t)r * cols + col0 + 64 * w + 8 * (lane % 8)) =
            *reinterpret_cast<const u32x4*>(mine + row * kPitch + 16 * (lane % 8));
    }
  }
}

}  // namespace sla2
