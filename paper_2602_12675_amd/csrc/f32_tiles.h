// Tile helpers of the fp32 kernels: products run on v_mfma_f32_32x32x2_f32 (fp32 operands, fp32 accumulation, twice the
// rate of plain FMA code and two operand registers per 4096 flops instead of one LDS read per FMA).
//
// Lane l = 32 g + l % 32 feeds row (A) / column (B) l % 32 with ONE contraction index, g; the 32 x 32 result puts column
// l % 32, rows 8 (v / 4) + 4 g + v % 4 (v = 0..15) on lane l.  Which two indices a product pairs up is free as long as
// both operands agree, and every contraction here uses one of two orders:
//   - over channels, product 4 j + x takes channels 8 j + 4 g + x: a lane reads 4 consecutive channels at a time, and a
//     result over channels is already in that order (row 32 t + 8 (v / 4) + 4 g + v % 4 = channel 8 j + 4 g + x of
//     j = 4 t + v / 4, x = v % 4), so results, Q^phi and K^phi meet in registers;
//   - over tokens of a result (keys or query rows), product v takes its rows as they lie: probabilities feed the next
//     product from registers.
#pragma once
#include <type_traits>

#include "common.h"

namespace sla2 {

constexpr int kF32Tokens = 64;                       // tokens per key/value block
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int e = 0; e < 16; e++) z[e] = 0.f;
  return z;
}
__device__ __forceinline__ float exp2_f32(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float both_halves_sum(float x) { return x + __shfl_xor(x, 32); }
__device__ __forceinline__ float both_halves_max(float x) { return fmaxf(x, __shfl_xor(x, 32)); }

// rows of D floats in LDS, padded by one 16-byte chunk: 16 consecutive rows of a 16-byte column fall on all 64 banks
template <int D> constexpr int kF32Ld = D + 4;

// Rows of a [rows][D] tile as 16-byte chunks over NT threads: thread tid always has chunk tid % (D / 4), rows
// tid / (D / 4) + i * kRows.
template <int D, int NT, int ROWS> struct ChunkMap {
  static constexpr int kChunks = D / 4;
  static constexpr int kRows = NT / kChunks;
  static constexpr int kLoads = ROWS / kRows;
  static_assert(kLoads >= 1 && kLoads * kRows == ROWS, "unsupported split");
  // rows past `valid` repeat the last existing one (never none: valid >= 1)
  __device__ static __forceinline__ void load(f32x4 (&r)[kLoads], const float* src, int row_stride, int valid, int tid) {
#pragma unroll
    for (int i = 0; i < kLoads; i++)
      r[i] = *reinterpret_cast<const f32x4*>(src + (size_t)min(tid / kChunks + i * kRows, valid - 1) * row_stride + 4 * (tid % kChunks));
  }
  // sum over the lanes that share a row (all of them get it)
  __device__ static __forceinline__ float row_sum(float v) {
#pragma unroll
    for (int o = 1; o < kChunks; o <<= 1) v += __shfl_xor(v, o);
    return v;
  }
  __device__ static __forceinline__ float row_max(float v) {
#pragma unroll
    for (int o = 1; o < kChunks; o <<= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
  }
};

// acc += A B over D channels, A rows from LDS (`row`: this lane's row), B from registers
template <int D>
__device__ __forceinline__ f32x16 channel_product(const float* row, const f32x4 (&b)[D / 8], f32x16 acc, int g) {
#pragma unroll
  for (int j = 0; j < D / 8; j++) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(row + 8 * j + 4 * g);
#pragma unroll
    for (int x = 0; x < 4; x++) acc = mfma_f32(a[x], b[j][x], acc);
  }
  return acc;
}
// the same with both operands from LDS
template <int D>
__device__ __forceinline__ f32x16 channel_product(const float* row_a, const float* row_b, f32x16 acc, int g) {
#pragma unroll
  for (int j = 0; j < D / 8; j++) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(row_a + 8 * j + 4 * g);
    const f32x4 b = *reinterpret_cast<const f32x4*>(row_b + 8 * j + 4 * g);
#pragma unroll
    for (int x = 0; x < 4; x++) acc = mfma_f32(a[x], b[x], acc);
  }
  return acc;
}

// How the (D/32)^2 tiles of a d x d state are spread over NW waves: wave w owns kTiles tiles from tile w * kTiles on
// (row-major); with more waves than tiles the last waves own none.
template <int D, int NW> struct StateSplit {
  static constexpr int kEdge = D / 32;
  static constexpr int kTiles = kEdge * kEdge / NW > 0 ? kEdge * kEdge / NW : 1;
  __device__ static bool active(int w) { return w * kTiles < kEdge * kEdge; }
  __device__ static int mt(int w) { return (w * kTiles) / kEdge; }
  __device__ static int nt(int w) { return (w * kTiles) % kEdge; }
  static_assert(kTiles <= kEdge, "the tiles of a wave share their rows");
};
// state[32 mt.., 32 nt..] += a^T b over `rows` rows (a, b: [rows][kF32Ld<D>] in LDS)
template <int D, int NW, int TILES>
__device__ __forceinline__ void state_product(f32x16 (&h)[TILES], const float* a, const float* b, int rows, int w, int lane) {
  typedef StateSplit<D, NW> S;
  static_assert(TILES == S::kTiles, "one accumulator per tile of the wave");
  const float* pa = a + (lane / 32) * kF32Ld<D> + 32 * S::mt(w) + lane % 32;
  const float* pb = b + (lane / 32) * kF32Ld<D> + 32 * S::nt(w) + lane % 32;
#pragma unroll 8
  for (int s = 0; s < rows / 2; s++) {
    const float av = pa[2 * s * kF32Ld<D>];
#pragma unroll
    for (int x = 0; x < S::kTiles; x++) h[x] = mfma_f32(av, pb[2 * s * kF32Ld<D> + 32 * x], h[x]);
  }
}

}  // namespace sla2
