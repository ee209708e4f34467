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
  // over the lanes that share a row (all of them get it); vector instructions: four or five exchanges through LDS in a row took 1 to 4 %
  // of a call (training step on 3 heads of 1,000 tokens 126.2 us, now 121.1; forward on 8 heads of 3,000, d = 64 61.2 / 60.5)
  __device__ static __forceinline__ float row_sum(float v) { return sla2::row_sum<kChunks>(v); }
  __device__ static __forceinline__ float row_max(float v) { return sla2::row_max<kChunks>(v); }
};

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
// state += a^T b over 64 rows: a [64][kF32Ld<D>] in LDS, b straight from memory, as only one wave (d = 128: all four, out of
// the L1) reads an entry.  Column of entry x of a lane: column() + x, so that a lane reads and stores kTiles floats at a time.
template <int D> struct StateProduct {
  typedef StateSplit<D, 4> SS;
  typedef __attribute__((ext_vector_type(SS::kTiles))) float Cols;
  static constexpr int kAhead = SS::kTiles == 1 ? 32 : 8;       // 2,048 matrix cycles
  Cols b[kAhead];
  const char* base;
  unsigned off, step, end;                // bytes: this lane's next row, two rows, the last row there is
  unsigned lane_off;
  __device__ static __forceinline__ int column(int w, int r) { return 32 * SS::nt(w) + SS::kTiles * r; }
  __device__ __forceinline__ Cols next() {
    const Cols c = *reinterpret_cast<const Cols*>(base + (off + lane_off));
    off = min(off + step, end);
    return c;
  }
  // rows from `rows` on, `valid` of them there (those past the end repeat the last one: a has zeros for them)
  __device__ __forceinline__ void begin(const float* rows, int n, int valid, int w, int lane) {
    base = reinterpret_cast<const char*>(rows);
    lane_off = 4u * (unsigned)column(w, lane % 32);
    step = 8u * (unsigned)n;
    end = 4u * (unsigned)n * (unsigned)(valid - 1);     // strides are below 2^24 elements
    off = min(4u * (unsigned)n * (unsigned)(lane / 32), end);
#pragma unroll
    for (int s = 0; s < kAhead; s++) b[s] = next();
  }
  __device__ __forceinline__ void add(f32x16 (&h)[SS::kTiles], const float* a, int w, int lane) {
    const float* pa = a + (lane / 32) * kF32Ld<D> + 32 * SS::mt(w) + lane % 32;
#pragma unroll
    for (int s = 0; s < 32; s++) {
      const float av = pa[2 * s * kF32Ld<D>];
      const Cols c = b[s % kAhead];
#pragma unroll
      for (int x = 0; x < SS::kTiles; x++) h[x] = mfma_f32(av, c[x], h[x]);
      if (s % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // else all rows are requested at once
      if (s + kAhead < 32) b[s % kAhead] = next();
    }
  }
  __device__ static __forceinline__ void store(const f32x16 (&h)[SS::kTiles], float scale, float* out, int w, int lane) {
    float* p = out + (32 * SS::mt(w) + 4 * (lane / 32)) * D + column(w, lane % 32);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      Cols c;
#pragma unroll
      for (int x = 0; x < SS::kTiles; x++) c[x] = scale * h[x][e];
      *reinterpret_cast<Cols*>(p + (8 * (e / 4) + e % 4) * D) = c;
    }
  }
};

// ---- four waves that share 32 rows (of queries or keys, one per lane pair) and split the blocks of a list ----
// Each has parts of the same D x 32 results in ET = D / 32 accumulators.  Which channel a row of tile x stands for is free:
// ET row + x, so that a lane reads ET consecutive channels of an operand row at a time.  After the loop wave w owns the
// entries v / 4 = w of all tiles: entry e < D / 8 of a lane is channel own_channel() + e.
__device__ __forceinline__ int own_channel(int D, int w, int g) { return D / 32 * (8 * w + 4 * g); }
template <int D, int ROUNDS = 1> constexpr int kMeetFloats = 4 * 3 * (D / 8) * kWave / ROUNDS;
// own = the sum of the four waves' parts, each times its wave's `scale`; `swap` holds kMeetFloats<D, ROUNDS>, free for
// everyone.  In ROUNDS rounds with a part of the tiles each; the last one ends with the reads.
template <int D, int ROUNDS = 1>
__device__ __forceinline__ void meet4(float (&own)[D / 8], const f32x16 (&acc)[D / 32], float scale, float* swap, int w, int lane) {
  constexpr int ET = D / 32, XT = ET / ROUNDS;
  auto part = [&](int owner, int from) { return swap + (owner * 3 + from - (from > owner)) * 4 * XT * kWave + lane; };
#pragma unroll
  for (int n = 0; n < ROUNDS; n++) {
    if (n) __syncthreads();               // the round before has been read
    auto put = [&](auto wave) {           // one branch a round, not one an entry
      constexpr int W = decltype(wave)::value;
#pragma unroll
      for (int o = 0; o < 4; o++)
#pragma unroll
        for (int y = 0; y < 4; y++)
#pragma unroll
          for (int x = 0; x < XT; x++) {
            const float p = acc[XT * n + x][4 * o + y] * scale;
            if (o == W) own[ET * y + XT * n + x] = p;
            else part(o, W)[(XT * y + x) * kWave] = p;
          }
    };
    if (w == 0) put(std::integral_constant<int, 0>());
    else if (w == 1) put(std::integral_constant<int, 1>());
    else if (w == 2) put(std::integral_constant<int, 2>());
    else put(std::integral_constant<int, 3>());
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 4; f++)
      if (f != w) {
#pragma unroll
        for (int y = 0; y < 4; y++)
#pragma unroll
          for (int x = 0; x < XT; x++) own[ET * y + XT * n + x] += part(w, f)[(XT * y + x) * kWave];
      }
  }
}
// 32 consecutive rows of a head from `first` (the same on all lanes) on, rows past `last` repeating it: as pieces of this
// lane's row, or as the same channels of 16 rows.  Bases are scalar, lane offsets 32 bits: made where they are used, so
// that the addresses of a phase do not take up registers.
struct RowPieces {
  const char* base;
  int stride, left;                       // bytes; rows behind the first one
  __device__ __forceinline__ RowPieces(const float* head, int first, int last, int n) : stride(4 * n) {
    const int f = min(first, last);
    base = reinterpret_cast<const char*>(head) + (size_t)(unsigned)f * (unsigned)stride;
    left = last - f;
  }
  // channels 8 j + 4 g .. of row r: at own(r, g), j
  __device__ __forceinline__ unsigned own(int r, int g) const { return (unsigned)min(r, left) * (unsigned)stride + 16u * (unsigned)g; }
  __device__ __forceinline__ f32x4 piece(unsigned own, int j) const { return *reinterpret_cast<const f32x4*>(base + own + 32 * j); }
  // channels ET r .. of rows 8 (e / 4) + 4 g + e % 4: four floats, of row e = j at d = 128, of e = 2 j, 2 j + 1 at d = 64
  template <int D> __device__ __forceinline__ f32x4 cols(int j, int r, int g) const {
    constexpr int ET = D / 32;
    typedef __attribute__((ext_vector_type(ET))) float Cols;
    f32x4 out;
#pragma unroll
    for (int y = 0; y < 4 / ET; y++) {
      const int e = 4 / ET * j + y, s = min(8 * (e / 4) + e % 4, left), up = min(4, left - s) * stride;
      const Cols c = *reinterpret_cast<const Cols*>(base + (size_t)(unsigned)s * (unsigned)stride +
                                                    ((unsigned)(g ? up : 0) + (unsigned)(4 * ET * r)));
#pragma unroll
      for (int x = 0; x < ET; x++) out[ET * y + x] = c[x];
    }
    return out;
  }
};
// What a wave streams for its products, 16 bytes a lane and four products an element, goes through kStream sets of
// registers: an element is requested into the set of the one kStream before it as soon as that has been consumed, 2,048 matrix
// cycles ahead (with a second wave on the SIMD, 4,096).  All 16 of a phase ahead took 64 registers, and spills where two results
// are accumulated.
constexpr int kStream = 8;
// acc[tile] += (element j of cols) x weights: m-th float of the element is row e = (4 j + m) / ET, tile (4 j + m) % ET
template <int D>
__device__ __forceinline__ void col_products(f32x16 (&acc)[D / 32], const f32x4& a, const f32x16& p, int j) {
#pragma unroll
  for (int m = 0; m < 4; m++) acc[(4 * j + m) % (D / 32)] = mfma_f32(a[m], p[(4 * j + m) / (D / 32)], acc[(4 * j + m) % (D / 32)]);
}
// A D x 32 product of which every wave wants just the channels it owns: 32-channel tile StatePart::tile(w) each, at d = 64
// two waves a tile with half of the contraction (channel steps StatePart::first(w) ..).  Operand row r of the tile is channel
// row(r), so that results lie on the entries the wave owns.
template <int D> struct StatePart {
  static constexpr int kShares = 128 / D, kSteps = D / 8 / kShares;      // waves per tile; steps of 8 channels each
  __device__ static int tile(int w) { return w / kShares; }
  __device__ static int first(int w) { return w % kShares * kSteps; }
  __device__ static __forceinline__ int row(int r) {
    return D == 128 ? 16 * (r >> 2 & 1) + 4 * (r >> 3) + (r & 3) : 16 * (r >> 4) + 8 * (r >> 2 & 1) + 4 * (r >> 3 & 1) + (r & 3);
  }
  static constexpr int kLds = D == 64 ? 4 * 8 * kWave : 0;               // floats
  // own entries of the product in `acc`; d = 64: the two waves of a tile exchange halves of their parts (a barrier inside)
  __device__ static __forceinline__ void own(float (&o)[D / 8], const f32x16& acc, float* lds, int w, int lane) {
    if constexpr (D == 128) {
#pragma unroll
      for (int e = 0; e < 16; e++) o[e] = acc[e];
    } else {
      auto exchange = [&](auto half) {
        constexpr int E0 = 8 * decltype(half)::value;
#pragma unroll
        for (int e = 0; e < 8; e++) lds[((w ^ 1) * 8 + e) * kWave + lane] = acc[8 - E0 + e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = acc[E0 + e] + lds[(w * 8 + e) * kWave + lane];
      };
      if (w % 2 == 0) exchange(std::integral_constant<int, 0>());
      else exchange(std::integral_constant<int, 1>());
    }
  }
};

}  // namespace sla2
