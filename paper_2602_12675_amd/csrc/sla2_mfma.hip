// bf16 / FP8 path of the SLA2 forward pass on the gfx950 matrix cores (Alg. 2 of the paper).
//
//   kv_state_bf16   per key block j of a head: K^phi_j = softmax_d(K_j - colmean K), written out as bf16
//                   MFMA operand fragments; z_j = colsum(K^phi_j); per-chunk partial sums of
//                   h_j = (K^phi_j)^T V_j and z_j (reduced to the per-head totals by kv_total); in the
//                   low-bit modes also the e4m3 or INT8 codes of K - colmean K with one scale per key
//                   block, and, when V is quantised too, the e4m3 codes of V in operand order (Sec. 5).
//   attn_mfma       one workgroup per query block i:
//                     sparse branch over the selected key/value blocks, ascending (online softmax);
//                     the d x d state of exactly those blocks, sum_sel (K^phi_j)^T V_j, from the stored
//                     K^phi fragments and the V tile that is already staged for P V;
//                     H_i = H_total - that sum, Z_i = Z_total - sum_sel z_j  (complement of the
//                     M_c[i,j] = 0 sum of Alg. 2; for long lists H_i is formed beforehand, by
//                     block_states_bf16);  O_l = Q^phi H_i / (Q^phi Z_i);
//                     out = alpha O_s + (1 - alpha) O_l                                     (Eq. 13)
//                   The same kernel with the block list replaced by 0..T_n-1 and the linear branch
//                   compiled out is the dense attention comparator.
//
// Products run as v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  In the low-bit modes (Sec. 5) Q K^T
// runs on 8-bit codes: 64-deep v_mfma_f32_32x32x64_f8f6f4 (e4m3) or 32-deep v_mfma_i32_32x32x32_i8 (INT8);
// with V quantised as well, P V is a 64-deep FP8 product too.  Scores are kept transposed (S^T = K Q^T) so that one lane owns one query row:
// row maxima and sums are in-lane reductions plus one exchange between the two lane halves, and
// the probabilities go back into the next product as its B operand without leaving registers.
#include "masked_sums.h"

namespace sla2 {

// four values already scaled into [-127, 127] -> their nearest integers (ties to even), one per byte
__device__ __forceinline__ int pack_int8(float a, float b, float c, float d) {
  const int ia = (int)__builtin_rintf(a), ib = (int)__builtin_rintf(b), ic = (int)__builtin_rintf(c), id = (int)__builtin_rintf(d);
  return (ia & 0xff) | ((ib & 0xff) << 8) | ((ic & 0xff) << 16) | (id << 24);
}

// How the (D/32)^2 32x32 tiles of the d x d state h are spread over NW waves: wave w owns
// kMtw x kNtw tiles starting at (mt0, nt0).
template <int D, int NW> struct HSplit {
  static constexpr int kMt = D / 32;
  static constexpr int kPerWave = kMt * kMt / NW;
  static constexpr int kMtw = kPerWave > kMt ? kPerWave / kMt : 1;
  static constexpr int kNtw = kPerWave / kMtw;
  static_assert(kPerWave >= 1 && kMtw * kNtw == kPerWave, "unsupported split");
  __device__ static int mt0(int w) { return (w * kPerWave) / kMt; }
  __device__ static int nt0(int w) { return (w * kPerWave) % kMt; }
};

// K^phi of one key block is stored as the A-operand fragments of the product K^phi^T V:
// [block][mt = channel tile][ks = 16-token step][lane][8 bf16], lane l holding channel 32 mt + l % 32
// and the 8 tokens of (ks, l / 32) in token order - 1 KB per fragment, 16 consecutive
// bytes a lane: the attention kernel's pipelined loop brings it into the wave's own part of LDS, its plain loop into
// registers.
template <int D>
__device__ __forceinline__ size_t kphi_offset(size_t block, int mt, int ks, int lane) {
  return (((block * (D / 32) + mt) * (kTileTokens / 16) + ks) * kWave + lane) * 8;
}

// =============================================================================================
// kv_state_bf16
// =============================================================================================
// QUANT: 0 none, 1 FP8 e4m3 codes of K - colmean K, 2 INT8 codes, 3 as 1 plus e4m3 codes of V.
// STATES: half of h_j of every key block is written too (masked_sums.h), in the place of K^phi, as the sum of three bf16 parts
// (8 + 8 + 8 bits: nothing of an fp32 entry is left out): rows 3 j to 3 j + 2 of `states`, each as the accumulators lie - [tile (mt, nt)][2][64 lanes][8], lane l of half y
// holding column e = 32 nt + l % 32, rows c = 32 mt + 16 y + 4 (l / 32) + {0..3, 8..11}.  The heads are those from bh0 on;
// `partial` and `states` hold theirs alone.
// A token's softmax is taken once, in registers: its K^phi goes to LDS rounded, for the fragments, and from the registers into z_j,
// the sum of what was not rounded.  Taken twice, for lnZ and again for the fragments, the exponentials and the sums around them were most
// of a tile's 9,000 cycles (two workgroups a CU).  us, before / now: FP8, 12 heads of 32,760 tokens 73.9 / 65.3 (0.35 GB at 5.4 TB/s),
// 48 heads of 4,096 46.8 / 39.5; bf16 63.0 / 58.5; 32 heads of 4,096, d = 64 19.6 / 17.0; FP8 with V, 12 heads of 32,760, d = 64
// 68.7 / 49.0.
// Threads: at d = 128 eight waves with two tiles of h each run four on a SIMD, four waves with four tiles two: those leave the vector
// unit and the memory idle in turn (us, four / eight waves: FP8, 12 heads of 32,760 tokens 67.5 / 65.4, 48 of 4,096 42.5 / 39.5).
// With the states or the codes of V four: what they add does not fit 128 registers (FP8 with V 95 / 106).
template <int D, int QUANT, bool STATES> constexpr int kKvThreads = D == 128 && QUANT != 3 && !STATES ? 512 : 256;
template <int D, int QUANT, bool STATES>
__global__ __launch_bounds__((kKvThreads<D, QUANT, STATES>), (D == 64 || kKvThreads<D, QUANT, STATES> == 512 ? 4 : 2)) void kv_state_bf16_kernel(const uint16_t* __restrict__ k,
                                                            const uint16_t* __restrict__ v,
                                                            const double* __restrict__ k_mean,
                                                            float* __restrict__ k_stats, float* __restrict__ partial,
                                                            uint16_t* __restrict__ k_phi, float* __restrict__ z_blocks,
                                                            uint8_t* __restrict__ k_codes, float* __restrict__ k_scale,
                                                            uint8_t* __restrict__ v_codes, float* __restrict__ v_scale,
                                                            uint16_t* __restrict__ states, Strides sin, int bh0, int H, int N,
                                                            int Tn, int chunks, int blocks_per_chunk) {
  constexpr int LD = TileGeom<D>::kLd;
  constexpr int NT = kKvThreads<D, QUANT, STATES>, NW = NT / kWave, TPT = NT / kTileTokens;   // TPT: threads a token
  typedef HSplit<D, NW> HS;
  __shared__ __attribute__((aligned(16))) uint16_t ptile[kTileTokens * LD];    // K^phi
  __shared__ __attribute__((aligned(16))) uint16_t vtile[kTileTokens * LD];
  __shared__ __attribute__((aligned(16))) float zpart[NW][D];                  // sums of K^phi over the tokens of a wave
  __shared__ __attribute__((aligned(16))) float mu_s[D];
  __shared__ float red[NW];
  __shared__ float red_v[NW];
  const int bh = bh0 + blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
  const uint16_t* kh = k + head_offset(sin, bh, H);
  const uint16_t* vh = v + head_offset(sin, bh, H);
  const int j0 = chunk * blocks_per_chunk, j1 = min(Tn, j0 + blocks_per_chunk);
  const int mt0 = HS::mt0(w), nt0 = HS::nt0(w);

  if (tid < D) mu_s[tid] = (float)k_mean[(size_t)bh * D + tid];
  __syncthreads();

  f32x16 hacc[HS::kMtw][HS::kNtw];
#pragma unroll
  for (int a = 0; a < HS::kMtw; a++)
#pragma unroll
    for (int b = 0; b < HS::kNtw; b++)
#pragma unroll
      for (int e = 0; e < 16; e++) hacc[a][b][e] = 0.f;
  float zacc = 0.f;                                    // of channel tid

  // TPT threads a token, each with 8 P channels from c0 on: K goes from memory to the registers its softmax is taken in, V through
  // registers to LDS.
  constexpr int P = D / 8 / TPT;
  const int t = tid / TPT, sub = tid % TPT, c0 = 8 * P * sub;
  typedef TileCopy<D, NT> TC;
  u32x4 kr[P], vr[TC::kLoads];
  auto load_k = [&](int j) {
    const int there = min(kTileTokens, N - j * kTileTokens);
    const uint16_t* row = kh + ((size_t)j * kTileTokens + min(t, there - 1)) * sin.n + c0;
#pragma unroll
    for (int i = 0; i < P; i++) kr[i] = *reinterpret_cast<const u32x4*>(row + 8 * i);
  };
  auto load_v = [&](int j) { TC::load(vr, vh + (size_t)j * kTileTokens * sin.n, sin.n, min(kTileTokens, N - j * kTileTokens), tid); };
  if (j0 < j1) {
    load_k(j0);
    load_v(j0);
  }
  for (int j = j0; j < j1; j++) {
    const int t0 = j * kTileTokens, valid = min(kTileTokens, N - t0);
    const bool ok = t < valid;
    float x[8 * P];
#pragma unroll
    for (int i = 0; i < P; i++) {
      const f32x4 mu[2] = {*reinterpret_cast<const f32x4*>(mu_s + c0 + 8 * i), *reinterpret_cast<const f32x4*>(mu_s + c0 + 8 * i + 4)};
#pragma unroll
      for (int e = 0; e < 4; e++) {
        x[8 * i + 2 * e] = __builtin_bit_cast(float, kr[i][e] << 16) - mu[e / 2][2 * (e % 2)];
        x[8 * i + 2 * e + 1] = __builtin_bit_cast(float, kr[i][e] & 0xFFFF0000u) - mu[e / 2][2 * (e % 2) + 1];
      }
    }
    if (j + 1 < j1) load_k(j + 1);
    // K^phi = softmax_d(k') of the token and lnZ, its log-partition
    float p[8 * P];
    {
      float m = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8 * P; e++) m = fmaxf(m, x[e]);
      m = quad_max(m);
      if (TPT == 8) m = fmaxf(m, dpp_move<0x141>(m));  // row_half_mirror: the other four lanes
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8 * P; e++) {
        p[e] = fast_exp2((x[e] - m) * kLog2e);
        sum += p[e];
      }
      sum = quad_sum(sum);
      if (TPT == 8) sum += dpp_move<0x141>(sum);
      if (ok && sub == 0) k_stats[(size_t)bh * N + t0 + t] = m + __log2f(sum) * 0.6931471805599453f;
      const float inv = 1.f / sum;
#pragma unroll
      for (int e = 0; e < 8 * P; e++) p[e] *= inv;
      if (valid < kTileTokens)                         // tokens past the end contribute nothing
#pragma unroll
        for (int e = 0; e < 8 * P; e++) p[e] = ok ? p[e] : 0.f;
    }
    float amax = 0.f;
    if (QUANT) {
#pragma unroll
      for (int e = 0; e < 8 * P; e++) amax = fmaxf(amax, fabsf(x[e]));
      amax = wave_max(ok ? amax : 0.f);
    }
    // Sums over the tokens of the wave (lanes TPT apart), in fp32: two exchanges that halve what a lane has left to sum, then
    // rotations within 16 lanes.  A lane ends up with 2 P channels from c0 + zc on.
    constexpr int Z = 2 * P;
    const int zc = 2 * Z * (lane / 32) + Z * (lane / 16 % 2);
    float z[Z];
    {
      float half[2 * Z];
#pragma unroll
      for (int e = 0; e < 2 * Z; e++) half[e] = swap32_add(p[e], p[2 * Z + e]);
#pragma unroll
      for (int e = 0; e < Z; e++) {
        z[e] = swap16_add(half[e], half[Z + e]);
        z[e] += rotate16<8>(z[e]);
        if (TPT == 4) z[e] += rotate16<4>(z[e]);
      }
    }
    __syncthreads();                                   // previous tile fully consumed
#pragma unroll
    for (int i = 0; i < P; i++) {
      bf16x8 y;
#pragma unroll
      for (int e = 0; e < 8; e++) y[e] = (__bf16)p[8 * i + e];
      *reinterpret_cast<bf16x8*>(ptile + t * LD + c0 + 8 * i) = y;
    }
    TC::store(vr, vtile, tid);
    if (j + 1 < j1) load_v(j + 1);
    if (lane % 16 < TPT) {
#pragma unroll
      for (int e = 0; e < Z; e += 4) *reinterpret_cast<f32x4*>(&zpart[w][c0 + zc + e]) = f32x4{z[e], z[e + 1], z[e + 2], z[e + 3]};
    }
    if (QUANT && lane == 0) red[w] = amax;
    __syncthreads();
    if (tid < D) {
      float zj = 0.f;
#pragma unroll
      for (int y = 0; y < NW; y++) zj += zpart[y][tid];
      zacc += zj;
      z_blocks[((size_t)bh * Tn + j) * D + tid] = zj;
    }
    if (QUANT) {
      // one scale per key block: amax over the block's existing tokens (Sec. 5; see sla2.h)
      constexpr float kCodeMax = QUANT == 2 ? kInt8Max : kE4M3Max;
#pragma unroll
      for (int y = 0; y < NW; y++) amax = fmaxf(amax, red[y]);
      const float inv = amax > 0.f ? kCodeMax / amax : 1.f;
      if (tid == 0) k_scale[(size_t)bh * Tn + j] = amax > 0.f ? amax / kCodeMax : 1.f;
      int codes[2 * P];
#pragma unroll
      for (int i = 0; i < P; i++) {
        int lo = 0, hi = 0;
        if (ok) {
          float y[8];
#pragma unroll
          for (int e = 0; e < 8; e++) y[e] = fminf(fmaxf(x[8 * i + e] * inv, -kCodeMax), kCodeMax);
          if constexpr (QUANT == 2) {
            lo = pack_int8(y[0], y[1], y[2], y[3]);
            hi = pack_int8(y[4], y[5], y[6], y[7]);
          } else {
            lo = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], lo, false);
            lo = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], lo, true);
            hi = __builtin_amdgcn_cvt_pk_fp8_f32(y[4], y[5], hi, false);
            hi = __builtin_amdgcn_cvt_pk_fp8_f32(y[6], y[7], hi, true);
          }
        }
        codes[2 * i] = lo;
        codes[2 * i + 1] = hi;
      }
      uint8_t* dst = k_codes + (((size_t)bh * Tn + j) * kTileTokens + t) * D + c0;
#pragma unroll
      for (int x = 0; x < P; x += 2) *reinterpret_cast<i32x4*>(dst + 8 * x) = i32x4{codes[2 * x], codes[2 * x + 1], codes[2 * x + 2], codes[2 * x + 3]};
    }
    if constexpr (QUANT == 3) {
      // quant(V_j) for the second product (Alg. 2): one e4m3 scale per block over its existing tokens,
      // codes stored channel-major with the tokens of a row in the order the 64-deep product consumes
      // them (layout: sla2.h, v_fp8).  The threads of token t find the maximum ...
      float vmax = 0.f;
      if (t < valid) {
#pragma unroll
        for (int i = 0; i < P; i++) {
          const uint4 u = *reinterpret_cast<const uint4*>(vtile + t * LD + c0 + 8 * i);
          const uint32_t wds[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
          for (int e = 0; e < 4; e++) {
            vmax = fmaxf(vmax, fabsf(__builtin_bit_cast(float, wds[e] << 16)));
            vmax = fmaxf(vmax, fabsf(__builtin_bit_cast(float, wds[e] & 0xFFFF0000u)));
          }
        }
      }
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, o));
      if (lane == 0) red_v[w] = vmax;
      __syncthreads();
#pragma unroll
      for (int y = 0; y < NW; y++) vmax = fmaxf(vmax, red_v[y]);
      const float vinv = vmax > 0.f ? kE4M3Max / vmax : 1.f;
      if (tid == 0) v_scale[(size_t)bh * Tn + j] = vmax > 0.f ? vmax / kE4M3Max : 1.f;
      // ... and four threads of channel c write 16 codes each of row c: bytes 16 part .. 16 part + 15
      for (int y = tid; y < 4 * D; y += NT) {
        const int c = y / 4, part = y % 4;
        int wd[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {                  // dword q = bytes 4 q .. 4 q + 3
          float x4[4];
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int b = 16 * (part % 2) + 4 * q + r; // byte of the half row part / 2
            const int tok = 32 * (b / 16) + 8 * ((b % 16) / 4) + 4 * (part / 2) + b % 4;
            const float v4 = __builtin_bit_cast(float, (uint32_t)vtile[tok * LD + c] << 16);
            x4[r] = tok < valid ? fminf(fmaxf(v4 * vinv, -kE4M3Max), kE4M3Max) : 0.f;
          }
          int d0 = 0;
          d0 = __builtin_amdgcn_cvt_pk_fp8_f32(x4[0], x4[1], d0, false);
          d0 = __builtin_amdgcn_cvt_pk_fp8_f32(x4[2], x4[3], d0, true);
          wd[q] = d0;
        }
        *reinterpret_cast<int4*>(v_codes + (((size_t)bh * Tn + j) * D + c) * kTileTokens + 16 * part) = make_int4(wd[0], wd[1], wd[2], wd[3]);
      }
    }
    // K^phi fragments (kept for the attention kernel), h += K^phi^T V on the matrix cores, z_j
    if constexpr (STATES) {
      static_assert(HS::kMtw == 1, "one row of tiles a wave");
      bf16x8 kf[kTileTokens / 16];
#pragma unroll
      for (int ks = 0; ks < kTileTokens / 16; ks++)
        kf[ks] = v_fragment<PaddedLayout<D>>(ptile, ks, 32 * mt0, lane);
      uint16_t* to = states + ((size_t)(bh - bh0) * Tn + j) * (kStateParts * D * D) + ((mt0 * (D / 32) + nt0) * 2 * kWave + lane) * 8;
#pragma unroll
      for (int b = 0; b < HS::kNtw; b++) {
        f32x16 h;
#pragma unroll
        for (int e = 0; e < 16; e++) h[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < kTileTokens / 16; ks++)
          h = mfma_bf16(kf[ks], v_fragment<PaddedLayout<D>>(vtile, ks, 32 * (nt0 + b), lane), h);
#pragma unroll
        for (int y = 0; y < 2; y++) {
          float left[8];
#pragma unroll
          for (int e = 0; e < 8; e++) left[e] = 0.5f * h[8 * y + e];
#pragma unroll
          for (int p = 0; p < kStateParts; p++) {
            bf16x8 part;
#pragma unroll
            for (int e = 0; e < 8; e++) {
              part[e] = (__bf16)left[e];
              const float rest = left[e] - (float)part[e];
              left[e] = p > 0 || __builtin_isfinite(left[e]) ? rest : 0.f;   // the first part has all of an infinite entry
            }
            *reinterpret_cast<bf16x8*>(to + p * (D * D) + (2 * b + y) * kWave * 8) = part;
          }
        }
        hacc[0][b] += h;
        __builtin_amdgcn_sched_barrier(0);             // one tile at a time: the registers
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < kTileTokens / 16; ks++) {
        bf16x8 kf[HS::kMtw];
#pragma unroll
        for (int a = 0; a < HS::kMtw; a++) {
          kf[a] = v_fragment<PaddedLayout<D>>(ptile, ks, 32 * (mt0 + a), lane);
          if (HS::kNtw == D / 32 || ks / 2 == nt0 / HS::kNtw)   // where two waves form the fragments of a channel tile: two steps each
            *reinterpret_cast<bf16x8*>(k_phi + kphi_offset<D>((size_t)bh * Tn + j, mt0 + a, ks, lane)) = kf[a];
        }
#pragma unroll
        for (int b = 0; b < HS::kNtw; b++) {
          bf16x8 vf = v_fragment<PaddedLayout<D>>(vtile, ks, 32 * (nt0 + b), lane);
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) hacc[a][b] = mfma_bf16(kf[a], vf, hacc[a][b]);
        }
      }
    }
  }
  float* ph = partial + (size_t)blockIdx.x * (D * D + D);   // head of the launch, chunk
#pragma unroll
  for (int a = 0; a < HS::kMtw; a++) {
#pragma unroll
    for (int b = 0; b < HS::kNtw; b++)
#pragma unroll
      for (int x = 0; x < 4; x++) {
        const f32x4 part = {hacc[a][b][4 * x], hacc[a][b][4 * x + 1], hacc[a][b][4 * x + 2], hacc[a][b][4 * x + 3]};
        *reinterpret_cast<f32x4*>(ph + (((mt0 + a) * (D / 32) + nt0 + b) * 4 + x) * 256 + 4 * lane) = part;   // as it lies (kv_total)
      }
  }
  if (tid < D) ph[D * D + tid] = zacc;
}

hipError_t launch_kv_state_bf16(const Shape& s, const uint16_t* k, const uint16_t* v, const double* k_mean,
                                float* k_stats, float* partial, uint16_t* k_phi, float* z_blocks, uint8_t* k_codes,
                                float* k_scale, uint8_t* v_codes, float* v_scale, hipStream_t stream) {
  dim3 grid((unsigned)(s.BH * s.chunks));
#define SLA2_KV(DD, QQ)                                                                                          \
  kv_state_bf16_kernel<DD, QQ, false><<<grid, kKvThreads<DD, QQ, false>, 0, stream>>>(k, v, k_mean, k_stats, partial, k_phi, z_blocks, k_codes, \
                                                                k_scale, v_codes, v_scale, nullptr, s.sin, 0, s.H, s.N, s.Tn, \
                                                                s.chunks, s.blocks_per_chunk)
#define SLA2_KV_D(DD)                                                                                  \
  do {                                                                                                 \
    if (s.quant == 3) SLA2_KV(DD, 3); else if (s.quant == 2) SLA2_KV(DD, 2);                           \
    else if (s.quant == 1) SLA2_KV(DD, 1); else SLA2_KV(DD, 0);                                        \
  } while (0)
  if (s.d == 128) SLA2_KV_D(128);
  else SLA2_KV_D(64);
#undef SLA2_KV_D
#undef SLA2_KV
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// H_i of all query blocks of a call as a product of the selection's complement with all h_j (masked_sums.h), for long lists:
// an h_j in three bf16 parts, which hold its fp32 entries whole, the sum in fp32, H_i as bf16 (as the attention kernel applies it)
// in the order of kv_state.  Two parts leave out 2^-18 of an entry: where 257 states cancel to 2^-9 of one, the output was off by
// 5e-2 with them, by the rounding of its operands with three (and with states rebuilt from bf16 operands).
// On 8 heads of 75,601 tokens: kv_state 244 us (0.9 GB written, K^phi left out), the product 534 us (549 GFLOP, 1.0 PFLOP/s, bound
// by the matrix cores); with two parts 173 and 349 us.  The attention kernel without the rebuilt states takes 35.4 instead of
// 48.4 ms on 80 of them at 85 % sparsity, the call 43.9 instead of 50.1 (two parts 41.6).
//
// block_bits: the complement as bits, 3 j to 3 j + 2 of a row for key block j; one workgroup per 64 rows of a head.
__global__ __launch_bounds__(256) void block_bits_kernel(const int32_t* __restrict__ block_idx, uint32_t* __restrict__ bits, int Tm, int Tn,
                                                         int ksel) {
  extern __shared__ uint32_t listed[];                // [words][64]
  const int words = masked_words(kStateParts * Tn), pitch = masked_pitch(Tm), r0 = blockIdx.x * 64, bh = blockIdx.y, rows = min(64, Tm - r0);
  for (int x = threadIdx.x; x < 64 * words; x += 256) listed[x] = 0u;
  __syncthreads();
  const int32_t* idx = block_idx + ((size_t)bh * Tm + r0) * ksel;
  for (int e = threadIdx.x; e < rows * ksel; e += 256) {
    for (int s = kStateParts * idx[e], end = s + kStateParts; s < end; s++)
      atomicOr(&listed[s / 32 * 64 + e / ksel], 1u << (s % 32));       // OR: the result does not depend on the order
  }
  __syncthreads();
  for (int x = threadIdx.x; x < 64 * words; x += 256) {
    const int y = x / 64, left = kStateParts * Tn - 32 * y;
    const uint32_t open = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
    bits[((size_t)bh * words + y) * pitch + r0 + x % 64] = ~listed[x] & open;
  }
}

// The tiles of one set of columns, which read the same states, run next to each other on one XCD.
__global__ __launch_bounds__(256, 2) void block_states_bf16_kernel(const uint16_t* __restrict__ states, const uint32_t* __restrict__ bits,
                                                                   uint16_t* __restrict__ h_i, int Tm, int Tn, int len) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tiles = (Tm + kMaskedRows - 1) / kMaskedRows, sets = len / kMaskedCols;
  const int y = blockIdx.x / kXcds, set = y / tiles * kXcds + blockIdx.x % kXcds, head = set / sets;   // sets: a multiple of 8
  const int S = kStateParts * Tn;
  masked_sums_tile(states + (size_t)head * S * len, bits + (size_t)head * masked_words(S) * masked_pitch(Tm),
                   h_i + (size_t)head * Tm * len, S, Tm, len, y % tiles * kMaskedRows, set % sets * kMaskedCols, smem);
}

// As many heads at a time as their states fill kStateBytes: with kv_state of a group, its totals and its product.
hipError_t launch_kv_states_bf16(const Shape& s, const uint16_t* k, const uint16_t* v, const double* k_mean, float* k_stats,
                                 float* partial, float* h_total, float* z_total, float* z_blocks, uint8_t* k_codes, float* k_scale,
                                 uint8_t* v_codes, float* v_scale, const int32_t* block_idx, const GivenStates& gs, hipStream_t stream) {
  const int words = masked_words(kStateParts * s.Tn), len = s.d * s.d, tiles = (s.Tm + kMaskedRows - 1) / kMaskedRows;
  block_bits_kernel<<<dim3((unsigned)((s.Tm + 63) / 64), (unsigned)s.BH), 256, 64 * words * sizeof(uint32_t), stream>>>(   // at most 48 KB
      block_idx, gs.bits, s.Tm, s.Tn, s.k);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)block_states_bf16_kernel, kMaskedLds); e != hipSuccess) return e;
  for (int bh0 = 0; bh0 < s.BH; bh0 += s.state_heads) {
    const int heads = s.BH - bh0 < s.state_heads ? s.BH - bh0 : s.state_heads;
#define SLA2_KV(QQ)                                                                                                        \
  kv_state_bf16_kernel<128, QQ, true><<<dim3((unsigned)(heads * s.chunks)), kKvThreads<128, QQ, true>, 0, stream>>>(                             \
      k, v, k_mean, k_stats, partial, nullptr, z_blocks, k_codes, k_scale, v_codes, v_scale, gs.states, s.sin, bh0, s.H, s.N, \
      s.Tn, s.chunks, s.blocks_per_chunk)
    if (s.quant == 3) SLA2_KV(3);
    else if (s.quant == 2) SLA2_KV(2);
    else if (s.quant == 1) SLA2_KV(1);
    else SLA2_KV(0);
#undef SLA2_KV
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (hipError_t e = launch_kv_total(s, heads, partial, h_total + (size_t)bh0 * len, z_total + (size_t)bh0 * s.d, nullptr, stream); e != hipSuccess) return e;
    block_states_bf16_kernel<<<dim3((unsigned)(heads * (len / kMaskedCols) * tiles)), 256, kMaskedLds, stream>>>(
        gs.states, gs.bits + (size_t)bh0 * words * masked_pitch(s.Tm), gs.h_i + (size_t)bh0 * s.Tm * len, s.Tm, s.Tn, len);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Totals over the chunks of a head (Alg. 2's sums of h_j and z_j over all key blocks).  A thread owns 4 consecutive entries
// of the partial sums; the 8 waves of a workgroup walk the chunks 8 apart and meet in LDS, always in the same
// order, so the totals are the same bits on every run.  Bound by the start of the launch and one pass over the partial sums
// (33 MB for 12 heads of 32k tokens).
// The h part of the partial sums lies as accumulator fragments (kv_state_bf16): [d/32 (c)][d/32 (e)][4][64 lanes][4],
// lane l of part x holding rows c = 8 x + 4 (l / 32) + 0..3 of column e = l % 32; h_frag takes -h_total in the same order, which
// is what the accumulators of the attention kernel start from (null where H_i is given to it).
constexpr int kTotalWaves = 8;
__global__ __launch_bounds__(64 * kTotalWaves) void kv_total_kernel(const float* __restrict__ partial, float* __restrict__ h_total,
                                                                    float* __restrict__ z_total, float* __restrict__ h_frag,
                                                                    int d, int chunks) {
  __shared__ f32x4 red[64 * kTotalWaves];
  const int per_head = d * d + d;
  const int bh = blockIdx.y, l = threadIdx.x % 64, cg = threadIdx.x / 64;
  const int e = (blockIdx.x * 64 + l) * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (e < per_head) {
    const float* p = partial + (size_t)bh * chunks * per_head + e;
#pragma unroll 4
    for (int c = cg; c < chunks; c += kTotalWaves) s += *reinterpret_cast<const f32x4*>(p + (size_t)c * per_head);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (cg == 0 && e < per_head) {
    for (int x = 1; x < kTotalWaves; x++) s += red[64 * x + l];
    if (e >= d * d) {
      *reinterpret_cast<f32x4*>(z_total + (size_t)bh * d + (e - d * d)) = s;
    } else {
      if (h_frag != nullptr) *reinterpret_cast<f32x4*>(h_frag + (size_t)bh * d * d + e) = -s;
      const int tile = e / 1024, x = e / 256 % 4, lane = e / 4 % 64;
      const int row = 32 * (tile / (d / 32)) + 8 * x + 4 * (lane / 32), col = 32 * (tile % (d / 32)) + lane % 32;
      for (int r = 0; r < 4; r++) h_total[((size_t)bh * d + row + r) * d + col] = s[r];
    }
  }
}

hipError_t launch_kv_total(const Shape& s, int heads, const float* partial, float* h_total, float* z_total, float* h_frag,
                           hipStream_t stream) {
  const dim3 grid((unsigned)((s.d * s.d + s.d + 255) / 256), (unsigned)heads);
  kv_total_kernel<<<grid, 64 * kTotalWaves, 0, stream>>>(partial, h_total, z_total, h_frag, s.d, s.chunks);
  return hipGetLastError();
}

// =============================================================================================
// attn_mfma
// =============================================================================================
enum AttnMode { kSparseBf16 = 0, kSparseFp8 = 1, kDenseBf16 = 2, kSparseInt8 = 3, kSparseFp8V = 4 };


// Shapes whose main loop can be the pipelined one (see there).  The others keep the plain loop: the dense comparator, and
// d = 64 with 128-row blocks, whose waves own single tiles of the d x d state.
template <int D, int BQ, int MODE> constexpr bool kPipelined = MODE != kDenseBf16 && HSplit<D, BQ / 32>::kNtw == D / 32;
// Shapes that take the plain loop for long lists over many key blocks all the same, and the line: k T_n above 2,500.  A tile
// is short there (d = 64, 64-row blocks, FP8 scores) and the loop bound by its transfers, so it lives on what the workgroups
// of a head find in the L2 of their XCD; that takes workgroups in step with each other, and the pipelined loop holds them
// there less well: 12 heads of 32,760 tokens, k = 61, L2 hits 45 % against 72 % (FP8), 42 % against 66 % (FP8 with V), bytes
// through the fabric 4.4 against 2.2 GB and 5.5 against 3.2.  Attention kernel, pipelined / plain, us at k T_n:
//            480 (6,144 tokens)  1,920 (12,288)  3,328 (16,384)  4,416 (12,288)  5,120 (32,760)  31,232 (32,760)
//   FP8      51.0 / 52.7         76.3 / 77.1     115.8 / 112.8   143.7 / 143.9   137.2 / 130.9   693 / 634
//   with V   55.5 / 57.6         85.5 / 87.5     126.3 / 125.4   153.8 / 149.0   156.4 / 147.8   789 / 619
// The other shapes do not lose with it: INT8 stays within 4 % either way, bf16 gains up to 10 %, d = 128 gains throughout.
template <int D, int BQ, int MODE> constexpr bool kPlainToo = D == 64 && BQ == 64 && (MODE == kSparseFp8 || MODE == kSparseFp8V);
constexpr int kPipelinedTiles = 2500;

// LDS carve-up.  Loop, in this order: K^phi fragments of one tile, each wave's own (pipelined loop only); two V tiles
// (bf16); codes of the first V tile (when V is quantised for the second product); two K tiles (bf16, or 8-bit codes);
// codes of the second V tile - all in the layouts the load unit fills directly.  Before the loop the query rows of
// waves 0, 1 pass through the place of the second V tile and those of waves 2, 3 through that from the second K tile on.
// Epilogue, over the same memory: H_i^T as bf16 [D][D+8], the output tile [BQ][D+8] and Z_i as fp32.  At
// d = 128 the loop takes at most 80 KB: two workgroups a CU.
template <int D, int BQ, bool FP8, bool VQ, bool PIPE, bool GIVEN> struct AttnSmem {
  static constexpr int kLd = TileGeom<D>::kLd, NW = BQ / 32;
  static constexpr int kVBytes = SwizzledLayout<D>::kTileBytes;
  static constexpr int kKBytes = FP8 ? SwizzledLayout8<D>::kTileBytes : kVBytes;
  static constexpr int kVqBytes = VQ ? SwizzledLayoutVq<D>::kTileBytes : 0;   // e4m3 codes of V, when P V is an FP8 product
  static constexpr int kQBytes = 32 * D * 2;                        // query rows of one wave
  static constexpr int kVOff = PIPE && !GIVEN ? kTileTokens * D * 2 : 0;      // behind the K^phi fragments
  static constexpr int kVq0Off = kVOff + 2 * kVBytes;
  static constexpr int kKOff = kVq0Off + kVqBytes;
  static constexpr int kVq1Off = kKOff + 2 * kKBytes;
  static constexpr int kTiles = kVq1Off + kVqBytes, kQEnd = kKOff + kKBytes + (NW - 2) * kQBytes;
  static constexpr int kLoopBytes = kTiles > kQEnd ? kTiles : kQEnd;
  static constexpr int kZsOff = (D + BQ) * kLd * 2;                 // fp32 [D]: Z_i (epilogue)
  static constexpr int kEpiBytes = kZsOff + D * 4;
  static constexpr int kBytes = kLoopBytes > kEpiBytes ? kLoopBytes : kEpiBytes;
  __device__ static unsigned q_rows(int w) { return w < 2 ? kVOff + kVBytes + w * kQBytes : kKOff + kKBytes + (w - 2) * kQBytes; }
};


// Waves per SIMD the register budget is set for (second launch bound): 2; 1 for d = 128 with 64-row blocks, whose
// two waves hold half of the d x d state each; 3 for d = 64 with 128-row blocks, where the accumulators are small
// enough for 168 registers (measured on a 32,760-token d = 64 input: 6 % faster in FP8 mode, 10 % in bf16 mode;
// with 64-row blocks three waves gain nothing).
// GIVEN (pipelined loop): H_i was formed before (launch_kv_states_bf16) and is not rebuilt from K^phi: in the slots of `h_save`,
// which the workgroup of the block turns into H_i^T at its end, or without it where `k_phi` points to.
template <int D, int BQ, int MODE, bool PIPE, bool GIVEN>
__global__ __launch_bounds__(BQ * 2, (D == 128 && BQ == 64) ? 1 : (D == 64 && BQ == 128) ? 3 : 2) void attn_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const double* __restrict__ k_mean, const uint16_t* __restrict__ k_phi, const float* __restrict__ z_blocks,
    const uint8_t* __restrict__ k_codes, const float* __restrict__ k_scale, const uint8_t* __restrict__ v_codes,
    const float* __restrict__ v_scale, const float* __restrict__ h_frag,
    const float* __restrict__ z_total, const int32_t* __restrict__ block_idx, const float* __restrict__ alpha,
    uint16_t* __restrict__ out, float* __restrict__ lse, uint16_t* __restrict__ o_s_save,
    uint16_t* __restrict__ o_l_save, float* __restrict__ lse_save, uint16_t* __restrict__ h_save,
    float* __restrict__ z_save, Strides sin, Strides sout, int H, int N, int Tm,
    int Tn, int ksel, int alpha_per_block) {
  // FP8 below means "8-bit codes of Q and K": everything the two low-bit modes share.  INT8 marks the
  // places where the integer mode differs (the quantiser of Q and the Q K^T product).
  // FP8V: V is quantised too and P V runs as an FP8 product (the linear branch still reads the bf16 V).
  constexpr bool DENSE = MODE == kDenseBf16, INT8 = MODE == kSparseInt8, FP8V = MODE == kSparseFp8V;
  constexpr bool FP8 = MODE == kSparseFp8 || INT8 || FP8V;
  constexpr int NW = BQ / 32, NT = NW * kWave;
  constexpr int LD = TileGeom<D>::kLd;
  constexpr int KS = D / 16;            // contraction steps over the head dimension
  constexpr int ET = D / 32;            // 32-wide tiles over the head dimension
  typedef HSplit<D, NW> HS;
  typedef AttnSmem<D, BQ, FP8, FP8V, PIPE, GIVEN> SM;
  // the layout without bank conflicts where the tile transfers of a workgroup's waves allow it
  typedef typename std::conditional<PIPE && D == 128 && NW == 4, SwizzledLayoutB<128>, SwizzledLayout<D>>::type SL;
  typedef SwizzledLayout8<D> SL8;
  // Loads and LDS reads are issued untracked and waited for by count (see load_untracked): in the pipelined loop always,
  // in the plain one in the low-bit modes.  Its two bf16 forms leave them to the compiler.
  constexpr bool kManual = FP8;
  // global -> LDS transfers (1 KB each) a wave issues per tile: K in bf16 or 8-bit codes, V with its codes, K^phi fragments
  constexpr int kKOps = kTileTokens * D * (FP8 ? 1 : 2) / 1024 / NW;
  constexpr int kVOps = kTileTokens * D * 2 / 1024 / NW + (FP8V ? kTileTokens * D / 1024 / NW : 0);
  constexpr int kDmaOps = kKOps + kVOps;
  constexpr int kSteps = kTileTokens / 16, kPhiOps = PIPE && !GIVEN ? HS::kMtw * kSteps : 0;
  constexpr int kQOps = SM::kQBytes / 1024;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned lds0 = lds_address(smem);
  auto kbuf = [&](int buf) { return lds0 + SM::kKOff + buf * SM::kKBytes; };
  auto vbuf = [&](int buf) { return lds0 + SM::kVOff + buf * SM::kVBytes; };
  auto vqbuf = [&](int buf) { return lds0 + SM::kVq0Off + buf * (SM::kVq1Off - SM::kVq0Off); };

  // The arguments that the requests below need, all at once: left to the compiler they come in three turns, each as long as a
  // scalar load.  (In the plain loop too, whose scalar registers they do not push out; d = 64, us, without / with: FP8, 128-row blocks,
  // 32 heads of 4,096 tokens 66.0 / 65.5, 24 of 16,384 215.8 / 215.3, FP8 with V, 64-row blocks, 12 of 32,760 at 61 tiles 729 / 719.)
  asm volatile("" ::"s"(q), "s"(k), "s"(v), "s"(block_idx), "s"(k_codes), "s"(k_phi), "s"(h_frag), "s"(z_total), "s"(sin.b), "s"(sin.h),
               "s"(sin.n), "s"(H), "s"(N), "s"(Tm), "s"(Tn), "s"(ksel));
  asm volatile("" ::"s"(k_scale), "s"(alpha), "s"(v_scale), "s"(v_codes), "s"(alpha_per_block), "s"(h_save), "s"(z_blocks));
  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Consecutive query blocks of
  // a head share key/value tiles: every head is cut into 8 runs of consecutive blocks, one per XCD, and
  // all XCDs work through the heads in the same order - the tiles in flight then belong to one or two
  // heads, which the memory-side cache holds whole.
  const int per_head = (Tm + kXcds - 1) / kXcds;
  const int bh = (blockIdx.x / kXcds) / per_head, i = (blockIdx.x % kXcds) * per_head + (blockIdx.x / kXcds) % per_head;
  if (i >= Tm) return;
  const int h = bh % H;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);   // wave index, known to be uniform
  const int row0 = i * BQ;
  const int rows_valid = min(BQ, N - row0);
  const uint16_t* qh = q + head_offset(sin, bh, H);
  const uint16_t* kh = k + head_offset(sin, bh, H);
  const uint16_t* vh = v + head_offset(sin, bh, H);
  const int tok_stride = sin.n;                      // elements between consecutive tokens of q, k, v
  const int32_t* sel = DENSE ? nullptr : block_idx + ((size_t)bh * Tm + i) * ksel;
  const int ntiles = DENSE ? Tn : ksel;
  const int mt0 = HS::mt0(w), nt0 = HS::nt0(w);
  const size_t blk0 = (size_t)bh * Tn;   // first key block of this head in the per-block arrays
  // Key block of tile s.  The indices (and the FP8 scales) are fetched one and two tiles ahead of
  // their use: a scalar load consumed right away stalls the wave for its whole latency.
  auto tile_block = [&](int s) { return DENSE ? min(s, Tn - 1) : scalar_load(sel + min(s, ntiles - 1)); };
  int j_cur = ntiles > 0 ? tile_block(0) : 0, j_nxt = ntiles > 0 ? tile_block(1) : 0;
  // FP8V: O^T is carried in units of the V scale of the tile being added (the factor between two tiles
  // joins the online-softmax correction); sv_cur is the scale of the coming tile, sv_prev of the last one
  float sk_cur = 1.f, sv_cur = 1.f, sv_prev = 1.f;

  // key block j: global memory -> LDS buffer `buf`, no registers involved (completion: vmcnt)
  const uint8_t* k_codes_h = FP8 ? k_codes + blk0 * (kTileTokens * D) : nullptr;
  const uint8_t* v_codes_h = FP8V ? v_codes + blk0 * (kTileTokens * D) : nullptr;
  const uint16_t* k_phi_h = DENSE || GIVEN ? nullptr : k_phi + kphi_offset<D>(blk0, mt0, 0, 0);
  const unsigned tile_stride = (unsigned)tok_stride * (kTileTokens * 2);   // bytes; below 2^31
  auto rows_at = [&](const uint16_t* head, int j) { return (const uint16_t*)((const char*)head + (size_t)(unsigned)j * tile_stride); };
  // what a lane adds to the base of its transfers; the pipelined loop keeps these in registers
  unsigned lane16 = 16u * lane;                            // consecutive bytes: K^phi fragments
  unsigned row_off = tile_lane_off<D, NW, SL>(tok_stride, w, lane);   // a whole tile of bf16 rows
  unsigned code_off = FP8 ? tile8_lane_off<D>(lane) : 0u;  // a tile of 8-bit codes
  auto dma_rows = [&](const uint16_t* head, int j, unsigned lds) {
    const int valid = min(kTileTokens, N - j * kTileTokens);
    if ((kManual || PIPE) && valid == kTileTokens) dma_tile_full<D, NW, SL>(rows_at(head, j), tok_stride, lds, w, row_off);
    else dma_tile<D, NW, SL>(rows_at(head, j), tok_stride, valid, lds, w, PIPE ? lane_again() : lane);
  };
  auto dma_k = [&](int j, int buf) {
    if constexpr (FP8) dma_tile8<D, NW>(k_codes_h + (unsigned)j * (kTileTokens * D), kbuf(buf), w, code_off);
    else dma_rows(kh, j, kbuf(buf));
  };
  auto dma_v = [&](int j, int buf) {
    dma_rows(vh, j, vbuf(buf));
    if constexpr (FP8V) dma_tile_vq<D, NW>(v_codes_h + (unsigned)j * (kTileTokens * D), vqbuf(buf), w, PIPE ? lane_again() : lane);
  };
  auto dma = [&](int j, int buf) {
    dma_k(j, buf);
    dma_v(j, buf);
  };
  // K^phi fragment (channel tile mt0 + a, 16-token step ks) of block j -> its place in this wave's part of LDS; the
  // fragments of a channel tile are consecutive on both sides
  const unsigned phi_lds = lds0 + w * (HS::kMtw * kSteps * 1024);
  auto dma_phi = [&](int j, int a, int ks) {
    dma_lane16_at(k_phi_h + (unsigned)j * (kTileTokens * D) + a * (kSteps * 512), lane16, phi_lds + a * (kSteps * 1024), ks);
  };
  // This wave's 32 query rows -> LDS at `lds` in the swizzled layout (whole lines of memory at a time; read as operand
  // fragments from there, every lane would touch lines of its own); rows past the end repeat the last one; never stored.
  // (The way for whole blocks makes the plain loop spill three to five scalars more; d = 64, us, with / without it there: 128-row blocks, FP8
  // 24 heads of 16,384 tokens 215.8 / 216.5, INT8 12 of 32,760 228.2 / 228.0, 64-row blocks, FP8 at 61 tiles 708.9 / 701.8.)
  auto dma_q = [&](unsigned lds) {
    typedef SwizzledLayout<D> L;
    constexpr int kRows = 1024 / (D * 2);
    const unsigned l = lane_again();
    if (rows_valid == BQ) {                            // two lane offsets at most, the rest is uniform
      const uint16_t* base = qh + (size_t)(row0 + 32 * w) * tok_stride;
      constexpr int kDiffer = kRows % 8 == 0 ? 1 : 2;  // the swizzle repeats every 8 rows
      static_assert(kDiffer * kRows == 8, "");
      unsigned off[kDiffer];
#pragma unroll
      for (int n = 0; n < kDiffer; n++)
        off[n] = ((int)l / L::kChunks) * (unsigned)(tok_stride * 2) + 16u * (((int)l % L::kChunks) ^ L::swz(n * kRows + (int)l / L::kChunks));
#pragma unroll
      for (int n = 0; n < kQOps; n++) dma_lane16(base + (size_t)(n * kRows) * (unsigned)tok_stride, off[n % kDiffer], lds + n * 1024);
      return;
    }
#pragma unroll
    for (int n = 0; n < kQOps; n++) {
      const int row = n * kRows + (int)l / L::kChunks;
      const unsigned r = (unsigned)min(32 * w + row, rows_valid - 1);
      dma_lane16(qh + (size_t)row0 * tok_stride, r * (unsigned)(tok_stride * 2) + 16u * (((int)l % L::kChunks) ^ L::swz(row)), lds + n * 1024);
    }
  };
  // fragment ks of those rows (B operand of S^T = K Q^T): lane <- row l % 32, 8 columns from column 8 * (chunk ^ XOR(ks))
  auto q_lane = [&](unsigned lds, int chunk) {
    typedef SwizzledLayout<D> L;
    const int row = (int)lane_again() % 32;
    return lds + row * (D * 2) + 16u * (chunk ^ L::swz(row));
  };
  auto read_q = [&](unsigned at, int x) { return lds_read16_untracked<0>(at ^ (16u * x)); };

  // Requests in the order their results are needed and can be made: the query rows and the d x d total need nothing but
  // the block index; the tiles need the block list.
  // Scales and alpha are asked for behind the tiles: the scalar loads return in any order, so the first one that is waited for
  // is a wait for all of them.
  float sk_nxt = 1.f, al;
  const int j_third = PIPE && ntiles > 0 ? tile_block(2) : 0;
  dma_q(lds0 + SM::q_rows(w));
  // The state accumulators start at -H_total (and -Z_total): the loop adds the h_j and z_j of the selected
  // blocks, which leaves -(H_total - sum) = -H_i.  The total lies there negated and as accumulator fragments
  // (kv_total): four 16-byte loads a tile.
  // GIVEN: H_i itself, 16 bytes of the slot per thread and kilobyte; it waits in registers for the epilogue.
  constexpr int kGivenLoads = GIVEN ? D * D / 8 / NT : 1;
  f32x4 hq[HS::kMtw][HS::kNtw][4], hgiven[kGivenLoads];
  float zsel[HS::kMtw];
  if constexpr (!DENSE) {
    if constexpr (GIVEN) {
      const float* slot = reinterpret_cast<const float*>((h_save ? h_save : k_phi) + ((size_t)bh * Tm + i) * D * D) + w * (D * D / 2 / NW);
#pragma unroll
      for (int x = 0; x < kGivenLoads; x++) hgiven[x] = load16_untracked_at(slot + 1024 * (x / 4), lane16, x % 4);
    } else {
#pragma unroll
    for (int a = 0; a < HS::kMtw; a++)
#pragma unroll
      for (int b = 0; b < HS::kNtw; b++)
#pragma unroll
        for (int x = 0; x < 4; x++)
          hq[a][b][x] = load16_untracked_at(h_frag + (size_t)bh * D * D + ((mt0 + a) * ET + nt0 + b) * 1024, lane16, x);
    }
#pragma unroll
    for (int a = 0; a < HS::kMtw; a++)
      zsel[a] = load_untracked_at(z_total + (size_t)bh * D + 32 * (mt0 + a), 4u * (unsigned)(lane % 32));
  }
  if (ntiles > 0) {
    dma(j_cur, 0);
    if constexpr (PIPE && !GIVEN) {
#pragma unroll
      for (int a = 0; a < HS::kMtw; a++)
#pragma unroll
        for (int ks = 0; ks < kSteps; ks++) dma_phi(j_cur, a, ks);
    }
    if constexpr (FP8) sk_cur = scalar_load(k_scale + blk0 + j_cur);
    if constexpr (FP8V) sv_cur = sv_prev = scalar_load(v_scale + blk0 + j_cur);
    if constexpr (PIPE && FP8) sk_nxt = scalar_load(k_scale + blk0 + j_nxt);
    al = DENSE ? 1.f : scalar_load(alpha + (alpha_per_block ? (size_t)h * Tm + i : (size_t)h));
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<kDmaOps + kPhiOps>();                 // query rows and totals are there
  } else {
    al = DENSE ? 1.f : scalar_load(alpha + (alpha_per_block ? (size_t)h * Tm + i : (size_t)h));
    wait_vmcnt<0>();
  }
  f32x16 hacc[HS::kMtw][HS::kNtw];
#pragma unroll
  for (int a = 0; a < HS::kMtw; a++) {
    if constexpr (!DENSE) {
      settle(zsel[a]);
      zsel[a] = -zsel[a];
    }
#pragma unroll
    for (int b = 0; b < HS::kNtw; b++)
      if constexpr (!DENSE && !GIVEN) {
#pragma unroll
        for (int x = 0; x < 4; x++) {
          settle(hq[a][b][x]);
#pragma unroll
          for (int e = 0; e < 4; e++) hacc[a][b][4 * x + e] = hq[a][b][x][e];
        }
        settle(hacc[a][b]);                          // one value from here on, not four
      }
  }
  if constexpr (GIVEN) {
#pragma unroll
    for (int x = 0; x < kGivenLoads; x++) settle(hgiven[x]);
  }
  // bf16 product: fragment ks = columns 16 ks + 8 g + 0..7.  FP8 product (64 deep): the lane's
  // operand of step ks2 is columns 64 ks2 + 32 g + 0..31, held as fragments 4 ks2 + 0..3.
  // INT8 product (32 deep): columns 32 ks4 + 16 g + 0..15, fragments 2 ks4 + 0..1.
  bf16x8 qf[KS];
  {
    u32x4 raw[KS];
    const unsigned at = q_lane(lds0 + SM::q_rows(w), INT8 ? 2 * g : FP8 ? 4 * g : g);
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
      raw[ks] = read_q(at, INT8 ? 4 * (ks / 2) + ks % 2 : FP8 ? 8 * (ks / 4) + ks % 4 : 2 * ks);
    wait_lgkmcnt(0);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      settle(raw[ks]);
      qf[ks] = __builtin_bit_cast(bf16x8, raw[ks]);
    }
  }
  // entry e of fragment ks in fp32: a shift or a mask (from elements of the vector the compiler makes sub-dword operations, which
  // wait for each other)
  auto q_value = [&](int ks, int e) {
    const unsigned two = __builtin_bit_cast(u32x4, qf[ks])[e / 2];
    return __builtin_bit_cast(float, e % 2 == 0 ? two << 16 : two & 0xFFFF0000u);
  };
  // FP8: quant(Q_i) with one scale for the whole query block (Sec. 5)
  long qf8[FP8 ? KS : 1];
  float s_q = 1.f;
  if constexpr (FP8) {
    float amax = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int e = 0; e < 8; e += 2) amax = max3_abs(amax, q_value(ks, e), q_value(ks, e + 1));
    amax = wave_max(amax);
    if (lane == 0) *reinterpret_cast<float*>(smem + SM::q_rows(w)) = amax;   // (this wave has read its rows)
    __syncthreads();
    amax = 0.f;
#pragma unroll
    for (int x = 0; x < NW; x++) amax = fmaxf(amax, *reinterpret_cast<const float*>(smem + SM::q_rows(x)));
    constexpr float kCodeMax = INT8 ? kInt8Max : kE4M3Max;
    const float inv = amax > 0.f ? kCodeMax / amax : 1.f;
    s_q = amax > 0.f ? amax / kCodeMax : 1.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      float y[8];
#pragma unroll
      for (int e = 0; e < 8; e++) y[e] = fminf(fmaxf(q_value(ks, e) * inv, -kCodeMax), kCodeMax);
      int lo = 0, hi = 0;
      if constexpr (INT8) {
        lo = pack_int8(y[0], y[1], y[2], y[3]);
        hi = pack_int8(y[4], y[5], y[6], y[7]);
      } else {
        lo = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], lo, false);
        lo = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], lo, true);
        hi = __builtin_amdgcn_cvt_pk_fp8_f32(y[4], y[5], hi, false);
        hi = __builtin_amdgcn_cvt_pk_fp8_f32(y[6], y[7], hi, true);
      }
      qf8[ks] = (long)(((unsigned long)(unsigned)hi << 32) | (unsigned)lo);
    }
  }
  if (PIPE && ntiles > 0) wait_vmcnt<kVOps + kPhiOps>();   // the first K tile (V and K^phi: in front of the loop)
  else wait_vmcnt<0>();
  __syncthreads();                                   // tile 0 is in LDS for everyone
  if constexpr (PIPE) {
    if (ntiles > 1) dma_k(j_nxt, 1);                 // (its place held query rows until here)
  }
  f32x16 oacc[ET];
#pragma unroll
  for (int et = 0; et < ET; et++)
#pragma unroll
    for (int e = 0; e < 16; e++) oacc[et][e] = 0.f;
  // running max and sum of this lane's query row, in the log2 domain.  In FP8 mode P is carried
  // scaled by 2^8 (the rounding grid of P, see sla2.h): the factor cancels in O / l.
  float m_run = -INFINITY, l_run = 0.f;
  constexpr float kPShift = FP8 ? 8.f : 0.f;
  const float c0 = kLog2e * rsqrtf((float)D);        // scores are used as S * log2(e) / sqrt(d)

  // Q^phi = softmax_d(Q) of this lane's row, in the order of its fragments - without its normaliser, which cancels
  // between Q^phi H_i and Q^phi Z_i.  In fp32: the numerator takes it rounded to bf16, the denominator as it is.
  // In pieces: the pipelined loop has them between the products of its last tile.
  // (The low-bit modes dropped the bf16 rows after quantisation; they come back through LDS, q_again.)
  f32x4 qx[DENSE ? 1 : KS][2];
  float qm = -INFINITY;
  auto q_max = [&]() {
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int e = 0; e < 8; e++) qm = fmaxf(qm, q_value(ks, e));
    qm = swap_halves_max(qm) * kLog2e;
  };
  auto q_exp = [&](int ks) {
#pragma unroll
    for (int x = 0; x < 2; x++) {
#pragma unroll
      for (int e = 0; e < 4; e++) qx[ks][x][e] = fast_exp2(q_value(ks, 4 * x + e) * kLog2e - qm);
      settle(qx[ks][x]);
    }
  };
  // where the query rows go at the last tile (V in vbuf(buf)): both K tiles and the other V tile are done with
  auto q_again = [&](int buf) { return w < 2 ? vbuf(buf ^ 1) + w * SM::kQBytes : kbuf(0) + (w - 2) * SM::kQBytes; };

  // S^T = K Q^T on the 8-bit codes, two 32-key halves; ka: this lane's first operand in the K tile.  The callbacks run
  // behind the operand reads and behind the matrix instructions.
  auto low_bit_scores = [&](unsigned ka, f32x16 (&sacc)[2], auto behind_reads, auto behind_product, auto behind_products) {
    if constexpr (INT8) {
      // 32-deep integer products (v_mfma_i32_32x32x32_i8: lane l holds row l % 32, contraction indices
      // 16 (l / 32) + 0..15): the operand of (step ks4, key half mt) is 16 consecutive codes of key row
      // 32 mt + l % 32 - one 16-byte read at (address of step 0) ^ 32 ks4 in the pair-swizzled tile.
      // Sums of 128 products of codes stay below 2^21: exact in the int32 accumulator and in fp32.
      constexpr int KS4 = D / 32;
      u32x4 kq[KS4][2];
#pragma unroll
      for (int ks4 = 0; ks4 < KS4; ks4++) {
        kq[ks4][0] = lds_read16_untracked<0>(ka ^ (32u * ks4));
        kq[ks4][1] = lds_read16_untracked<32 * D>(ka ^ (32u * ks4));
      }
      behind_reads();
      i32x16 iacc[2];
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int e = 0; e < 16; e++) iacc[mt][e] = 0;
#pragma unroll
      for (int ks4 = 0; ks4 < KS4; ks4++)
#pragma unroll
        for (int mt = 0; mt < 2; mt++) {
          wait_lgkmcnt(2 * (KS4 - 1 - ks4) + 1 - mt);
          settle(kq[ks4][mt]);
          const i32x4 a = __builtin_bit_cast(i32x4, kq[ks4][mt]);
          const i32x4 b = {(int)(unsigned)((unsigned long)qf8[2 * ks4]), (int)(unsigned)((unsigned long)qf8[2 * ks4] >> 32),
                           (int)(unsigned)((unsigned long)qf8[2 * ks4 + 1]), (int)(unsigned)((unsigned long)qf8[2 * ks4 + 1] >> 32)};
          iacc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, iacc[mt], 0, 0, 0);
          if (mt == 1) behind_product(ks4);
        }
      behind_products();
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int e = 0; e < 16; e++) sacc[mt][e] = (float)iacc[mt][e];
    } else {
      // 64-deep products: the operand of (step ks2, key half mt) is 32 consecutive codes of key row
      // 32 mt + l % 32, two 16-byte reads.  The swizzle is an XOR on the pair bits of the address,
      // so step ks2 sits at (address of step 0) ^ 64 ks2; all reads of a tile are issued up front.
      static_assert(D % 64 == 0, "the FP8 product consumes the head dimension 64 at a time");
      constexpr int KS2 = D / 64;
      u32x4 klo[KS2][2], khi[KS2][2];
#pragma unroll
      for (int ks2 = 0; ks2 < KS2; ks2++) {
        klo[ks2][0] = lds_read16_untracked<0>(ka ^ (64u * ks2));
        khi[ks2][0] = lds_read16_untracked<16>(ka ^ (64u * ks2));
        klo[ks2][1] = lds_read16_untracked<32 * D>(ka ^ (64u * ks2));
        khi[ks2][1] = lds_read16_untracked<32 * D + 16>(ka ^ (64u * ks2));
      }
      behind_reads();
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int e = 0; e < 16; e++) sacc[mt][e] = 0.f;
#pragma unroll
      for (int ks2 = 0; ks2 < KS2; ks2++)
#pragma unroll
        for (int mt = 0; mt < 2; mt++) {
          wait_lgkmcnt(2 * (2 * (KS2 - 1 - ks2) + 1 - mt));
          settle(klo[ks2][mt]);
          settle(khi[ks2][mt]);
          const u32x4 lo = klo[ks2][mt], hi = khi[ks2][mt];
          const i32x8 a = {(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
          i32x8 b;
#pragma unroll
          for (int x = 0; x < 4; x++) {
            b[2 * x] = (int)(unsigned)((unsigned long)qf8[4 * ks2 + x]);
            b[2 * x + 1] = (int)(unsigned)((unsigned long)qf8[4 * ks2 + x] >> 32);
          }
          sacc[mt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, sacc[mt], 0, 0, 0, 0, 0, 0);   // e4m3 x e4m3, no scales
          behind_product(2 * ks2 + mt);
        }
      behind_products();
    }
  };

  if constexpr (PIPE) {
    // The pipelined loop.  Pass s forms S of tile s + 1, then runs the products of tile s, P V and K^phi^T V, with the
    // softmax of tile s + 1 in between them: a matrix product holds the issue port of its SIMD for about a third of its
    // time, and what fits into the rest - a wave's own vector instructions included - costs nothing (micro-benchmark: one
    // product alone 33 cycles, with four multiply-adds behind it 34).  P replaces its predecessor 16 tokens at a time,
    // right after the products that read it, so it takes no second set of registers.
    // Measured on 12 heads of 32,760 tokens, d = 128, 128-row blocks: bf16, 26 tiles a block 520 -> 480 us; FP8, 15 tiles
    // 287 -> 276 us.  The clock falls as the loop gets denser and the launch longer: 1.96 GHz over the FP8 launch, now of 265 us,
    // 1.76 over the bf16 one of 459, 1.65 over 4.7 ms on 40 heads of 75,600 tokens (GRBM_GUI_ACTIVE over the launch): there work
    // counts, not latency.
    // Transfers, all global -> LDS: K of tile s + 2 and V of tile s + 1 are requested at the top of pass s, into places
    // read for the last time before the barrier above, and have a whole pass to land; the K^phi fragments of tile s + 1
    // are requested one by one as those of tile s leave the wave's part of LDS.  Counts: requests at the top are older
    // than the kPhiOps fragment requests of the same pass and younger than those of the pass before.
    // What the lanes derive from their index stays in registers too; the compiler would work it out again in every pass.
    unsigned k_lane = FP8 ? SL8::offset(lane % 32, (INT8 ? 16 : 32) * g) : 2 * SL::offset(lane % 32, 8 * g);
    constexpr bool kPeel = FP8;
    // A V fragment is two transposing reads, 8 rows apart: the row permutation is the same there, or differs in one bit.
    unsigned v_lane = 2 * SL::offset(4 * g + (lane % 16) / 4, 16 * ((lane / 16) % 2) + 4 * (lane % 4));
    constexpr unsigned kHiXor = std::is_same<SL, SwizzledLayout<D>>::value ? 0u : 32u;
    settle(lane16);
    settle(row_off);
    if constexpr (FP8) settle(code_off);
    settle(k_lane);
    settle(v_lane);
    f32x16 sacc[2];
    // S^T = K Q^T of the tile in kbuf(buf), two 32-key halves
    auto scores = [&](int buf, auto behind_reads, auto behind_product) {
      const unsigned ka = kbuf(buf) + k_lane;
      if constexpr (FP8) {
        low_bit_scores(ka, sacc, behind_reads, behind_product, [] {});
      } else {
        // the operand of (step ks, key half mt): 16 bytes of key row 32 mt + l % 32, step ks at (address of step 0) ^ 32 ks
        constexpr int kItems = 2 * KS, kAhead = 3, kSlots = kAhead + 1;
        u32x4 ring[kSlots];
        auto issue = [&](int n) {
          if (n % 2 == 0) ring[n % kSlots] = lds_read16_untracked<0>(ka ^ (32u * (n / 2)));
          else ring[n % kSlots] = lds_read16_untracked<32 * D * 2>(ka ^ (32u * (n / 2)));
        };
#pragma unroll
        for (int n = 0; n < kAhead; n++) issue(n);
        behind_reads();
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int e = 0; e < 16; e++) sacc[mt][e] = 0.f;
#pragma unroll
        for (int n = 0; n < kItems; n++) {
          if (n + kAhead < kItems) issue(n + kAhead);
          wait_lgkmcnt(n + kAhead < kItems ? kAhead : kItems - 1 - n);
          settle(ring[n % kSlots]);
          sacc[n % 2] = mfma_bf16(__builtin_bit_cast(bf16x8, ring[n % kSlots]), qf[n / 2], sacc[n % 2]);
        }
      }
    };
    // Online softmax of this lane's query row over the 64 keys in sacc, in pieces.
    float c1 = 1.f, mx = 0.f, m_new = 0.f, m_off = 0.f, corr = 1.f, rs = 0.f;
    bool rescale = false;
    bf16x8 pf[FP8V ? 1 : kSteps];                    // P^T fragments, token order
    i32x8 pb, pb_new;                                // FP8V: the e4m3 codes of P^T, byte 16 mt + e of the lane's half
    int codes = 0;
    auto mask_tail = [&](int valid) {
      if (valid < kTileTokens) {
        const int g4 = 4 * (int)(lane_again() / 32);
        asm volatile("" : "+s"(valid));              // none of the comparisons below is to be hoisted out of this rare branch
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int e = 0; e < 16; e++) {
            sacc[mt][e] = 32 * mt + 8 * (e / 4) + e % 4 < valid - g4 ? sacc[mt][e] : -INFINITY;
            __builtin_amdgcn_sched_barrier(0);       // one comparison at a time: 32 at once take 64 scalar registers
          }
      }
    };
    // The reference of the exponentials.  With P rounded to a grid (low-bit modes) it is the running maximum,
    // as Alg. 2 states it.  Otherwise any reference gives the same O / l, and the one in use is kept while the
    // maximum of the row stays within 2^kLazy of it (the weights reach at most 2^kLazy, harmless in bf16 and fp32).
    // O^T and l are rescaled when any row of the wave moves its reference.
    constexpr float kLazy = FP8 ? 0.f : 8.f;
    auto soft_max = [&](int mt) {
      if (mt == 0) mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 16; e++) mx = fmaxf(mx, sacc[mt][e]);
    };
    auto soft_reference = [&]() {
      mx = swap_halves_max(mx) * c1;
      rescale = __builtin_amdgcn_ballot_w64(mx > m_run + kLazy) != 0;   // first tile: m_run = -inf
      m_new = rescale ? fmaxf(m_run, mx) : m_run;    // finite: a tile holds at least one key
      m_off = m_new - kPShift;
      corr = fast_exp2(m_run - m_new);               // 0 on the first tile
      rs = 0.f;
    };
    auto soft_pair = [&](int n) {                    // probabilities 2 n, 2 n + 1 of the lane
      const int mt = n / 8, e = 2 * (n % 8);
      const float p0 = fast_exp2(sacc[mt][e] * c1 - m_off);
      const float p1 = fast_exp2(sacc[mt][e + 1] * c1 - m_off);
      rs += p0 + p1;                                 // the denominator keeps the un-rounded P
      settle(rs);                                    // (summed here: left for later, 32 addends stay in registers)
      if constexpr (FP8V) {
        const int q = 4 * mt + e / 4;                // two codes into the lower or upper half of dword q
        if (e % 4 == 0) pb_new[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, 0, false);
        else pb_new[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, pb_new[q], true);
      } else if constexpr (FP8) {
        // quant(P): e4m3 grid.  The instruction keeps the other half of its destination; feeding it the
        // previous pair's register (dead by now) instead of a zero saves a register move per pair
        codes = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, codes, false);
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const bf16x2 pq = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, false);
        pf[2 * mt + e / 8][e % 8] = pq[0];
        pf[2 * mt + e / 8][e % 8 + 1] = pq[1];
      } else {
        pf[2 * mt + e / 8][e % 8] = (__bf16)p0;
        pf[2 * mt + e / 8][e % 8 + 1] = (__bf16)p1;
      }
    };
    // The weights are made where they stand: left to itself the compiler moves the conversions behind the products, to
    // their first use in the next pass.
    auto soft_keep = [&](int ks) {
      if constexpr (FP8V) settle(pb_new);
      else settle(pf[ks]);
    };
    auto soft_end = [&]() {                          // the last step's probabilities, and the sums
#pragma unroll
      for (int n = 0; n < 4; n++) soft_pair(4 * (kSteps - 1) + n);
      soft_keep(kSteps - 1);
      l_run = l_run * corr + swap_halves_sum(rs);
      m_run = m_new;
      if constexpr (FP8V) pb = pb_new;
    };

    int j1 = j_nxt;                                  // key block of tile s + 1
    int j2 = j_third;
    float sk1 = sk_nxt;                              // scale of tile s + 1
    // Of the two waves of a SIMD the one that has its products and their softmax before it is served first: it has work for both units,
    // the other waits for requests or scores.  us, without / with: bf16, 12 heads of 32,760 tokens at 26 tiles a block 598.2 / 588.5,
    // with H_i given (80 heads of 75,601, 177 tiles) 44,852 / 44,181, FP8 at 15 tiles 406.9 / 404.5, INT8 416.2 / 413.2; d = 64, 64-row
    // blocks, INT8, 12 heads of 32,000 372.8 / 361.2.  With 64-row blocks and bf16 scores, where both waves have products most of the
    // time, it loses (d = 64, 12 heads of 16,000 104.6 / 105.4; d = 128, 12 of 32,760 909 / 925).
    constexpr bool kFirst = FP8 || BQ == 128;
    // At d = 128 with 128-row blocks in the low-bit modes the last quarter of a tile's softmax stands in the next pass, behind the operand reads of its
    // scores: ahead of the barrier nothing ran beside it (us: FP8, 40 heads of 75,600 tokens 5,767 -> 5,718, 12 of 32,760 410.5 ->
    // 406.9, INT8 418.8 -> 415.2; 64-row blocks 624 -> 625, bf16 602 -> 604; d = 64, 64-row blocks, training step 198.2 -> 200.9).
    // With V in FP8 only where H_i is given (24 heads of 16,384, 84 tiles 1,296 -> 1,286): its tile is the largest, and on long heads the
    // workgroups then share less of what they gather (40 heads of 75,600, 95 tiles 13,786 -> 13,893, 20 of them at 118 8,068 -> 8,129,
    // 40 of 45,000 at 56 4,976 -> 5,020; 48 of 4,096 178.6 / 178.4).
    constexpr bool kDefer = FP8 && D == 128 && BQ == 128 && (!FP8V || GIVEN);
    // The last tile has a copy of the pass of its own, with Q^phi in the place of the softmax - in the low-bit modes; bf16
    // operands, whose query fragments take 16 registers more, leave none for what the two copies would exchange.
    auto pass = [&](int s, auto last_pass) {
      constexpr bool LAST = decltype(last_pass)::value;
      const int buf = s & 1;
      const bool more = kPeel ? !LAST : s + 1 < ntiles;
      // In the low-bit modes the requests and the rescale of O^T stand in the score product, behind its operand reads and its four
      // 64-cycle instructions, which leave the issue port to them: ahead of it they held up the wave by some 400 cycles of 3,900 a pass
      // (us: FP8, 12 heads of 32,760 tokens 412.7 -> 407.8, 40 of 75,600 5,700 -> 5,622).  bf16 tensors rescale rarely, and have no gain;
      // nor has FP8 with V at d = 128 with 64-row blocks, one wave a SIMD, which loses on long heads (within / ahead of the product: 12 heads
      // of 2,048 tokens 49.4 / 49.4, 48 of 4,096 230.5 / 230.4, 12 of 16,384 461.4 / 461.6, 12 of 32,760 at 51 tiles 1,537 / 1,526, 30 of
      // 56,000 at 88 12,120 / 11,846, 40 of 75,600 at 118 31,899 / 31,621).
      constexpr bool kWithin = FP8 && !(FP8V && D == 128 && BQ == 64);
      float zj[HS::kMtw];
      int j3;
      float sk2 = 1.f, sv1 = 1.f;
      auto requests = [&]() {
        if (s + 2 < ntiles) dma_k(j2, buf);
        if (more) dma_v(j1, buf ^ 1);
        if constexpr (LAST) dma_q(q_again(buf));
#pragma unroll
        for (int a = 0; a < HS::kMtw; a++)
          zj[a] = load_untracked_at(z_blocks + (blk0 + j_cur) * D + 32 * (mt0 + a), (lane16 >> 2) & 124u);
        j3 = tile_block(s + 3);                        // indices and scales are fetched a pass ahead of their use
        if constexpr (FP8) sk2 = scalar_load(k_scale + blk0 + j2);
        if constexpr (FP8V) sv1 = scalar_load(v_scale + blk0 + j1);
      };
      // O^T in units of the new reference, 32 channels at a time
      const float co = FP8V ? corr * (sv_prev / sv_cur) : corr;
      auto rescale_o = [&](int et) {
        if (FP8V || rescale)
#pragma unroll
          for (int e = 0; e < 16; e++) oacc[et][e] *= co;
      };
      if (kWithin && !LAST) {
        scores(buf ^ 1,
               [&] {
                 requests();
                 if (kDefer) soft_end();
                 rescale_o(0);
               },
               [&](int n) {
                 if (n + 1 < ET) rescale_o(n + 1);
                 __builtin_amdgcn_sched_barrier(0);
               });
      } else {
        requests();
        if (kDefer) soft_end();
#pragma unroll
        for (int et = 0; et < ET; et++) rescale_o(et);
        if (more) scores(buf ^ 1, [] {}, [](int) {});
      }
      if constexpr (FP8V) {
        sv_prev = sv_cur;
        sv_cur = sv1;
      }
      if (more) mask_tail(N - j1 * kTileTokens);
      if constexpr (kFirst) __builtin_amdgcn_s_setprio(1);
      c1 = FP8 ? c0 * s_q * sk1 : c0;
      // the K^phi fragments of this tile have landed
      if constexpr (LAST) wait_vmcnt<kQOps + HS::kMtw>();
      else if (!more) wait_vmcnt<HS::kMtw>();
      else if (s + 2 < ntiles) wait_vmcnt<kKOps + kVOps + HS::kMtw>();
      else wait_vmcnt<kVOps + HS::kMtw>();
      // ---- O^T += V^T P^T and h += K^phi^T V of tile s; softmax of tile s + 1, or Q^phi ----
      const unsigned va = vbuf(buf) + v_lane, pa = phi_lds + lane16;
      constexpr int kFrags = kSteps * ET, kVAhead = 2;
      // reads are counted as they are issued; everything here is a constant once the loops are unrolled
      int issued = 0, v_at[kFrags], q_at = 0;
      u32x2 vlo[kVAhead + 1], vhi[kVAhead + 1];
      u32x4 ph[2][HS::kMtw];
      auto read_v = [&](int f) {
        vlo[f % (kVAhead + 1)] = lds_read_tr_untracked_at<16 * D>(va ^ (64u * (f % ET)), 2 * (f / ET));
        vhi[f % (kVAhead + 1)] = lds_read_tr_untracked_at<16 * D>(va ^ (64u * (f % ET) ^ kHiXor), 2 * (f / ET) + 1);
        v_at[f] = issued += 2;
      };
      auto read_phi = [&](int ks) {
        if constexpr (GIVEN) return;
#pragma unroll
        for (int a = 0; a < HS::kMtw; a++) ph[ks % 2][a] = lds_read16_untracked_at<1024>(pa + a * (kSteps * 1024), ks);
        issued += HS::kMtw;
      };
      if constexpr (FP8V) {
        // O^T += Vhat^T Ptilde^T as 64-deep FP8 products, one per 32-channel tile: the operand is the half
        // row (l / 32) of channel row 32 et + l % 32 of the code tile, two 16-byte reads
        typedef SwizzledLayoutVq<D> SLV;
        const unsigned qa = vqbuf(buf) + SLV::offset(lane % 32, 2 * g);
        u32x4 vq_lo[ET], vq_hi[ET];
#pragma unroll
        for (int et = 0; et < ET; et++) {
          vq_lo[et] = lds_read16_untracked_at<32 * kTileTokens>(qa, et);
          vq_hi[et] = lds_read16_untracked_at<32 * kTileTokens>(qa ^ 16u, et);
        }
#pragma unroll
        for (int et = 0; et < ET; et++) {
          wait_lgkmcnt(2 * (ET - 1 - et));
          settle(vq_lo[et]);
          settle(vq_hi[et]);
          const u32x4 lo = vq_lo[et], hi = vq_hi[et];
          const i32x8 a = {(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
          oacc[et] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, pb, oacc[et], 0, 0, 0, 0, 0, 0);
        }
      }
      constexpr int kQFrom = kFrags / 2;             // LAST: fragment from which on Q^phi is made of the query rows, back by then
      u32x4 raw[KS];
      read_phi(0);
#pragma unroll
      for (int f = 0; f < kVAhead; f++) read_v(f);
      unrolled<kFrags>([&](auto frag) {
        constexpr int f = decltype(frag)::value, ks = f / ET, et = f % ET;
        if (LAST && f == kQFrom - 1) {
          wait_vmcnt<HS::kMtw>();
          const unsigned at = q_lane(q_again(buf), g);
#pragma unroll
          for (int x = 0; x < KS; x++) raw[x] = read_q(at, 2 * x);
          q_at = issued += KS;
        }
        // K^phi of the next step before the V fragment it meets first: the wait for that one covers both
        static_assert(kVAhead == 2, "");
        if (et == ET - 2 && ks + 1 < kSteps) read_phi(ks + 1);
        if (f + kVAhead < kFrags) read_v(f + kVAhead);
        wait_lgkmcnt(issued - v_at[f]);
        settle(vlo[f % (kVAhead + 1)]);
        settle(vhi[f % (kVAhead + 1)]);
        if (!GIVEN && et == 0) {
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) settle(ph[ks % 2][a]);
          asm volatile("" ::: "memory");             // the fragments have left LDS: their successors may be requested
          if constexpr (!LAST) {
#pragma unroll
            for (int a = 0; a < HS::kMtw; a++) dma_phi(j1, a, ks);   // (bf16, past the last tile: that one again, never read)
          }
        }
        if (LAST && f == kQFrom) {
          wait_lgkmcnt(issued - q_at);
#pragma unroll
          for (int x = 0; x < KS; x++) {
            settle(raw[x]);
            qf[x] = __builtin_bit_cast(bf16x8, raw[x]);
          }
        }
        const u32x4 v4 = {vlo[f % (kVAhead + 1)][0], vlo[f % (kVAhead + 1)][1], vhi[f % (kVAhead + 1)][0], vhi[f % (kVAhead + 1)][1]};
        const bf16x8 vf = __builtin_bit_cast(bf16x8, v4);
        if constexpr (!FP8V) oacc[et] = mfma_bf16(vf, pf[ks], oacc[et]);
        if constexpr (!GIVEN) {
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) hacc[a][et] = mfma_bf16(__builtin_bit_cast(bf16x8, ph[ks % 2][a]), vf, hacc[a][et]);
        }
        if constexpr (LAST) {
          if (f == kQFrom) q_max();
          if (f > kQFrom) {
#pragma unroll
            for (int x = 2 * (f - kQFrom - 1); x < 2 * (f - kQFrom); x++)
              if (x < KS) q_exp(x);
          }
        } else if (ks == 0) {
          // softmax of the next tile: maximum and reference in step 0, then the probabilities of the step just done with
          if (et == 0) soft_max(0);
          if (et == (ET > 2 ? 1 : 0)) soft_max(1);
          if (et == (ET > 2 ? 2 : 1)) soft_reference();
        } else {
#pragma unroll
          for (int n = 4 / ET * et; n < 4 / ET * (et + 1); n++) soft_pair(4 * (ks - 1) + n);
          if (et == ET - 1) soft_keep(ks - 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (LAST) {
        wait_vmcnt<0>();                             // z_j
      } else {
        if (!kDefer && more) soft_end();
        wait_vmcnt<kPhiOps>();                       // the next K and V tiles have landed (and z_j) ...
      }
#pragma unroll
      for (int a = 0; a < HS::kMtw; a++) {
        settle(zj[a]);
        zsel[a] += zj[a];
      }
      phase_barrier();                               // ... for everyone, and this pass's tiles are free
      if constexpr (kFirst) __builtin_amdgcn_s_setprio(0);
      j_cur = j1;
      j1 = j2;
      j2 = j3;
      sk1 = sk2;
    };
    if (ntiles > 0) {
      scores(0, [] {}, [](int) {});
      c1 = FP8 ? c0 * s_q * sk_cur : c0;             // dequantisation folded into the score scale
      mask_tail(N - j_cur * kTileTokens);
      soft_max(0);
      soft_max(1);
      soft_reference();
#pragma unroll
      for (int n = 0; n < 4 * (kSteps - 1); n++) soft_pair(n);
      if (!kDefer) soft_end();
      rescale = false;                               // O^T is zero
      __builtin_amdgcn_s_waitcnt(kVmcnt0);           // V and K^phi of the first tile, K of the second have landed
      phase_barrier();                               // everyone is done with the first K tile
      for (int s = 0; s < ntiles - (kPeel ? 1 : 0); s++) pass(s, std::integral_constant<bool, false>());
      if constexpr (kPeel) pass(ntiles - 1, std::integral_constant<bool, true>());
      else __builtin_amdgcn_s_waitcnt(kVmcnt0);      // the last fragment requests: the epilogue reuses their place
    }
  } else {
  for (int s = 0; s < ntiles; s++) {
      const int buf = s & 1;
      const int j = j_cur;
      const int valid = min(kTileTokens, N - j * kTileTokens);
      const float sk = sk_cur;
      const int j_nn = tile_block(s + 2);                // consumed in the next iteration
      if constexpr (FP8) sk_cur = scalar_load(k_scale + blk0 + j_nxt);
      const float sv = sv_cur;
      if constexpr (FP8V) sv_cur = scalar_load(v_scale + blk0 + j_nxt);
      // K^phi fragments and z_j of this tile straight from global memory into registers (no other
      // wave needs them); they are consumed after the softmax.  They are issued before the next
      // tile's transfer and, since vmcnt retires in order, are complete once at most kDmaOps
      // operations are outstanding.  The loads are opaque to the compiler on purpose: its own
      // bookkeeping across the conditional transfer below falls back to vmcnt(0) at their first
      // use, which stalls every iteration on the tile that was just requested.
      bf16x8 kphi[DENSE ? 1 : HS::kMtw][kTileTokens / 16];
      float zj[DENSE ? 1 : HS::kMtw];
      auto state_loads = [&]() {
        if constexpr (!DENSE) {
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) {
#pragma unroll
            for (int ks = 0; ks < kTileTokens / 16; ks++)
              kphi[a][ks] = load_maybe_tracked<bf16x8, kManual>(k_phi + kphi_offset<D>(blk0 + j, mt0 + a, ks, lane));
            zj[a] = load_maybe_tracked<float, kManual>(z_blocks + (blk0 + j) * D + 32 * (mt0 + a) + lane % 32);
            if constexpr (!kManual) zsel[a] += zj[a];
          }
        }
      };
      auto next_tile = [&]() {
        if (s + 1 < ntiles) dma(j_nxt, buf ^ 1);             // next tile -> other buffer
      };
      // With the reads under this kernel's own control (low-bit modes) the requests for the rest of the
      // tile's data are placed inside the score product: the fragment loads behind its operand reads, the
      // next tile's transfer behind its matrix instructions - some hundred instructions that otherwise
      // stand in front of it, on a wave whose progress is bound by its own chain of dependent steps.
      if constexpr (!kManual) {
        state_loads();
        next_tile();
      }
      const uint16_t* vt = reinterpret_cast<const uint16_t*>(smem + SM::kVOff + buf * SM::kVBytes);
      // Two waves share a SIMD.  The one that is issuing matrix products is given the higher issue priority, so
      // that the matrix pipe is fed while the other wave's softmax fills the gaps (measured: 2 % on the
      // sparse modes; the dense comparator, all of whose waves are in step, loses with it).
      if constexpr (!DENSE) __builtin_amdgcn_s_setprio(2);
      // ---- S^T = K Q^T (keys x query rows), two 32-key halves ----
      f32x16 sacc[2];
      if constexpr (FP8) {
        low_bit_scores(kbuf(buf) + SL8::offset(lane % 32, (INT8 ? 16 : 32) * g), sacc, state_loads, [](int) {}, next_tile);
      } else {
        const uint16_t* kt = reinterpret_cast<const uint16_t*>(smem + SM::kKOff + buf * SM::kKBytes);
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int e = 0; e < 16; e++) sacc[mt][e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
          for (int mt = 0; mt < 2; mt++)
            sacc[mt] = mfma_bf16(row_fragment<SL>(kt, 32 * mt + lane % 32, 16 * ks + 8 * g), qf[ks], sacc[mt]);
      }
      j_cur = j_nxt;
      j_nxt = j_nn;
      if constexpr (!DENSE) __builtin_amdgcn_s_setprio(0);   // softmax: the other wave's matrix products go first
      // ---- online softmax of this lane's query row over the 64 keys ----
      const float c1 = FP8 ? c0 * s_q * sk : c0;       // dequantisation folded into the score scale
      if (valid < kTileTokens) {
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int e = 0; e < 16; e++)
            if (32 * mt + 8 * (e / 4) + 4 * g + e % 4 >= valid) sacc[mt][e] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int e = 0; e < 16; e++) mx = fmaxf(mx, sacc[mt][e]);
      mx = swap_halves_max(mx) * c1;
      // The reference of the exponentials.  With P rounded to a grid (low-bit modes) it is the running maximum,
      // as Alg. 2 states it.  Otherwise any reference gives the same O / l, and the one in use is kept while the
      // maximum of the row stays within 2^kLazy of it: O^T, l then need no rescaling in most tiles (the weights
      // reach at most 2^kLazy, harmless in bf16 and fp32).  The decision is taken for the whole wave.
      constexpr float kLazy = 8.f;
      bool rescale = true;
      if constexpr (!FP8) rescale = __builtin_amdgcn_ballot_w64(mx > m_run + kLazy) != 0;   // first tile: m_run = -inf
      const float m_new = rescale ? fmaxf(m_run, mx) : m_run;   // finite: a tile holds at least one key
      const float m_off = m_new - kPShift;
      float rs = 0.f;
      bf16x8 pf[FP8V ? 1 : 4];                         // P^T fragments, token order
      i32x8 pb;                                        // FP8V: the e4m3 codes of P^T, byte 16 mt + e of the lane's half
      int codes = 0;
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const float p0 = fast_exp2(sacc[mt][e] * c1 - m_off);
          const float p1 = fast_exp2(sacc[mt][e + 1] * c1 - m_off);
          rs += p0 + p1;                               // the denominator keeps the un-rounded P
          if constexpr (FP8V) {
            const int q = 4 * mt + e / 4;              // two codes into the lower or upper half of dword q
            if (e % 4 == 0) pb[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, 0, false);
            else pb[q] = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, pb[q], true);
          } else if constexpr (FP8) {
            // quant(P): e4m3 grid.  The instruction keeps the other half of its destination; feeding it the
            // previous pair's register (dead by now) instead of a zero saves a register move per pair
            codes = __builtin_amdgcn_cvt_pk_fp8_f32(p0, p1, codes, false);
            typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
            const bf16x2 pq = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, false);
            pf[2 * mt + e / 8][e % 8] = pq[0];
            pf[2 * mt + e / 8][e % 8 + 1] = pq[1];
          } else {
            pf[2 * mt + e / 8][e % 8] = (__bf16)p0;
            pf[2 * mt + e / 8][e % 8 + 1] = (__bf16)p1;
          }
        }
      rs = swap_halves_sum(rs);
      if (rescale) {
        const float corr = fast_exp2(m_run - m_new);   // 0 on the first tile
        l_run *= corr;
        m_run = m_new;
        const float corr_o = FP8V ? corr * (sv_prev / sv) : corr;   // FP8V: also from the last tile's V scale to this one's
        sv_prev = sv;
#pragma unroll
        for (int et = 0; et < ET; et++)
#pragma unroll
          for (int e = 0; e < 16; e++) oacc[et][e] *= corr_o;
      }
      l_run += rs;

      if constexpr (!DENSE) __builtin_amdgcn_s_setprio(2);   // matrix products again
      if constexpr (!DENSE) {
        if constexpr (kManual) {
          // the register loads issued at the top have landed; the tile transfer may still be in flight
          if (s + 1 < ntiles) wait_vmcnt<kDmaOps>();
          else wait_vmcnt<0>();
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) {
#pragma unroll
            for (int ks = 0; ks < kTileTokens / 16; ks++) settle(kphi[a][ks]);
            settle(zj[a]);
          }
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) zsel[a] += zj[a];
        }
      }
      if constexpr (FP8V) {
        // O^T += Vhat^T Ptilde^T as 64-deep FP8 products, one per 32-channel tile: the operand is the half
        // row (l / 32) of channel row 32 et + l % 32 of the code tile, two 16-byte reads
        typedef SwizzledLayoutVq<D> SLV;
        const unsigned qa = vqbuf(buf) + SLV::offset(lane % 32, 2 * g);
        u32x4 vq_lo[ET], vq_hi[ET];
#pragma unroll
        for (int et = 0; et < ET; et++) {
          vq_lo[et] = lds_read16_untracked_at<32 * kTileTokens>(qa, et);
          vq_hi[et] = lds_read16_untracked_at<32 * kTileTokens>(qa ^ 16u, et);
        }
#pragma unroll
        for (int et = 0; et < ET; et++) {
          wait_lgkmcnt(2 * (ET - 1 - et));
          settle(vq_lo[et]);
          settle(vq_hi[et]);
          const u32x4 lo = vq_lo[et], hi = vq_hi[et];
          const i32x8 a = {(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
          oacc[et] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, pb, oacc[et], 0, 0, 0, 0, 0, 0);
        }
      }
      // ---- O^T += V^T P^T, and the d x d state of this block: h += K^phi^T V ----
      if constexpr (!DENSE && HS::kNtw == ET) {        // every V fragment feeds both products
        // fragment f = ks ET + et: two transposing reads (tokens 16 ks + 4 g.. and + 8), kept kVAhead fragments ahead of the
        // products; (ks, et) sits at (address of the first) ^ 64 et, + 32 D ks.
        constexpr int kVAhead = 2, kFrags = (kTileTokens / 16) * ET;
        const unsigned va = lds_address(vt + SL::offset(4 * g + (lane % 16) / 4, 16 * ((lane / 16) % 2) + 4 * (lane % 4)));
        u32x2 vlo[kVAhead + 1], vhi[kVAhead + 1];
        auto read_v = [&](int f) {
          vlo[f % (kVAhead + 1)] = lds_read_tr_untracked_at<16 * D>(va ^ (64u * (f % ET)), 2 * (f / ET));
          vhi[f % (kVAhead + 1)] = lds_read_tr_untracked_at<16 * D>(va ^ (64u * (f % ET)), 2 * (f / ET) + 1);
        };
#pragma unroll
        for (int f = 0; f < kVAhead; f++) read_v(f);
#pragma unroll
        for (int f = 0; f < kFrags; f++) {
          if (f + kVAhead < kFrags) read_v(f + kVAhead);
          const int ks = f / ET, et = f % ET, left = kFrags - 1 - f;
          wait_lgkmcnt(2 * (left < kVAhead ? left : kVAhead));
          u32x2 &lo = vlo[f % (kVAhead + 1)], &hi = vhi[f % (kVAhead + 1)];
          settle(lo);
          settle(hi);
          const u32x4 v4 = {lo[0], lo[1], hi[0], hi[1]};
          const bf16x8 vf = __builtin_bit_cast(bf16x8, v4);
          if constexpr (!FP8V) oacc[et] = mfma_bf16(vf, pf[ks], oacc[et]);
#pragma unroll
          for (int a = 0; a < HS::kMtw; a++) hacc[a][et] = mfma_bf16(kphi[a][ks], vf, hacc[a][et]);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < kTileTokens / 16; ks++) {
#pragma unroll
          for (int et = 0; et < ET; et++) {
            bf16x8 vf = v_fragment<SL>(vt, ks, 32 * et, lane);
            if constexpr (!FP8V) oacc[et] = mfma_bf16(vf, pf[ks], oacc[et]);
          }
          if constexpr (!DENSE) {
#pragma unroll
            for (int b = 0; b < HS::kNtw; b++) {
              bf16x8 vf = v_fragment<SL>(vt, ks, 32 * (nt0 + b), lane);
#pragma unroll
              for (int a = 0; a < HS::kMtw; a++) hacc[a][b] = mfma_bf16(kphi[a][ks], vf, hacc[a][b]);
            }
          }
        }
      }
      __builtin_amdgcn_s_waitcnt(kVmcnt0);             // the next tile has landed in LDS ...
      __syncthreads();                                 // ... for everyone, and this tile's buffer is free
    }
  }

  if constexpr (!DENSE) __builtin_amdgcn_s_setprio(0);
  // ================= epilogue =================
  const float inv_l = l_run > 0.f ? 1.f / l_run : 0.f;
  const int qrow = 32 * w + lane % 32;               // this lane's query row inside the block
  if (!DENSE && (!PIPE || !FP8 || ntiles == 0)) {
    if constexpr (FP8) {
      dma_q(q_again(0));
      wait_vmcnt<0>();
      u32x4 raw[KS];
      const unsigned at = q_lane(q_again(0), g);
#pragma unroll
      for (int ks = 0; ks < KS; ks++) raw[ks] = read_q(at, 2 * ks);
      wait_lgkmcnt(0);
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        settle(raw[ks]);
        qf[ks] = __builtin_bit_cast(bf16x8, raw[ks]);
      }
    }
    q_max();
#pragma unroll
    for (int ks = 0; ks < KS; ks++) q_exp(ks);
    __syncthreads();                                 // the rows have left LDS
  }
  uint16_t* ht = reinterpret_cast<uint16_t*>(smem);  // H_i^T as bf16 [e][c], row stride LD
  uint16_t* os = ht + D * LD;                        // output tile [BQ][LD]
  float* zs = reinterpret_cast<float*>(smem + SM::kZsOff);   // Z_i
  f32x16 lacc[ET];
  float inv_den = 0.f;
  if constexpr (!DENSE) {
    // H_i^T = -(accumulated)^T as bf16, Z_i likewise
#pragma unroll
    for (int a = 0; a < HS::kMtw; a++) {
#pragma unroll
      for (int b = 0; b < (GIVEN ? 0 : HS::kNtw); b++) {
        const int e_col = 32 * (nt0 + b) + lane % 32;
#pragma unroll
        for (int v4 = 0; v4 < 4; v4++) {
          const int cc = 32 * (mt0 + a) + 8 * v4 + 4 * g;
          bf16x4 pk;
#pragma unroll
          for (int r = 0; r < 4; r++) pk[r] = (__bf16)(-hacc[a][b][4 * v4 + r]);
          *reinterpret_cast<bf16x4*>(ht + e_col * LD + cc) = pk;
        }
      }
      // zsel holds the same sum on both lane halves (each half added z_j of channel l % 32)
      if (g == 0 && nt0 == 0) {
        const int c = 32 * (mt0 + a) + lane;
        const float z = -zsel[a];
        if (z_save != nullptr) z_save[((size_t)bh * Tm + i) * D + c] = z;
        zs[c] = z;
      }
    }
    if constexpr (GIVEN) {
#pragma unroll
      for (int x = 0; x < kGivenLoads; x++) {
        const int n = w * kGivenLoads + x, t = n / 2;  // kilobyte of the slot, tile of h
        const bf16x8 y = __builtin_bit_cast(bf16x8, hgiven[x]);
        uint16_t* dst = ht + (32 * (t % ET) + lane % 32) * LD + 32 * (t / ET) + 16 * (n % 2) + 4 * g;
        *reinterpret_cast<bf16x4*>(dst) = bf16x4{y[0], y[1], y[2], y[3]};
        *reinterpret_cast<bf16x4*>(dst + 8) = bf16x4{y[4], y[5], y[6], y[7]};
      }
    }
    __syncthreads();                                 // H_i^T and Z_i visible
    // Q^phi Z_i in fp32 from the un-rounded Q^phi, in four sums side by side, and O_l^T = H_i^T Q^phi^T.  The denominator
    // is no matrix product (Z_i in three bf16 parts against the fragments of Q^phi): that rounds the weights, each by up
    // to 2^-8 of itself, and where they round to one side the output is off by as much (1.2e-3 in the mean on rows of
    // two weights).  It would save nothing either: 8 products of 33 cycles against 64 multiply-adds of 4, and the times
    // of both are equal (12 heads of 32,760 tokens, FP8: 443.6 us with the product, 443.0 us so).
    f32x4 den4 = {0.f, 0.f, 0.f, 0.f};
    const float* zlane = zs + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const f32x4 z4 = *reinterpret_cast<const f32x4*>(zlane + 16 * ks + 4 * x);
#pragma unroll
        for (int e = 0; e < 4; e++) {
          den4[e] += qx[ks][x][e] * z4[e];
          qf[ks][4 * x + e] = (__bf16)qx[ks][x][e];
        }
      }
    const float den = swap_halves_sum((den4[0] + den4[1]) + (den4[2] + den4[3]));
#pragma unroll
    for (int et = 0; et < ET; et++)
#pragma unroll
      for (int e = 0; e < 16; e++) lacc[et][e] = 0.f;
    const uint16_t* hrow = ht + (lane % 32) * LD + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int et = 0; et < ET; et++)
        lacc[et] = mfma_bf16(*reinterpret_cast<const bf16x8*>(hrow + 32 * et * LD + 16 * ks), qf[ks], lacc[et]);
    inv_den = ksel >= Tn ? 0.f : 1.f / den;          // every block selected: nothing left for the linear branch
  }
  // ---- mix (Eq. 13), transpose through LDS, coalesced store ----
  const float ws = al * inv_l * (FP8V ? sv_prev : 1.f), wl = (1.f - al) * inv_den;   // FP8V: back from the last tile's V scale
#pragma unroll
  for (int et = 0; et < ET; et++)
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      bf16x4 pk;
#pragma unroll
      for (int r = 0; r < 4; r++) {
        float o = ws * oacc[et][4 * v4 + r];
        if constexpr (!DENSE) o += wl * lacc[et][4 * v4 + r];
        pk[r] = (__bf16)o;
      }
      *reinterpret_cast<bf16x4*>(os + qrow * LD + 32 * et + 8 * v4 + 4 * g) = pk;
    }
  wave_lds_fence();                                  // (a wave stores the 32 rows that it wrote itself: no barrier)
  uint16_t* oh = out + head_offset(sout, bh, H) + (size_t)row0 * sout.n;
#pragma unroll
  for (int x = 0; x < D / 16; x++) {
    const int r = 32 * w + (x * kWave + lane) / (D / 8), ch = lane % (D / 8);
    if (r < rows_valid) store_streamed(reinterpret_cast<u32x4*>(oh + (size_t)r * sout.n + 8 * ch), *reinterpret_cast<const u32x4*>(os + r * LD + 8 * ch));
  }
  if constexpr (!DENSE) {
    if (h_save != nullptr) {
      // H_i^T (bf16 [e][c], as the product above consumed it) and Z_i, kept for the backward pass
      uint16_t* dst = h_save + ((size_t)bh * Tm + i) * D * D;
      for (int idx = tid; idx < D * (D / 8); idx += NT) {
        const int e = idx / (D / 8), ch = idx % (D / 8);
        store_streamed(reinterpret_cast<u32x4*>(dst + e * D + 8 * ch), *reinterpret_cast<const u32x4*>(ht + e * LD + 8 * ch));
      }
    }
  }
  if (o_s_save != nullptr) {
    // O^s (and O^l, if asked for) on its own ([BH, N, d] contiguous), kept for the backward pass: same
    // route through the transposing tile as the mixed output
    for (int which = 0; which < (o_l_save != nullptr ? 2 : 1); which++) {
      wave_lds_fence();                              // the tile has been read out
#pragma unroll
      for (int et = 0; et < ET; et++)
#pragma unroll
        for (int v4 = 0; v4 < 4; v4++) {
          bf16x4 pk;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            float o = which == 0 ? oacc[et][4 * v4 + r] * inv_l * (FP8V ? sv_prev : 1.f) : 0.f;
            if constexpr (!DENSE) {
              if (which == 1) o = lacc[et][4 * v4 + r] * inv_den;
            }
            pk[r] = (__bf16)o;
          }
          *reinterpret_cast<bf16x4*>(os + qrow * LD + 32 * et + 8 * v4 + 4 * g) = pk;
        }
      wave_lds_fence();
      uint16_t* dst = (which == 0 ? o_s_save : o_l_save) + ((size_t)bh * N + row0) * D;
#pragma unroll
      for (int x = 0; x < D / 16; x++) {
        const int r = 32 * w + (x * kWave + lane) / (D / 8), ch = lane % (D / 8);
        if (r < rows_valid) store_streamed(reinterpret_cast<u32x4*>(dst + (size_t)r * D + 8 * ch), *reinterpret_cast<const u32x4*>(os + r * LD + 8 * ch));
      }
    }
  }
  if (lse != nullptr || lse_save != nullptr) {
    // Alg. 2 defines L on the smoothed keys.  The bf16 products use the raw K, whose scores are larger by
    // q . colmean(K) / sqrt(d) in every column of a row (the softmax cancels it); the low-bit codes are those of
    // the smoothed K already.  (The rows are read again: the fragments hold Q^phi by now.)
    float qmu = 0.f;
    if constexpr (!DENSE && !FP8) {
      const uint16_t* src = qh + (size_t)(row0 + min(qrow, rows_valid - 1)) * tok_stride + 8 * g;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(src + 16 * ks);
#pragma unroll
        for (int e = 0; e < 8; e++) qmu += (float)x[e] * (float)k_mean[(size_t)bh * D + 16 * ks + 8 * g + e];
      }
      qmu = swap_halves_sum(qmu);
    }
    if (g == 0 && qrow < rows_valid) {
      const float L =
          l_run > 0.f ? (m_run - kPShift + __log2f(l_run)) * 0.6931471805599453f - qmu * rsqrtf((float)D) : -INFINITY;
      if (lse != nullptr) lse[(size_t)bh * N + row0 + qrow] = L;
      if (lse_save != nullptr) lse_save[(size_t)bh * N + row0 + qrow] = L;
    }
  }
}

struct AttnArgs {
  const uint16_t *q, *k, *v;
  const double* k_mean;
  const uint16_t* k_phi;
  const float* z_blocks;
  const uint8_t* k_fp8;
  const float* k_scale;
  const uint8_t* v_codes;
  const float *v_scale, *h_frag, *z_total;
  const int32_t* block_idx;
  const float* alpha;
  uint16_t* out;
  float* lse;
  SavedForBackward sv;
};

template <int D, int BQ, int MODE, bool PIPE, bool GIVEN = false>
static hipError_t launch_attn_loop(const Shape& s, const AttnArgs& a, hipStream_t stream) {
  constexpr int smem = AttnSmem<D, BQ, MODE == kSparseFp8 || MODE == kSparseInt8 || MODE == kSparseFp8V, MODE == kSparseFp8V, PIPE, GIVEN>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)attn_mfma_kernel<D, BQ, MODE, PIPE, GIVEN>, smem); e != hipSuccess) return e;
  const int Tm = (s.N + BQ - 1) / BQ;
  const int grid = ((Tm + kXcds - 1) / kXcds) * kXcds * s.BH;   // some workgroups of the last run of a head may have no block
  attn_mfma_kernel<D, BQ, MODE, PIPE, GIVEN><<<dim3((unsigned)grid), BQ * 2, smem, stream>>>(
      a.q, a.k, a.v, a.k_mean, a.k_phi, a.z_blocks, a.k_fp8, a.k_scale, a.v_codes, a.v_scale, a.h_frag, a.z_total,
      a.block_idx, a.alpha,
      a.out, a.lse, (uint16_t*)a.sv.o_s, (uint16_t*)a.sv.o_l, a.sv.lse, (uint16_t*)a.sv.h_i, a.sv.z_i, s.sin, s.sout, s.H, s.N, Tm, s.Tn, s.k,
      s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

template <int D, int BQ, int MODE>
static hipError_t launch_attn_t(const Shape& s, const AttnArgs& a, hipStream_t stream) {
  if constexpr (D == 128 && BQ == 128 && MODE != kDenseBf16)
    if (s.state_heads > 0) return launch_attn_loop<D, BQ, MODE, true, true>(s, a, stream);
  if constexpr (kPlainToo<D, BQ, MODE>)
    if (s.k * s.Tn > kPipelinedTiles) return launch_attn_loop<D, BQ, MODE, false>(s, a, stream);   // below 2^22
  return launch_attn_loop<D, BQ, MODE, kPipelined<D, BQ, MODE>>(s, a, stream);
}

hipError_t launch_attn_bf16(const Shape& s, const uint16_t* q, const uint16_t* k, const uint16_t* v,
                            const double* k_mean, const uint16_t* k_phi, const float* z_blocks, const uint8_t* k_fp8,
                            const float* k_scale, const uint8_t* v_codes, const float* v_scale,
                            const float* h_frag, const float* z_total,
                            const int32_t* block_idx, const float* alpha, uint16_t* out, float* lse,
                            const SavedForBackward& sv, hipStream_t stream) {
  AttnArgs a{q, k, v, k_mean, k_phi, z_blocks, k_fp8, k_scale, v_codes, v_scale, h_frag, z_total, block_idx, alpha, out, lse, sv};
#define SLA2_ATTN(DD, QQ)                                                  \
  return s.quant == 3 ? launch_attn_t<DD, QQ, kSparseFp8V>(s, a, stream)   \
       : s.quant == 2 ? launch_attn_t<DD, QQ, kSparseInt8>(s, a, stream)   \
       : s.quant == 1 ? launch_attn_t<DD, QQ, kSparseFp8>(s, a, stream)    \
                      : launch_attn_t<DD, QQ, kSparseBf16>(s, a, stream)
  if (s.d == 128 && s.bq == 128) SLA2_ATTN(128, 128);
  if (s.d == 128 && s.bq == 64) SLA2_ATTN(128, 64);
  if (s.d == 64 && s.bq == 128) SLA2_ATTN(64, 128);
  SLA2_ATTN(64, 64);
#undef SLA2_ATTN
}

hipError_t launch_dense_bf16(const Shape& s, const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out,
                             hipStream_t stream) {
  AttnArgs a{q, k, v, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, out, nullptr,
             SavedForBackward{nullptr, nullptr, nullptr, nullptr, nullptr}};
  // d = 128: the kernel of its own in sla2_dense.hip (256 query rows per workgroup, the two waves of a SIMD
  // in opposite phases)
  if (s.d == 128) return launch_dense_pp(s, q, k, v, out, stream);
  return launch_attn_t<64, 128, kDenseBf16>(s, a, stream);
}

}  // namespace sla2
