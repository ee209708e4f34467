// fp32 path of the SLA2 forward pass (Alg. 2 of the paper), used when q, k, v are stored in fp32.  The data flow is the
// one of the bf16 / FP8 path - per-head totals of h_j, z_j first, then one pass per query block that runs the sparse
// branch over the selected key/value blocks, rebuilds the h_j, z_j of exactly those blocks, subtracts them from the
// totals, and mixes the two branches - in fp32 throughout: products on the fp32 matrix instruction (f32_tiles.h).
#include "f32_tiles.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// kv_state_f32: for a chunk of key blocks of one head
//   k' = k - colmean(K);  stats[token] = lnZ = log sum_c exp(k'_c);
//   K^phi = softmax_d(k');  partial h += (K^phi_j)^T V_j,  partial z += colsum(K^phi_j)
// (Alg. 2: K^phi, h, z).  Tokens past N contribute nothing.  A token's channels sit on neighbouring lanes, 4 each, so
// the softmax is taken in registers on the way into LDS.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void kv_state_f32_kernel(const float* __restrict__ k, const float* __restrict__ v,
                                                           const double* __restrict__ k_mean,
                                                           float* __restrict__ k_stats, float* __restrict__ partial,
                                                           Strides sin, int H, int N, int Tn, int chunks,
                                                           int blocks_per_chunk) {
  constexpr int LD = kF32Ld<D>;
  typedef ChunkMap<D, 256, kF32Tokens> CM;
  typedef StateSplit<D, 4> SS;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* kp = smem;                       // [64][LD]  K^phi tile
  float* vs = smem + kF32Tokens * LD;     // [64][LD]  V tile
  const int bh = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const float* kh = k + head_offset(sin, bh, H);
  const float* vh = v + head_offset(sin, bh, H);
  const int j0 = chunk * blocks_per_chunk, j1 = min(Tn, j0 + blocks_per_chunk);
  f32x4 mu;
#pragma unroll
  for (int x = 0; x < 4; x++) mu[x] = (float)k_mean[(size_t)bh * D + 4 * ch + x];

  f32x16 hacc[SS::kTiles];
#pragma unroll
  for (int x = 0; x < SS::kTiles; x++) hacc[x] = zero16();
  f32x4 zacc = {0.f, 0.f, 0.f, 0.f};
  f32x4 kr[CM::kLoads], vr[CM::kLoads];
  auto fetch = [&](int j) {
    const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
    CM::load(kr, kh + (size_t)t0 * sin.n, sin.n, valid, tid);
    CM::load(vr, vh + (size_t)t0 * sin.n, sin.n, valid, tid);
  };
  if (j0 < j1) fetch(j0);
  for (int j = j0; j < j1; j++) {
    const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
    __syncthreads();                      // previous tile fully consumed
#pragma unroll
    for (int i = 0; i < CM::kLoads; i++) {
      const int t = trow + i * CM::kRows;
      const bool ok = t < valid;
      f32x4 x = kr[i] - mu;
      const float m = CM::row_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      f32x4 e;
#pragma unroll
      for (int c = 0; c < 4; c++) e[c] = exp2_f32((x[c] - m) * kLog2e);
      const float sum = CM::row_sum((e[0] + e[1]) + (e[2] + e[3]));
      const float inv = ok ? 1.f / sum : 0.f;
      e *= inv;
      zacc += e;
      *reinterpret_cast<f32x4*>(kp + t * LD + 4 * ch) = e;
      *reinterpret_cast<f32x4*>(vs + t * LD + 4 * ch) = vr[i];
      if (ok && ch == 0) k_stats[(size_t)bh * N + t0 + t] = m + __log2f(sum) * kLn2;
    }
    if (j + 1 < j1) fetch(j + 1);
    __syncthreads();
    state_product<D, 4>(hacc, kp, vs, kF32Tokens, w, lane);
  }
  float* ph = partial + (size_t)blockIdx.x * (D * D + D);
#pragma unroll
  for (int x = 0; x < SS::kTiles; x++)
#pragma unroll
    for (int e = 0; e < 16; e++)
      ph[(32 * SS::mt(w) + 8 * (e / 4) + 4 * g + e % 4) * D + 32 * (SS::nt(w) + x) + lane % 32] = hacc[x][e];
  __syncthreads();                        // the last tile fully consumed: its place takes the column sums
  *reinterpret_cast<f32x4*>(kp + trow * D + 4 * ch) = zacc;
  __syncthreads();
  if (tid < D) {
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < CM::kRows; r++) z += kp[r * D + tid];
    ph[D * D + tid] = z;
  }
}

// Totals over the chunks of a head (Alg. 2's sums of h_j and z_j over all key blocks).  A thread owns 4 consecutive entries
// of the partial sums; the 8 waves of a workgroup walk the chunks 8 apart and meet in LDS, always in the same
// order, so the totals are the same bits on every run.  Bound by the start of the launch and one pass over the partial sums
// (33 MB for 12 heads of 32k tokens).
// FRAG: the h part of the partial sums lies as accumulator fragments (kv_state_bf16): [d/32 (c)][d/32 (e)][4][64 lanes][4],
// lane l of part x holding rows c = 8 x + 4 (l / 32) + 0..3 of column e = l % 32; h_frag takes -h_total in the same order, which
// is what the accumulators of the attention kernel start from.
constexpr int kTotalWaves = 8;
template <bool FRAG>
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
    } else if (!FRAG) {
      *reinterpret_cast<f32x4*>(h_total + (size_t)bh * d * d + e) = s;
    } else {
      *reinterpret_cast<f32x4*>(h_frag + (size_t)bh * d * d + e) = -s;
      const int tile = e / 1024, x = e / 256 % 4, lane = e / 4 % 64;
      const int row = 32 * (tile / (d / 32)) + 8 * x + 4 * (lane / 32), col = 32 * (tile % (d / 32)) + lane % 32;
      for (int r = 0; r < 4; r++) h_total[((size_t)bh * d + row + r) * d + col] = s[r];
    }
  }
}

hipError_t launch_kv_total(const Shape& s, const float* partial, float* h_total, float* z_total, float* h_frag, hipStream_t stream) {
  const dim3 grid((unsigned)((s.d * s.d + s.d + 255) / 256), (unsigned)s.BH);
  if (s.bf16) kv_total_kernel<true><<<grid, 64 * kTotalWaves, 0, stream>>>(partial, h_total, z_total, h_frag, s.d, s.chunks);
  else kv_total_kernel<false><<<grid, 64 * kTotalWaves, 0, stream>>>(partial, h_total, z_total, nullptr, s.d, s.chunks);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_kv_state_f32_t(const Shape& s, const float* k, const float* v, const double* k_mean, float* k_stats,
                                        float* partial, hipStream_t stream) {
  constexpr int smem = 2 * kF32Tokens * kF32Ld<D> * (int)sizeof(float);
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)kv_state_f32_kernel<D>, smem); e != hipSuccess) return e;
  kv_state_f32_kernel<D><<<dim3((unsigned)(s.BH * s.chunks)), 256, smem, stream>>>(k, v, k_mean, k_stats, partial, s.sin, s.H, s.N,
                                                                                s.Tn, s.chunks, s.blocks_per_chunk);
  return hipGetLastError();
}
hipError_t launch_kv_state_f32(const Shape& s, const float* k, const float* v, const double* k_mean, float* k_stats,
                               float* partial, hipStream_t stream) {
  return s.d == 128 ? launch_kv_state_f32_t<128>(s, k, v, k_mean, k_stats, partial, stream)
                    : launch_kv_state_f32_t<64>(s, k, v, k_mean, k_stats, partial, stream);
}

// ---------------------------------------------------------------------------------------------
// attn_f32: one workgroup per query block i, BQ / 16 waves.
//   sparse branch  : for j in sel(i), ascending: S^T = K'_j Q_i^T / sqrt(d), online softmax, O^T += V_j^T P^T
//   linear branch  : H_i = H_total - sum_{j in sel(i)} h_j (h_j rebuilt from the staged tiles and the
//                    per-token log-partition lnZ), Z_i likewise; O_l^T = H_i^T Q^phi^T
//   mix            : out = alpha O_s / l + (1 - alpha) O_l                                   (Eq. 13)
// Wave (rg, kh) owns query rows 32 rg.. and, in the sparse branch, keys 32 kh.. of every tile: the two waves of a row
// group keep running maxima of their own and meet once, after the loop, like two halves of a split softmax.  A lane owns
// one query row, so its probabilities feed O^T += V^T P^T from registers.  The bound is the fp32 matrix rate: on 12 heads
// of 4,096 tokens (d = 128, 10 % kept) 12 GFLOP.
// ---------------------------------------------------------------------------------------------
template <int D, int BQ> struct AttnF32Smem {
  static constexpr int NW = BQ / 16, NT = NW * kWave;
  static constexpr int kTile = kF32Tokens * kF32Ld<D>;                     // floats
  static constexpr int kState = D * kF32Ld<D>;                             // H_i, over the K' and K^phi tiles
  static_assert(kState <= 2 * kTile, "H_i takes the place of the K' and K^phi tiles");
  static constexpr int kSwap = NW * (D / 64) * 16 * kWave;                 // half of every wave's O^T tiles
  static constexpr int kSwapOff = 2 * kTile;                               // over the V tile and behind it
  static constexpr int kZred = NT * 4;                                     // column sums of K^phi, before the swap
  static constexpr int kBig = kTile > kSwap ? (kTile > kZred ? kTile : kZred) : (kSwap > kZred ? kSwap : kZred);
  static constexpr int kMlOff = kSwapOff + kBig;                           // [NW][2][32] m and l
  static constexpr int kZsOff = kMlOff + NW * 64;                          // [D] Z_i
  static constexpr int kBytes = (kZsOff + D) * (int)sizeof(float);
};

template <int D, int BQ>
__global__ __launch_bounds__(BQ * 4, BQ / 64) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const double* __restrict__ k_mean,
    const float* __restrict__ k_stats, const float* __restrict__ h_total, const float* __restrict__ z_total,
    const int32_t* __restrict__ block_idx, const float* __restrict__ alpha, float* __restrict__ out, float* __restrict__ lse,
    float* __restrict__ o_s_save, float* __restrict__ o_l_save, float* __restrict__ lse_save, float* __restrict__ h_save,
    float* __restrict__ z_save, Strides sin, Strides sout, int H, int N, int Tm, int Tn, int ksel, int alpha_per_block) {
  typedef AttnF32Smem<D, BQ> SM;
  constexpr int NW = SM::NW, NT = SM::NT, LD = kF32Ld<D>, ET = D / 32, J = D / 8;
  typedef ChunkMap<D, NT, kF32Tokens> CM;
  typedef StateSplit<D, NW> SS;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* ks = smem;                       // [64][LD]  K' tile
  float* kp = smem + SM::kTile;           // [64][LD]  K^phi tile
  float* vs = smem + 2 * SM::kTile;       // [64][LD]  V tile
  float* hs = smem;                       // [D][LD]   H_i
  float* swap = smem + SM::kSwapOff;
  float* ml = smem + SM::kMlOff;
  float* zs = smem + SM::kZsOff;

  const int i = blockIdx.x % Tm, bh = blockIdx.x / Tm, h = bh % H;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int rg = w >> 1, kh = w & 1;
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const int row0 = i * BQ, rows_valid = min(BQ, N - row0);
  const int qrow = 32 * rg + lane % 32;
  const bool row_ok = qrow < rows_valid;
  const float* kh_ = k + head_offset(sin, bh, H);
  const float* vh = v + head_offset(sin, bh, H);
  const int32_t* sel = block_idx + ((size_t)bh * Tm + i) * ksel;

  f32x4 kr[CM::kLoads], vr[CM::kLoads];
  float zr[CM::kLoads];
  auto fetch = [&](int j) {
    const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
    CM::load(kr, kh_ + (size_t)t0 * sin.n, sin.n, valid, tid);
    CM::load(vr, vh + (size_t)t0 * sin.n, sin.n, valid, tid);
#pragma unroll
    for (int x = 0; x < CM::kLoads; x++) zr[x] = k_stats[(size_t)bh * N + t0 + min(trow + x * CM::kRows, valid - 1)];
  };
  if (ksel > 0) fetch(sel[0]);
  f32x4 qf[J];                            // this lane's query row, channels 8 j + 4 g ..
  {
    const float* src = q + head_offset(sin, bh, H) + (size_t)(row0 + min(qrow, rows_valid - 1)) * sin.n + 4 * g;
#pragma unroll
    for (int j = 0; j < J; j++) qf[j] = *reinterpret_cast<const f32x4*>(src + 8 * j);
  }
  f32x4 mu;
#pragma unroll
  for (int x = 0; x < 4; x++) mu[x] = (float)k_mean[(size_t)bh * D + 4 * ch + x];

  f32x16 oacc[ET], hacc[SS::kTiles];
#pragma unroll
  for (int e = 0; e < ET; e++) oacc[e] = zero16();
#pragma unroll
  for (int x = 0; x < SS::kTiles; x++) hacc[x] = zero16();
  f32x4 zacc = {0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;   // this lane's row over this wave's keys, log2 domain
  const float c0 = kLog2e * rsqrtf((float)D);

  for (int s = 0; s < ksel; s++) {
    const int valid = min(kF32Tokens, N - sel[s] * kF32Tokens);
    __syncthreads();                      // previous tile fully consumed
#pragma unroll
    for (int x = 0; x < CM::kLoads; x++) {
      const int t = trow + x * CM::kRows;
      const bool ok = t < valid;
      f32x4 a = kr[x] - mu, e;
#pragma unroll
      for (int c = 0; c < 4; c++) e[c] = ok ? exp2_f32((a[c] - zr[x]) * kLog2e) : 0.f;
      zacc += e;
      *reinterpret_cast<f32x4*>(ks + t * LD + 4 * ch) = a;
      *reinterpret_cast<f32x4*>(kp + t * LD + 4 * ch) = e;
      *reinterpret_cast<f32x4*>(vs + t * LD + 4 * ch) = vr[x];   // rows past the end: finite, weighted with 0
    }
    if (s + 1 < ksel) fetch(sel[s + 1]);
    __syncthreads();
    f32x16 sacc = channel_product<D>(ks + (32 * kh + lane % 32) * LD, qf, zero16(), g);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const bool ok = 32 * kh + 8 * (e / 4) + 4 * g + e % 4 < valid;
      sacc[e] = ok ? sacc[e] * c0 : -INFINITY;
      mx = fmaxf(mx, sacc[e]);
    }
    mx = both_halves_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;        // no key of this half seen yet (short last block)
    const float corr = exp2_f32(m_run - m_ref);
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      sacc[e] = exp2_f32(sacc[e] - m_ref);
      rs += sacc[e];
    }
    l_run = l_run * corr + both_halves_sum(rs);
    m_run = m_new;
#pragma unroll
    for (int et = 0; et < ET; et++) oacc[et] *= corr;
    const float* va = vs + (32 * kh + 4 * g) * LD + lane % 32;
#pragma unroll
    for (int e = 0; e < 16; e++)
#pragma unroll
      for (int et = 0; et < ET; et++) oacc[et] = mfma_f32(va[(8 * (e / 4) + e % 4) * LD + 32 * et], sacc[e], oacc[et]);
    if (SS::active(w)) state_product<D, NW>(hacc, kp, vs, kF32Tokens, w, lane);
  }
  __syncthreads();

  // ---- H_i = H_total - sum, Z_i likewise; the two key halves exchange m and l ----
  if (SS::active(w)) {
    const float* ht = h_total + (size_t)bh * D * D;
    float* hsv = h_save != nullptr ? h_save + ((size_t)bh * Tm + i) * D * D : nullptr;
#pragma unroll
    for (int x = 0; x < SS::kTiles; x++)
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int c = 32 * SS::mt(w) + 8 * (e / 4) + 4 * g + e % 4, col = 32 * (SS::nt(w) + x) + lane % 32;
        const float y = ht[c * D + col] - hacc[x][e];
        hs[c * LD + col] = y;
        if (hsv != nullptr) hsv[c * D + col] = y;
      }
  }
  *reinterpret_cast<f32x4*>(swap + trow * D + 4 * ch) = zacc;
  if (g == 0) {
    ml[w * 64 + lane] = m_run;
    ml[w * 64 + 32 + lane] = l_run;
  }
  __syncthreads();
  if (tid < D) {
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < CM::kRows; r++) z += swap[r * D + tid];
    z = z_total[(size_t)bh * D + tid] - z;
    zs[tid] = z;
    if (z_save != nullptr) z_save[((size_t)bh * Tm + i) * D + tid] = z;
  }
  const float m_o = ml[(w ^ 1) * 64 + lane % 32], l_o = ml[(w ^ 1) * 64 + 32 + lane % 32];
  const float m_all = fmaxf(m_run, m_o), m_ref = m_all == -INFINITY ? 0.f : m_all;
  const float mine = exp2_f32(m_run - m_ref), l = l_run * mine + l_o * exp2_f32(m_o - m_ref);
#pragma unroll
  for (int et = 0; et < ET; et++) oacc[et] *= mine;
  // Q^phi = softmax_d(Q) of this lane's row
  float qm = -INFINITY;
#pragma unroll
  for (int j = 0; j < J; j++)
#pragma unroll
    for (int x = 0; x < 4; x++) qm = fmaxf(qm, qf[j][x]);
  qm = both_halves_max(qm);
  float qs = 0.f;
#pragma unroll
  for (int j = 0; j < J; j++)
#pragma unroll
    for (int x = 0; x < 4; x++) {
      qf[j][x] = exp2_f32((qf[j][x] - qm) * kLog2e);
      qs += qf[j][x];
    }
  const float qinv = 1.f / both_halves_sum(qs);
#pragma unroll
  for (int j = 0; j < J; j++) qf[j] *= qinv;
  __syncthreads();                        // Z_i visible, the column sums have been read
  float den = 0.f;
#pragma unroll
  for (int j = 0; j < J; j++) {
    const f32x4 z = *reinterpret_cast<const f32x4*>(zs + 8 * j + 4 * g);
#pragma unroll
    for (int x = 0; x < 4; x++) den += qf[j][x] * z[x];
  }
  den = both_halves_sum(den);
  const bool all_selected = ksel >= Tn;   // nothing left for the linear branch: O_l = 0
  const float inv_l = l > 0.f ? 1.f / l : 0.f, inv_den = all_selected ? 0.f : 1.f / den;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];

  // Each of the two waves of a row group finishes half of the channel tiles: it hands the other half of its O^T over.
  float* mine_out = swap + (size_t)w * (ET / 2) * 16 * kWave + lane;
  const float* other = swap + (size_t)(w ^ 1) * (ET / 2) * 16 * kWave + lane;
  auto finish = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2), F0 = ET / 2 - E0;      // own tiles, tiles handed over
#pragma unroll
    for (int x = 0; x < ET / 2; x++)
#pragma unroll
      for (int e = 0; e < 16; e++) mine_out[(x * 16 + e) * kWave] = oacc[F0 + x][e];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < ET / 2; x++) {
      constexpr int et0 = E0;
      const int et = et0 + x;
#pragma unroll
      for (int e = 0; e < 16; e++) oacc[et][e] += other[(x * 16 + e) * kWave];
      f32x16 lacc = zero16();
      const float* ha = hs + 4 * g * LD + 32 * et + lane % 32;
#pragma unroll
      for (int j = 0; j < J; j++)
#pragma unroll
        for (int y = 0; y < 4; y++) lacc = mfma_f32(ha[(8 * j + y) * LD], qf[j][y], lacc);
      if (row_ok) {
        float* o = out + head_offset(sout, bh, H) + (size_t)(row0 + qrow) * sout.n + 32 * et + 4 * g;
        const size_t at = ((size_t)bh * N + row0 + qrow) * D + 32 * et + 4 * g;
#pragma unroll
        for (int v4 = 0; v4 < 4; v4++) {
          f32x4 os, ol;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            os[r] = oacc[et][4 * v4 + r] * inv_l;
            ol[r] = lacc[4 * v4 + r] * inv_den;
          }
          *reinterpret_cast<f32x4*>(o + 8 * v4) = al * os + (1.f - al) * ol;
          if (o_s_save != nullptr) {      // the two branches, kept for the backward pass
            *reinterpret_cast<f32x4*>(o_s_save + at + 8 * v4) = os;
            *reinterpret_cast<f32x4*>(o_l_save + at + 8 * v4) = ol;
          }
        }
      }
    }
  };
  if (kh == 0) finish(std::integral_constant<int, 0>());
  else finish(std::integral_constant<int, 1>());
  if (kh == 0 && g == 0 && row_ok) {
    const float L = l > 0.f ? (m_all + __log2f(l)) * kLn2 : -INFINITY;
    if (lse != nullptr) lse[(size_t)bh * N + row0 + qrow] = L;
    if (lse_save != nullptr) lse_save[(size_t)bh * N + row0 + qrow] = L;
  }
}

template <int D, int BQ>
static hipError_t launch_attn_f32_t(const Shape& s, const float* q, const float* k, const float* v,
                                    const double* k_mean, const float* k_stats, const float* h_total,
                                    const float* z_total, const int32_t* block_idx, const float* alpha, float* out,
                                    float* lse, const SavedForBackward& sv, hipStream_t stream) {
  constexpr int smem = AttnF32Smem<D, BQ>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)attn_f32_kernel<D, BQ>, smem); e != hipSuccess) return e;
  attn_f32_kernel<D, BQ><<<dim3((unsigned)(s.BH * s.Tm)), BQ * 4, smem, stream>>>(
      q, k, v, k_mean, k_stats, h_total, z_total, block_idx, alpha, out, lse, (float*)sv.o_s, (float*)sv.o_l, sv.lse,
      (float*)sv.h_i, sv.z_i, s.sin, s.sout, s.H, s.N, s.Tm, s.Tn, s.k, s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_attn_f32(const Shape& s, const float* q, const float* k, const float* v, const double* k_mean,
                           const float* k_stats, const float* h_total, const float* z_total, const int32_t* block_idx,
                           const float* alpha, float* out, float* lse, const SavedForBackward& sv,
                           hipStream_t stream) {
#define SLA2_F32(DD, QQ) \
  return launch_attn_f32_t<DD, QQ>(s, q, k, v, k_mean, k_stats, h_total, z_total, block_idx, alpha, out, lse, sv, stream)
  if (s.d == 128 && s.bq == 128) SLA2_F32(128, 128);
  if (s.d == 128) SLA2_F32(128, 64);
  if (s.bq == 128) SLA2_F32(64, 128);
  SLA2_F32(64, 64);
#undef SLA2_F32
}

}  // namespace sla2
