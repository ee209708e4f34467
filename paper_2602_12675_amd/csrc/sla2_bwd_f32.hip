// The two heavy steps of the backward pass for fp32 tensors (Alg. 3 of the paper's appendix with the steps it leaves to
// automatic differentiation written out): products on the fp32 matrix instruction, everything fp32 (f32_tiles.h).
//
//   bwd_q_f32   one workgroup per query block i:  D^s, D^l, d alpha;  over the selected key blocks, scores transposed as
//               in the forward kernel (a lane owns a query row):  P^T = exp(S^T - L), dP^T = V dO^T,
//               dS^T = P^T (.) (alpha dP^T - D^s), dQ^T += K'^T dS^T;  then from the H_i, Z_i the forward pass kept
//               dQ^phi^T = ((1 - alpha) H_i dO^T - Z_i D^l^T) / (Q^phi Z_i), dQ += softmax-backward(dQ^phi),
//               dH_i = (1 - alpha) (Q^phi / (Q^phi Z_i))^T dO, dZ_i.
//   bwd_kv_f32  one workgroup per key block j, over the query blocks that selected it, 64 rows a step:  S = Q K'^T (a lane
//               owns a key), dV^T += dO^T (alpha P), dK'^T += Q^T dS;  then dH = dH_total - sum of those blocks' dH_i
//               (the M_c[i, j] = 0 sum of Alg. 3, by complement), dK^phi^T = dH V^T + dZ 1^T, dV^T += dH^T K^phi^T,
//               dK' += softmax-backward(dK^phi).
//
// The waves of a workgroup share the work as in the forward kernel: two waves own the same 32 query rows (keys) and one
// half of the contraction each - keys of a tile, query rows of a step - and add their results once, after the loop.
#include "f32_tiles.h"

namespace sla2 {

template <int D, int BQ> struct BwdQF32Smem {
  static constexpr int NW = BQ / 16, NT = NW * kWave, LD = kF32Ld<D>;
  static constexpr int kTile = kF32Tokens * LD;                            // floats
  // K' and V tiles; after the loop the swapped halves of dQ^T, then H_i, then w = Q^phi / (Q^phi Z_i)
  static constexpr int kSwap = NW * (D / 64) * 16 * kWave;
  static constexpr int kA0 = 2 * kTile > kSwap ? 2 * kTile : kSwap;
  static constexpr int kA1 = kA0 > D * LD ? kA0 : D * LD;
  static constexpr int kBig = kA1 > BQ * LD ? kA1 : BQ * LD;
  static constexpr int kDoOff = kBig;                                      // [BQ][LD] dO
  static constexpr int kRowOff = kDoOff + BQ * LD;                         // [2][BQ] dO . O^s and dO . O^l per row
  static constexpr int kDotOff = kRowOff + 2 * BQ;                         // [NW][32] halves of row sums
  static constexpr int kZsOff = kDotOff + NW * 32;                         // [D] Z_i
  static constexpr int kRedOff = kZsOff + D;                               // [NT]
  static constexpr int kBytes = (kRedOff + NT) * (int)sizeof(float);
  static_assert(kBytes <= 160 * 1024, "LDS of a CU");
};

template <int D, int BQ>
__global__ __launch_bounds__(BQ * 4, BQ / 64) void bwd_q_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ o_s, const float* __restrict__ o_l, const float* __restrict__ lse,
    const double* __restrict__ k_mean, const float* __restrict__ h_i, const float* __restrict__ z_i,
    const int32_t* __restrict__ block_idx, const float* __restrict__ alpha, float* __restrict__ dq, float* __restrict__ ds_out,
    float* __restrict__ l2_out, float* __restrict__ dh_out, float* __restrict__ dz_out, float* __restrict__ dalpha_part,
    Strides sin, Strides sout, int H, int N, int Tm, int Tn, int ksel, int alpha_per_block) {
  typedef BwdQF32Smem<D, BQ> SM;
  constexpr int NW = SM::NW, NT = SM::NT, LD = SM::LD, ET = D / 32, J = D / 8;
  typedef ChunkMap<D, NT, kF32Tokens> CM;
  typedef ChunkMap<D, NT, BQ> RM;
  typedef StateSplit<D, NW> SS;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* ks = smem;                       // [64][LD] K' tile
  float* vs = smem + SM::kTile;           // [64][LD] V tile
  float* hs = smem;                       // [D][LD]  H_i
  float* wt = smem;                       // [BQ][LD] w
  float* swap = smem;
  float* dos = smem + SM::kDoOff;
  float* rows = smem + SM::kRowOff;
  float* dots = smem + SM::kDotOff;
  float* zs = smem + SM::kZsOff;
  float* red = smem + SM::kRedOff;

  const int i = blockIdx.x % Tm, bh = blockIdx.x / Tm, h = bh % H;
  const size_t slot = (size_t)bh * Tm + i;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int rg = w >> 1, kh = w & 1;
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const int row0 = i * BQ, rows_valid = min(BQ, N - row0);
  const int qrow = 32 * rg + lane % 32;
  const bool row_ok = qrow < rows_valid;
  const float* kh_ = k + head_offset(sin, bh, H);
  const float* vh = v + head_offset(sin, bh, H);
  const int32_t* sel = block_idx + slot * ksel;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
  const float rscale = rsqrtf((float)D);

  f32x4 kr[CM::kLoads], vr[CM::kLoads];
  auto fetch = [&](int j) {
    const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
    CM::load(kr, kh_ + (size_t)t0 * sin.n, sin.n, valid, tid);
    CM::load(vr, vh + (size_t)t0 * sin.n, sin.n, valid, tid);
  };
  if (ksel > 0) fetch(sel[0]);
  f32x4 mu;
#pragma unroll
  for (int x = 0; x < 4; x++) mu[x] = (float)k_mean[(size_t)bh * D + 4 * ch + x];
  f32x4 qf[J];                            // this lane's query row, channels 8 j + 4 g ..
  {
    const float* src = q + head_offset(sin, bh, H) + (size_t)(row0 + min(qrow, rows_valid - 1)) * sin.n + 4 * g;
#pragma unroll
    for (int j = 0; j < J; j++) qf[j] = *reinterpret_cast<const f32x4*>(src + 8 * j);
  }
  {  // dO into LDS (zero rows past the end), dO . O^s and dO . O^l per row
    const float* doh = dout + head_offset(sout, bh, H) + (size_t)row0 * sout.n;
    const float* osh = o_s + ((size_t)bh * N + row0) * D;
    const float* olh = o_l + ((size_t)bh * N + row0) * D;
    float mix = 0.f;
#pragma unroll
    for (int x = 0; x < RM::kLoads; x++) {
      const int r = trow + x * RM::kRows, rc = min(r, rows_valid - 1);
      const float keep = r < rows_valid ? 1.f : 0.f;
      f32x4 go = *reinterpret_cast<const f32x4*>(doh + (size_t)rc * sout.n + 4 * ch);
      const f32x4 os = *reinterpret_cast<const f32x4*>(osh + (size_t)rc * D + 4 * ch);
      const f32x4 ol = *reinterpret_cast<const f32x4*>(olh + (size_t)rc * D + 4 * ch);
      go *= keep;
      *reinterpret_cast<f32x4*>(dos + r * LD + 4 * ch) = go;
      float s_s = 0.f, s_l = 0.f;
#pragma unroll
      for (int c = 0; c < 4; c++) {
        s_s += go[c] * os[c];
        s_l += go[c] * ol[c];
        mix += go[c] * (os[c] - ol[c]);
      }
      s_s = RM::row_sum(s_s);
      s_l = RM::row_sum(s_l);
      if (ch == 0) {
        rows[r] = s_s;
        rows[BQ + r] = s_l;
      }
    }
    red[tid] = mix;
  }
  __syncthreads();
  if (tid < kWave) {                      // d alpha: the sum over the block's tokens of dO . (O^s - O^l)
    float t = 0.f;
#pragma unroll
    for (int x = 0; x < NW; x++) t += red[tid + x * kWave];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) t += __shfl_xor(t, o);
    if (tid == 0) dalpha_part[slot] = t;
  }
  const float Ds = al * rows[qrow], Dl = (1.f - al) * rows[BQ + qrow];
  const float L2 = lse[(size_t)bh * N + row0 + min(qrow, rows_valid - 1)] * kLog2e;
  if (kh == 0 && g == 0) {                // as the key-side kernel uses them: rows past the end get exp2(-inf) = 0 there
    ds_out[slot * BQ + qrow] = row_ok ? Ds : 0.f;
    l2_out[slot * BQ + qrow] = row_ok ? L2 : INFINITY;
  }

  f32x16 dqacc[ET];
#pragma unroll
  for (int e = 0; e < ET; e++) dqacc[e] = zero16();
  const float c0 = kLog2e * rscale;
  for (int s = 0; s < ksel; s++) {
    const int valid = min(kF32Tokens, N - sel[s] * kF32Tokens);
    __syncthreads();                      // previous tile fully consumed
#pragma unroll
    for (int x = 0; x < CM::kLoads; x++) {
      const int t = trow + x * CM::kRows;
      *reinterpret_cast<f32x4*>(ks + t * LD + 4 * ch) = kr[x] - mu;
      *reinterpret_cast<f32x4*>(vs + t * LD + 4 * ch) = vr[x];
    }
    if (s + 1 < ksel) fetch(sel[s + 1]);
    __syncthreads();
    f32x16 ds = channel_product<D>(ks + (32 * kh + lane % 32) * LD, qf, zero16(), g);
    const f32x16 dp = channel_product<D>(vs + (32 * kh + lane % 32) * LD, dos + qrow * LD, zero16(), g);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const bool ok = row_ok && 32 * kh + 8 * (e / 4) + 4 * g + e % 4 < valid;
      const float p = ok ? exp2_f32(ds[e] * c0 - L2) : 0.f;
      ds[e] = p * (al * dp[e] - Ds);
    }
    const float* ka = ks + (32 * kh + 4 * g) * LD + lane % 32;
#pragma unroll
    for (int e = 0; e < 16; e++)
#pragma unroll
      for (int et = 0; et < ET; et++) dqacc[et] = mfma_f32(ka[(8 * (e / 4) + e % 4) * LD + 32 * et], ds[e], dqacc[et]);
  }

  // ---- linear branch ----
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
  float* mine_out = swap + (size_t)w * (ET / 2) * 16 * kWave + lane;
  const float* other = swap + (size_t)(w ^ 1) * (ET / 2) * 16 * kWave + lane;
  f32x16 dqo[ET / 2];                     // dQ^T of the channel tiles this wave finishes
  auto exchange = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2), F0 = ET / 2 - E0;
    __syncthreads();                      // the tiles are free
#pragma unroll
    for (int x = 0; x < ET / 2; x++)
#pragma unroll
      for (int e = 0; e < 16; e++) mine_out[(x * 16 + e) * kWave] = dqacc[F0 + x][e];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < ET / 2; x++)
#pragma unroll
      for (int e = 0; e < 16; e++) dqo[x][e] = dqacc[E0 + x][e] + other[(x * 16 + e) * kWave];
  };
  if (kh == 0) exchange(std::integral_constant<int, 0>());
  else exchange(std::integral_constant<int, 1>());
  __syncthreads();                        // the swapped halves have been read
  for (int idx = tid; idx < D * (D / 4); idx += NT)
    *reinterpret_cast<f32x4*>(hs + (idx / (D / 4)) * LD + 4 * (idx % (D / 4))) =
        *reinterpret_cast<const f32x4*>(h_i + slot * D * D + 4 * (size_t)idx);
  if (tid < D) zs[tid] = z_i[slot * D + tid];
  __syncthreads();
  float den = 0.f;
#pragma unroll
  for (int j = 0; j < J; j++) {
    const f32x4 z = *reinterpret_cast<const f32x4*>(zs + 8 * j + 4 * g);
#pragma unroll
    for (int x = 0; x < 4; x++) den += qf[j][x] * z[x];
  }
  den = both_halves_sum(den);
  // every block selected: the linear branch receives and passes no gradient
  const float inv_den = (ksel >= Tn || !row_ok) ? 0.f : 1.f / den;
  f32x16 dqp[ET / 2];
  float dot = 0.f;
  auto state_grad = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2);
#pragma unroll
    for (int x = 0; x < ET / 2; x++) {
      dqp[x] = channel_product<D>(hs + (32 * (E0 + x) + lane % 32) * LD, dos + qrow * LD, zero16(), g);
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int c = 32 * (E0 + x) + 8 * (e / 4) + 4 * g + e % 4;
        dqp[x][e] = ((1.f - al) * dqp[x][e] - Dl * zs[c]) * inv_den;
        dot += dqp[x][e] * qf[4 * (E0 + x) + e / 4][e % 4];
      }
    }
  };
  if (kh == 0) state_grad(std::integral_constant<int, 0>());
  else state_grad(std::integral_constant<int, 1>());
  dot = both_halves_sum(dot);
  if (g == 0) dots[w * 32 + lane] = dot;
  __syncthreads();                        // the row sums are visible; H_i has been read
  dot += dots[(w ^ 1) * 32 + lane % 32];
  auto store = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2);
    float* dst = dq + head_offset(sin, bh, H) + (size_t)(row0 + qrow) * sin.n + 4 * g;
#pragma unroll
    for (int x = 0; x < ET / 2; x++)
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        const f32x4 qp = qf[4 * (E0 + x) + v4];
        f32x4 y;
#pragma unroll
        for (int r = 0; r < 4; r++) y[r] = dqo[x][4 * v4 + r] * rscale + qp[r] * (dqp[x][4 * v4 + r] - dot);
        if (row_ok) *reinterpret_cast<f32x4*>(dst + 32 * (E0 + x) + 8 * v4) = y;
        *reinterpret_cast<f32x4*>(wt + qrow * LD + 32 * (E0 + x) + 8 * v4 + 4 * g) = qp * inv_den;
      }
  };
  if (kh == 0) store(std::integral_constant<int, 0>());
  else store(std::integral_constant<int, 1>());
  __syncthreads();                        // w complete
  if (SS::active(w)) {
    f32x16 dh[SS::kTiles];
#pragma unroll
    for (int x = 0; x < SS::kTiles; x++) dh[x] = zero16();
    state_product<D, NW>(dh, wt, dos, BQ, w, lane);
#pragma unroll
    for (int x = 0; x < SS::kTiles; x++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        dh_out[slot * D * D + (32 * SS::mt(w) + 8 * (e / 4) + 4 * g + e % 4) * D + 32 * (SS::nt(w) + x) + lane % 32] =
            (1.f - al) * dh[x][e];
  }
  {  // dZ_i[c] = -sum_r w[r][c] D^l_r, a share of the rows per thread
    constexpr int kParts = NT / D;
    const int c = tid % D, part = tid / D;
    float dz = 0.f;
#pragma unroll 4
    for (int r = part * (BQ / kParts); r < (part + 1) * (BQ / kParts); r++) dz -= wt[r * LD + c] * rows[BQ + r];
    red[tid] = dz;
    __syncthreads();
    if (tid < D) {
      float t = 0.f;
#pragma unroll
      for (int x = 0; x < kParts; x++) t += red[x * D + tid];
      dz_out[slot * D + tid] = (1.f - al) * t;
    }
  }
}

template <int D, int BQ>
static hipError_t launch_q(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdQF32Smem<D, BQ>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_q_f32_kernel<D, BQ>, smem); e != hipSuccess) return e;
  bwd_q_f32_kernel<D, BQ><<<dim3((unsigned)(s.BH * s.Tm)), BQ * 4, smem, stream>>>(
      (const float*)a.q, (const float*)a.k, (const float*)a.v, (const float*)a.dout, (const float*)a.o_s, (const float*)a.o_l,
      a.lse, a.k_mean, (const float*)a.h_i, a.z_i, a.block_idx, a.alpha, (float*)a.dq, a.ds, a.lraw, (float*)a.dh, a.dz,
      a.dalpha_part, s.sin, s.sout, s.H, s.N, s.Tm, s.Tn, s.k, s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_bwd_q_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (s.d == 128) return s.bq == 128 ? launch_q<128, 128>(s, a, stream) : launch_q<128, 64>(s, a, stream);
  return s.bq == 128 ? launch_q<64, 128>(s, a, stream) : launch_q<64, 64>(s, a, stream);
}

// ---------------------------------------------------------------------------------------------
template <int D> struct BwdKvF32Smem {
  static constexpr int LD = kF32Ld<D>;
  static constexpr int kTile = 64 * LD;                                    // floats
  // Q and dO rows of a step; after the loop the swapped halves of dV^T and dK^T, then dH, then the outputs
  static constexpr int kSwap = 4 * 2 * (D / 64) * 16 * kWave;
  static constexpr int kA0 = 2 * kTile > kSwap ? 2 * kTile : kSwap;
  static constexpr int kBig = kA0 > D * LD ? kA0 : D * LD;
  static constexpr int kRowOff = kBig;                                     // [2][64] L log2(e) and D^s of a step's rows
  static constexpr int kDzOff = kRowOff + 128;                             // [D]
  static constexpr int kDotOff = kDzOff + D;                               // [4][32]
  static constexpr int kBytes = (kDotOff + 128) * (int)sizeof(float);
};

template <int D, int BQ>
__global__ __launch_bounds__(256, 1) void bwd_kv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ l2_in, const float* __restrict__ ds_in, const double* __restrict__ k_mean,
    const float* __restrict__ k_stats, const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ col_idx, const int32_t* __restrict__ order,
    const float* __restrict__ dh_in, const float* __restrict__ dz_in, const float* __restrict__ dh_total,
    const float* __restrict__ dz_total, const float* __restrict__ alpha, float* __restrict__ dk, float* __restrict__ dv,
    float* __restrict__ colsum, Strides sin, Strides sout, int H, int N, int Tm, int Tn, int ksel, int alpha_per_block) {
  typedef BwdKvF32Smem<D> SM;
  constexpr int NT = 256, LD = SM::LD, ET = D / 32, J = D / 8, HP = BQ / 64;
  typedef ChunkMap<D, NT, 64> CM;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* qs = smem;                       // [64][LD] Q rows of the step
  float* dos = smem + SM::kTile;          // [64][LD] dO rows of the step
  float* dhs = smem;                      // [D][LD]  dH
  float* okt = smem;                      // [64][LD] dK', then dV behind it
  float* ovt = smem + SM::kTile;
  float* rows = smem + SM::kRowOff;
  float* dzs = smem + SM::kDzOff;
  float* dots = smem + SM::kDotOff;

  const int entry = __builtin_amdgcn_readfirstlane(order[blockIdx.x]);
  if (entry < 0) return;
  const int j = entry & (kMaxKeyBlocks - 1), bh = entry / kMaxKeyBlocks, h = bh % H;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kh = w >> 1, rh = w & 1;      // 32 keys of the block, 32 rows of a step
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const int t0 = j * kF32Tokens, valid = min(kF32Tokens, N - t0);
  const int mykey = 32 * kh + lane % 32;
  const bool key_ok = mykey < valid;
  const float* qh = q + head_offset(sin, bh, H);
  const float* doh = dout + head_offset(sout, bh, H);
  const float rscale = rsqrtf((float)D), c0 = kLog2e * rscale;

  const int32_t* cp = col_ptr + (size_t)bh * (Tn + 1);
  const int l0 = __builtin_amdgcn_readfirstlane(cp[j]), listed = __builtin_amdgcn_readfirstlane(cp[j + 1]) - l0;
  const int32_t* ci = col_idx + (size_t)bh * Tm * ksel + l0;   // the query blocks that selected this key block
  const int nsteps = listed * HP;
  // Step t: rows [64 (t % HP), +64) of query block ci[t / HP].  Rows past the end repeat an existing one; their L is
  // +inf, so their probabilities are 0.
  f32x4 qr[CM::kLoads], gr[CM::kLoads];
  float lr = 0.f, dr = 0.f;
    auto fetch = [&](int t) {
    const int i = ci[t / HP], r0 = i * BQ + 64 * (t % HP), src = r0 < N ? r0 : i * BQ, n = max(1, min(64, N - r0));
    CM::load(qr, qh + (size_t)src * sin.n, sin.n, n, tid);
    CM::load(gr, doh + (size_t)src * sout.n, sout.n, n, tid);
    if (tid < 64) {
      const size_t at = (size_t)bh * Tm * BQ + r0 + tid;
      lr = l2_in[at];
      dr = ds_in[at];
    }
  };
  if (nsteps > 0) fetch(0);

  f32x4 kf[J], vf[J];                     // K' and V of this lane's key, channels 8 j + 4 g ..
  {
    const size_t at = head_offset(sin, bh, H) + (size_t)(t0 + min(mykey, valid - 1)) * sin.n + 4 * g;
    const double* mu = k_mean + (size_t)bh * D + 4 * g;
#pragma unroll
    for (int x = 0; x < J; x++) {
      kf[x] = *reinterpret_cast<const f32x4*>(k + at + 8 * x);
      vf[x] = *reinterpret_cast<const f32x4*>(v + at + 8 * x);
#pragma unroll
      for (int y = 0; y < 4; y++) kf[x][y] -= (float)mu[8 * x + y];
    }
  }
  f32x16 dvacc[ET], dkacc[ET];
#pragma unroll
  for (int e = 0; e < ET; e++) { dvacc[e] = zero16(); dkacc[e] = zero16(); }

  for (int t = 0; t < nsteps; t++) {
    const int i = ci[t / HP];
    const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
    __syncthreads();                      // previous step fully consumed
#pragma unroll
    for (int x = 0; x < CM::kLoads; x++) {
      *reinterpret_cast<f32x4*>(qs + (trow + x * CM::kRows) * LD + 4 * ch) = qr[x];
      *reinterpret_cast<f32x4*>(dos + (trow + x * CM::kRows) * LD + 4 * ch) = gr[x];
    }
    if (tid < 64) {
      rows[tid] = lr;
      rows[64 + tid] = dr;
    }
    if (t + 1 < nsteps) fetch(t + 1);
    __syncthreads();
    f32x16 p = channel_product<D>(qs + (32 * rh + lane % 32) * LD, kf, zero16(), g);
    f32x16 ds = channel_product<D>(dos + (32 * rh + lane % 32) * LD, vf, zero16(), g);
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const int r = 32 * rh + 8 * v4 + 4 * g;
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(rows + r);
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(rows + 64 + r);
#pragma unroll
      for (int y = 0; y < 4; y++) {
        const int e = 4 * v4 + y;
        const float pv = exp2_f32(p[e] * c0 - l4[y]);   // keys past the end: columns of their own, not stored
        ds[e] = pv * (al * ds[e] - d4[y]);
        p[e] = al * pv;
      }
    }
    const float* ga = dos + (32 * rh + 4 * g) * LD + lane % 32;
    const float* qa = qs + (32 * rh + 4 * g) * LD + lane % 32;
#pragma unroll
    for (int e = 0; e < 16; e++)
#pragma unroll
      for (int et = 0; et < ET; et++) {
        dvacc[et] = mfma_f32(ga[(8 * (e / 4) + e % 4) * LD + 32 * et], p[e], dvacc[et]);
        dkacc[et] = mfma_f32(qa[(8 * (e / 4) + e % 4) * LD + 32 * et], ds[e], dkacc[et]);
      }
  }

  // the two row halves add up: each wave finishes half of the channel tiles
  f32x16 dvo[ET / 2], dko[ET / 2];
  {
    float* mine_out = smem + (size_t)w * ET * 16 * kWave + lane;
    const float* other = smem + (size_t)(w ^ 1) * ET * 16 * kWave + lane;
    auto exchange = [&](auto half) {
      constexpr int E0 = decltype(half)::value * (ET / 2), F0 = ET / 2 - E0;
      __syncthreads();                    // the last step fully consumed
#pragma unroll
      for (int x = 0; x < ET / 2; x++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          mine_out[(x * 16 + e) * kWave] = dvacc[F0 + x][e];
          mine_out[((ET / 2 + x) * 16 + e) * kWave] = dkacc[F0 + x][e];
        }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < ET / 2; x++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          dvo[x][e] = dvacc[E0 + x][e] + other[(x * 16 + e) * kWave];
          dko[x][e] = dkacc[E0 + x][e] + other[((ET / 2 + x) * 16 + e) * kWave];
        }
    };
    if (rh == 0) exchange(std::integral_constant<int, 0>());
    else exchange(std::integral_constant<int, 1>());
  }

  // ---- linear branch: dH = dH_total - sum over the query blocks that selected j of dH_i ----
  const bool all_selected = ksel >= Tn;
  {
    constexpr int NC = D * D / 4 / NT;    // 16-byte chunks per thread
    f32x4 acc[NC];
    const float* tot = dh_total + (size_t)bh * D * D + 4 * tid;
#pragma unroll
    for (int x = 0; x < NC; x++) acc[x] = *reinterpret_cast<const f32x4*>(tot + 4 * NT * x);
    float dz = tid < D ? dz_total[(size_t)bh * D + tid] : 0.f;
    for (int l = 0; l < listed; l++) {
      const size_t slot = (size_t)bh * Tm + ci[l];
      const float* src = dh_in + slot * D * D + 4 * tid;
#pragma unroll
      for (int x = 0; x < NC; x++) acc[x] -= *reinterpret_cast<const f32x4*>(src + 4 * NT * x);
      if (tid < D) dz -= dz_in[slot * D + tid];
    }
    __syncthreads();                      // the swapped halves have been read
#pragma unroll
    for (int x = 0; x < NC; x++) {
      const int idx = tid + NT * x;
      *reinterpret_cast<f32x4*>(dhs + (idx / (D / 4)) * LD + 4 * (idx % (D / 4))) = all_selected ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[x];
    }
    if (tid < D) dzs[tid] = all_selected ? 0.f : dz;
  }
  {  // K' -> K^phi = exp(K' - lnZ) (keys past the end: 0)
    const float lnz = k_stats[(size_t)bh * N + t0 + min(mykey, valid - 1)];
#pragma unroll
    for (int x = 0; x < J; x++)
#pragma unroll
      for (int y = 0; y < 4; y++) kf[x][y] = key_ok ? exp2_f32((kf[x][y] - lnz) * kLog2e) : 0.f;
  }
  __syncthreads();
  f32x16 dkp[ET / 2];
  float dot = 0.f;
  auto state_grad = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2);
#pragma unroll
    for (int x = 0; x < ET / 2; x++) {
      dkp[x] = channel_product<D>(dhs + (32 * (E0 + x) + lane % 32) * LD, vf, zero16(), g);    // over e
      const float* ha = dhs + 4 * g * LD + 32 * (E0 + x) + lane % 32;
#pragma unroll
      for (int jj = 0; jj < J; jj++)
#pragma unroll
        for (int y = 0; y < 4; y++) dvo[x] = mfma_f32(ha[(8 * jj + y) * LD], kf[jj][y], dvo[x]);   // over c
#pragma unroll
      for (int e = 0; e < 16; e++) {
        dkp[x][e] += dzs[32 * (E0 + x) + 8 * (e / 4) + 4 * g + e % 4];
        dot += dkp[x][e] * kf[4 * (E0 + x) + e / 4][e % 4];
      }
    }
  };
  if (rh == 0) state_grad(std::integral_constant<int, 0>());
  else state_grad(std::integral_constant<int, 1>());
  dot = both_halves_sum(dot);
  if (g == 0) dots[w * 32 + lane] = dot;
  __syncthreads();                        // row sums visible; dH has been read
  dot += dots[(w ^ 1) * 32 + lane % 32];
  auto park = [&](auto half) {
    constexpr int E0 = decltype(half)::value * (ET / 2);
#pragma unroll
    for (int x = 0; x < ET / 2; x++)
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        const f32x4 kp = kf[4 * (E0 + x) + v4];
        f32x4 yk, yv;
#pragma unroll
        for (int r = 0; r < 4; r++) {
          yk[r] = dko[x][4 * v4 + r] * rscale + kp[r] * (dkp[x][4 * v4 + r] - dot);
          yv[r] = dvo[x][4 * v4 + r];
        }
        *reinterpret_cast<f32x4*>(okt + mykey * LD + 32 * (E0 + x) + 8 * v4 + 4 * g) = yk;
        *reinterpret_cast<f32x4*>(ovt + mykey * LD + 32 * (E0 + x) + 8 * v4 + 4 * g) = yv;
      }
  };
  if (rh == 0) park(std::integral_constant<int, 0>());
  else park(std::integral_constant<int, 1>());
  __syncthreads();
  float* dkh = dk + head_offset(sin, bh, H) + (size_t)t0 * sin.n + 4 * ch;
  float* dvh = dv + head_offset(sin, bh, H) + (size_t)t0 * sin.n + 4 * ch;
#pragma unroll
  for (int x = 0; x < CM::kLoads; x++) {
    const int t = trow + x * CM::kRows;
    if (t < valid) {
      *reinterpret_cast<f32x4*>(dkh + (size_t)t * sin.n) = *reinterpret_cast<const f32x4*>(okt + t * LD + 4 * ch);
      *reinterpret_cast<f32x4*>(dvh + (size_t)t * sin.n) = *reinterpret_cast<const f32x4*>(ovt + t * LD + 4 * ch);
    }
  }
  if (tid < D) {                          // column sums of dK' for the smoothing term
    float sum = 0.f;
    for (int t = 0; t < valid; t++) sum += okt[t * LD + tid];
    colsum[((size_t)bh * Tn + j) * D + tid] = sum;
  }
}

template <int D, int BQ>
static hipError_t launch_kv(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdKvF32Smem<D>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_kv_f32_kernel<D, BQ>, smem); e != hipSuccess) return e;
  bwd_kv_f32_kernel<D, BQ><<<dim3((unsigned)bwd_kv_grid(s)), 256, smem, stream>>>(
      (const float*)a.q, (const float*)a.k, (const float*)a.v, (const float*)a.dout, a.lraw, a.ds, a.k_mean, a.k_stats,
      a.col_ptr, a.col_idx, a.order, (const float*)a.dh, a.dz, a.dh_total, a.dz_total, a.alpha, (float*)a.dk, (float*)a.dv, a.colsum, s.sin, s.sout,
      s.H, s.N, s.Tm, s.Tn, s.k, s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_bwd_kv_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (s.d == 128) return s.bq == 128 ? launch_kv<128, 128>(s, a, stream) : launch_kv<128, 64>(s, a, stream);
  return s.bq == 128 ? launch_kv<64, 128>(s, a, stream) : launch_kv<64, 64>(s, a, stream);
}

}  // namespace sla2
