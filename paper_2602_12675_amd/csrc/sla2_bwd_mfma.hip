// Backward pass of SLA2 on the matrix cores, for bf16 tensors (Alg. 3 of the paper's appendix with the
// steps it leaves to automatic differentiation written out; Sec. 5: the backward pass is never
// quantised).  Products run as v_mfma_f32_32x32x16_bf16 with fp32 accumulation; everything between
// them (exp, the D^s / D^l terms, both softmax-backward steps) is fp32.
//
// In each kernel the scores are laid out so that the probabilities feed the next product from registers:
//
//   bwd_q_mfma   one workgroup per query block i (b_q rows, one wave per 32 rows), scores transposed as
//                in the forward kernel, S^T = K Q^T (keys x query rows): one lane owns one query row, so
//                L and D^s are per-lane scalars and dS^T is the B operand of the product that contracts
//                over keys.  Over the selected key blocks: P^T = exp(S^T - L), dP^T = V dO^T,
//                dS^T = P^T (.) (alpha dP^T - D^s), dQ^T += K^T dS^T.  Then the linear branch from the
//                H_i^T, Z_i the forward pass kept: dQ^phi^T = (1 - alpha) H_i dO^T - Z_i D^l^T (over
//                Q^phi Z_i), dQ += softmax-backward(dQ^phi), dH_i = (Q^phi / (Q^phi Z_i))^T dO^l, dZ_i.
//   bwd_kv_mfma  one workgroup per key block j, over the query blocks that selected it, 64 rows a
//                step: here S = Q K^T (rows x keys), so that P and dS are already laid out as the
//                B operands of dV^T += dO^T (alpha P), dK'^T += Q^T dS.  Then the linear branch:
//                dH = the sum of dH_i over the other query blocks (Alg. 3's M_c[i, j] = 0 sum, a matrix product
//                in bwd_totals), dK^phi^T = dH V^T + dZ 1^T, dV^T += dH^T K^phi^T,
//                dK' += softmax-backward(dK^phi).
#include <type_traits>

#include "bwd_columns.h"
#include "mfma_tiles.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// Two buffers of (K, V) tiles.  Before the loop: the query rows and then the dO rows of every wave pass through the first one,
// which then takes w = Q^phi / (Q^phi Z_i); H_i^T arrives in the second, dO takes its place.  After it, dQ.  Rows of D
// elements throughout, in the layout of the tiles.
template <int D, int BQ> struct BwdQSmem {
  static constexpr int kTile = SwizzledLayout<D>::kTileBytes;                  // one 64 x D bf16 tile
  static constexpr int kTiles = 4 * kTile;
  static_assert(D * D * 2 <= 2 * kTile && BQ * D * 2 <= 2 * kTile, "a buffer holds H_i^T, and the rows of a query block");
  static constexpr int kZsOff = kTiles;                                        // float [D]   Z_i
  static constexpr int kMuOff = kZsOff + D * 4;                                // float [D]   colmean(K)
  static constexpr int kDlOff = kMuOff + D * 4;                                // float [BQ]  dO . O^s, later D^l, per row
  static constexpr int kRedOff = kDlOff + BQ * 4;                              // float [8]
  static constexpr int kBytes = kRedOff + 32;
  static_assert(kBwdColumnsLds <= kBytes, "the lists are made by workgroups of the same launch");
};

template <int D, int BQ>
__global__ __launch_bounds__(BQ * 2, 2) void bwd_q_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const uint16_t* __restrict__ o_s, const float* __restrict__ lse,
    const double* __restrict__ k_mean, const uint16_t* __restrict__ h_i,
    const float* __restrict__ z_i, const int32_t* __restrict__ block_idx, const float* __restrict__ alpha,
    uint16_t* __restrict__ dq, float* __restrict__ ds_out, float* __restrict__ lraw_out, uint16_t* __restrict__ dh_out,
    float* __restrict__ dz_out, float* __restrict__ dalpha_part, Strides sin, Strides sout, int H, int N, int Tm, int Tn,
    int ksel, int alpha_per_block, BwdColumns columns) {
  constexpr int NW = BQ / 32;
  constexpr int KS = D / 16, ET = D / 32;
  constexpr float kWScale = D == 64 ? 8.f : 16.f;    // of w in LDS: a power of two, at least sqrt(d)
  typedef typename std::conditional<D == 128 && BQ == 128, SwizzledLayoutB<128>, SwizzledLayout<D>>::type SL;
  // (at d = 128 free of bank conflicts, which were half of the LDS cycles: 435 -> 427 us on 12 heads of 32,760 tokens; its
  // rows repeat every 16, which the two waves of a 64-row block do not cover with one transfer)
  typedef BwdQSmem<D, BQ> SM;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  if ((int)blockIdx.x < columns.blocks) return bwd_columns_job<BQ * 2>(columns, blockIdx.x, smem);
  const int block = blockIdx.x - columns.blocks;
  float* zs = reinterpret_cast<float*>(smem + SM::kZsOff);
  float* mus = reinterpret_cast<float*>(smem + SM::kMuOff);
  float* dls = reinterpret_cast<float*>(smem + SM::kDlOff);
  float* red = reinterpret_cast<float*>(smem + SM::kRedOff);
  auto kbuf = [&](int buf) { return reinterpret_cast<uint16_t*>(smem + buf * 2 * SM::kTile); };
  auto vbuf = [&](int buf) { return reinterpret_cast<uint16_t*>(smem + buf * 2 * SM::kTile + SM::kTile); };

  // consecutive query blocks of a head share key/value tiles: every head is cut into 8 runs of
  // consecutive blocks, one per XCD (own L2), and all XCDs work through the heads in the same order
  const int per_head = (Tm + kXcds - 1) / kXcds;
  const int bh = (block / kXcds) / per_head, i = (block % kXcds) * per_head + (block / kXcds) % per_head;
  if (i >= Tm) return;
  const int h = bh % H;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int row0 = i * BQ;
  const int rows_valid = min(BQ, N - row0);
  const int qrow = 32 * w + lane % 32;               // this lane's query row inside the block
  const bool row_ok = qrow < rows_valid;
  const int r_ld = min(qrow, rows_valid - 1);        // rows past the end repeat the last one; never stored
  const uint16_t* qh = q + head_offset(sin, bh, H);
  const uint16_t* kh = k + head_offset(sin, bh, H);
  const uint16_t* vh = v + head_offset(sin, bh, H);
  const uint16_t* doh = dout + head_offset(sout, bh, H);
  const int tok_stride = sin.n;
  const int32_t* sel = block_idx + ((size_t)bh * Tm + i) * ksel;
  const int ntiles = ksel;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
  const float rscale = rsqrtf((float)D);
  const size_t slot = (size_t)bh * Tm + i;

  auto dma = [&](int j, int buf) {
    const int t0 = j * kTileTokens, valid = min(kTileTokens, N - t0);
    dma_tile<D, NW, SL>(kh + (size_t)t0 * tok_stride, tok_stride, valid, lds_address(kbuf(buf)), w, lane);
    dma_tile<D, NW, SL>(vh + (size_t)t0 * tok_stride, tok_stride, valid, lds_address(vbuf(buf)), w, lane);
  };
#pragma unroll
  for (int x = 0; x < D / 64; x++)                   // H_i^T [e][c]
    dma_tile<D, NW, SL>(h_i + slot * D * D + x * 64 * D, D, 64, lds_address(kbuf(1)) + x * SM::kTile, w, lane);
  int j_cur = ntiles > 0 ? sel[0] : 0, j_nxt = ntiles > 1 ? sel[1] : 0;

  // ---- prologue: Q and dO as B-operand fragments (alpha is applied to the products); dO . O^s per row ----
  // A wave loads its rows whole, 1 KB of consecutive bytes a request, and turns them through LDS: with every lane loading
  // pieces of its own row, a request is 32 cache lines and takes four times as long.
  bf16x8 qf[KS], gof[KS];
  float dot_s = 0.f;                                 // dO . O^s of this lane's row;  D^s = alpha dot_s
  {
    constexpr int kChunks = D / 8, kLoads = 32 * kChunks / kWave, kRows = kWave / kChunks;
    const int ch = lane % kChunks, first = 32 * w + lane / kChunks;
    u32x4 qr[kLoads], gr[kLoads], sr[kLoads];
#pragma unroll
    for (int x = 0; x < kLoads; x++) {
      const int row = row0 + min(first + kRows * x, rows_valid - 1);
      qr[x] = *reinterpret_cast<const u32x4*>(qh + (size_t)row * tok_stride + 8 * ch);
      gr[x] = *reinterpret_cast<const u32x4*>(doh + (size_t)row * sout.n + 8 * ch);
      sr[x] = *reinterpret_cast<const u32x4*>(o_s + ((size_t)bh * N + row) * D + 8 * ch);
    }
    if (tid < D) {
      mus[tid] = (float)k_mean[(size_t)bh * D + tid];
      zs[tid] = z_i[slot * D + tid];
    }
    uint16_t* turn = kbuf(0);
    auto turned = [&](const u32x4 (&from)[kLoads], bf16x8 (&to)[KS]) {
#pragma unroll
      for (int x = 0; x < kLoads; x++) *reinterpret_cast<u32x4*>(turn + SL::offset(first + kRows * x, 8 * ch)) = from[x];
      wave_lds_fence();
#pragma unroll
      for (int ks = 0; ks < KS; ks++) to[ks] = row_fragment<SL>(turn, qrow, 16 * ks + 8 * g);
      wave_lds_fence();
    };
    turned(qr, qf);
    turned(gr, gof);
    float dots[kLoads];
#pragma unroll
    for (int x = 0; x < kLoads; x++) {
      const bf16x8 go = __builtin_bit_cast(bf16x8, gr[x]), os = __builtin_bit_cast(bf16x8, sr[x]);
      float part = 0.f;
#pragma unroll
      for (int e = 0; e < 8; e++) part += (float)go[e] * (float)os[e];
      dots[x] = row_sum<kChunks>(part);
    }
    if (ch == 0)
#pragma unroll
      for (int x = 0; x < kLoads; x++) dls[first + kRows * x] = dots[x];
    wave_lds_fence();
    dot_s = dls[qrow];
    wave_lds_fence();
  }
  const float Ds = al * dot_s;
  const float L = lse[(size_t)bh * N + row0 + r_ld];
  __builtin_amdgcn_s_waitcnt(kVmcnt0);               // H_i^T and everything above have landed
  __syncthreads();                                   // ... for everyone; mus is visible
  // The forward pass defines L on the smoothed keys; the products below use the raw K, whose scores are
  // larger by q . colmean(K) / sqrt(d) in every column of a row.
  f32x4 qx[KS][2];                                   // the row in fp32, taken apart once: Q, then Q^phi without its normaliser
  float qmu = 0.f;
  lds_stream<FragmentChannels, 2 * KS, 8>(lds_address(mus + 8 * g), [&](auto n, const u32x4& raw) {
    constexpr int ks = decltype(n)::value / 2, x = decltype(n)::value % 2;
    const u32x4 two = __builtin_bit_cast(u32x4, qf[ks]);
    const f32x4 m = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      qx[ks][x][e] = __builtin_bit_cast(float, e % 2 == 0 ? two[2 * x + e / 2] << 16 : two[2 * x + e / 2] & 0xFFFF0000u);
      qmu += qx[ks][x][e] * m[e];
    }
    settle(qx[ks][x]);
  });
  qmu = swap_halves_sum(qmu);
  const float Lraw = L + qmu * rscale;
  const float L2 = Lraw * kLog2e;
  if (g == 0) {                                      // as the key-side kernel uses them: L on the raw keys, times log2(e);
    ds_out[slot * BQ + qrow] = row_ok ? Ds : 0.f;    // rows past the end get a probability of exp2(-inf) = 0 there
    lraw_out[slot * BQ + qrow] = row_ok ? L2 : INFINITY;
  }

  // ================= linear branch =================
  // First, while the scores of the loop take no registers: behind the loop it spilled up to a hundred, each waited for by itself.
  // 12 heads of 32,760 tokens: 438 -> 385 us with 15 tiles a block, 250 -> 177 without any (0.6 GB at 3.4 TB/s); 32 heads of
  // 4,096, d = 64, 64-row blocks: 56 -> 51 us.
  // What it costs is vector instructions and round trips to LDS: Q taken apart once, exponentials in place, what is read per channel kept
  // in flight (lds_stream), no second term of the softmax-backward step.  Training step, us: 1,472.6 -> 1,455.7 and 200.5 -> 198.7.
  uint16_t* ta = kbuf(1);                                           // H_i^T [e][c]; then dO [row][e]
  uint16_t* tb = kbuf(0);                                           // w = Q^phi / (Q^phi Z_i) as [row][c]
  // Byte offsets of this lane's row: 16 bytes of channels 16 ks + 8 g .. at (full) ^ 32 ks, 8 of 8 c + 4 g .. at (quarter) ^ 16 c
  // (made opaque before every loop over them: sixteen addresses are not to be kept)
  unsigned full = 2u * (unsigned)SL::offset(qrow, 8 * g), quarter = 2u * (unsigned)SL::offset(qrow, 4 * g);
  unsigned char *pa = reinterpret_cast<unsigned char*>(ta), *pb = reinterpret_cast<unsigned char*>(tb);
  // Q^phi = softmax_d(Q) of this lane's row (channels 16 ks + 8 g + 0..7) as exp(q - max); the normalisation is applied where it is
  // used.  The difference comes first: in q log2(e) - max log2(e) as a multiply-add one of the two products is rounded and the other is
  // not, which from entries of 1e9 on leaves more than an exponent holds.
  float qm = -INFINITY;
#pragma unroll
  for (int ks = 0; ks < KS; ks++)
#pragma unroll
    for (int e = 0; e < 8; e++) qm = fmaxf(qm, qx[ks][e / 4][e % 4]);
  qm = swap_halves_max(qm);
  float qs = 0.f, den = 0.f;
  lds_stream<FragmentChannels, 2 * KS, 8>(lds_address(zs + 8 * g), [&](auto n, const u32x4& raw) {
    constexpr int ks = decltype(n)::value / 2, x = decltype(n)::value % 2;
    const f32x4 z = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int e = 0; e < 4; e++) {
      qx[ks][x][e] = fast_exp2((qx[ks][x][e] - qm) * kLog2e);
      qs += qx[ks][x][e];
      den += qx[ks][x][e] * z[e];
    }
    settle(qx[ks][x]);
  });
  const float qinv = 1.f / swap_halves_sum(qs);
  den = swap_halves_sum(den) * qinv;
  // every block selected: the linear branch receives and passes no gradient
  const float inv_den = (ksel >= Tn || !row_ok) ? 0.f : 1.f / den;
  // w as a [row][c] tile (zero rows past the end), times kWScale; the softmax-backward step reads it back in the layout of the
  // accumulators.  The loop's sums are scaled by 1 / sqrt(d) at the end, so what is added to them ahead of it takes a factor sqrt(d),
  // which on H_i dO and D^l would take entries past the largest number and as an operation of its own costs 0.1 to 0.4 % of a training step.
  {
    const float wscale = qinv * inv_den * kWScale;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      bf16x8 wv;
#pragma unroll
      for (int e = 0; e < 8; e++) wv[e] = (__bf16)(qx[ks][e / 4][e % 4] * wscale);
      *reinterpret_cast<bf16x8*>(pb + (full ^ (32u * ks))) = wv;
    }
  }
  // dQ^phi^T = (1 - alpha) H_i dO^T: A = H_i read transposed out of the H_i^T tile, B = the dO fragments
  // (in the accumulators of dQ: what they end up with before the loop is added to by it)
  f32x16 dqacc[ET];
#pragma unroll
  for (int ct = 0; ct < ET; ct++)
#pragma unroll
    for (int e = 0; e < 16; e++) dqacc[ct][e] = 0.f;
  // (fragment ks ET + ct: two transposing reads, kept kAhead fragments ahead, cf. nat_fragment; left to the compiler each is waited
  // for right in front of its product)
  const int tr_row = (lane % 16) / 4, tr_col = 16 * ((lane / 16) % 2) + 4 * (lane % 4);
  {
    constexpr int kFrags = KS * ET, kAhead = 4, kSlots = kAhead + 1;
    const unsigned at[2] = {lds_address(ta + SL::offset(8 * g + tr_row, tr_col)), lds_address(ta + SL::offset(8 * g + 4 + tr_row, tr_col))};
    u32x2 ring[kSlots][2];
    auto issue = [&](int n) {
#pragma unroll
      for (int y = 0; y < 2; y++) ring[n % kSlots][y] = lds_read_tr_untracked_at<32 * D>(at[y] ^ (64u * (n % ET)), n / ET);
    };
#pragma unroll
    for (int n = 0; n < kAhead; n++) issue(n);
#pragma unroll
    for (int n = 0; n < kFrags; n++) {
      if (n + kAhead < kFrags) issue(n + kAhead);
      wait_lgkmcnt(2 * (n + kAhead < kFrags ? kAhead : kFrags - 1 - n));
      settle(ring[n % kSlots][0]);
      settle(ring[n % kSlots][1]);
      const u32x4 a = {ring[n % kSlots][0][0], ring[n % kSlots][0][1], ring[n % kSlots][1][0], ring[n % kSlots][1][1]};
      dqacc[n % ET] = mfma_bf16(__builtin_bit_cast(bf16x8, a), gof[n / ET], dqacc[n % ET]);
    }
  }
  wave_lds_fence();                                  // (w rows: the wave's own)
  settle(quarter);
  // O^l is not kept by the forward pass: dO . O^l of a row equals sum_c w[r][c] (H_i dO^T)[c][r], both at
  // hand.  D^l = (1 - alpha) dO . O^l; the row's part of d alpha is dO . (O^s - O^l).
  u32x2 wq[4 * ET];                                  // w in the layout of the accumulators
#pragma unroll
  for (int c = 0; c < 4 * ET; c++) wq[c] = lds_read8_untracked(lds_address(pb) + (quarter ^ (16u * c)));
  wait_lgkmcnt(0);
#pragma unroll
  for (int c = 0; c < 4 * ET; c++) settle(wq[c]);
  auto w_value = [&](int c, int r) { return __builtin_bit_cast(float, r % 2 == 0 ? wq[c][r / 2] << 16 : wq[c][r / 2] & 0xFFFF0000u); };
  float dot_l = 0.f, wz = 0.f;
  lds_stream<AccumulatorChannels, 4 * ET, 8>(lds_address(zs + 4 * g), [&](auto n, const u32x4& raw) {
    constexpr int ct = decltype(n)::value / 4, v4 = decltype(n)::value % 4;
    const f32x4 z = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int r = 0; r < 4; r++) {
      dot_l += w_value(4 * ct + v4, r) * dqacc[ct][4 * v4 + r];
      wz += w_value(4 * ct + v4, r) * z[r];
    }
  });
  wz = swap_halves_sum(wz);                          // kWScale but for the rounding of w, which is taken out again (a row of zeros stays 0)
  dot_l = swap_halves_sum(dot_l) * (wz != 0.f ? 1.f / wz : 0.f);
  const float Dl = (1.f - al) * dot_l;
  if (g == 0) dls[qrow] = Dl;
  {
    float mix = (row_ok && g == 0) ? dot_s - dot_l : 0.f;
    mix = wave_sum(mix);
    if (lane == 0) red[w] = mix;
  }
  // dQ^phi = ((1 - alpha) H_i dO - D^l Z_i) / (Q^phi Z_i) is orthogonal to Q^phi: O^l does not change with the length of Q^phi.  So the
  // softmax-backward step, Q^phi (.) (dQ^phi - <dQ^phi, Q^phi>), has no second term, and Q^phi / (Q^phi Z_i) is w.  With D^l formed
  // as above that holds for the rounded w too.
  const float rest = sqrtf((float)D) / kWScale, from_h = (1.f - al) * rest, from_z = Dl * rest;    // rest: at most 1
  lds_stream<AccumulatorChannels, 4 * ET, 8>(lds_address(zs + 4 * g), [&](auto n, const u32x4& raw) {
    constexpr int ct = decltype(n)::value / 4, v4 = decltype(n)::value % 4;
    const f32x4 z = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int r = 0; r < 4; r++) dqacc[ct][4 * v4 + r] = w_value(4 * ct + v4, r) * (from_h * dqacc[ct][4 * v4 + r] - from_z * z[r]);
    if (v4 == 3) settle(dqacc[ct]);                  // here: moved behind the products below, its operands go through scratch memory
  });
  __syncthreads();                                   // nobody reads H_i^T any more
#pragma unroll
  for (int ks = 0; ks < KS; ks++) *reinterpret_cast<bf16x8*>(pa + (full ^ (32u * ks))) = gof[ks];   // dO as [row][e]
  __syncthreads();                                   // dO and w complete; the waves' d alpha parts are visible
  if (tid == 0) {
    float t = 0.f;
#pragma unroll
    for (int x = 0; x < NW; x++) t += red[x];
    dalpha_part[slot] = t;
  }
  // dH_i[c][e] = (1 - alpha) sum_r w[r][c] dO[r][e]: both operands read transposed, contraction over the rows.  Formed as
  // dH_i^T tiles and stored as they lie in the accumulators, 16 bytes a lane and a whole kilobyte per store: lane l holds
  // channel c = 32 ct + l % 32 and, in half x of tile (ct, et), e = 32 et + 16 x + 4 (l / 32) + {0..3, 8..11}.
  // dZ_i[c] = -sum_r w[r][c] D^l_r from the same operands of w.
  constexpr int kTilesPerWave = ET * ET / NW, kEts = kTilesPerWave < ET ? kTilesPerWave : ET, kCts = kTilesPerWave / kEts;
  static_assert(kTilesPerWave >= 1, "unsupported split");
  uint16_t* dh_slot = dh_out + slot * D * D;
  const float dh_scale = 0.5f / kWScale * (1.f - al);   // w without its factor; a half of it, for masked_sums.h
#pragma unroll 1
  for (int x = 0; x < kCts; x++) {
    const int t0 = w * kTilesPerWave + x * kEts, ct = t0 / ET, et0 = t0 % ET;
    f32x16 acc[kEts];
#pragma unroll
    for (int y = 0; y < kEts; y++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[y][e] = 0.f;
    float dz = 0.f;
    // fragments in turn: w of a step of 16 rows, then dO of the tiles (cf. v_fragment)
    constexpr int kPer = 1 + kEts, kFrags = BQ / 16 * kPer, kAhead = 4, kSlots = kAhead + 1;
    const unsigned at[2] = {2u * (unsigned)SL::offset(4 * g + tr_row, tr_col), 2u * (unsigned)SL::offset(4 * g + 8 + tr_row, tr_col)};
    const unsigned w_at = lds_address(tb), g_at = lds_address(ta);
    u32x2 ring[kSlots][2];
    auto issue = [&](int n) {
      const int y = n % kPer;
#pragma unroll
      for (int hi = 0; hi < 2; hi++)
        ring[n % kSlots][hi] = lds_read_tr_untracked_at<32 * D>(y == 0 ? (w_at + at[hi]) ^ (64u * ct) : (g_at + at[hi]) ^ (64u * et0) ^ (64u * (y - 1)), n / kPer);
    };
    bf16x8 wf;
#pragma unroll
    for (int n = 0; n < kAhead; n++) issue(n);
#pragma unroll
    for (int n = 0; n < kFrags; n++) {
      if (n + kAhead < kFrags) issue(n + kAhead);
      wait_lgkmcnt(2 * (n + kAhead < kFrags ? kAhead : kFrags - 1 - n));
      settle(ring[n % kSlots][0]);
      settle(ring[n % kSlots][1]);
      const u32x4 a = {ring[n % kSlots][0][0], ring[n % kSlots][0][1], ring[n % kSlots][1][0], ring[n % kSlots][1][1]};
      const int y = n % kPer;
      if (y > 0) {
        acc[y - 1] = mfma_bf16(__builtin_bit_cast(bf16x8, a), wf, acc[y - 1]);
      } else {
        wf = __builtin_bit_cast(bf16x8, a);
        const f32x4 d0 = *reinterpret_cast<const f32x4*>(dls + 16 * (n / kPer) + 4 * g), d1 = *reinterpret_cast<const f32x4*>(dls + 16 * (n / kPer) + 8 + 4 * g);
#pragma unroll
        for (int e = 0; e < 8; e++) dz -= __builtin_bit_cast(float, e % 2 == 0 ? a[e / 2] << 16 : a[e / 2] & 0xFFFF0000u) * (e < 4 ? d0[e] : d1[e - 4]);
      }
    }
#pragma unroll
    for (int y = 0; y < kEts; y++)
#pragma unroll
      for (int half = 0; half < 2; half++) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = (__bf16)(dh_scale * acc[y][8 * half + e]);
        *reinterpret_cast<bf16x8*>(dh_slot + (((t0 + y) * 2 + half) * kWave + lane) * 8) = o;
      }
    dz = swap_halves_sum(dz);
    if (et0 == 0 && g == 0) dz_out[slot * D + 32 * ct + lane] = dz * (1.f / kWScale);
  }
  __syncthreads();                                   // w and dO consumed
  if (ntiles > 0) dma(j_cur, 0);

  // LDS byte offsets of this lane's operand reads inside a K or V tile: row-wise reads (key row
  // l % 32, channel step ks at (offset of step 0) ^ 32 ks) and transposing reads (cf. read_tr4): rows 4 g + (l % 16) / 4 (lo)
  // and 8 further (hi), channel tile et at (offset of tile 0) ^ 64 et, 16-token step ks 32 D ks further
  const unsigned b_off = (unsigned)SL::offset(lane % 32, 8 * g) * 2;
  const unsigned a_off[2] = {(unsigned)SL::offset(4 * g + tr_row, tr_col) * 2, (unsigned)SL::offset(4 * g + tr_row + 8, tr_col) * 2};
  __builtin_amdgcn_s_waitcnt(kVmcnt0);               // tile 0 has landed ...
  __syncthreads();                                   // ... for everyone
  float sumds = 0.f;
  const float c0 = kLog2e * rscale;

  auto tile = [&](int s, auto is_short) {
    constexpr bool kShort = decltype(is_short)::value;
    const int buf = s & 1;
    const int valid = kShort ? N - j_cur * kTileTokens : kTileTokens;
    const int j_nn = sel[min(s + 2, ntiles - 1)];
    if (s + 1 < ntiles) dma(j_nxt, buf ^ 1);
    j_cur = j_nxt;
    j_nxt = j_nn;
    const unsigned ka = lds_address(kbuf(buf)), va = lds_address(vbuf(buf));
    f32x16 sacc[2], dpacc[2];
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
      for (int e = 0; e < 16; e++) { sacc[mt][e] = 0.f; dpacc[mt][e] = 0.f; }
    // Element x of the tile: P^T = exp(S^T - L), in the place of the score, and dS^T = P^T (.) (alpha dP^T - D^s), as
    // B-operand fragments in token order.  Both run between the products of other elements: the exponentials behind
    // those of dP^T, dS^T of the first 32 keys behind those of the second half, the rest behind dQ's first products.
    // The matrix and the vector unit then work side by side within a wave too: a training step on 12 heads of 32,760
    // tokens 1,730 -> 1,711 us.
    bf16x8 dsf[4];
    constexpr int kPer = 16 / KS;                      // elements per product
    auto prob = [&](int x) {
      float p = fast_exp2(sacc[x / 16][x % 16] * c0 - L2);
      if (kShort && 32 * (x / 16) + 8 * (x % 16 / 4) + 4 * g + x % 4 >= valid) p = 0.f;
      settle(p);                                       // here, not where the compiler would gather them
      sacc[x / 16][x % 16] = p;
    };
    auto grad = [&](int x) {
      const float dsv = sacc[x / 16][x % 16] * (al * dpacc[x / 16][x % 16] - Ds);
      sumds += dsv;
      dsf[x / 8][x % 8] = (__bf16)dsv;
    };
    // S^T = K Q^T and dP^T = V dO^T (keys x query rows; alpha joins below), two 32-key halves each.  One operand read
    // (16 bytes of key row 32 mt + l % 32) per product, issued untracked and kept kAhead deep in flight:
    // a tracked read would be waited for right before its product, one LDS round trip per product.
    {
      constexpr int kItems = 4 * KS, kAhead = 6, kSlots = kAhead + 1;
      u32x4 ring[kSlots];
      auto issue = [&](int n) {                      // item n: (K | V, key half, channel step)
        const int grp = n / KS, ks = n % KS;
        const unsigned base = (grp < 2 ? ka : va) + b_off;
        if (grp % 2 == 0) ring[n % kSlots] = lds_read16_untracked<0>(base ^ (32u * ks));
        else ring[n % kSlots] = lds_read16_untracked<32 * D * 2>(base ^ (32u * ks));
      };
#pragma unroll
      for (int n = 0; n < kAhead; n++) issue(n);
#pragma unroll
      for (int n = 0; n < kItems; n++) {
        if (n + kAhead < kItems) issue(n + kAhead);
        wait_lgkmcnt(n + kAhead < kItems ? kAhead : kItems - 1 - n);
        settle(ring[n % kSlots]);
        const bf16x8 a = __builtin_bit_cast(bf16x8, ring[n % kSlots]);
        const int grp = n / KS, ks = n % KS;
        if (grp < 2) sacc[grp] = mfma_bf16(a, qf[ks], sacc[grp]);
        else dpacc[grp - 2] = mfma_bf16(a, gof[ks], dpacc[grp - 2]);
        if (grp >= 2)
#pragma unroll
          for (int x = 0; x < kPer; x++) prob(kPer * (n - 2 * KS) + x);
        if (grp == 3)
#pragma unroll
          for (int x = 0; x < kPer; x++) grad(kPer * ks + x);
      }
    }
    // dQ^T += K^T dS^T: transposing reads of the K tile, those of the next 16-token step in flight
    // while the products of this one run
    {
      constexpr int kReads = 2 * ET;
      u32x2 rk[2][ET][2];
      auto issue = [&](int ks, int slot) {
#pragma unroll
        for (int et = 0; et < ET; et++)
#pragma unroll
          for (int hi = 0; hi < 2; hi++) rk[slot][et][hi] = lds_read_tr_untracked_at<32 * D>((ka + a_off[hi]) ^ (64u * et), ks);
      };
      issue(0, 0);
#pragma unroll
      for (int ks = 0; ks < kTileTokens / 16; ks++) {
        const int slot = ks & 1;
        if (ks + 1 < kTileTokens / 16) issue(ks + 1, slot ^ 1);
        wait_lgkmcnt(ks + 1 < kTileTokens / 16 ? kReads : 0);
#pragma unroll
        for (int et = 0; et < ET; et++) {
          settle(rk[slot][et][0]);
          settle(rk[slot][et][1]);
          const u32x4 v4 = {rk[slot][et][0][0], rk[slot][et][0][1], rk[slot][et][1][0], rk[slot][et][1][1]};
          dqacc[et] = mfma_bf16(__builtin_bit_cast(bf16x8, v4), dsf[ks], dqacc[et]);
          if (ks < 2)
#pragma unroll
            for (int x = 0; x < 8 / ET; x++) grad(16 + 8 * ks + (8 / ET) * et + x);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(kVmcnt0);             // the next tile has landed in LDS ...
    __syncthreads();                                 // ... for everyone, and this tile's buffer is free
  };
  // indices ascend: only the last tile of the list can be the short one at the end of the sequence
  const int whole = ntiles - (ntiles > 0 && N % kTileTokens != 0 && sel[ntiles - 1] == Tn - 1 ? 1 : 0);
  for (int s = 0; s < whole; s++) tile(s, std::false_type());
  if (whole < ntiles) tile(whole, std::true_type());

  // ================= epilogue =================
  // dS K' = dS K - rowsum(dS) colmean(K)^T; transposed through LDS for a coalesced store of the wave's own rows
  sumds = swap_halves_sum(sumds);
  const int ln = (int)lane_again();                  // addresses are made here, not kept from the start of the kernel
  const unsigned row_at = 2u * (unsigned)SL::offset(32 * w + ln % 32, 4 * (ln / 32));
#pragma unroll
  for (int et = 0; et < ET; et++)
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const f32x4 m = *reinterpret_cast<const f32x4*>(mus + 32 * et + 8 * v4 + 4 * (ln / 32));
      bf16x4 pk;
#pragma unroll
      for (int r = 0; r < 4; r++) pk[r] = (__bf16)((dqacc[et][4 * v4 + r] - sumds * m[r]) * rscale);
      *reinterpret_cast<bf16x4*>(smem + (row_at ^ (16u * (4 * et + v4)))) = pk;
    }
  wave_lds_fence();
  {
    uint16_t* dst = dq + head_offset(sin, bh, H) + (size_t)row0 * tok_stride;
#pragma unroll
    for (int x = 0; x < D / 16; x++) {
      const int r = 32 * w + (x * kWave + ln) / (D / 8), ch = ln % (D / 8);
      if (r < rows_valid)
        store_streamed(reinterpret_cast<u32x4*>(dst + (size_t)r * tok_stride + 8 * ch), *reinterpret_cast<const u32x4*>(kbuf(0) + SL::offset(r, 8 * ch)));
    }
  }
}

template <int D, int BQ>
static hipError_t launch_bwd_q_mfma(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdQSmem<D, BQ>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_q_mfma_kernel<D, BQ>, smem); e != hipSuccess) return e;
  const int grid = ((s.Tm + kXcds - 1) / kXcds) * kXcds * s.BH;
  const BwdColumns columns = bwd_columns(s, a);
  bwd_q_mfma_kernel<D, BQ><<<dim3((unsigned)(columns.blocks + grid)), BQ * 2, smem, stream>>>(
      (const uint16_t*)a.q, (const uint16_t*)a.k, (const uint16_t*)a.v, (const uint16_t*)a.dout, (const uint16_t*)a.o_s,
      a.lse, a.k_mean, (const uint16_t*)a.h_i, a.z_i, a.block_idx, a.alpha, (uint16_t*)a.dq, a.ds, a.lraw,
      (uint16_t*)a.dh, a.dz, a.dalpha_part, s.sin, s.sout, s.H, s.N, s.Tm, s.Tn, s.k, s.alpha_per_block ? 1 : 0, columns);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// 16 bytes of a step's row quantities: the 32-byte groups 8 rows apart, L at n = 0 .. 3 and D^s, 256 bytes on, at 8 .. 11
__device__ __forceinline__ u32x4 stat_read(unsigned base, int n) {
  switch (n) {
    case 0: return lds_read16_untracked<0>(base);
    case 1: return lds_read16_untracked<32>(base);
    case 2: return lds_read16_untracked<64>(base);
    case 3: return lds_read16_untracked<96>(base);
    case 8: return lds_read16_untracked<256>(base);
    case 9: return lds_read16_untracked<288>(base);
    case 10: return lds_read16_untracked<320>(base);
    default: return lds_read16_untracked<352>(base);
  }
}

template <int D> struct BwdKvSmem {
  static constexpr int kLd = D + 8;
  static constexpr int kTile = SwizzledLayout<D>::kTileBytes;                  // one 64 x D bf16 tile
  static constexpr int kStepBytes = 4 * kTile;                                 // two buffers of (Q rows, dO rows); before the loop
                                                                               // K_j, V_j and dH_j, after it the outputs
  static constexpr int kStatOff = kStepBytes;                                  // float [2][2][64]: L log2(e) and D^s of a step's rows
                                                                               // (before the loop parts of dZ_j, after it of sums)
  static constexpr int kMuOff = kStatOff + 2 * 2 * 64 * 4;                     // float [D]  colmean(K)
  static constexpr int kDotOff = kMuOff + D * 4;                               // float [D / 32][64]
  static constexpr int kBytes = kDotOff + 256 * 4;
  static_assert(D * D * 2 <= 2 * kTile && 2 * 64 * kLd * 2 <= kStepBytes, "dH_j and the outputs in the place of the steps");
  static_assert(kStatOff + 512 * 4 <= kBytes, "parts of the column sums");
};

// Scores are computed as S = Q K^T (query rows x keys) here: a lane of the result then owns one key
// and 16 of the 32 query rows of the tile, which is the B-operand layout of the products that contract
// over query rows (dV^T += dO^T P, dK^T += Q^T dS) - P and dS never leave registers.  Wave (kh, rh) owns the
// key half kh and, of every 64-row step, the row half rh: it forms 32 x 32 scores and contracts over its 32 rows
// into all channels; the two waves of a key half add their dV^T, dK^T once, after the loop, and share the channel
// tiles of the linear branch.  (Owning 64 rows and half of the channels instead, a wave formed every score twice:
// 48 products and 32 exponentials per lane and step where 32 and 16 do, and read 48 KB of operands from LDS instead
// of 32: LDS feeds 128 bytes a cycle, one operand per product and SIMD.)  The price is registers: 128 accumulators
// next to the 64 of the K_j, V_j fragments, so the operand reads run only a few ahead.
template <int D, int BQ>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void bwd_kv_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const uint16_t* __restrict__ dout, const float* __restrict__ lraw2, const float* __restrict__ ds_in,
    const double* __restrict__ k_mean, const float* __restrict__ k_stats, const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ col_idx,
    const int32_t* __restrict__ order, const uint16_t* __restrict__ dh_in, const float* __restrict__ dz_in,
    const float* __restrict__ dz_total, const float* __restrict__ alpha,
    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, float* __restrict__ colsum, Strides sin, Strides sout, int H,
    int N, int Tm, int Tn, int ksel, int alpha_per_block) {
  constexpr int NW = 4, NT = 256;
  constexpr int LD = D + 8, KS = D / 16, ET = D / 32;
  constexpr int HP = BQ / 64;                        // 64-row steps per query block
  constexpr int CT = ET / 2;                         // 32-channel tiles a wave finishes after the loop
  typedef typename std::conditional<D == 128, SwizzledLayoutB<128>, SwizzledLayout<64>>::type SL;   // no bank conflicts
  typedef BwdKvSmem<D> SM;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  auto qbuf = [&](int buf) { return reinterpret_cast<uint16_t*>(smem + buf * 2 * SM::kTile); };
  auto gbuf = [&](int buf) { return reinterpret_cast<uint16_t*>(smem + buf * 2 * SM::kTile + SM::kTile); };
  float* stat = reinterpret_cast<float*>(smem + SM::kStatOff);
  float* mus = reinterpret_cast<float*>(smem + SM::kMuOff);
  float* dred = reinterpret_cast<float*>(smem + SM::kDotOff);

  const int entry = __builtin_amdgcn_readfirstlane(order[blockIdx.x]);
  if (entry < 0) return;
  const int j = entry & (kMaxKeyBlocks - 1), bh = entry / kMaxKeyBlocks, h = bh % H;   // longest lists first, see sla2_bwd.hip
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kh = w >> 1, rh = w & 1;                 // rh: also the half of the channel tiles finished after the loop
  const int t0 = j * kTileTokens, valid = min(kTileTokens, N - t0);
  const int mykey = 32 * kh + lane % 32;             // this lane's key inside the block
  const uint16_t* qh = q + head_offset(sin, bh, H);
  const uint16_t* kh_ = k + head_offset(sin, bh, H);
  const uint16_t* vh = v + head_offset(sin, bh, H);
  const uint16_t* doh = dout + head_offset(sout, bh, H);
  const int tok_stride = sin.n;
  const float rscale = rsqrtf((float)D);
  const float c0 = kLog2e * rscale;

  // K_j and V_j (rows past the end repeat the last one)
  dma_tile<D, NW, SL>(kh_ + (size_t)t0 * tok_stride, tok_stride, valid, lds_address(qbuf(0)), w, lane);
  dma_tile<D, NW, SL>(vh + (size_t)t0 * tok_stride, tok_stride, valid, lds_address(gbuf(0)), w, lane);
  const int32_t* cp = col_ptr + (size_t)bh * (Tn + 1);
  const int32_t* ci = col_idx + (size_t)bh * Tm * ksel;
  const int l0 = __builtin_amdgcn_readfirstlane(cp[j]), l1 = __builtin_amdgcn_readfirstlane(cp[j + 1]);
  const int nsteps = (l1 - l0) * HP;

  // Step t covers rows [64 (t % HP), +64) of query block ci[l0 + t / HP].  Rows past the end (a short last query block)
  // repeat an existing one; their L is +inf, so their probabilities are 0.
  // The rows of step t + 1 (and L log2 e, D^s of those rows) are requested at the start of step t,
  // straight into LDS; the query block index is read one step before that.
  struct Step { int i, row0; float al; };
  auto block_of = [&](int t) { return ci[l0 + min(t, nsteps - 1) / HP]; };
  auto place = [&](int t, int i) {
    return Step{i, i * BQ + 64 * (t % HP), alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h]};
  };
  auto request = [&](const Step& st, int buf) {
    const int ln = (int)lane_again();                 // lane addresses are made here each time, not kept through the loop
    const int src = st.row0 < N ? st.row0 : st.i * BQ, rows = max(1, min(64, N - st.row0));
    dma_tile<D, NW, SL>(qh + (size_t)src * tok_stride, tok_stride, rows, lds_address(qbuf(buf)), w, ln);
    dma_tile<D, NW, SL>(doh + (size_t)src * sout.n, sout.n, rows, lds_address(gbuf(buf)), w, ln);
    // every wave fetches the same 2 x 64 floats (same values to the same place: the counts of
    // outstanding transfers stay equal across the waves)
    const size_t at = (size_t)bh * Tm * BQ + st.row0;
    dma_lane4(lraw2 + at, 4u * (unsigned)ln, lds_address(stat + buf * 128));
    dma_lane4(ds_in + at, 4u * (unsigned)ln, lds_address(stat + buf * 128 + 64));
  };

  f32x16 dvall[ET], dkall[ET];
#pragma unroll
  for (int x = 0; x < ET; x++)
#pragma unroll
    for (int e = 0; e < 16; e++) { dvall[x][e] = 0.f; dkall[x][e] = 0.f; }

  // ================= linear branch =================
  // First: behind the loop every one of its steps (the lists' dZ_i, dH_j, its place in LDS, products, row sums) waits for the
  // one before with nothing else to do, and takes registers from the accumulators.  What it gives is what they start from,
  // each wave's half of the channel tiles.  12 heads of 32,760 tokens: 597 -> 566 us, 207 -> 188 without any list entry.
  bf16x8 kfr[KS], vfr[KS];                           // K_j and V_j rows of this lane's key as operand fragments
  {
    const bool all_selected = ksel >= Tn;            // no gradient, whatever dO holds
    uint16_t* dht = qbuf(1);                         // dH [c][e]
    // dH (Alg. 3's M_c[i, j] = 0 sum, from bwd_totals) in the order in which the query-side kernel leaves dH_i
    constexpr int NCH = D * D / 8 / NT;
    const uint16_t* src = dh_in + ((size_t)bh * Tn + j) * D * D + (size_t)tid * 8;
    bf16x8 x[NCH];
#pragma unroll
    for (int n = 0; n < NCH; n++) x[n] = *reinterpret_cast<const bf16x8*>(src + NT * n * 8);
    const float lnz2 = k_stats[(size_t)bh * N + t0 + min(mykey, valid - 1)] * kLog2e;
    if (tid < D) mus[tid] = (float)k_mean[(size_t)bh * D + tid];
    // dZ_j = dZ_total less the dZ_i of the list, NT / D parts side by side and four entries each at a time on their way
    constexpr int kParts = NT / D;
    {
      const int c = tid % D, part = tid / D, last = all_selected ? l0 : l1;
      float dzj = (part == 0 && !all_selected) ? dz_total[(size_t)bh * D + c] : 0.f;
      for (int l = l0 + 4 * part; l < last; l += 4 * kParts) {
        float z[4];
#pragma unroll
        for (int y = 0; y < 4; y++) z[y] = dz_in[((size_t)bh * Tm + ci[min(l + y, last - 1)]) * D + c];
#pragma unroll
        for (int y = 0; y < 4; y++)
          if (l + y < last) dzj -= z[y];
      }
      stat[tid] = dzj;
    }
#pragma unroll
    for (int n = 0; n < NCH; n++) {
      const int idx = tid + NT * n, l = idx % kWave, half = idx / kWave % 2, t = idx / (2 * kWave);
      const int row = 32 * (t / ET) + l % 32, col = 32 * (t % ET) + 16 * half + 4 * (l / 32);
#pragma unroll
      for (int y = 0; y < 2; y++) {
        bf16x4 four = {x[n][4 * y], x[n][4 * y + 1], x[n][4 * y + 2], x[n][4 * y + 3]};
        if (all_selected) four = bf16x4{};
        *reinterpret_cast<bf16x4*>(dht + SL::offset(row, col + 8 * y)) = four;
      }
    }
    wait_vmcnt<0>();
    __syncthreads();                                 // K_j, V_j, dH, parts of dZ_j and mus are in LDS for everyone
    // K^phi_j = exp(K - colmean(K) - lnZ).  (Keys past the end repeat the last one here and need no zeros, see the loop; asked for, they
    // became a branch around every exponential.)
    bf16x8 pfr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      kfr[ks] = row_fragment<SL>(qbuf(0), mykey, 16 * ks + 8 * g);
      vfr[ks] = row_fragment<SL>(gbuf(0), mykey, 16 * ks + 8 * g);
      const f32x4 m0 = *reinterpret_cast<const f32x4*>(mus + 16 * ks + 8 * g);
      const f32x4 m1 = *reinterpret_cast<const f32x4*>(mus + 16 * ks + 8 * g + 4);
#pragma unroll
      for (int e = 0; e < 8; e++)
        pfr[ks][e] = (__bf16)fast_exp2(((float)kfr[ks][e] - (e < 4 ? m0[e] : m1[e - 4])) * kLog2e - lnz2);
      settle(pfr[ks]);                               // one fragment at a time: the registers
      __builtin_amdgcn_sched_barrier(0);
    }
    // dK^phi^T = dH V^T (+ dZ 1^T below) and dV^T += dH^T K^phi^T, both channels x keys
    f32x16 dkp[CT], dvl[CT];
#pragma unroll
    for (int y = 0; y < CT; y++)
#pragma unroll
      for (int e = 0; e < 16; e++) { dkp[y][e] = 0.f; dvl[y][e] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
#pragma unroll
      for (int y = 0; y < CT; y++) {
        const int ct = CT * rh + y;
        dkp[y] = mfma_bf16(row_fragment<SL>(dht, 32 * ct + lane % 32, 16 * ks + 8 * g), vfr[ks], dkp[y]);   // over e
        dvl[y] = mfma_bf16(nat_fragment<SL>(dht, ks, 32 * ct, lane), pfr[ks], dvl[y]);                     // over c
      }
      if (D == 64) __builtin_amdgcn_sched_barrier(0);
    }
    // back through phi: dK' += K^phi (.) (dK^phi - rowsum(dK^phi (.) K^phi)); the row sum spans all channels
    float kp[CT][16];
#pragma unroll
    for (int y = 0; y < CT; y++) {
      const int ct = CT * rh + y;
      float part = 0.f;
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        const int c = 32 * ct + 8 * v4 + 4 * g;
        const bf16x4 kk = *reinterpret_cast<const bf16x4*>(qbuf(0) + SL::offset(mykey, c));
        const f32x4 m = *reinterpret_cast<const f32x4*>(mus + c);
        f32x4 dz = *reinterpret_cast<const f32x4*>(stat + c);
#pragma unroll
        for (int n = 1; n < kParts; n++) dz += *reinterpret_cast<const f32x4*>(stat + n * D + c);
#pragma unroll
        for (int r = 0; r < 4; r++) {
          kp[y][4 * v4 + r] = (float)(__bf16)fast_exp2(((float)kk[r] - m[r]) * kLog2e - lnz2);
          dkp[y][4 * v4 + r] += dz[r];
          part += dkp[y][4 * v4 + r] * kp[y][4 * v4 + r];
        }
      }
      part = swap_halves_sum(part);
      if (g == 0) dred[ct * 64 + mykey] = part;
    }
    __syncthreads();                                 // row sums complete; the tiles have been read
    float dot = 0.f;
#pragma unroll
    for (int c2 = 0; c2 < ET; c2++) dot += dred[c2 * 64 + mykey];
    const float unscale = sqrtf((float)D);           // the loop's sums are scaled by 1 / sqrt(d) at the end
    auto start_from = [&](auto half) {
      constexpr int E0 = decltype(half)::value * CT;
#pragma unroll
      for (int y = 0; y < CT; y++) {
        dvall[E0 + y] = dvl[y];
#pragma unroll
        for (int e = 0; e < 16; e++) dkall[E0 + y][e] = kp[y][e] * (dkp[y][e] - dot) * unscale;
      }
    };
    if (rh == 0) start_from(std::integral_constant<int, 0>());
    else start_from(std::integral_constant<int, 1>());
  }

  Step cur{0, 0, 0.f};
  int i_nxt = 0;
  if (nsteps > 0) {
    cur = place(0, block_of(0));
    i_nxt = block_of(1);
    request(cur, 0);
  }
  wait_vmcnt<0>();
#pragma unroll
  for (int ks = 0; ks < KS; ks++) { settle(kfr[ks]); settle(vfr[ks]); }
  __syncthreads();                                   // step 0 is in LDS for everyone

  // LDS byte offsets of this lane's operand reads inside a Q or dO tile.  Row-wise reads: row 32 rh + l % 32, channel
  // step ks at (offset of step 0) ^ 32 ks.  Transposing reads (cf. read_tr4): rows 32 rh + 4 g + (l % 16) / 4 (lo) and
  // 8 further (hi), channel tile et at (offset of tile 0) ^ 64 et, 16-row step ks 32 D ks further.
  const unsigned b_off = (unsigned)SL::offset(32 * rh + lane % 32, 8 * g) * 2;
  const int tr_row = 32 * rh + 4 * g + (lane % 16) / 4, tr_col = 16 * ((lane / 16) % 2) + 4 * (lane % 4);
  const unsigned a_lo = (unsigned)SL::offset(tr_row, tr_col) * 2, a_hi = (unsigned)SL::offset(tr_row + 8, tr_col) * 2;

  for (int t = 0; t < nsteps; t++) {
    const int buf = t & 1;
    Step nxt = cur;
    if (t + 1 < nsteps) {
      nxt = place(t + 1, i_nxt);
      request(nxt, buf ^ 1);
    }
    i_nxt = block_of(t + 2);
    const unsigned qa = lds_address(qbuf(buf)), ga = lds_address(gbuf(buf));
    const unsigned st = lds_address(stat + buf * 128 + 32 * rh + 4 * g);
    // S = Q K^T and dP = dO V^T: this wave's 32 rows x its 32 keys; alpha P and dS = P (.) (alpha dP - D^s), as B-operand
    // fragments over the 32 rows (token order).  One stream of LDS reads, kAhead of them in flight: the operand reads, each
    // feeding one product, and among them the row quantities - L of four rows behind every KS / 4 products of dP, whose
    // exponentials then run beside the products, and D^s at the end (12 heads of 32,760 tokens: 860 -> 852 us).  Keys past the end of a short key block need no
    // mask: their columns mix with no others and are not stored.
    f32x16 sacc, dpacc;
    bf16x8 pf[2], dsf[2];
#pragma unroll
    for (int e = 0; e < 16; e++) { sacc[e] = 0.f; dpacc[e] = 0.f; }
    {
      constexpr int kGroup = KS / 4 + 1, kItems = KS + 4 * kGroup + 4, kAhead = 4, kSlots = kAhead + 1;
      u32x4 ring[kSlots];
      auto pin = [](bf16x8& f) {                       // converted here: eight registers less than the fp32 values
        u32x4 u = __builtin_bit_cast(u32x4, f);
        settle(u);
        f = __builtin_bit_cast(bf16x8, u);
      };
      // items: KS of S; four groups of (KS / 4 of dP, L of rows 8 v4 + 4 g ..); D^s of the same rows, v4 = 0 .. 3
      auto issue = [&](int n) {
        const int m = n - KS, v4 = m / kGroup;
        if (n < KS) ring[n % kSlots] = lds_read16_untracked<0>((qa + b_off) ^ (32u * n));
        else if (m >= 4 * kGroup) ring[n % kSlots] = stat_read(st, 8 + m - 4 * kGroup);
        else if (m % kGroup == kGroup - 1) ring[n % kSlots] = stat_read(st, v4);
        else ring[n % kSlots] = lds_read16_untracked<0>((ga + b_off) ^ (32u * (v4 * (kGroup - 1) + m % kGroup)));
      };
#pragma unroll
      for (int n = 0; n < kAhead; n++) issue(n);
#pragma unroll
      for (int n = 0; n < kItems; n++) {
        if (n + kAhead < kItems) issue(n + kAhead);
        wait_lgkmcnt(n + kAhead < kItems ? kAhead : kItems - 1 - n);
        settle(ring[n % kSlots]);
        const int m = n - KS, v4 = m / kGroup;
        if (n < KS) {
          sacc = mfma_bf16(__builtin_bit_cast(bf16x8, ring[n % kSlots]), kfr[n], sacc);
        } else if (m >= 4 * kGroup) {
          const int q = m - 4 * kGroup;
          const f32x4 d4 = __builtin_bit_cast(f32x4, ring[n % kSlots]);
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int e = 4 * q + r;
            pf[q / 2][e % 8] = (__bf16)(cur.al * sacc[e]);
            dsf[q / 2][e % 8] = (__bf16)(sacc[e] * (cur.al * dpacc[e] - d4[r]));
          }
          if (q % 2 == 1) {
            pin(pf[q / 2]);
            pin(dsf[q / 2]);
          }
        } else if (m % kGroup == kGroup - 1) {
          const f32x4 l4 = __builtin_bit_cast(f32x4, ring[n % kSlots]);
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int e = 4 * v4 + r;
            float p = fast_exp2(sacc[e] * c0 - l4[r]);
            settle(p);                                 // here, not where the compiler would gather them
            sacc[e] = p;
          }
        } else {
          const int ks = v4 * (kGroup - 1) + m % kGroup;
          dpacc = mfma_bf16(__builtin_bit_cast(bf16x8, ring[n % kSlots]), vfr[ks], dpacc);
        }
      }
    }
    // dV^T += dO^T (alpha P), dK'^T += Q^T dS: contraction over the 32 rows.  Fragment n: 16-row step, tensor, channel tile.
    {
      constexpr int kFrags = 4 * ET, kAhead = 3, kSlots = kAhead + 1;
      u32x2 lo[kSlots], hi[kSlots];
      auto issue = [&](int n) {
        const int ks = n / (2 * ET), et = n % ET;
        const unsigned base = (n / ET) % 2 == 0 ? ga : qa;
        lo[n % kSlots] = lds_read_tr_untracked_at<32 * D>((base + a_lo) ^ (64u * et), ks);
        hi[n % kSlots] = lds_read_tr_untracked_at<32 * D>((base + a_hi) ^ (64u * et), ks);
      };
#pragma unroll
      for (int n = 0; n < kAhead; n++) issue(n);
#pragma unroll
      for (int n = 0; n < kFrags; n++) {
        if (n + kAhead < kFrags) issue(n + kAhead);
        wait_lgkmcnt(2 * (n + kAhead < kFrags ? kAhead : kFrags - 1 - n));
        settle(lo[n % kSlots]);
        settle(hi[n % kSlots]);
        const u32x4 v4 = {lo[n % kSlots][0], lo[n % kSlots][1], hi[n % kSlots][0], hi[n % kSlots][1]};
        const bf16x8 f = __builtin_bit_cast(bf16x8, v4);
        const int ks = n / (2 * ET), et = n % ET;
        if ((n / ET) % 2 == 0) dvall[et] = mfma_bf16(f, pf[ks], dvall[et]);
        else dkall[et] = mfma_bf16(f, dsf[ks], dkall[et]);
      }
    }
    wait_vmcnt<0>();                                 // the next step's rows have landed ...
    asm volatile("s_barrier" ::: "memory");          // ... for everyone; this step's tiles are free
    cur = nxt;
  }

  // the two row halves add up: each wave finishes half of the channel tiles and hands the other half over
  const int ln = (int)lane_again(), thread = w * kWave + ln;   // (not kept through the loop)
  f32x16 dvacc[CT], dkacc[CT];
  {
    float* mine = reinterpret_cast<float*>(smem) + (size_t)w * (2 * CT * 16 * kWave) + ln;
    const float* other = reinterpret_cast<float*>(smem) + (size_t)(w ^ 1) * (2 * CT * 16 * kWave) + ln;
    auto exchange = [&](auto half) {
      constexpr int E0 = decltype(half)::value * CT, F0 = CT - E0;
      __syncthreads();                               // the last step fully consumed
#pragma unroll
      for (int x = 0; x < CT; x++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          mine[(x * 16 + e) * kWave] = dvall[F0 + x][e];
          mine[((CT + x) * 16 + e) * kWave] = dkall[F0 + x][e];
        }
      __syncthreads();
#pragma unroll
      for (int x = 0; x < CT; x++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          dvacc[x][e] = dvall[E0 + x][e] + other[(x * 16 + e) * kWave];
          dkacc[x][e] = dkall[E0 + x][e] + other[((CT + x) * 16 + e) * kWave];
        }
    };
    if (rh == 0) exchange(std::integral_constant<int, 0>());
    else exchange(std::integral_constant<int, 1>());
  }
  __syncthreads();                                   // the halves have been read

  uint16_t* okt = reinterpret_cast<uint16_t*>(smem);                     // dK' [key][c], then dV [key][e] behind it, row stride LD
  uint16_t* ovt = okt + 64 * LD;
  {
#pragma unroll
    for (int x = 0; x < CT; x++) {
      const int ct = CT * rh + x;
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        bf16x4 pk, pv;
#pragma unroll
        for (int r = 0; r < 4; r++) {
          pk[r] = (__bf16)(dkacc[x][4 * v4 + r] * rscale);
          pv[r] = (__bf16)dvacc[x][4 * v4 + r];
        }
        *reinterpret_cast<bf16x4*>(okt + (32 * kh + ln % 32) * LD + 32 * ct + 8 * v4 + 4 * (ln / 32)) = pk;
        *reinterpret_cast<bf16x4*>(ovt + (32 * kh + ln % 32) * LD + 32 * ct + 8 * v4 + 4 * (ln / 32)) = pv;
      }
    }
  }
  __syncthreads();
  {
    uint16_t* dkh = dk + head_offset(sin, bh, H) + (size_t)t0 * tok_stride;
    uint16_t* dvh = dv + head_offset(sin, bh, H) + (size_t)t0 * tok_stride;
    for (int idx = thread; idx < kTileTokens * (D / 8); idx += NT) {
      const int t = idx / (D / 8), ch = idx % (D / 8);
      if (t < valid) {
        *reinterpret_cast<u32x4*>(dkh + (size_t)t * tok_stride + 8 * ch) = *reinterpret_cast<const u32x4*>(okt + t * LD + 8 * ch);
        store_streamed(reinterpret_cast<u32x4*>(dvh + (size_t)t * tok_stride + 8 * ch), *reinterpret_cast<const u32x4*>(ovt + t * LD + 8 * ch));
      }
    }
    // column sums of dK' (as stored) for the smoothing term: two channels and 64 / kParts rows per thread
    constexpr int kParts = 2 * NT / D, kRows = 64 / kParts;
    const int c2 = thread % (D / 2), part = thread / (D / 2);
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int y = 0; y < kRows; y++) {
      const int t = part * kRows + y;
      const unsigned two = *reinterpret_cast<const unsigned*>(okt + t * LD + 2 * c2);
      s0 += t < valid ? bf16_bits_to_f32((uint16_t)two) : 0.f;
      s1 += t < valid ? bf16_bits_to_f32((uint16_t)(two >> 16)) : 0.f;
    }
    *reinterpret_cast<float2*>(stat + part * D + 2 * c2) = float2{s0, s1};
    __syncthreads();
    if (thread < D) {
      float sum = 0.f;
#pragma unroll
      for (int y = 0; y < kParts; y++) sum += stat[y * D + thread];
      colsum[((size_t)bh * Tn + j) * D + thread] = sum;
    }
  }
}

template <int D, int BQ>
static hipError_t launch_bwd_kv_mfma(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdKvSmem<D>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_kv_mfma_kernel<D, BQ>, smem); e != hipSuccess) return e;
  bwd_kv_mfma_kernel<D, BQ><<<dim3((unsigned)bwd_kv_grid(s)), 256, smem, stream>>>(
      (const uint16_t*)a.q, (const uint16_t*)a.k, (const uint16_t*)a.v, (const uint16_t*)a.dout, a.lraw, a.ds, a.k_mean,
      a.k_stats, a.col_ptr, a.col_idx, a.order, (const uint16_t*)a.dh_sum, a.dz, a.dz_total, a.alpha, (uint16_t*)a.dk,
      (uint16_t*)a.dv, a.colsum, s.sin, s.sout, s.H, s.N, s.Tm, s.Tn, s.k, s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_bwd_kv_bf16(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (s.d == 128 && s.bq == 128) return launch_bwd_kv_mfma<128, 128>(s, a, stream);
  if (s.d == 128 && s.bq == 64) return launch_bwd_kv_mfma<128, 64>(s, a, stream);
  if (s.d == 64 && s.bq == 128) return launch_bwd_kv_mfma<64, 128>(s, a, stream);
  return launch_bwd_kv_mfma<64, 64>(s, a, stream);
}

hipError_t launch_bwd_q_bf16(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (s.d == 128 && s.bq == 128) return launch_bwd_q_mfma<128, 128>(s, a, stream);
  if (s.d == 128 && s.bq == 64) return launch_bwd_q_mfma<128, 64>(s, a, stream);
  if (s.d == 64 && s.bq == 128) return launch_bwd_q_mfma<64, 128>(s, a, stream);
  return launch_bwd_q_mfma<64, 64>(s, a, stream);
}

}  // namespace sla2
