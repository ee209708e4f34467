// The heavy steps of the backward pass for fp32 tensors (Alg. 3 of the paper's appendix with the steps it leaves to
// automatic differentiation written out): products on the fp32 matrix instruction, everything fp32 (f32_tiles.h).
//
//   bwd_q_f32     one workgroup per 32 rows of a query block i:  D^s, D^l, d alpha;  over the selected key blocks, scores
//                 transposed as in the forward kernel (a lane owns a query row):  P^T = exp(S^T - L), dP^T = V dO^T,
//                 dS^T = P^T (.) (alpha dP^T - D^s), dQ^T += K'^T dS^T;  then from the H_i, Z_i the forward pass kept
//                 dQ^phi^T = ((1 - alpha) H_i dO^T - Z_i D^l^T) / (Q^phi Z_i), dQ += softmax-backward(dQ^phi).
//   bwd_state_f32 one workgroup per query block:  dH_i = (1 - alpha) (Q^phi / (Q^phi Z_i))^T dO, dZ_i;  and the order of work
//                 of bwd_kv_f32 (work_order.h).  Then dH_j, dZ_j, their sums over the query blocks that did not select key
//                 block j (the M_c[i, j] = 0 sum of Alg. 3): masked_states_f32 in sla2_f32.hip.
//   bwd_kv_f32    one workgroup per 32 keys of a key block j, over the query blocks that selected it:  S = Q K'^T (a lane
//                 owns a key), dV^T += dO^T (alpha P), dK'^T += Q^T dS;  then dK^phi^T = dH_j V^T + dZ_j 1^T,
//                 dV^T += dH_j^T K^phi^T, dK' += softmax-backward(dK^phi).
//
// The four waves of a workgroup of bwd_q and bwd_kv share 32 rows (keys) and take every fourth 32-token piece of the list, as
// in the forward kernel: no tile in LDS and no barrier in the loop; what a lane streams, 16-byte pieces of its row or the same
// channels of 16 rows, is requested kStream elements ahead.  The parts meet once, after the loop (meet4).
// 12 heads of 4,096 tokens, d = 128, 128-row blocks, 6 of 64 blocks a list, against 128-row (64-key) workgroups with the tiles
// in LDS between two barriers, two waves to each 32 rows: bwd_q 235 -> 164 us
// and bwd_state 36, bwd_kv 290 -> 222 us and the sums of states 21 (the gathers of dH_i and lists of unequal length took their
// time at the end of few workgroups).  A longer list costs bwd_q 18.3 us a block and bwd_kv 22.0, where the products alone take
// 16.0 and 21.4; without a list they take 51 and 71 us, which is HBM and the meeting of the parts.
#include "bwd_columns.h"
#include "f32_tiles.h"
#include "work_order.h"

namespace sla2 {

template <int D> struct BwdQF32Smem {
  static constexpr int LD = kF32Ld<D>;
  // query rows and dO rows; after the loop, when both are consumed, the parts of dQ^T
  static constexpr int kRounds = D / 64;                                   // of meet4
  static constexpr int kDoOff = 32 * LD;
  static constexpr int kRowsEnd = 2 * 32 * LD;
  static constexpr int kA = kRowsEnd > kMeetFloats<D, kRounds> ? kRowsEnd : kMeetFloats<D, kRounds>;
  static constexpr int kLSwapOff = kA;
  static constexpr int kMuOff = kLSwapOff + StatePart<D>::kLds;            // [D] colmean(K)
  static constexpr int kZsOff = kMuOff + D;                                // [D] Z_i
  static constexpr int kRowOff = kZsOff + D;                               // [3][32] dO . O^s, dO . O^l, their difference
  static constexpr int kDotOff = kRowOff + 96;                             // [4][32] parts of row sums
  static constexpr int kBytes = (kDotOff + 128) * (int)sizeof(float);
  static_assert(kBytes <= 80 * 1024, "two workgroups a CU");
  static_assert(kBwdColumnsLds <= kBytes, "the lists are made by workgroups of the same launch");
};

template <int D>
__global__ __launch_bounds__(256, 2) void bwd_q_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ o_s, const float* __restrict__ o_l, const float* __restrict__ lse,
    const double* __restrict__ k_mean, const float* __restrict__ h_i, const float* __restrict__ z_i,
    const int32_t* __restrict__ block_idx, const float* __restrict__ alpha, float* __restrict__ dq, float* __restrict__ ds_out,
    float* __restrict__ l2_out, float* __restrict__ inv_den_out, float* __restrict__ dl_out, float* __restrict__ dalpha_part,
    Strides sin, Strides sout, int BH, int H, int N, int Tm, int Tn, int bq, int ksel, int alpha_per_block,
    BwdColumns columns) {
  typedef BwdQF32Smem<D> SM;
  typedef StatePart<D> SP;
  constexpr int LD = SM::LD, ET = D / 32, J = D / 8, NW = 4;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  if ((int)blockIdx.x < columns.blocks) return bwd_columns_job<256>(columns, blockIdx.x, reinterpret_cast<unsigned char*>(smem));
  const int block = blockIdx.x - columns.blocks;
  float* qs = smem;
  float* dos = smem + SM::kDoOff;
  float* mus = smem + SM::kMuOff;
  float* zs = smem + SM::kZsOff;
  float* rows = smem + SM::kRowOff;
  float* dots = smem + SM::kDotOff;

  const int groups = (N + 31) / 32, all = BH * groups, run = (all + kXcds - 1) / kXcds;   // as in the forward kernel
  const int at = block % kXcds * run + block / kXcds;
  if (at >= all) return;
  const int bh = at / groups, grp = at % groups, h = bh % H;
  const int row0 = 32 * grp, rows_valid = min(32, N - row0), i = row0 / bq;
  const size_t slot = (size_t)bh * Tm + i;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, r = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool row_ok = r < rows_valid;
  const float* kh = k + head_offset(sin, bh, H);
  const float* vh = v + head_offset(sin, bh, H);
  const int32_t* sel = block_idx + slot * ksel;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
  const float rscale = rsqrtf((float)D);

  typedef ChunkMap<D, 256, 32> QM;
  {  // Q and dO into LDS (dO: zero rows past the end), dO . O^s and dO . O^l per row
    const int ch = tid % QM::kChunks, trow = tid / QM::kChunks;
    f32x4 qr[QM::kLoads], gr[QM::kLoads], sr[QM::kLoads], lr[QM::kLoads];
    QM::load(qr, q + head_offset(sin, bh, H) + (size_t)row0 * sin.n, sin.n, rows_valid, tid);
    QM::load(gr, dout + head_offset(sout, bh, H) + (size_t)row0 * sout.n, sout.n, rows_valid, tid);
    QM::load(sr, o_s + ((size_t)bh * N + row0) * D, D, rows_valid, tid);
    QM::load(lr, o_l + ((size_t)bh * N + row0) * D, D, rows_valid, tid);
    if (tid < D) {
      mus[tid] = (float)k_mean[(size_t)bh * D + tid];
      zs[tid] = z_i[slot * D + tid];
    }
#pragma unroll
    for (int y = 0; y < QM::kLoads; y++) {
      const int row = trow + y * QM::kRows;
      const float keep = row < rows_valid ? 1.f : 0.f;
      gr[y] *= keep;
      *reinterpret_cast<f32x4*>(qs + row * LD + 4 * ch) = qr[y];
      *reinterpret_cast<f32x4*>(dos + row * LD + 4 * ch) = gr[y];
      float s_s = 0.f, s_l = 0.f, mix = 0.f;
#pragma unroll
      for (int c = 0; c < 4; c++) {
        s_s += gr[y][c] * sr[y][c];
        s_l += gr[y][c] * lr[y][c];
        mix += gr[y][c] * (sr[y][c] - lr[y][c]);
      }
      s_s = QM::row_sum(s_s);
      s_l = QM::row_sum(s_l);
      mix = QM::row_sum(mix);
      if (ch == 0) {
        rows[row] = s_s;
        rows[32 + row] = s_l;
        rows[64 + row] = mix;
      }
    }
  }
  const int items = 2 * ksel;             // halves of the selected blocks; an odd one of the last block may hold no key
  auto first_key = [&](int t) { return __builtin_amdgcn_readfirstlane(sel[t / 2]) * kF32Tokens + 32 * (t % 2); };
  auto rows_of = [&](const float* head, int first) { return RowPieces(head, first, N - 1, sin.n); };
  int t = w, key0 = 0;
  f32x4 st[kStream];                      // per piece of 32 keys: J elements of K by lane, J of V, J of the columns of K
  if (t < items) {
    key0 = first_key(t);
    const RowPieces kp = rows_of(kh, key0);
    const unsigned own = kp.own(r, g);
#pragma unroll
    for (int n = 0; n < kStream; n++) st[n] = kp.piece(own, n);
  }
  const float L2 = lse[(size_t)bh * N + row0 + min(r, rows_valid - 1)] * kLog2e;
  f32x16 dqacc[ET];
#pragma unroll
  for (int e = 0; e < ET; e++) dqacc[e] = zero16();
  const float c0 = kLog2e * rscale;
  const float *qrow = qs + r * LD + 4 * g, *grow = dos + r * LD + 4 * g, *mrow = mus + 4 * g;
  const int j0 = SP::first(w);            // H_i: channels c of dQ^phi by rows, contracted over e
  const float* hsrc = h_i + slot * D * D + (size_t)(32 * SP::tile(w) + SP::row(r)) * D + 8 * j0 + 4 * g;
  __syncthreads();
  const float Ds = al * rows[r], Dl = (1.f - al) * rows[32 + r];
  if (w == 0) {                           // d alpha: the sum over the tokens of dO . (O^s - O^l)
    float x = g == 0 ? rows[64 + r] : 0.f;
    x = wave_sum(x);
    const int parts = bq / 32, part = grp % parts;
    if (lane == 0) dalpha_part[slot * parts + part] = x;
    if (grp == groups - 1 && lane > part && lane < parts) dalpha_part[slot * parts + lane] = 0.f;   // groups past the end
  }
  if (w == 0 && g == 0) {                 // as the key-side kernel uses them: rows past the end get exp2(-inf) = 0 there
    ds_out[slot * bq + row0 % bq + r] = row_ok ? Ds : 0.f;
    l2_out[slot * bq + row0 % bq + r] = row_ok ? L2 : INFINITY;
    dl_out[slot * bq + row0 % bq + r] = row_ok ? Dl : 0.f;
  }
  f32x4 mc;                               // colmean(K) as it meets an element of the columns
#pragma unroll
  for (int x = 0; x < 4; x++) mc[x] = mus[ET * r + x % ET];

  int key_next = t + NW < items ? first_key(t + NW) : 0;
  auto pass = [&](auto more) {
    constexpr bool MORE = decltype(more)::value;
    const int valid = N - key0;
    const RowPieces kp = rows_of(kh, key0), vp = rows_of(vh, key0), np = rows_of(kh, MORE ? key_next : key0);
    const unsigned own_k = kp.own(r, g), own_v = vp.own(r, g), own_n = np.own(r, g);
    auto request = [&](int n) {           // element n of the piece, behind the last one of the next
      const int j = n % J;
      if (n < J) st[n % kStream] = kp.piece(own_k, j);
      else if (n < 2 * J) st[n % kStream] = vp.piece(own_v, j);
      else if (n < 3 * J) st[n % kStream] = kp.cols<D>(j, r, g);
      else if (MORE) st[n % kStream] = np.piece(own_n, j);
    };
    f32x16 ds = zero16(), dp = zero16();
    f32x4 bb = *reinterpret_cast<const f32x4*>(qrow), mb = *reinterpret_cast<const f32x4*>(mrow);
#pragma unroll
    for (int j = 0; j < J; j++) {         // S^T = K' Q^T
      const f32x4 a = st[j % kStream] - mb, b = bb;
      bb = *reinterpret_cast<const f32x4*>(j + 1 < J ? qrow + 8 * (j + 1) : grow);
      if (j + 1 < J) mb = *reinterpret_cast<const f32x4*>(mrow + 8 * (j + 1));
#pragma unroll
      for (int x = 0; x < 4; x++) ds = mfma_f32(a[x], b[x], ds);
      __builtin_amdgcn_sched_barrier(0);
      request(j + kStream);
    }
#pragma unroll
    for (int j = 0; j < J; j++) {         // dP^T = V dO^T
      const f32x4 a = st[(J + j) % kStream], b = bb;
      if (j + 1 < J) bb = *reinterpret_cast<const f32x4*>(grow + 8 * (j + 1));
#pragma unroll
      for (int x = 0; x < 4; x++) dp = mfma_f32(a[x], b[x], dp);
      __builtin_amdgcn_sched_barrier(0);
      request(J + j + kStream);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const bool ok = row_ok && 8 * (e / 4) + 4 * g + e % 4 < valid;
      float p = exp2_f32(ds[e] * c0 - L2);
      asm volatile("" : "+v"(p));         // taken in any case: no branch around each of them
      ds[e] = (ok ? p : 0.f) * (al * dp[e] - Ds);
    }
#pragma unroll
    for (int j = 0; j < J; j++) {         // dQ^T += K'^T dS^T
      col_products<D>(dqacc, st[(2 * J + j) % kStream] - mc, ds, j);
      __builtin_amdgcn_sched_barrier(0);
      request(2 * J + j + kStream);
    }
    if constexpr (MORE) {
      key0 = key_next;
      if (t + 2 * NW < items) key_next = first_key(t + 2 * NW);
    }
  };
  for (; t + NW < items; t += NW) pass(std::integral_constant<bool, true>());
  if (t < items) pass(std::integral_constant<bool, false>());
#pragma unroll
  for (int j = 0; j < kStream; j++)
    if (j < SP::kSteps) st[j] = *reinterpret_cast<const f32x4*>(hsrc + 8 * j);

  // ---- linear branch ----
  // Q^phi = softmax_d(Q) of this lane's row: its normaliser, Q^phi Z_i, and the channels this wave owns
  float qm = -INFINITY;
#pragma unroll
  for (int j = 0; j < J; j++) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(qrow + 8 * j);
#pragma unroll
    for (int y = 0; y < 4; y++) qm = fmaxf(qm, x[y]);
  }
  qm = swap_halves_max(qm);
  float qsum = 0.f, den = 0.f;
#pragma unroll
  for (int j = 0; j < J; j++) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(qrow + 8 * j), z = *reinterpret_cast<const f32x4*>(zs + 8 * j + 4 * g);
#pragma unroll
    for (int y = 0; y < 4; y++) {
      const float e = exp2_f32((x[y] - qm) * kLog2e);
      qsum += e;
      den += e * z[y];
    }
  }
  const float qinv = 1.f / swap_halves_sum(qsum);
  den = swap_halves_sum(den) * qinv;
  // every block selected: the linear branch receives and passes no gradient
  const float inv_den = (ksel >= Tn || !row_ok) ? 0.f : 1.f / den;
  if (w == 0 && g == 0) inv_den_out[slot * bq + row0 % bq + r] = inv_den;
  const int c_own = own_channel(D, w, g);
  f32x4 qp[ET];
#pragma unroll
  for (int y = 0; y < ET; y++) {
    qp[y] = *reinterpret_cast<const f32x4*>(qs + r * LD + c_own + 4 * y);
#pragma unroll
    for (int x = 0; x < 4; x++) qp[y][x] = exp2_f32((qp[y][x] - qm) * kLog2e) * qinv;
  }
  f32x16 hacc = zero16();
#pragma unroll
  for (int j = 0; j < SP::kSteps; j++) {
    const f32x4 a = st[j % kStream], b = *reinterpret_cast<const f32x4*>(grow + 8 * (j0 + j));
#pragma unroll
    for (int x = 0; x < 4; x++) hacc = mfma_f32(a[x], b[x], hacc);
    if (j + kStream < SP::kSteps) st[j % kStream] = *reinterpret_cast<const f32x4*>(hsrc + 8 * (j + kStream));
  }
  float dqp[D / 8], dqo[D / 8];
  SP::own(dqp, hacc, smem + SM::kLSwapOff, w, lane);
  float dot = 0.f;
#pragma unroll
  for (int e = 0; e < D / 8; e++) {
    dqp[e] = ((1.f - al) * dqp[e] - Dl * zs[c_own + e]) * inv_den;
    dot += dqp[e] * qp[e / 4][e % 4];
  }
  dot = swap_halves_sum(dot);
  if (g == 0) dots[w * 32 + r] = dot;
  __syncthreads();                        // everyone is done with the Q and dO rows
  meet4<D, SM::kRounds>(dqo, dqacc, 1.f, smem, w, lane);
  dot = (dots[r] + dots[32 + r]) + (dots[64 + r] + dots[96 + r]);
  __syncthreads();                        // the parts have been read: their place takes dQ, to leave in whole rows
#pragma unroll
  for (int y = 0; y < ET; y++) {
    f32x4 o;
#pragma unroll
    for (int x = 0; x < 4; x++) o[x] = dqo[4 * y + x] * rscale + qp[y][x] * (dqp[4 * y + x] - dot);
    *reinterpret_cast<f32x4*>(smem + r * LD + c_own + 4 * y) = o;
  }
  __syncthreads();
#pragma unroll
  for (int y = 0; y < QM::kLoads; y++) {
    const int row = tid / QM::kChunks + y * QM::kRows, c = 4 * (tid % QM::kChunks);
    if (row < rows_valid)
      *reinterpret_cast<f32x4*>(dq + head_offset(sin, bh, H) + (size_t)(row0 + row) * sin.n + c) =
          *reinterpret_cast<const f32x4*>(smem + row * LD + c);
  }
}

// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256, 2) void bwd_state_f32_kernel(const WorkOrder order, const float* __restrict__ q,
                                                               const float* __restrict__ dout, const float* __restrict__ inv_den,
                                                               const float* __restrict__ dl, const float* __restrict__ alpha,
                                                               float* __restrict__ dh, Strides sin, Strides sout, int H, int N,
                                                               int Tm, int bq, int alpha_per_block) {
  constexpr int LD = kF32Ld<D>;
  typedef ChunkMap<D, 256, 64> CM;
  typedef StateSplit<D, 4> SS;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  __shared__ int places[2 * kXcds];
  if ((int)blockIdx.x <= order.groups) return order_job(order, blockIdx.x, reinterpret_cast<int*>(smem), places);
  float* wt = smem;                       // [64][LD] w = Q^phi / (Q^phi Z_i)
  const int slot = blockIdx.x - order.groups - 1, bh = slot / Tm, i = slot % Tm, h = bh % H;
  const int tid = threadIdx.x, lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int ch = tid % CM::kChunks, trow = tid / CM::kChunks;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
  f32x16 hacc[SS::kTiles];
#pragma unroll
  for (int x = 0; x < SS::kTiles; x++) hacc[x] = zero16();
  f32x4 zacc = {0.f, 0.f, 0.f, 0.f};
  const int end = min((i + 1) * bq, N);
  f32x4 qr[CM::kLoads];
  StateProduct<D> sp;                     // dO
  auto fetch = [&](int t0) {
    CM::load(qr, q + head_offset(sin, bh, H) + (size_t)t0 * sin.n, sin.n, min(64, end - t0), tid);
  };
  fetch(i * bq);
#pragma unroll 1
  for (int t0 = i * bq; t0 < end; t0 += 64) {
    const int valid = min(64, end - t0);
    const size_t row = (size_t)slot * bq + t0 % bq;
    sp.begin(dout + head_offset(sout, bh, H) + (size_t)t0 * sout.n, sout.n, valid, w, lane);
    __syncthreads();                      // previous rows fully consumed
#pragma unroll
    for (int y = 0; y < CM::kLoads; y++) {
      const int t = trow + y * CM::kRows;
      const bool ok = t < valid;
      const f32x4 x = qr[y];
      const float m = CM::row_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      f32x4 e;
#pragma unroll
      for (int c = 0; c < 4; c++) e[c] = exp2_f32((x[c] - m) * kLog2e);
      const float sum = CM::row_sum((e[0] + e[1]) + (e[2] + e[3]));
      const float scale = ok ? inv_den[row + t] / sum : 0.f, l = ok ? dl[row + t] : 0.f;
      e *= scale;
      zacc -= e * l;                      // dZ_i = -sum_r w[r] D^l_r
      *reinterpret_cast<f32x4*>(wt + t * LD + 4 * ch) = e;
    }
    if (t0 + 64 < end) fetch(t0 + 64);
    __syncthreads();
    sp.add(hacc, wt, w, lane);
  }
  float* out = dh + (size_t)slot * (D * D + D);
  StateProduct<D>::store(hacc, 1.f - al, out, w, lane);
  __syncthreads();                        // the last rows fully consumed: their place takes the column sums
  *reinterpret_cast<f32x4*>(wt + trow * D + 4 * ch) = zacc;
  __syncthreads();
  if (tid < D) {
    float z = 0.f;
#pragma unroll
    for (int y = 0; y < CM::kRows; y++) z += wt[y * D + tid];
    out[D * D + tid] = z;
  }
}

// ---------------------------------------------------------------------------------------------
template <int D> struct BwdKvF32Smem {
  static constexpr int LD = kF32Ld<D>;
  // K' (later K^phi) and V rows; the parts of dV^T and of dK^T, then dK'
  static constexpr int kRounds = D / 64;                                   // of meet4: two workgroups a CU
  static constexpr int kVOff = 32 * LD, kSwapOff = 2 * 32 * LD;
  static constexpr int kA = kSwapOff + kMeetFloats<D, kRounds>;
  static constexpr int kLSwapOff = kA;
  static constexpr int kStatOff = kLSwapOff + StatePart<D>::kLds;          // [4 waves][2][32] L log2(e) and D^s of a piece's rows
  static constexpr int kDzOff = kStatOff + 256;                            // [D] dZ_j
  static constexpr int kDotOff = kDzOff + D;                               // [4][32] parts of row sums
  static constexpr int kBytes = (kDotOff + 128) * (int)sizeof(float);
  static_assert(kBytes <= 80 * 1024, "two workgroups a CU");
  static_assert(32 * LD <= kMeetFloats<D, kRounds>, "dK' takes the place of the parts");
};

template <int D>
__global__ __launch_bounds__(256, 2) void bwd_kv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const float* __restrict__ dout,
    const float* __restrict__ l2_in, const float* __restrict__ ds_in, const double* __restrict__ k_mean,
    const float* __restrict__ k_stats, const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ col_idx,
    const int32_t* __restrict__ order, const float* __restrict__ dh_sum, const float* __restrict__ dz_sum,
    const float* __restrict__ alpha, float* __restrict__ dk, float* __restrict__ dv, float* __restrict__ colsum, Strides sin,
    Strides sout, int H, int N, int Tm, int Tn, int bq, int ksel, int alpha_per_block) {
  typedef BwdKvF32Smem<D> SM;
  typedef StatePart<D> SP;
  constexpr int LD = SM::LD, ET = D / 32, J = D / 8, NW = 4;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* ks = smem;
  float* vs = smem + SM::kVOff;
  float* dzs = smem + SM::kDzOff;
  float* dots = smem + SM::kDotOff;

  // the two halves of a key block next to each other on the block's XCD
  const int y2 = blockIdx.x / kXcds, entry = __builtin_amdgcn_readfirstlane(order[y2 / 2 * kXcds + blockIdx.x % kXcds]);
  if (entry < 0) return;
  const int j = entry & (kMaxKeyBlocks - 1), bh = entry / kMaxKeyBlocks, h = bh % H, half = y2 % 2;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, r = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const size_t sums = (((size_t)bh * Tn + j) * 2 + half) * D;
  const int t0 = j * kF32Tokens + 32 * half, valid = min(32, N - t0);
  if (valid <= 0) {                       // no key in this half of the last block
    if (tid < D) colsum[sums + tid] = 0.f;
    return;
  }
  float* stat = smem + SM::kStatOff + 64 * w;
  const float* qh = q + head_offset(sin, bh, H);
  const float* doh = dout + head_offset(sout, bh, H);
  const float rscale = rsqrtf((float)D), c0 = kLog2e * rscale;

  const int32_t* cp = col_ptr + (size_t)bh * (Tn + 1);
  const int l0 = __builtin_amdgcn_readfirstlane(cp[j]), listed = __builtin_amdgcn_readfirstlane(cp[j + 1]) - l0;
  const int32_t* ci = col_idx + (size_t)bh * Tm * ksel + l0;   // the query blocks that selected this key block
  const int per = bq / 32;
  // Piece t: rows [32 (t % per), +32) of query block ci[t / per].  Rows past the end repeat the last one; their L is +inf,
  // so their probabilities are 0.  A piece with no row at all (only in the last query block) has the last row throughout.
  const int items = listed * per;
  typedef ChunkMap<D, 256, 32> KM;
  const int ch = tid % KM::kChunks, trow = tid / KM::kChunks;
  {
    f32x4 kr[KM::kLoads], vr[KM::kLoads], mu;
    KM::load(kr, k + head_offset(sin, bh, H) + (size_t)t0 * sin.n, sin.n, valid, tid);
    KM::load(vr, v + head_offset(sin, bh, H) + (size_t)t0 * sin.n, sin.n, valid, tid);
#pragma unroll
    for (int x = 0; x < 4; x++) mu[x] = (float)k_mean[(size_t)bh * D + 4 * ch + x];
    if (tid < D) dzs[tid] = ksel >= Tn ? 0.f : dz_sum[((size_t)bh * Tn + j) * D + tid];
#pragma unroll
    for (int y = 0; y < KM::kLoads; y++) {
      *reinterpret_cast<f32x4*>(ks + (trow + y * KM::kRows) * LD + 4 * ch) = kr[y] - mu;
      *reinterpret_cast<f32x4*>(vs + (trow + y * KM::kRows) * LD + 4 * ch) = vr[y];
    }
  }
  f32x16 dvacc[ET], dkacc[ET];
#pragma unroll
  for (int e = 0; e < ET; e++) { dvacc[e] = zero16(); dkacc[e] = zero16(); }
  const float *krow = ks + r * LD + 4 * g, *vrow = vs + r * LD + 4 * g;
  f32x4 st[kStream];                      // per piece: J elements of Q by lane, J of dO, J of the columns of dO, J of those of Q
  int t = w, i = 0, i_next = 0;
  auto block_of = [&](int x) { return __builtin_amdgcn_readfirstlane(ci[x / per]); };
  auto first_row = [&](int x, int block) { return block * bq + 32 * (x % per); };
  auto row_stat = [&](int r0) {           // L log2(e) (g = 0) or D^s (g = 1) of a row of the piece
    const size_t row = (size_t)bh * Tm * bq + min(r0 + r, N - 1);
    const float x = g == 0 ? l2_in[row] : ds_in[row];
    return r0 + r < N ? x : g == 0 ? INFINITY : 0.f;
  };
  float stat_next = 0.f;
  if (t < items) {
    i = block_of(t);
    const RowPieces qp(qh, first_row(t, i), N - 1, sin.n);
    const unsigned own = qp.own(r, g);
#pragma unroll
    for (int n = 0; n < kStream; n++) st[n] = qp.piece(own, n);
    stat_next = row_stat(first_row(t, i));
    if (t + NW < items) i_next = block_of(t + NW);
  }
  __syncthreads();

  auto pass = [&](auto more) {
    constexpr bool MORE = decltype(more)::value;
    const int r0 = first_row(t, i), r0_next = MORE ? first_row(t + NW, i_next) : r0;
    const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
    stat[32 * g + r] = stat_next;
    if constexpr (MORE) stat_next = row_stat(r0_next);
    const RowPieces qp(qh, r0, N - 1, sin.n), gp(doh, r0, N - 1, sout.n), np(qh, r0_next, N - 1, sin.n);
    const unsigned own_q = qp.own(r, g), own_g = gp.own(r, g), own_n = np.own(r, g);
    auto request = [&](int n) {           // element n of the piece, behind the last one of the next
      const int x = n % J;
      if (n < J) st[n % kStream] = qp.piece(own_q, x);
      else if (n < 2 * J) st[n % kStream] = gp.piece(own_g, x);
      else if (n < 3 * J) st[n % kStream] = gp.cols<D>(x, r, g);
      else if (n < 4 * J) st[n % kStream] = qp.cols<D>(x, r, g);
      else if (MORE) st[n % kStream] = np.piece(own_n, x);
    };
    f32x16 p = zero16(), ds = zero16();
    f32x4 bb = *reinterpret_cast<const f32x4*>(krow);
#pragma unroll
    for (int x = 0; x < J; x++) {         // S = Q K'^T
      const f32x4 a = st[x % kStream], b = bb;
      bb = *reinterpret_cast<const f32x4*>(x + 1 < J ? krow + 8 * (x + 1) : vrow);
#pragma unroll
      for (int y = 0; y < 4; y++) p = mfma_f32(a[y], b[y], p);
      __builtin_amdgcn_sched_barrier(0);
      request(x + kStream);
    }
    wave_lds_fence();
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const f32x4 l4 = *reinterpret_cast<const f32x4*>(stat + 8 * v4 + 4 * g);
#pragma unroll
      for (int y = 0; y < 4; y++) p[4 * v4 + y] = exp2_f32(p[4 * v4 + y] * c0 - l4[y]);   // keys past the end: columns of their own, not stored
    }
#pragma unroll
    for (int x = 0; x < J; x++) {         // dP = dO V^T
      const f32x4 a = st[(J + x) % kStream], b = bb;
      if (x + 1 < J) bb = *reinterpret_cast<const f32x4*>(vrow + 8 * (x + 1));
#pragma unroll
      for (int y = 0; y < 4; y++) ds = mfma_f32(a[y], b[y], ds);
      __builtin_amdgcn_sched_barrier(0);
      request(J + x + kStream);
    }
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const f32x4 d4 = *reinterpret_cast<const f32x4*>(stat + 32 + 8 * v4 + 4 * g);
#pragma unroll
      for (int y = 0; y < 4; y++) {
        const int e = 4 * v4 + y;
        ds[e] = p[e] * (al * ds[e] - d4[y]);
        p[e] *= al;
      }
    }
    wave_lds_fence();                     // read before the next piece's take their place
#pragma unroll
    for (int x = 0; x < J; x++) {         // dV^T += dO^T (alpha P)
      col_products<D>(dvacc, st[(2 * J + x) % kStream], p, x);
      __builtin_amdgcn_sched_barrier(0);
      request(2 * J + x + kStream);
    }
#pragma unroll
    for (int x = 0; x < J; x++) {         // dK'^T += Q^T dS
      col_products<D>(dkacc, st[(3 * J + x) % kStream], ds, x);
      __builtin_amdgcn_sched_barrier(0);
      request(3 * J + x + kStream);
    }
    if constexpr (MORE) {
      i = i_next;
      if (t + 2 * NW < items) i_next = block_of(t + 2 * NW);
    }
  };
  for (; t + NW < items; t += NW) pass(std::integral_constant<bool, true>());
  if (t < items) pass(std::integral_constant<bool, false>());

  // ---- linear branch ----
  const bool all_selected = ksel >= Tn;   // no gradient, whatever dO holds
  const int j0 = SP::first(w), tile = SP::tile(w), c_own = own_channel(D, w, g);
  const float* dhj = dh_sum + ((size_t)bh * Tn + j) * D * D;
  f32x4 hf[SP::kSteps];                   // dH_j: channels c of dK^phi by rows, contracted over e
  {
    const float* src = dhj + (size_t)(32 * tile + SP::row(r)) * D + 8 * j0 + 4 * g;
#pragma unroll
    for (int x = 0; x < SP::kSteps; x++) hf[x] = *reinterpret_cast<const f32x4*>(src + 8 * x);
  }
  float dvo[D / 8], dko[D / 8];
  float* swap = smem + SM::kSwapOff;
  meet4<D, SM::kRounds>(dvo, dvacc, 1.f, swap, w, lane);
  __syncthreads();                        // everyone is done with K', and the parts have been read
  meet4<D, SM::kRounds>(dko, dkacc, 1.f, swap, w, lane);
#pragma unroll
  for (int y = 0; y < KM::kLoads; y++) {  // K' -> K^phi = exp(K' - lnZ) (keys past the end: 0)
    const int row = trow + y * KM::kRows;
    const float lnz = k_stats[(size_t)bh * N + t0 + min(row, valid - 1)];
    f32x4 x = *reinterpret_cast<const f32x4*>(ks + row * LD + 4 * ch);
#pragma unroll
    for (int c = 0; c < 4; c++) {
      float p = exp2_f32((x[c] - lnz) * kLog2e);
      asm volatile("" : "+v"(p));         // taken in any case: no branch around each of them
      x[c] = row < valid ? p : 0.f;
    }
    *reinterpret_cast<f32x4*>(ks + row * LD + 4 * ch) = x;
  }
  f32x16 acc = zero16();
#pragma unroll
  for (int x = 0; x < SP::kSteps; x++) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(vrow + 8 * (j0 + x));
#pragma unroll
    for (int y = 0; y < 4; y++) acc = mfma_f32(all_selected ? 0.f : hf[x][y], b[y], acc);
  }
  {  // dH_j^T: channels e of dV by rows, contracted over c
    const float* src = dhj + (size_t)(8 * j0 + 4 * g) * D + 32 * tile + SP::row(r);
#pragma unroll
    for (int x = 0; x < SP::kSteps; x++)
#pragma unroll
      for (int y = 0; y < 4; y++) hf[x][y] = src[(8 * x + y) * D];
  }
  float dkp[D / 8], dvl[D / 8];
  SP::own(dkp, acc, smem + SM::kLSwapOff, w, lane);
  __syncthreads();                        // K^phi complete
  acc = zero16();
#pragma unroll
  for (int x = 0; x < SP::kSteps; x++) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(krow + 8 * (j0 + x));
#pragma unroll
    for (int y = 0; y < 4; y++) acc = mfma_f32(all_selected ? 0.f : hf[x][y], b[y], acc);
  }
  SP::own(dvl, acc, smem + SM::kLSwapOff, w, lane);
  f32x4 kp[ET];
  float dot = 0.f;
#pragma unroll
  for (int y = 0; y < ET; y++) {
    kp[y] = *reinterpret_cast<const f32x4*>(ks + r * LD + c_own + 4 * y);
#pragma unroll
    for (int x = 0; x < 4; x++) {
      dkp[4 * y + x] += dzs[c_own + 4 * y + x];
      dot += dkp[4 * y + x] * kp[y][x];
    }
  }
  dot = swap_halves_sum(dot);
  if (g == 0) dots[w * 32 + r] = dot;
  __syncthreads();                        // the row sums are there
  dot = (dots[r] + dots[32 + r]) + (dots[64 + r] + dots[96 + r]);
#pragma unroll
  for (int y = 0; y < ET; y++) {          // to leave in whole rows
    f32x4 ok, ov;
#pragma unroll
    for (int x = 0; x < 4; x++) {
      ok[x] = dko[4 * y + x] * rscale + kp[y][x] * (dkp[4 * y + x] - dot);
      ov[x] = dvo[4 * y + x] + dvl[4 * y + x];
    }
    *reinterpret_cast<f32x4*>(swap + r * LD + c_own + 4 * y) = r < valid ? ok : f32x4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4*>(vs + r * LD + c_own + 4 * y) = ov;
  }
  __syncthreads();
#pragma unroll
  for (int y = 0; y < KM::kLoads; y++) {
    const int row = trow + y * KM::kRows;
    const size_t dst = head_offset(sin, bh, H) + (size_t)(t0 + row) * sin.n + 4 * ch;
    if (row < valid) {
      *reinterpret_cast<f32x4*>(dk + dst) = *reinterpret_cast<const f32x4*>(swap + row * LD + 4 * ch);
      *reinterpret_cast<f32x4*>(dv + dst) = *reinterpret_cast<const f32x4*>(vs + row * LD + 4 * ch);
    }
  }
  if (tid < D) {                          // column sums of dK' for the smoothing term
    float sum = 0.f;
#pragma unroll
    for (int x = 0; x < 32; x++) sum += swap[x * LD + tid];
    colsum[sums + tid] = sum;
  }
}

// ---------------------------------------------------------------------------------------------
template <int D>
static hipError_t launch_q(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdQF32Smem<D>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_q_f32_kernel<D>, smem); e != hipSuccess) return e;
  const int run = (s.BH * ((s.N + 31) / 32) + kXcds - 1) / kXcds;
  const BwdColumns columns = bwd_columns(s, a);
  bwd_q_f32_kernel<D><<<dim3((unsigned)(columns.blocks + run * kXcds)), 256, smem, stream>>>(
      (const float*)a.q, (const float*)a.k, (const float*)a.v, (const float*)a.dout, (const float*)a.o_s, (const float*)a.o_l,
      a.lse, a.k_mean, (const float*)a.h_i, a.z_i, a.block_idx, a.alpha, (float*)a.dq, a.ds, a.lraw, a.inv_den, a.dl,
      a.dalpha_part, s.sin, s.sout, s.BH, s.H, s.N, s.Tm, s.Tn, s.bq, s.k, s.alpha_per_block ? 1 : 0, columns);
  return hipGetLastError();
}
hipError_t launch_bwd_q_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.d == 128 ? launch_q<128>(s, a, stream) : launch_q<64>(s, a, stream);
}

template <int D>
static hipError_t launch_state(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = 64 * kF32Ld<D> * (int)sizeof(float);
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_state_f32_kernel<D>, smem); e != hipSuccess) return e;
  const WorkOrder o = make_order(s, a);
  bwd_state_f32_kernel<D><<<dim3((unsigned)(1 + o.groups + s.BH * s.Tm)), 256, smem, stream>>>(
      o, (const float*)a.q, (const float*)a.dout, a.inv_den, a.dl, a.alpha, (float*)a.dh, s.sin, s.sout, s.H, s.N, s.Tm, s.bq,
      s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}
hipError_t launch_bwd_totals_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  if (hipError_t e = s.d == 128 ? launch_state<128>(s, a, stream) : launch_state<64>(s, a, stream); e != hipSuccess) return e;
  return launch_key_states_f32(s, a, stream);
}

template <int D>
static hipError_t launch_kv(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  constexpr int smem = BwdKvF32Smem<D>::kBytes;
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)bwd_kv_f32_kernel<D>, smem); e != hipSuccess) return e;
  bwd_kv_f32_kernel<D><<<dim3((unsigned)(2 * bwd_kv_grid(s))), 256, smem, stream>>>(
      (const float*)a.q, (const float*)a.k, (const float*)a.v, (const float*)a.dout, a.lraw, a.ds, a.k_mean, a.k_stats,
      a.col_ptr, a.col_idx, a.order, (const float*)a.dh_sum, a.dz_sum, a.alpha, (float*)a.dk, (float*)a.dv, a.colsum, s.sin,
      s.sout, s.H, s.N, s.Tm, s.Tn, s.bq, s.k, s.alpha_per_block ? 1 : 0);
  return hipGetLastError();
}
hipError_t launch_bwd_kv_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  return s.d == 128 ? launch_kv<128>(s, a, stream) : launch_kv<64>(s, a, stream);
}

}  // namespace sla2
