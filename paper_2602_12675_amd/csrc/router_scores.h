// Router scores of 16 query blocks of one head against all of its key blocks (Eq. 16), fp64 on the matrix cores;
// shared by the hard selection (sla2_router.hip) and the soft one (sla2_router_soft.hip).
//
//   R[i][j] = proj_q(Qbar_i) . proj_k(Kbar_j) / sqrt(d),   proj(x) = x W
//
// Two identities keep the work small.  (1) R = (Qbar M) Kbar^T with M = Wq Wk^T / sqrt(d), a d x d matrix formed once
// per call (fold_router_row, run by spare workgroups of the pooling launch): only the 16 query rows of a workgroup are
// projected, the pooled keys are used as they are.  (2) Kbar is pooled from K - colmean(K), which shifts every score
// of a row by the same amount, (Qbar Wq Wk^T) . colmean(K): neither a row-wise top-k nor a row softmax sees it, so the
// raw block sums of K are scored and the mean never enters.  The scores formed here therefore differ from R by one
// constant per row.
//
// A workgroup has 16 waves.  Scores are formed (v_mfma_f64_16x16x4) 256 key blocks at a time: wave w multiplies the
// projected 16 x d tile with key blocks [256 r + 16 w, +16), parks its 16 x 16 result in LDS, and wave i then picks up
// row i, so that after the last round every wave holds one complete score row in registers (4 values per lane and
// round).  Scores never touch HBM.  Two LDS tiles take the rounds in turn: one barrier a round, and a wave that has its row
// starts on the next products while others still collect (a workgroup has its CU to itself by its registers, so the second
// tile costs no place).
//
// What bounds it: the chain of a workgroup, half of it the fp64 products themselves (64 cycles each), the rest the phases
// between barriers.  The second tile, the divisions left to ragged blocks (they ran for every score before) and the order
// of the workgroups below: soft router on 12 heads of 256 x 512 blocks 73.4 -> 71.1 us with its pooling, selection on 40
// heads of 591 x 1,182 315 -> 309 us, on 2 heads of 16 x 16 (d = 64) the whole forward call 25.2 -> 24.9 us; at 12 heads of 256 x 512
// the hard selection, one workgroup on three quarters of the CUs, is where it was.
#pragma once
#include "common.h"

namespace sla2 {

constexpr int kRouterRows = 16;                       // query blocks per workgroup = waves per workgroup
constexpr int kColsPerRound = 256;                    // key blocks scored per round (16 waves x 16)
typedef __attribute__((ext_vector_type(2))) double f64x2;

template <int D> constexpr size_t router_lds_bytes() {
  return sizeof(double) * (kRouterRows * (D + 2) + 2 * kRouterRows * (kColsPerRound + 8));
}

// The (head, row tile) of a selection workgroup: all of them, head by head, in kXcds runs, one per XCD, so that the workgroups
// that an XCD runs at a time read the pooled keys of a head or two (1.2 MB a head of 1,182 key blocks) from its L2.
__device__ __forceinline__ int router_tile(int block, int blocks) {
  const int x = block % kXcds;
  return x * (blocks / kXcds) + min(x, blocks % kXcds) + block / kXcds;
}

// C[16][D] = A[16][D] M on the matrix cores, M fp64 [D][D] row-major in global memory.  All 16 waves
// work: wave w forms kTiles column tiles over a share of the contraction range; the shares are written side by side (C has room for
// kShares copies) and added by the reader.  At d = 128 a wave has two tiles, the even and the odd ones of 32 columns: 16 bytes of a
// row of M then serve both, and M, 128 KB a workgroup, comes in half as many requests (with them issued in front of the first pooled
// keys: soft router on 12 heads of 256 x 512 blocks 62.2 -> 61.1 us, on 20 heads of 32 x 63 25.7 -> 24.6; behind a fill of 1 GB, with
// nothing left in a cache, 102.7 -> 101.6 and 37.9 -> 36.7).  At d = 64, where M is a quarter of that, it loses 1 %.  The shares decide the
// order in which fp64 sums are added, so scores differ in their last bits between two shares and four; lists and stored masks did not.
template <int D> struct ProjGeom {
  static constexpr int kTiles = D == 128 ? 2 : 1;
  static constexpr int kNt = D / 16 / kTiles;        // column tiles or pairs of them
  static constexpr int kShares = 16 / kNt;           // waves each: 4
  static constexpr int kSteps = D / 4 / kShares;     // 4-wide contraction steps per wave
  typedef __attribute__((ext_vector_type(kTiles))) double Row;
  __device__ static __forceinline__ int col(int wave, int lane) { return kTiles * (16 * (wave % kNt) + lane % 16); }
};
template <int D>
__device__ __forceinline__ void project16_fetch(typename ProjGeom<D>::Row (&b)[ProjGeom<D>::kSteps], const double* __restrict__ M, int wave,
                                                int lane) {
  typedef ProjGeom<D> G;
#pragma unroll
  for (int i = 0; i < G::kSteps; i++)
    b[i] = *reinterpret_cast<const typename G::Row*>(M + (size_t)(4 * (wave / G::kNt * G::kSteps + i) + lane / 16) * D + G::col(wave, lane));
}
template <int D>
__device__ __forceinline__ void project16(const double (*A)[D + 2], double (*C)[D + 2] /* [kShares*16][D+2] */,
                                          const typename ProjGeom<D>::Row (&b)[ProjGeom<D>::kSteps], int wave, int lane) {
  typedef ProjGeom<D> G;
  const int share = wave / G::kNt;
  f64x4 acc[G::kTiles];
#pragma unroll
  for (int x = 0; x < G::kTiles; x++) acc[x] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < G::kSteps; i++) {
    const double a = A[lane % 16][4 * (share * G::kSteps + i) + lane / 16];
#pragma unroll
    for (int x = 0; x < G::kTiles; x++) acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[i][x], acc[x], 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < 4; v++) {
    typename G::Row y;
#pragma unroll
    for (int x = 0; x < G::kTiles; x++) y[x] = acc[x][v];
    *reinterpret_cast<typename G::Row*>(&C[share * 16 + lane / 16 + 4 * v][G::col(wave, lane)]) = y;
  }
}

// Leaves row (row0 + wave) in `score`: slot 4 r + x of lane l is key block 256 r + 64 x + l (slots past T_n hold
// -infinity).  All 16 waves of the workgroup call it; `lds` holds router_lds_bytes<D>().
template <int D, int SLOTS>
__device__ __forceinline__ void router_scores(double (&score)[SLOTS], const double* __restrict__ q_sum,
                                              const double* __restrict__ k_frag, const double* __restrict__ M, double* lds,
                                              int bh, int row0, int N, int bq, int bk, int Tm, int Tn) {
  // LDS: xa [16][D+2] pooled queries, later Qbar M | tile [2][16][264] the scores of a round (the partial projections
  // before the first round)
  double (*xa)[D + 2] = reinterpret_cast<double (*)[D + 2]>(lds);
  typedef double Tile[kRouterRows][kColsPerRound + 8];
  Tile* tiles = reinterpret_cast<Tile*>(lds + kRouterRows * (D + 2));
  static_assert(ProjGeom<D>::kShares * (D + 2) <= 2 * (kColsPerRound + 8), "projection shares must fit the score tiles");
  double (*xb)[D + 2] = reinterpret_cast<double (*)[D + 2]>(&tiles[0][0][0]);   // partial Qbar M; dead before the first round
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int rounds = (Tn + kColsPerRound - 1) / kColsPerRound;

  // Operand B of a round: lane l feeds key block col0 + l % 16.  The contraction runs in an order of its own (the
  // same for both operands): product 2 j + x takes channels 8 j + 2 (l / 16) + x, so that one 16-byte load serves two
  // products; the pooled keys lie in that order (k_frag).  The loads go straight to registers, kBatch of them ahead of
  // the products.
  constexpr int kLoads = D / 8, kBatch = SLOTS > 16 ? 4 : 8;
  f64x2 pre[2][kBatch];
  const double* kb = k_frag + (size_t)bh * Tn * D;
  auto fetch = [&](int r, int batch) {
    const int first = min(r * kColsPerRound + wave * 16, (Tn - 1) / 16 * 16), n = min(16, Tn - first);   // past the end: the last group again
    const double* p = kb + (size_t)first * D + 8 * n * kBatch * batch + 2 * (lane / 16 * n + min(lane % 16, n - 1));
#pragma unroll
    for (int i = 0; i < kBatch; i++) pre[batch & 1][i] = *reinterpret_cast<const f64x2*>(p + 8 * n * i);
  };

  // requested in the order of use: block sums of Q, operands of the projection; the first pooled keys once those are there, behind
  // the projection's products
  constexpr int kQLoads = kRouterRows * D / 1024;
  double qv[kQLoads];
  typename ProjGeom<D>::Row mb[ProjGeom<D>::kSteps];
#pragma unroll
  for (int x = 0; x < kQLoads; x++) {
    const int r = (threadIdx.x + 1024 * x) / D, c = threadIdx.x % D;
    qv[x] = q_sum[((size_t)bh * Tm + min(row0 + r, Tm - 1)) * D + c];     // rows past the end repeat the last one; never stored
  }
  project16_fetch<D>(mb, M, wave, lane);
  // Mean pooling (Eq. 15).  Blocks are powers of two: for full ones the product with 1 / b_q is the exact quotient; only the
  // tile that holds a ragged last block divides.
  const double inv_bq = 1.0 / bq;
  const bool ragged_q = row0 + kRouterRows >= Tm && Tm * bq != N;
#pragma unroll
  for (int x = 0; x < kQLoads; x++) {
    const int r = (threadIdx.x + 1024 * x) / D, c = threadIdx.x % D;
    if (ragged_q) qv[x] /= (double)min(bq, N - min(row0 + r, Tm - 1) * bq);
    else qv[x] *= inv_bq;
    xa[r][c] = qv[x];
  }
  __syncthreads();
  fetch(0, 0);
  project16<D>(xa, xb, mb, wave, lane);                                   // Qbar (Wq Wk^T / sqrt(d)), in shares
  __syncthreads();
  for (int e = threadIdx.x; e < kRouterRows * D; e += 1024) {
    const int r = e / D, c = e % D;
    double v = xb[r][c];
#pragma unroll
    for (int sh = 1; sh < ProjGeom<D>::kShares; sh++) v += xb[sh * 16 + r][c];
    xa[r][c] = v;
  }
  __syncthreads();

#pragma unroll
  for (int s = 0; s < SLOTS; s++) score[s] = -INFINITY;
  const double inv_bk = 1.0 / bk;                      // bk = 64: the product is the exact quotient
  const bool ragged_k = Tn * bk != N;
#pragma unroll
  for (int r = 0; r < SLOTS / 4; r++) {
    if (r < rounds) {
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      if (r * kColsPerRound + wave * 16 < Tn) {        // uniform per wave
#pragma unroll
        for (int b = 0; b < kLoads / kBatch; b++) {
          if (b + 1 < kLoads / kBatch) fetch(r, b + 1);
#pragma unroll
          for (int i = 0; i < kBatch; i++) {
            const f64x2 a = *reinterpret_cast<const f64x2*>(&xa[lane % 16][8 * (b * kBatch + i) + 2 * (lane / 16)]);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], pre[b & 1][i][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], pre[b & 1][i][1], acc, 0, 0, 0);
          }
        }
      }
      if (r + 1 < rounds) fetch(r + 1, 0);
      Tile& tile = tiles[r & 1];
      // result layout: lane l, register v holds C[l/16 + 4 v][l%16]
#pragma unroll
      for (int v = 0; v < 4; v++) tile[lane / 16 + 4 * v][wave * 16 + lane % 16] = acc[v];
      __syncthreads();
      // wave i collects row i; block sums -> block means (only a ragged last block differs)
#pragma unroll
      for (int x = 0; x < 4; x++) {
        const int col = r * kColsPerRound + x * kWave + lane;
        const double sum = tile[wave][x * kWave + lane];
        double sc = sum * inv_bk;
        if (ragged_k && col / kWave == (Tn - 1) / kWave)                  // one slot of the row: the others spend no division
          if (col == Tn - 1) sc = sum / (double)(N - (Tn - 1) * bk);
        score[4 * r + x] = col < Tn ? sc : -INFINITY;
      }
    }
  }
}

}  // namespace sla2
