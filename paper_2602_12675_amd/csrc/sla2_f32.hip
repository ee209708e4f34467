// fp32 path of the SLA2 forward pass (Alg. 2 of the paper), used when q, k, v are stored in fp32.  h_j, z_j of every key
// block are formed once and kept; their sums over the blocks that a query block did not select, H_i and Z_i, come out of a
// product of the selection's complement with all of them; one pass per query block then runs the sparse branch over the
// selected key/value blocks, applies H_i, Z_i and mixes the two branches.  fp32 throughout: products on the fp32 matrix
// instruction (f32_tiles.h).
#include "kv_state_f32.h"

namespace sla2 {

// ---------------------------------------------------------------------------------------------
// kv_state_f32: one workgroup per key block, where the block selection's launch has no room for them
template <int D>
__global__ __launch_bounds__(256, 4) void kv_state_f32_kernel(const KvStateArgs a, const double* __restrict__ k_mean, int H, int N, int Tn) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  kv_state_f32_job<D, false>(a, k_mean, smem, a.first + (int)blockIdx.x, threadIdx.x, H, N, Tn, 1);
}
template <int D>
static hipError_t launch_kv_state_f32_t(const Shape& s, int heads, const KvStateArgs& a, const double* k_mean, hipStream_t stream) {
  constexpr int smem = kKvStateFloats<D> * (int)sizeof(float);
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)kv_state_f32_kernel<D>, smem); e != hipSuccess) return e;
  kv_state_f32_kernel<D><<<dim3((unsigned)(heads * s.Tn)), 256, smem, stream>>>(a, k_mean, s.H, s.N, s.Tn);
  return hipGetLastError();
}
hipError_t launch_kv_state_f32(const Shape& s, const HeadGroup& hg, const float* k, const float* v, const double* k_mean,
                               float* k_stats, float* states, hipStream_t stream) {
  const KvStateArgs a{k, v, k_stats, states, s.sin, hg.bh0 * s.Tn};
  return s.d == 128 ? launch_kv_state_f32_t<128>(s, hg.heads, a, k_mean, stream) : launch_kv_state_f32_t<64>(s, hg.heads, a, k_mean, stream);
}

// ---------------------------------------------------------------------------------------------
// masked_states_f32: sums of states over the blocks that a list does not name - H_i, Z_i over the key blocks that query block
// i did not select, and in the backward pass dH_j, dZ_j over the query blocks that did not select key block j.  A wave forms
// 32 such sums for 128 of the d^2 + d entries of a state: the 32 x S matrix of 0 (listed) and 1 times the S states of the
// head; and the sums over all of them.  A lane has four consecutive entries, so a state is read 512 bytes at a time and
// stored the same way; the mask operand of 32 blocks is one word per lane, put together in LDS from the lists.
// Bound by the states, read once per 32 sums, and the sums written: 18 us on 12 heads of 64 key and 32 query blocks
// (d = 128; 50 MB read, 25 MB written).  The query blocks used to rebuild the h_j of their lists, a third of the products
// of the attention kernel, and to form K^phi of every tile again; the key blocks gathered one dH_i per list entry.
// ---------------------------------------------------------------------------------------------
// R lists a head over S blocks: offsets ptr [R + 1] into idx [S k] (key side), or k entries each (query side, ptr null)
struct BlockLists {
  const int32_t *ptr, *idx;
  int R, S, k;
  __device__ __forceinline__ const int32_t* begin(int bh, int r) const {
    return ptr ? idx + (size_t)bh * S * k + ptr[(size_t)bh * (R + 1) + r] : idx + ((size_t)bh * R + r) * k;
  }
  __device__ __forceinline__ int length(int bh, int r) const {
    return ptr ? ptr[(size_t)bh * (R + 1) + r + 1] - ptr[(size_t)bh * (R + 1) + r] : k;
  }
};
// sums: h [R][d * d] and z [R][d] per head; totals likewise with R = 1 (null: not wanted)
struct StateSums {
  float *h, *z, *h_total, *z_total;
};
constexpr int kStateCols = 128;           // entries of a state per wave
template <int D, bool TOTALS_ONLY>
__global__ __launch_bounds__(256, 2) void masked_states_f32_kernel(const float* __restrict__ states, const BlockLists lists,
                                                                   const StateSums out, int BH, int row_tiles) {
  constexpr int P = f32_state(D), kSets = (P + 4 * kStateCols - 1) / (4 * kStateCols);   // of four waves
  extern __shared__ uint32_t bits[];      // [W][32] bit s % 32 of word s / 32 of a row: block s is listed
  const int R = lists.R, S = lists.S, W = (S + 31) / 32;
  // the workgroups that read the same entries run next to each other on one XCD
  const int y = blockIdx.x / kXcds, set = y / row_tiles * kXcds + blockIdx.x % kXcds, tile = y % row_tiles;
  if (set >= BH * kSets) return;
  const int bh = set / kSets, row0 = 32 * tile;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, w = tid / kWave;
  const int col = (set % kSets * 4 + w) * kStateCols + 4 * (lane % 32);
  const float* src = states + (size_t)bh * S * P + min(col, P - 4);
  f32x4 b[16];                            // blocks 32 sw + 2 n + g; past the end the last one, taken as 0
  auto request = [&](int sw, int n) { b[n] = *reinterpret_cast<const f32x4*>(src + (size_t)min(32 * sw + 2 * n + g, S - 1) * P); };
#pragma unroll
  for (int n = 0; n < 16; n++) request(0, n);
  if constexpr (!TOTALS_ONLY) {
    for (int x = tid; x < 32 * W; x += 256) bits[x] = 0u;
    __syncthreads();
    const int row = tid / 8;
    if (row0 + row < R) {
      const int32_t* list = lists.begin(bh, row0 + row);
      const int n = lists.length(bh, row0 + row);
      for (int e = tid % 8; e < n; e += 8) {
        const int s = list[e];
        atomicOr(&bits[s / 32 * 32 + row], 1u << (s % 32));   // OR: the result does not depend on the order
      }
    }
    __syncthreads();
  }
  f32x16 acc[4];
#pragma unroll
  for (int x = 0; x < 4; x++) acc[x] = zero16();
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  const bool total = tile == 0 && out.h_total != nullptr;
  for (int sw = 0; sw < W; sw++) {
    const uint32_t word = TOTALS_ONLY ? 0u : bits[32 * sw + lane % 32];
    if (sw > 0) {
#pragma unroll
      for (int n = 0; n < 16; n++) request(sw, n);
    }
#pragma unroll
    for (int half = 0; half < 2; half++) {
      if (32 * sw + 16 * half < S) {
#pragma unroll
        for (int n = 8 * half; n < 8 * half + 8; n++) {
          const bool exists = 32 * sw + 2 * n + g < S;
          if (!exists) b[n] = f32x4{0.f, 0.f, 0.f, 0.f};   // (0 times an infinite entry is NaN)
          if (total) sum += b[n];
          if constexpr (!TOTALS_ONLY) {
            const float a = (word >> (2 * n + g) & 1u) == 0u ? 1.f : 0.f;
#pragma unroll
            for (int x = 0; x < 4; x++) acc[x] = mfma_f32(a, b[n][x], acc[x]);
          }
        }
      }
    }
  }
  if (col >= P) return;
  if (total) {
#pragma unroll
    for (int x = 0; x < 4; x++) sum[x] = swap_halves_sum(sum[x]);
    if (g == 0) *reinterpret_cast<f32x4*>(col < D * D ? out.h_total + (size_t)bh * D * D + col : out.z_total + (size_t)bh * D + (col - D * D)) = sum;
  }
  if constexpr (!TOTALS_ONLY) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int r = row0 + 8 * (v / 4) + 4 * g + v % 4;
      const size_t slot = (size_t)bh * R + r;
      if (r < R)
        *reinterpret_cast<f32x4*>(col < D * D ? out.h + slot * D * D + col : out.z + slot * D + (col - D * D)) =
            f32x4{acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
    }
  }
}

// The same sums as the totals less the states of the listed blocks: 1,024 entries of one sum per workgroup.
template <int D>
__global__ __launch_bounds__(256) void gather_states_f32_kernel(const float* __restrict__ states, const BlockLists lists, const StateSums out) {
  constexpr int P = f32_state(D), kParts = (P + 1023) / 1024;
  const int part = blockIdx.x % kParts, slot = blockIdx.x / kParts, bh = slot / lists.R;
  const int col = 1024 * part + 4 * (int)threadIdx.x;
  if (col >= P) return;
  const int32_t* list = lists.begin(bh, slot % lists.R);
  const int n = lists.length(bh, slot % lists.R);
  const float* src = states + (size_t)bh * lists.S * P + col;
  f32x4 a = *reinterpret_cast<const f32x4*>(col < D * D ? out.h_total + (size_t)bh * D * D + col : out.z_total + (size_t)bh * D + (col - D * D));
#pragma unroll 8
  for (int s = 0; s < n; s++) a -= *reinterpret_cast<const f32x4*>(src + (size_t)list[s] * P);
  *reinterpret_cast<f32x4*>(col < D * D ? out.h + (size_t)slot * D * D + col : out.z + (size_t)slot * D + (col - D * D)) = a;
}

// The product costs S per sum whatever is listed, the gather the length of the list, and a launch of its own behind the
// totals: it pays where the lists are a small part of many blocks.  In k / T_n the line lies in the same place on both sides (a
// key block's list is k T_m / T_n of T_m blocks on average) and for few and many heads; states of 64 KB and of 16 KB have lines
// of their own.  Calls, us, product / totals + gather:
//   query side (forward)                       d = 128                                   d = 64
//     12 heads, T_n = 64                       k = 1 129 / 130    k = 4 155 / 165        k = 1 66 / 64      k = 4 83 / 85
//     12 heads, T_n = 128, 64-row blocks       k = 4 341 / 335    k = 8 437 / 456        k = 4 146 / 142    k = 8 198 / 199
//     12 heads, T_n = 256                      k = 8 869 / 845    k = 16 1,272 / 1,335   k = 8 403 / 367    k = 16 618 / 598
//      8 heads, T_n = 512                      k = 16 1,855 / 1,791   k = 32 2,943 / 3,158   k = 16 904 / 810   k = 32 1,475 / 1,461
//      1 head, T_n = 512, 64-row blocks        k = 16 334 / 300   k = 32 470 / 503       k = 16 175 / 142   k = 32 248 / 225
//      2 heads, T_n = 1,182                    k = 36 2,223 / 2,141   k = 72 3,722 / 3,987   k = 36 1,217 / 1,039   k = 72 1,979 / 1,984
//   key side (training step, product on the query side)
//     12 heads, T_n = 128, 64-row blocks       k = 2 874 / 857    k = 4 1,090 / 1,094    k = 2 415 / 409    k = 4 500 / 500
//     12 heads, T_n = 256                      k = 8 2,911 / 2,893   k = 16 4,646 / 4,685   k = 8 1,472 / 1,446   k = 16 2,360 / 2,367
//      8 heads, T_n = 512                      k = 16 6,628 / 6,551  k = 32 11,422 / 11,666   k = 16 3,336 / 3,278   k = 32 5,809 / 5,811
//      2 heads, T_n = 1,182                    k = 36 8,103 / 8,018  k = 72 14,565 / 14,964   k = 36 4,312 / 4,140   k = 72 7,640 / 7,629
constexpr int kGatherBlocks = 64;
template <int D> constexpr int kGatherRatio = D == 128 ? 25 : 16;
template <int D>
static hipError_t launch_states_f32(const Shape& s, int heads, const float* states, const BlockLists& lists, StateSums out, bool totals,
                                    hipStream_t stream) {
  constexpr int P = f32_state(D), kSets = (P + 4 * kStateCols - 1) / (4 * kStateCols);
  const int sets = (heads * kSets + kXcds - 1) / kXcds * kXcds;
  if (s.Tn <= kGatherBlocks || s.Tn <= kGatherRatio<D> * s.k) {
    if (!totals) out.h_total = out.z_total = nullptr;
    const int tiles = (lists.R + 31) / 32, smem = (lists.S + 31) / 32 * 32 * (int)sizeof(uint32_t);   // at most 8 KB
    masked_states_f32_kernel<D, false><<<dim3((unsigned)(sets * tiles)), 256, smem, stream>>>(states, lists, out, heads, tiles);
    return hipGetLastError();
  }
  masked_states_f32_kernel<D, true><<<dim3((unsigned)sets), 256, 0, stream>>>(states, lists, out, heads, 1);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  gather_states_f32_kernel<D><<<dim3((unsigned)((size_t)heads * lists.R * ((P + 1023) / 1024))), 256, 0, stream>>>(states, lists, out);
  return hipGetLastError();
}
hipError_t launch_block_states_f32(const Shape& s, const HeadGroup& hg, const float* states, const int32_t* block_idx, float* h_total,
                                   float* z_total, float* h_i, float* z_i, hipStream_t stream) {
  const size_t b = hg.bh0;
  const BlockLists lists{nullptr, block_idx + b * s.Tm * s.k, s.Tm, s.Tn, s.k};
  const StateSums out{h_i, z_i, h_total + b * s.d * s.d, z_total + b * s.d};
  return s.d == 128 ? launch_states_f32<128>(s, hg.heads, states, lists, out, true, stream)
                    : launch_states_f32<64>(s, hg.heads, states, lists, out, true, stream);
}
hipError_t launch_key_states_f32(const Shape& s, const BwdArgs& a, hipStream_t stream) {
  const BlockLists lists{a.col_ptr, a.col_idx, s.Tn, s.Tm, s.k};
  const StateSums out{(float*)a.dh_sum, a.dz_sum, a.dh_total, a.dz_total};
  return s.d == 128 ? launch_states_f32<128>(s, s.BH, (const float*)a.dh, lists, out, false, stream)
                    : launch_states_f32<64>(s, s.BH, (const float*)a.dh, lists, out, false, stream);
}

// ---------------------------------------------------------------------------------------------
// attn_f32: one workgroup of four waves per 32 query rows of a query block i
//   sparse branch  : for j in sel(i): S^T = K'_j Q^T / sqrt(d), online softmax, O^T += V_j^T P^T
//   linear branch  : O_l^T = H_i^T Q^phi^T / (Q^phi Z_i)
//   mix            : out = alpha O_s / l + (1 - alpha) O_l                                   (Eq. 13)
// Wave w takes every fourth half (32 keys) of the selected blocks, with a running maximum and sum of its own; the four
// meet once, after the loop, like the parts of a split softmax.  A wave's K rows and V rows are its own, so they come
// straight from global memory into operand registers: no tile in LDS, no barrier in the loop, and four times as many
// workgroups as with 128 rows each.
// Bound by the fp32 matrix rate in the loop (a wave needs 64 products, 4,096 cycles, for every 16 loads of 1 KB; 85 % of the
// time of a longer list) and by HBM outside: 12 heads of 4,096 tokens, d = 128, keeping O^s and O^l, 6 blocks a list 125 us, none
// 46 us; 128-row workgroups with K', K^phi and V tiles in LDS, which rebuilt H_i, took 245 us.  2 heads of 1,024, d = 64: 20.5 ->
// 9.8 us (with the states' sums in it 12.8).
// ---------------------------------------------------------------------------------------------
template <int D> struct AttnF32Smem {
  static constexpr int LD = kF32Ld<D>, ET = D / 32, NW = 4;
  static constexpr int kQOff = 0;                                          // [32][LD] query rows
  static constexpr int kMuOff = kQOff + 32 * LD;                           // [D] colmean(K)
  static constexpr int kZsOff = kMuOff + D;                                // [D] Z_i
  static constexpr int kMlOff = kZsOff + D;                                // [NW][2][32] m and l
  static constexpr int kRounds = D / 64;                                   // of meet4
  static constexpr int kSwapOff = kMlOff + NW * 64;                        // parts of O^T
  static constexpr int kLSwapOff = kSwapOff + kMeetFloats<D, kRounds>;     // parts of O_l^T
  static constexpr int kBytes = (kLSwapOff + StatePart<D>::kLds) * (int)sizeof(float);
  static_assert(kBytes <= 80 * 1024, "two workgroups a CU");
  static_assert(32 * LD <= kMeetFloats<D, kRounds>, "O_l takes the place of the parts");
};

// OWN (small calls at d = 64): H_i, Z_i of the workgroup's query block formed here, from the states of the head's key blocks,
// into LDS: 16 KB a state, four states requested at a time.  Kept for the backward pass by one workgroup of the query block,
// the totals written by one of the head.
struct OwnStates {
  const float* states;
  float *h_i, *z_i, *h_total, *z_total;   // h_i, z_i: null unless kept
};
constexpr int kOwnBlocks = 16;            // attn_forms_states
constexpr int kOwnLd = 64 + 8;            // rows 4 apart meet the other half of the banks
__device__ __forceinline__ void own_states(const OwnStates& o, float* hs, float* zs, const int32_t* sel, int ksel, int Tn, int bh,
                                           size_t slot, bool keep, bool total) {
  constexpr int D = 64, P = f32_state(D), S = 4, U = 4;                     // U pieces of 1,024 entries: h; then z
  const int tid = threadIdx.x, zcol = min(4 * tid, D - 4);
  uint32_t listed = 0u;
  for (int e = 0; e < ksel; e++) listed |= 1u << __builtin_amdgcn_readfirstlane(sel[e]);
  const float* src = o.states + (size_t)bh * Tn * P;
  f32x4 sum[U + 1], all[U + 1];
#pragma unroll
  for (int u = 0; u <= U; u++) sum[u] = all[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < Tn; s0 += S) {
    f32x4 x[S][U + 1];
#pragma unroll
    for (int n = 0; n < S; n++) {
      const float* p = src + (size_t)min(s0 + n, Tn - 1) * P;
#pragma unroll
      for (int u = 0; u < U; u++) x[n][u] = *reinterpret_cast<const f32x4*>(p + 1024 * u + 4 * tid);
      x[n][U] = *reinterpret_cast<const f32x4*>(p + D * D + zcol);
    }
#pragma unroll
    for (int n = 0; n < S; n++)
      if (s0 + n < Tn) {
        if ((listed >> (s0 + n) & 1u) == 0u)
#pragma unroll
          for (int u = 0; u <= U; u++) sum[u] += x[n][u];
        if (total)
#pragma unroll
          for (int u = 0; u <= U; u++) all[u] += x[n][u];
      }
  }
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int e = 1024 * u + 4 * tid;
    *reinterpret_cast<f32x4*>(hs + e / D * kOwnLd + e % D) = sum[u];
    if (keep) *reinterpret_cast<f32x4*>(o.h_i + slot * D * D + e) = sum[u];
    if (total) *reinterpret_cast<f32x4*>(o.h_total + (size_t)bh * D * D + e) = all[u];
  }
  if (4 * tid < D) {
    *reinterpret_cast<f32x4*>(zs + zcol) = sum[U];
    if (keep) *reinterpret_cast<f32x4*>(o.z_i + slot * D + zcol) = sum[U];
    if (total) *reinterpret_cast<f32x4*>(o.z_total + (size_t)bh * D + zcol) = all[U];
  }
}

template <int D, bool OWN>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v, const double* __restrict__ k_mean,
    const float* __restrict__ h_i, const float* __restrict__ z_i, const int32_t* __restrict__ block_idx,
    const float* __restrict__ alpha, float* __restrict__ out, float* __restrict__ lse, float* __restrict__ o_s_save,
    float* __restrict__ o_l_save, float* __restrict__ lse_save, Strides sin, Strides sout, HeadGroup hg, int H, int N, int Tm, int Tn, int bq,
    int ksel, int alpha_per_block, const OwnStates own) {
  typedef AttnF32Smem<D> SM;
  constexpr int LD = SM::LD, ET = SM::ET, J = D / 8, NW = SM::NW;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* qs = smem + SM::kQOff;
  float* mus = smem + SM::kMuOff;
  float* zs = smem + SM::kZsOff;
  float* ml = smem + SM::kMlOff;
  float* swap = smem + SM::kSwapOff;

  // All row groups in runs of consecutive ones, one run per XCD: what runs there at a time gathers from a head or two
  const int groups = (N + 31) / 32, all = hg.heads * groups, run = (all + kXcds - 1) / kXcds;
  const int at = blockIdx.x % kXcds * run + blockIdx.x / kXcds;
  if (at >= all) return;
  const int bh = hg.bh0 + at / groups, grp = at % groups, h = bh % H;
  const int row0 = 32 * grp, rows_valid = min(32, N - row0), i = row0 / bq;
  const int tid = threadIdx.x, lane = tid % kWave, g = lane / 32, r = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const size_t slot = (size_t)(at / groups) * Tm + i;    // of H_i, Z_i
  const float* kh = k + head_offset(sin, bh, H);
  const float* vh = v + head_offset(sin, bh, H);
  const int32_t* sel = block_idx + ((size_t)bh * Tm + i) * ksel;

  const int items = 2 * ksel;             // halves of the selected blocks; an odd one of the last block may hold no key
  auto first_key = [&](int t) { return __builtin_amdgcn_readfirstlane(sel[t / 2]) * kF32Tokens + 32 * (t % 2); };
  auto rows_of = [&](const float* head, int first) { return RowPieces(head, first, N - 1, sin.n); };
  f32x4 st[kStream];                      // per piece of 32 keys: J elements of K by lane, J of the columns of V; then H_i
  typedef ChunkMap<D, 256, 32> QM;
  f32x4 qr[QM::kLoads];
  QM::load(qr, q + head_offset(sin, bh, H) + (size_t)row0 * sin.n, sin.n, rows_valid, tid);
  const double mu = tid < D ? k_mean[(size_t)bh * D + tid] : 0.0;
  const float zi = !OWN && tid < D ? z_i[slot * D + tid] : 0.f;
  __builtin_amdgcn_sched_barrier(0);
  int t = w, key0 = 0;
  if (t < items) {
    key0 = first_key(t);
    const RowPieces kp = rows_of(kh, key0);
    const unsigned own = kp.own(r, g);
#pragma unroll
    for (int n = 0; n < kStream; n++) st[n] = kp.piece(own, n);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int y = 0; y < QM::kLoads; y++)
    *reinterpret_cast<f32x4*>(qs + (tid / QM::kChunks + y * QM::kRows) * LD + 4 * (tid % QM::kChunks)) = qr[y];
  if (tid < D) {
    mus[tid] = (float)mu;
    if (!OWN) zs[tid] = zi;
  }
  float* hs = smem + SM::kBytes / sizeof(float);
  if constexpr (OWN) own_states(own, hs, zs, sel, ksel, Tn, bh, slot, own.h_i != nullptr && row0 % bq == 0, grp == 0);
  f32x16 oacc[ET];
#pragma unroll
  for (int e = 0; e < ET; e++) oacc[e] = zero16();
  float m_run = -INFINITY, l_run = 0.f;   // this lane's row over this wave's keys, log2 domain
  const float c0 = kLog2e * rsqrtf((float)D);
  const float *qrow = qs + r * LD + 4 * g, *mrow = mus + 4 * g;
  // H_i^T: channels of O_l^T by rows, contracted over c
  typedef StatePart<D> SP;
  constexpr int JW = SP::kSteps;
  const int j0 = SP::first(w);
  constexpr int LH = OWN ? kOwnLd : D;
  const float* hsrc = (OWN ? hs : h_i + slot * D * D) + (size_t)(8 * j0 + 4 * g) * LH + 32 * SP::tile(w) + SP::row(r);
  __syncthreads();

  int key_next = t + NW < items ? first_key(t + NW) : 0;
  // Requests are made one by one between the products: sixteen K requests in a row (32 cache lines each) hold the issue of
  // a wave, and of the others of its CU, for as long as the products they feed take.  The last pass has a copy of its own:
  // where a request may or may not have been made, the wait for one in front of it is a wait for that one.
  auto pass = [&](auto more) {
    constexpr bool MORE = decltype(more)::value;
    const int valid = N - key0;           // keys of this half that exist: below 32 only at the end of the sequence
    const RowPieces kp = rows_of(kh, key0), vp = rows_of(vh, key0), np = rows_of(kh, MORE ? key_next : key0);
    const unsigned own_k = kp.own(r, g), own_n = np.own(r, g);
    auto request = [&](int n) {           // element n of the piece, behind the last one of the next
      const int j = n % J;
      if (n < J) st[n % kStream] = kp.piece(own_k, j);
      else if (n < 2 * J) st[n % kStream] = vp.cols<D>(j, r, g);
      else if (MORE) st[n % kStream] = np.piece(own_n, j);
    };
    f32x16 sacc = zero16();
    f32x4 qb = *reinterpret_cast<const f32x4*>(qrow), mb = *reinterpret_cast<const f32x4*>(mrow);
#pragma unroll
    for (int j = 0; j < J; j++) {
      const f32x4 a = st[j % kStream] - mb, b = qb;
      if (j + 1 < J) {
        qb = *reinterpret_cast<const f32x4*>(qrow + 8 * (j + 1));
        mb = *reinterpret_cast<const f32x4*>(mrow + 8 * (j + 1));
      }
#pragma unroll
      for (int x = 0; x < 4; x++) sacc = mfma_f32(a[x], b[x], sacc);
      __builtin_amdgcn_sched_barrier(0);
      request(j + kStream);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      sacc[e] = 8 * (e / 4) + 4 * g + e % 4 < valid ? sacc[e] * c0 : -INFINITY;
      mx = fmaxf(mx, sacc[e]);
    }
    mx = swap_halves_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;        // no key seen yet
    const float corr = exp2_f32(m_run - m_ref);
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      sacc[e] = exp2_f32(sacc[e] - m_ref);
      rs += sacc[e];
    }
    l_run = l_run * corr + swap_halves_sum(rs);
    m_run = m_new;
#pragma unroll
    for (int x = 0; x < ET; x++) oacc[x] *= corr;
#pragma unroll
    for (int j = 0; j < J; j++) {
      col_products<D>(oacc, st[(J + j) % kStream], sacc, j);
      __builtin_amdgcn_sched_barrier(0);
      request(J + j + kStream);
    }
    if constexpr (MORE) {
      key0 = key_next;
      if (t + 2 * NW < items) key_next = first_key(t + 2 * NW);
    }
  };
  for (; t + NW < items; t += NW) pass(std::integral_constant<bool, true>());
  if (t < items) pass(std::integral_constant<bool, false>());
  auto h_piece = [&](int j) { return f32x4{hsrc[8 * j * LH], hsrc[(8 * j + 1) * LH], hsrc[(8 * j + 2) * LH], hsrc[(8 * j + 3) * LH]}; };
#pragma unroll
  for (int j = 0; j < kStream; j++)
    if (j < JW) st[j] = h_piece(j);

  // ---- linear branch ----
  // Q^phi = softmax_d(Q) of this lane's row: its normaliser and Q^phi Z_i
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
  const bool all_selected = ksel >= Tn;   // nothing left for the linear branch: O_l = 0
  const float inv_den = all_selected ? 0.f : 1.f / den;
  f32x16 lacc = zero16();
#pragma unroll
  for (int j = 0; j < JW; j++) {
    const f32x4 a = st[j % kStream], q4 = *reinterpret_cast<const f32x4*>(qrow + 8 * (j0 + j));
#pragma unroll
    for (int x = 0; x < 4; x++) lacc = mfma_f32(a[x], exp2_f32((q4[x] - qm) * kLog2e) * qinv, lacc);
    if (j + kStream < JW) st[j % kStream] = h_piece(j + kStream);
  }

  // ---- the four parts of the softmax meet ----
  if (g == 0) {
    ml[w * 64 + r] = m_run;
    ml[w * 64 + 32 + r] = l_run;
  }
  __syncthreads();
  float m_all = -INFINITY, l = 0.f;
#pragma unroll
  for (int x = 0; x < NW; x++) m_all = fmaxf(m_all, ml[x * 64 + r]);
  const float m_ref = m_all == -INFINITY ? 0.f : m_all, mine = exp2_f32(m_run - m_ref);
#pragma unroll
  for (int x = 0; x < NW; x++) l += ml[x * 64 + 32 + r] * exp2_f32(ml[x * 64 + r] - m_ref);
  float os[4 * ET], ol[4 * ET];
  meet4<D, SM::kRounds>(os, oacc, mine, swap, w, lane);
  SP::own(ol, lacc, smem + SM::kLSwapOff, w, lane);
  const float inv_l = l > 0.f ? 1.f / l : 0.f;
  const float al = alpha[alpha_per_block ? (size_t)h * Tm + i : (size_t)h];
  // through LDS: a lane's 16 bytes of a row each are a request of their own, whole rows are not
  const int c_own = own_channel(D, w, g);
  __syncthreads();                        // the parts have been read, and the query rows
#pragma unroll
  for (int y = 0; y < ET; y++) {
    f32x4 s4, l4;
#pragma unroll
    for (int x = 0; x < 4; x++) {
      s4[x] = os[4 * y + x] * inv_l;
      l4[x] = ol[4 * y + x] * inv_den;
    }
    *reinterpret_cast<f32x4*>(qs + r * LD + c_own + 4 * y) = s4;
    *reinterpret_cast<f32x4*>(swap + r * LD + c_own + 4 * y) = l4;
  }
  __syncthreads();
#pragma unroll
  for (int y = 0; y < QM::kLoads; y++) {
    const int row = tid / QM::kChunks + y * QM::kRows, c = 4 * (tid % QM::kChunks);
    if (row < rows_valid) {
      const f32x4 s4 = *reinterpret_cast<const f32x4*>(qs + row * LD + c), l4 = *reinterpret_cast<const f32x4*>(swap + row * LD + c);
      *reinterpret_cast<f32x4*>(out + head_offset(sout, bh, H) + (size_t)(row0 + row) * sout.n + c) = al * s4 + (1.f - al) * l4;
      if (o_s_save != nullptr) {          // the two branches, kept for the backward pass
        const size_t kept = ((size_t)bh * N + row0 + row) * D + c;
        *reinterpret_cast<f32x4*>(o_s_save + kept) = s4;
        *reinterpret_cast<f32x4*>(o_l_save + kept) = l4;
      }
    }
  }
  if (w == 0 && g == 0 && r < rows_valid) {
    const float L = l > 0.f ? (m_all + __log2f(l)) * kLn2 : -INFINITY;
    if (lse != nullptr) lse[(size_t)bh * N + row0 + r] = L;
    if (lse_save != nullptr) lse_save[(size_t)bh * N + row0 + r] = L;
  }
}

// Small calls form H_i in the attention kernel: a launch fewer, for T_n x 16 KB that every workgroup reads from L2 where the masked
// product reads them once per 32 query blocks.  The call with own states / with the product, us, d = 64, a tenth of the blocks kept:
//   T_n = 4, 4 heads 16.6 / 19.8      T_n = 8, 2 heads 20.7 / 23.0, 12 heads 21.6 / 24.4
//   T_n = 16, 2 heads 23.6 / 25.0, 4 heads 24.0 / 25.5, 10 heads 30.3 / 31.3 (128-row blocks 29.4 / 29.5)
//   T_n = 24, 2 heads 25.3 / 26.4, 6 heads 32.4 / 32.0      T_n = 32, 2 heads 29.6 / 29.8, 5 heads 40.2 / 38.1
// and at d = 128, where a state is 64 KB, 31.4 / 31.5 at T_n = 4, 47.5 / 40.8 at 16 (4 heads each).
bool attn_forms_states(const Shape& s) { return s.d == 64 && s.Tn <= kOwnBlocks && router_has_room(s); }

template <int D, bool OWN>
static hipError_t launch_attn_f32_t(const Shape& s, const HeadGroup& hg, const float* q, const float* k, const float* v, const double* k_mean,
                                    const float* h_i, const float* z_i, const int32_t* block_idx, const float* alpha, float* out,
                                    float* lse, const SavedForBackward& sv, const OwnStates& own, hipStream_t stream) {
  constexpr int smem = AttnF32Smem<D>::kBytes + (OWN ? D * kOwnLd * (int)sizeof(float) : 0);
  static OncePerDevice once;
  if (hipError_t e = allow_dynamic_lds(once, (const void*)attn_f32_kernel<D, OWN>, smem); e != hipSuccess) return e;
  const int run = (hg.heads * ((s.N + 31) / 32) + kXcds - 1) / kXcds;
  attn_f32_kernel<D, OWN><<<dim3((unsigned)(run * kXcds)), 256, smem, stream>>>(
      q, k, v, k_mean, h_i, z_i, block_idx, alpha, out, lse, (float*)sv.o_s, (float*)sv.o_l, sv.lse, s.sin, s.sout, hg, s.H, s.N, s.Tm,
      s.Tn, s.bq, s.k, s.alpha_per_block ? 1 : 0, own);
  return hipGetLastError();
}

hipError_t launch_attn_f32(const Shape& s, const HeadGroup& hg, const float* q, const float* k, const float* v, const double* k_mean,
                           const float* states, float* h_i, float* z_i, float* h_total, float* z_total, const int32_t* block_idx,
                           const float* alpha, float* out, float* lse, const SavedForBackward& sv, hipStream_t stream) {
  const OwnStates own{states, s.save ? h_i : nullptr, s.save ? z_i : nullptr, h_total, z_total};
#define SLA2_ATTN(DD, OO) launch_attn_f32_t<DD, OO>(s, hg, q, k, v, k_mean, h_i, z_i, block_idx, alpha, out, lse, sv, own, stream)
  if (attn_forms_states(s)) return SLA2_ATTN(64, true);
  return s.d == 128 ? SLA2_ATTN(128, false) : SLA2_ATTN(64, false);
#undef SLA2_ATTN
}

}  // namespace sla2
