// Shared declarations of the SLA2 HIP kernels (gfx950 only).
#pragma once
#include <type_traits>

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "../../include/sla2.h"

namespace sla2 {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // 16 bytes in flight (a native vector: stays in registers)
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(8))) int i32x8;            // operand of the 64-deep FP8 product
typedef __attribute__((ext_vector_type(4))) int i32x4;            // operand of the 32-deep INT8 product
typedef __attribute__((ext_vector_type(16))) int i32x16;          // its 32 x 32 accumulator

constexpr int kWave = 64;
constexpr int kXcds = 8;                // L2 domains; workgroups are dealt to them round-robin
constexpr int kMaxKeyBlocks = 2048;   // router keeps a whole score row in registers
constexpr float kE4M3Max = 448.0f;
constexpr float kInt8Max = 127.0f;   // symmetric INT8 code range of Q and K
constexpr float kLog2e = 1.4426950408889634f;

// Where (batch b, head h, token t) of a [.., d] tensor starts, in elements: b * b_ + h * h_ + t * n.
struct Strides {
  long long b, h;
  int n;
};
__host__ __device__ __forceinline__ size_t head_offset(const Strides& st, int bh, int H) {
  return (size_t)(bh / H) * (size_t)st.b + (size_t)(bh % H) * (size_t)st.h;
}

// hipFuncSetAttribute(MaxDynamicSharedMemorySize) once per kernel and device.  Safe to call from several
// threads: the flag is atomic and setting the attribute twice is harmless.
struct OncePerDevice { std::atomic<unsigned long long> done{0}; };
inline hipError_t allow_dynamic_lds(OncePerDevice& once, const void* kernel, int bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (once.done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) once.done.fetch_or(bit, std::memory_order_release);
  return e;
}

// Host-side description of one call, derived from sla2_params.
struct Shape {
  Strides sin, sout;                         // q, k, v share `sin`; out has `sout`
  int B, H, N, d, bq, bk;
  int BH, Tm, Tn, k;
  bool bf16, smooth, w_per_head, alpha_per_block;
  bool save;                                 // keep O^s, O^l, L for the backward pass
  int quant;                                 // sla2_quant: 0 none, 1 FP8 e4m3, 2 INT8 codes of Q and K, 3 FP8 with V in e4m3 too
  // kv precompute: each workgroup reduces `blocks_per_chunk` key blocks; `chunks` per head
  int blocks_per_chunk, chunks;
  // the states of this many heads at a time.  bf16 tensors: long lists, H_i formed before the attention kernel (0: rebuilt there);
  // fp32 tensors: always, the attention kernel with them
  int state_heads;
};

// sla2_api.cpp: parameter validation (SLA2_OK or a negative sla2_status) and the workspace carve-up
int make_shape(const sla2_params* p, Shape* s);
void make_layout(const Shape& s, sla2_ws_layout* L);

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __builtin_bit_cast(float, (uint32_t)b << 16);
}

// A load of what is the same for the whole wave, through the scalar cache: the compiler does so by itself only where it can prove that
// nothing was written in between, which it cannot behind inline assembly.  For memory that no workgroup of the launch writes.
template <class T>
__device__ __forceinline__ T scalar_load(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// A store past the caches, for results that no kernel of the same pass reads (out, what is kept for the backward pass, gradients):
// left in the 256 MB memory-side cache they push out the tiles that are gathered from it, and their way to memory falls into the
// next kernels that stream through HBM.  Forward, us, cached / past the caches: 48 heads of 4,096 tokens (FP8) 169.2 / 164.5,
// 12 heads of 32,760 434 / 428, bf16 at 26 blocks a list 616 / 609; with an elementwise kernel that reads `out` at once behind the
// call 182.2 / 180.4 and 457 / 454; training steps 1,510 / 1,499 and 209.3 / 206.9 (32 heads of 4,096 tokens, d = 64).  With four sets
// of inputs in turn, none of which is left in a cache, as much: 159.3 / 155.5, 409.6 / 404.8, 608.7 / 605.9, 1,449 / 1,442, 202.7 / 199.9.
template <class T>
__device__ __forceinline__ void store_streamed(T* p, T x) { __builtin_nontemporal_store(x, p); }

// lanes l and l ^ 32 combine their values through v_permlane32_swap; both get the same bits.  A vector instruction: no LDS round trip,
// whose latency a wave that has the vector unit to itself would sit out (us, with a round trip / so, in the plain loop of the attention
// kernel at d = 64, 128-row blocks: FP8, 24 heads of 16,384 tokens 195.5 / 192.7; dense, 24 heads of 8,192 471 / 464).
__device__ __forceinline__ float swap_halves_max(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // r[0] = low half twice, r[1] = high half twice
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float swap_halves_sum(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// max(x, |a|, |b|) as the one instruction it is: of values that come from bit operations the compiler takes maxima with themselves first
__device__ __forceinline__ float max3_abs(float x, float a, float b) {
  float r;
  asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(x), "v"(a), "v"(b));
  return r;
}
// Maximum over the wave, on every lane; vector instructions only.
__device__ __forceinline__ float wave_max(float x) {
  auto dpp = [&](auto ctrl) {
    const int i = __builtin_bit_cast(int, x);
    x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, decltype(ctrl)::value, 0xf, 0xf, false)));
  };
  dpp(std::integral_constant<int, 0xB1>());          // quad_perm 1 0 3 2
  dpp(std::integral_constant<int, 0x4E>());          // quad_perm 2 3 0 1
  dpp(std::integral_constant<int, 0x141>());         // row_half_mirror
  dpp(std::integral_constant<int, 0x140>());         // row_mirror
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
  return swap_halves_max(x);
}

// x of another lane: DPP controls, vector instructions only
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
  const int i = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}
template <int N> __device__ __forceinline__ float rotate16(float x) { return dpp_move<0x120 + N>(x); }   // within 16 lanes
// over four neighbouring lanes, on all of them
__device__ __forceinline__ float quad_max(float x) {
  x = fmaxf(x, dpp_move<0xB1>(x));
  return fmaxf(x, dpp_move<0x4E>(x));
}
__device__ __forceinline__ float quad_sum(float x) {
  x += dpp_move<0xB1>(x);
  return x + dpp_move<0x4E>(x);
}
// over 8, 16 or 32 neighbouring lanes and over the wave, on all of them, in the order of a butterfly.  (As four exchanges through LDS a row,
// each waited for, the sums of dO . O^s of the backward pass's query side took as long as reading its tiles.)
template <int LANES> __device__ __forceinline__ float row_sum(float x) {
  static_assert(LANES == 8 || LANES == 16 || LANES == 32, "");
  x = quad_sum(x);
  x += dpp_move<0x141>(x);                             // row_half_mirror
  if (LANES > 8) x += dpp_move<0x140>(x);              // row_mirror
  if (LANES < 32) return x;
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
template <int LANES> __device__ __forceinline__ float row_max(float x) {
  static_assert(LANES == 16 || LANES == 32, "");
  x = quad_max(x);
  x = fmaxf(x, dpp_move<0x141>(x));
  x = fmaxf(x, dpp_move<0x140>(x));
  if (LANES < 32) return x;
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float wave_sum(float x) { return swap_halves_sum(row_sum<32>(x)); }
// a of lanes l and l ^ 32 added up on the lower half of the wave, b on the upper one; the same with l ^ 16 on the even and odd
// 16 lanes
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// What the lanes of a wave wrote to LDS ahead of it the other lanes of that wave may read behind it, and the other way
// round.  LDS serves the accesses of a wave in order, so this is no instruction: it tells the compiler to keep them so.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where sla2_forward keeps O^s, O^l ([BH, N, d], element type of out; o_l may be null on its own) and
// L ([BH, N]) for the backward pass; all null when nothing is to be kept.  With them goes the state of the linear branch
// per query block: Z_i [BH, T_m, d] and H_i, bf16 tensors: H_i^T as bf16 [BH, T_m, d(e), d(c)], fp32 tensors: H_i as fp32
// [BH, T_m, d(c), d(e)].
struct SavedForBackward {
  void *o_s, *o_l;
  float* lse;
  void* h_i;
  float* z_i;
};

// Everything the backward kernels touch (device pointers).
struct BwdArgs {
  const void *q, *k, *v, *dout, *o_s, *o_l;
  const float* lse;
  const double* k_mean;
  const float* k_stats;
  const int32_t* block_idx;
  const float* alpha;
  void *dq, *dk, *dv;
  float* dalpha;
  const void* h_i;                           // as SavedForBackward
  const float* z_i;
  // scratch.  dh: one d x d slot per query block (bf16 tensors: dH_i / 2; fp32 tensors: dZ_i behind each); lraw: L log2(e) per row (bf16: on the raw keys)
  float *ds, *lraw, *dz /* bf16 tensors */, *dz_total, *colsum, *dk_mean, *dalpha_part;
  void* dh;
  int32_t *col_ptr, *col_idx, *col_cnt;      // per key block the query blocks that selected it: offsets, lists, lengths
  // bf16 tensors: the query blocks that did not, as a bit matrix (masked_sums.h)
  uint32_t* col_bits;
  void* dh_sum;                              // dH_j, the sum of their dH_i, one d x d slot per key block in the element order of dh
  float *dz_sum, *dh_total;                  // fp32 tensors: dZ_j per key block; the sum of all dH_i
  float *inv_den, *dl;                       // fp32 tensors, per row: 1 / (Q^phi Z_i) and D^l
  int32_t* order;                            // [bwd_kv_grid] the key block (bh kMaxKeyBlocks + j, or -1) of every bwd_kv workgroup
};
inline size_t bwd_kv_grid(const Shape& s) { return (size_t)s.BH * kXcds * ((s.Tn + kXcds - 1) / kXcds); }
// parts of d alpha per query block, column sums of dK' per head: fp32 kernels work on 32 rows and 32 keys at a time
inline int bwd_alpha_parts(const Shape& s) { return s.bf16 ? 1 : s.bq / 32; }
inline int bwd_colsums(const Shape& s) { return s.bf16 ? s.Tn : 2 * s.Tn; }
// the backward pass in the order it runs: query side (with the lists), totals, key side, finish
hipError_t launch_bwd_q(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_totals(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_kv(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_finish(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_q_bf16(const Shape& s, const BwdArgs& a, hipStream_t stream);   // matrix-core kernels, bf16 tensors
hipError_t launch_bwd_kv_bf16(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_totals_f32(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_q_f32(const Shape& s, const BwdArgs& a, hipStream_t stream);
hipError_t launch_bwd_kv_f32(const Shape& s, const BwdArgs& a, hipStream_t stream);

// ---- launchers (one per kernel file); all enqueue on `stream` and return hipGetLastError() ----
// k_frag [BH, T_n, d]: the block sums of K once more, as the operand fragments of the router's products: for each group of
// 16 key blocks of a head (the last group of a head: of the n it has) [d / 8][4][16 (n)][2], entry (j, g, b, x) being channel
// 8 j + 2 g + x of block b.  The router reads whole kilobytes; from the row-major sums each of the 16 lanes of a quarter
// wave would touch a cache line of its own, which took 60 cycles a load.  k_sum may be null: only callers of the library
// read it (sla2_ws_layout.k_sum).
__host__ __device__ __forceinline__ size_t k_frag_offset(int bh, int j, int c, int Tn, int d) {
  const int first = j - j % 16, n = Tn - first < 16 ? Tn - first : 16;
  return ((size_t)bh * Tn + first) * d + (c / 2 * n + j % 16) * 2 + c % 2;
}
hipError_t launch_block_sums(const Shape& s, const void* q, const void* k, const float* router_w, double* q_sum,
                             double* k_sum, double* k_frag, double* router_m, hipStream_t stream);
hipError_t launch_router_topk(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                              int32_t* block_idx, double* k_mean, hipStream_t stream);
// fp32 tensors, where every workgroup finds a CU of its own (router_has_room): with it states [BH, T_n, d * d + d], h_j and z_j of every
// key block, and lnZ of every token; `states` may not be where k_frag is
bool router_has_room(const Shape& s);
hipError_t launch_router_topk_f32(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                                  int32_t* block_idx, double* k_mean, const float* k, const float* v, float* k_stats, float* states,
                                  hipStream_t stream);
hipError_t launch_router_soft(const Shape& s, const double* q_sum, const double* k_frag, const double* router_m,
                              float* mask, double tau, hipStream_t stream);
// The three steps of the fp32 forward pass behind the selection work on `heads` heads from bh0 on; states, h_i and z_i are of those
// heads alone, everything else of all.
struct HeadGroup {
  int bh0, heads;
};
hipError_t launch_kv_state_f32(const Shape& s, const HeadGroup& hg, const float* k, const float* v, const double* k_mean,
                               float* k_stats, float* states, hipStream_t stream);
// h_i [heads, T_m, d, d], z_i [heads, T_m, d]: the sums of the states over the key blocks that a query block did not select
hipError_t launch_block_states_f32(const Shape& s, const HeadGroup& hg, const float* states, const int32_t* block_idx, float* h_total,
                                   float* z_total, float* h_i, float* z_i, hipStream_t stream);
// the same on the key side of the backward pass: dH_j, dZ_j from dH_i, dZ_i of the query blocks that did not select j
hipError_t launch_key_states_f32(const Shape& s, const BwdArgs& a, hipStream_t stream);
// small calls: the attention kernel forms them (and the totals) itself, from the states; all heads are one group then
bool attn_forms_states(const Shape& s);
hipError_t launch_attn_f32(const Shape& s, const HeadGroup& hg, const float* q, const float* k, const float* v, const double* k_mean,
                           const float* states, float* h_i, float* z_i, float* h_total, float* z_total, const int32_t* block_idx,
                           const float* alpha, float* out, float* lse, const SavedForBackward& sv, hipStream_t stream);

hipError_t launch_kv_total(const Shape& s, int heads, const float* partial, float* h_total, float* z_total, float* h_frag, hipStream_t stream);
hipError_t launch_kv_state_bf16(const Shape& s, const uint16_t* k, const uint16_t* v, const double* k_mean,
                                float* k_stats, float* partial, uint16_t* k_phi, float* z_blocks, uint8_t* k_codes,
                                float* k_scale, uint8_t* v_codes, float* v_scale, hipStream_t stream);
// bf16 tensors with Shape::state_heads: kv_state with the states of the key blocks, the totals, and H_i from the states
constexpr int kStateParts = 3;               // bf16 numbers that hold an fp32 entry of h_j exactly
struct GivenStates {
  uint16_t* states;                          // [state_heads][T_n][kStateParts][d * d]: h_j / 2 in bf16 parts, scratch
  uint16_t* h_i;                             // [BH][T_m][d * d], in the order in which kv_state leaves the parts
  uint32_t* bits;                            // scratch
};
hipError_t launch_kv_states_bf16(const Shape& s, const uint16_t* k, const uint16_t* v, const double* k_mean, float* k_stats,
                                 float* partial, float* h_total, float* z_total, float* z_blocks, uint8_t* k_codes, float* k_scale,
                                 uint8_t* v_codes, float* v_scale, const int32_t* block_idx, const GivenStates& gs, hipStream_t stream);
// k_phi: with Shape::state_heads H_i in its place (read from sv.h_i where that is not null)
hipError_t launch_attn_bf16(const Shape& s, const uint16_t* q, const uint16_t* k, const uint16_t* v,
                            const double* k_mean, const uint16_t* k_phi, const float* z_blocks, const uint8_t* k_codes,
                            const float* k_scale, const uint8_t* v_codes, const float* v_scale,
                            const float* h_frag, const float* z_total,
                            const int32_t* block_idx, const float* alpha, uint16_t* out, float* lse,
                            const SavedForBackward& sv, hipStream_t stream);
hipError_t launch_dense_pp(const Shape& s, const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out,
                           hipStream_t stream);
hipError_t launch_dense_bf16(const Shape& s, const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out,
                             hipStream_t stream);

}  // namespace sla2
