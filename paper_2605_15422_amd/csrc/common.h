// Shared device helpers for the gfx950 shared-prompt attention kernels.
//
// MFMA conventions (wave64).  v_mfma_f32_32x32x16_bf16 (dK/dV, head dims 192 and up; 16x16x32 beside mfma16 below):
//   A operand (M x K = 32 x 16): lane l holds row  i = l % 32, k = 8*(l/32) .. 8*(l/32)+7
//   B operand (K x N = 16 x 32): lane l holds col  j = l % 32, k = 8*(l/32) .. 8*(l/32)+7
//   C/D       (M x N = 32 x 32): lane l holds col  j = l % 32, and register r (0..15) holds
//                                row i = 8*(r/4) + 4*(l/32) + r%4
// Because the contraction index only has to agree between A and B, an accumulator tile can be fed
// back as the K-indexed operand of the next MFMA without leaving registers: registers 8t..8t+7 of a
// C tile are 16 distinct rows {16t + 8a + 4*(l/32) + c}, and the matching operand of the other
// matrix is read from LDS with the same permutation of the contraction index (the row pairs of tr_pair).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dkv {

typedef unsigned short u16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;      // finite "minus infinity" for running maxima

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16: A lane l holds row l % 16, B lane l column l % 16, both k = 8*(l/16) .. 8*(l/16)+7; C lane l holds
// column l % 16, register r (0..3) row 4*(l/16) + r.  Two C tiles of 16 rows are the 32-deep K-indexed operand of the next
// MFMA (lane group g holds rows 4g..4g+3 and 16+4g..16+4g+3).
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack2_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// eight consecutive fp32 values of an accumulator tile -> one MFMA operand
__device__ __forceinline__ bf16x8 pack8_bf16(const float* v) {
  u32x4 r;
  r.x = pack2_bf16(v[0], v[1]);
  r.y = pack2_bf16(v[2], v[3]);
  r.z = pack2_bf16(v[4], v[5]);
  r.w = pack2_bf16(v[6], v[7]);
  return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// Combine a value with the one held by lane ^ 32.  v_permlane32_swap exchanges, in place, the upper
// 32 lanes of its first operand with the lower 32 lanes of its second; fed two copies of the same value,
// every lane ends up with its own value in one register and its partner's in the other (no LDS round
// trip).  Written as inline asm with both registers as read-write operands; the leading s_nop covers
// the VALU-write -> permlane-read hazard the compiler cannot see.
// NEVER feed an MFMA result straight into an inline-asm VALU instruction: the wait states between an MFMA and
// a VALU read of its destination are inserted by the compiler, and it does not insert them for inline asm (the
// instruction then reads the registers before the MFMA has written them; seen as run-to-run differences).
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float xor32_max(float x) {
  float a = x, b = x;
  swap32(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float xor32_sum(float x) {
  float a = x, b = x;
  swap32(a, b);
  return a + b;
}

// D = rowsum(dO * O) is formed by the dQ kernels or by a kernel of its own (aux.hip), bit for bit alike: the eight products
// of a 16-byte chunk first, then the chunks in a butterfly from the widest distance down.
__device__ __forceinline__ float dot8_bf16(u32x4 x, u32x4 y) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) s += bf16_lo(x[i]) * bf16_lo(y[i]) + bf16_hi(x[i]) * bf16_hi(y[i]);
  return s;
}
__device__ __forceinline__ float dot8_bf16(bf16x8 a, bf16x8 b) {
  return dot8_bf16(__builtin_bit_cast(u32x4, a), __builtin_bit_cast(u32x4, b));
}
// the levels of that butterfly whose chunks one lane holds: t[i] + t[i + h], h = the next power of two's half, ..., 1
template <int N>
__device__ __forceinline__ float butterfly_sum(float (&t)[N]) {
  constexpr int top = N <= 4 ? 2 : N <= 8 ? 4 : 8;
  static_assert(N >= 2 && N <= 16, "");
#pragma unroll
  for (int h = top; h >= 1; h >>= 1)
#pragma unroll
    for (int i = 0; i < h; ++i)
      if (i + h < N) t[i] += t[i + h];
  return t[0];
}

// Row of a C tile held in register r by this lane.
__device__ __forceinline__ int crow(int r, int hi) { return 8 * (r >> 2) + 4 * hi + (r & 3); }

// A bf16 tensor view: element strides.
struct TView {
  const u16* ptr;
  int64_t ts, hs;
};
struct TViewOut {
  u16* ptr;
  int64_t ts, hs;
};

// Parameters shared by the three attention kernels.  "rows" are response rows (Call 2) or prompt
// rows (Call 1, run as N = 1, ctx_len = 0).
struct AttnParams {
  TView q, kc, vc, kd, vd, o, dout;     // o / dout only used by the backward kernels
  TViewOut out_o;                        // fwd: O
  TViewOut dq, dkc, dvc, dkd, dvd;       // bwd outputs (bf16)
  float* lse;                            // (H, total) fwd: written, bwd: read
  float* dvec;                           // (H, total) D = rowsum(dO * O), bwd only
  float* lse2;                           // (H, total) LSE * log2(e), written with D
  float* dkc_acc;                        // optional fp32 (P, Hk, d) accumulators (atomic adds)
  float* dvc_acc;
  float* dkd_acc;                        // optional fp32 (rows, Hk, d) accumulators for response-region keys
  float* dvd_acc;
  const int32_t* cu;                     // (N+1) or nullptr => one sequence [0, total)
  // Several prompt groups in one launch (Sec. 2.2): grp = n_groups x {first prompt row, P_g, first sequence, end
  // sequence} (device), seq_ctx = per sequence {first prompt row, P_g} expanded from it; both nullptr for one group,
  // whose prompt is rows [0, ctx_len) of kc / vc.  With groups, ctx_len is the largest P_g (grid sizing only).
  const int32_t* grp;
  const int32_t* seq_ctx;
  int n_groups;
  int n_seqs, ctx_len, total, max_rows;
  int H, Hk, G;
  int window;                            // > 0: sliding window
  float scale;                           // softmax scale
  float scale_log2;                      // scale * log2(e)
  // Q-stationary kernels: head packing of one workgroup
  int GP, RSH, BMR, MB, HC;              // heads packed, row-subtiles per head, rows per block, blocks, head chunks
  // KV-stationary kernel
  int n_ctx_tiles, n_dec_tiles;          // per sequence upper bound for dec
  int n_split;                           // ctx tiles: the sequence loop is cut in n_split parts

  // dQ kernels: D is formed from dO and O and written with LSE * log2(e), unless the row statistics are given (o.ptr nullptr).
  // Not a field: one more argument word shifts the blocks that the others arrive in, and the head-dim 512 dK/dV kernel, short of
  // scalar registers, then spills two and a half times as many (backward of Call 2 at N = 8, P = 1136, R ~ U(100, 400), 16 / 16
  // heads: 530 us; as it is, 515).
  __host__ __device__ bool make_stats() const { return o.ptr != nullptr; }
};

// A value whose origin the compiler does not see: what is formed from it is neither hoisted out of a loop into registers nor shared.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A scalar kernel argument in scalar registers of its own.  The arguments arrive in blocks of up to sixteen registers;
// a value used inside a loop keeps its whole block alive, and when scalar registers run short the block is spilled and
// reloaded as a whole for it.  The copy ends the block's life here.
__device__ __forceinline__ int own_sgpr(int v) {
  int r;
  asm volatile("s_mov_b32 %0, %1" : "=s"(r) : "s"(v));
  return r;
}
__device__ __forceinline__ int64_t own_sgpr(int64_t v) {
  int64_t r;
  asm volatile("s_mov_b64 %0, %1" : "=s"(r) : "s"(v));
  return r;
}

}  // namespace dkv
