// Output of the KV-stationary kernels: a tile's gradients from the accumulators to bf16 rows or, added, to fp32 sums.
//
// Every element is one store or atomic add of its own, so what bounds the end of a workgroup is the instructions around them: with
// 64-bit addresses formed per element, a bounds check per key and kernel arguments spilled across the main loop it took 1300 to 2600 of
// them a wave.  Here an element takes its product, its conversion and, once a row, one addition: buffer instructions add a
// 32-bit lane offset to a base in scalar registers and drop what lies past the tile's last key, and the arguments are read again
// behind the loop, which leaves their registers to it (head dim 512: 52 scalar registers spilled instead of 109, 63 -> 40 KB of code,
// an instruction cache of 64).  Layers, before -> after: 8 x U(100, 300) behind 300, 16 / 4 heads, d = 256 234 -> 216 us, d = 512 336 -> 317;
// 8 x U(65, 256) behind 1021, 32 / 8 heads, d = 128 347 -> 328.
#pragma once
#include "common.h"

namespace dkv {

// The kernel's first argument, read again here (a pointer that the compiler cannot trace to the arguments it has already loaded).
typedef const __attribute__((address_space(4))) AttnParams ArgParams;
__device__ __forceinline__ ArgParams* args_again() {
  uint64_t a = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return reinterpret_cast<ArgParams*>(a);
}

struct GradStore {
  __amdgpu_buffer_rsrc_t k, v;
  uint32_t row_k, row_v;   // bytes from one key to the next
  float scale_k;           // the dK accumulators hold -dK / scale
  bool sums;               // fp32 sums: add

  // keys [0, n) of the tile are rows key_row ... of the gradients of KV head hk (n > 0)
  template <typename Args>
  __device__ __forceinline__ GradStore(Args* a, bool is_ctx, int64_t key_row, int n, int hk, int D) {
    float* const acc_k = is_ctx ? a->dkc_acc : a->dkd_acc;
    float* const acc_v = is_ctx ? a->dvc_acc : a->dvd_acc;
    scale_k = -a->scale;
    sums = acc_k != nullptr;
    if (sums) {
      const int64_t at = (key_row * a->Hk + hk) * D;
      row_k = row_v = (uint32_t)a->Hk * D * 4;
      k = rows(acc_k + at, n, row_k, D * 4);
      v = rows(acc_v + at, n, row_v, D * 4);
    } else {
      const int64_t kts = is_ctx ? a->dkc.ts : a->dkd.ts, vts = is_ctx ? a->dvc.ts : a->dvd.ts;
      u16* const kp = is_ctx ? a->dkc.ptr : a->dkd.ptr;
      u16* const vp = is_ctx ? a->dvc.ptr : a->dvd.ptr;
      row_k = (uint32_t)kts * 2;
      row_v = (uint32_t)vts * 2;
      k = rows(kp + key_row * kts + hk * (is_ctx ? a->dkc.hs : a->dkd.hs), n, row_k, D * 2);
      v = rows(vp + key_row * vts + hk * (is_ctx ? a->dvc.hs : a->dvd.hs), n, row_v, D * 2);
    }
  }
  // n rows of `bytes` each, `row` >= bytes apart: an offset into a later row lies past the end
  __device__ __forceinline__ static __amdgpu_buffer_rsrc_t rows(void* base, int n, uint32_t row, uint32_t bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(uniform(base));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, __builtin_amdgcn_readfirstlane((int)((n - 1) * row + bytes)), 0x00020000);
  }
  __device__ __forceinline__ static void* uniform(void* ptr) {
    const uint64_t v = reinterpret_cast<uint64_t>(ptr);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  }
  // the elements `col` columns behind the byte offsets at_k and at_v; SUMS: the same offset for both
  template <bool SUMS>
  __device__ __forceinline__ void put(uint32_t at_k, uint32_t at_v, int col, float gk, float gv) const {
    gk *= scale_k;
    if (SUMS) {
      __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(gk, k, at_k + col * 4, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(gv, v, at_k + col * 4, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b16((short)(pack2_bf16(gk, 0.f) & 0xffffu), k, at_k + col * 2, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b16((short)(pack2_bf16(gv, 0.f) & 0xffffu), v, at_v + col * 2, 0, 0);
    }
  }
  // f(r, at_k, at_v): register r = 0 ... 15 of a 32x32 accumulator tile and the offsets of its row, the first row's at the start
  template <bool SUMS, typename F>
  __device__ __forceinline__ void tile32(uint32_t& at_k, uint32_t& at_v, F&& f) const {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      f(r, at_k, at_v);
      at_k += (r & 3) == 3 ? 5 * row_k : row_k;   // crow: 0 1 2 3 8 9 10 11 16 ...
      if (!SUMS) at_v += (r & 3) == 3 ? 5 * row_v : row_v;
    }
  }
};

}  // namespace dkv
