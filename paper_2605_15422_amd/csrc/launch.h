// Host-side launch entry points of the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "kvsched.h"

namespace dkv {

// tuned forward for head dims 64 / 96 / 128
hipError_t launch_fwd2(const AttnParams& p, int head_dim, hipStream_t st);
// tuned backward kernels for head dims 64 / 96 / 128
hipError_t launch_dq2(const AttnParams& p, int head_dim, hipStream_t st);
hipError_t launch_dkdv4(const AttnParams& p, int head_dim, hipStream_t st);
// dK/dV of Call 2 at head dims 96 and 128 without a window, two workgroups a CU
hipError_t launch_dkdvw(const AttnParams& p, int head_dim, hipStream_t st);
// dK/dV and dQ in one launch (row statistics given), by the rules of dq_beside (rules.h)
hipError_t launch_dkdv4_dq(const AttnParams& p, int head_dim, int dq_waves, bool dq_first, hipStream_t st);
hipError_t launch_dkdv256_dq(const AttnParams& p, int head_dim, bool dq_first, hipStream_t st);
hipError_t launch_dkdv512_dq(const AttnParams& p, bool dq_first, hipStream_t st);
// kernels for head dims 192 / 256 (forward, dQ: 128 rows per workgroup; dK/dV: 64-key tile)
hipError_t launch_fwd256(const AttnParams& p, int head_dim, hipStream_t st);
hipError_t launch_dq256(const AttnParams& p, int head_dim, hipStream_t st);
hipError_t launch_dkdv256(const AttnParams& p, int head_dim, hipStream_t st);
// tuned dK/dV kernel for head dim 512 (32-key tile, 16-row blocks)
hipError_t launch_dkdv512(const AttnParams& p, hipStream_t st);
// tuned dQ kernel for head dim 512 (64 rows per workgroup, 16-key tiles)
hipError_t launch_dq512(const AttnParams& p, hipStream_t st);
hipError_t launch_fwd512(const AttnParams& p, hipStream_t st);
// key tile (rows of K/V owned by one workgroup) of the dK/dV kernel for a head dim
inline int dkdv_key_tile(int head_dim) { return head_dim <= 128 ? 128 : head_dim <= 256 ? 64 : 32; }

hipError_t launch_dot_do_o(const TView& dout, const TView& o, const float* lse, float* dvec, float* lse2, int total,
                           int H, int head_dim, hipStream_t st);
hipError_t launch_group_offsets(const int32_t* grp, int n_groups, int total_ctx, int32_t* cu, hipStream_t st);
hipError_t launch_expand_groups(const int32_t* grp, int n_groups, int n_seqs, int32_t* seq_ctx, hipStream_t st);
hipError_t launch_clear2_f32(float* ptr0, float* ptr1, int64_t n, hipStream_t st);
hipError_t launch_convert2_ctx(const float* acc0, const TViewOut& out0, const float* acc1, const TViewOut& out1, int P, int Hk,
                               int head_dim, hipStream_t st);
hipError_t launch_rows_copy(bool to_packed, int n_seqs, int ctx_len, int total_resp, const int32_t* cu,
                            int64_t row_bytes, const void* src, void* dst, int32_t* pos_ids, hipStream_t st);
hipError_t launch_label_map(int n_seqs, int ctx_len, int total_resp, const int32_t* cu, int32_t* next_index,
                            int32_t* first_token_index, hipStream_t st);

// Raises the dynamic-LDS limit of a kernel instantiation once per process (a host API call; not repeated on
// every launch, so that nothing but kernel launches is issued on a stream under capture after the first use).
template <auto Kern>
inline hipError_t ensure_dynamic_lds(size_t bytes) {
  static hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  return once;
}

// HIP takes fewer than 2^32 work items a launch.  Row blocks or key tiles count with the longest sequence, so that a call with many
// sequences and a long one may need more of them: its sequences go out in several launches of per_seq workgroups each.
template <typename F>
inline hipError_t launch_sequences(const AttnParams& p, int64_t per_seq, int threads, F launch) {
  if (per_seq == 0) return hipSuccess;
  const int64_t fit = ((int64_t)1 << 32) / threads - 1, step = fit > per_seq ? fit / per_seq : 1;
  hipError_t e = hipSuccess;
  for (int64_t s = 0; s < p.n_seqs && e == hipSuccess; s += step) {
    AttnParams q = p;
    q.n_seqs = (int)std::min(step, p.n_seqs - s);
    if (s) q.cu += s;
    if (s && q.seq_ctx) q.seq_ctx += 2 * s;
    e = launch(q, (unsigned)(q.n_seqs * per_seq));
  }
  return e;
}
// dK/dV: the prompt tiles go out by groups (they see all sequences of theirs), then the response tiles
template <typename F>
inline hipError_t launch_key_tiles(const AttnParams& p, int64_t prompt, int64_t per_seq, int threads, F launch) {
  const int64_t n = prompt + p.n_seqs * per_seq, fit = ((int64_t)1 << 32) / threads - 1;
  if (n == 0) return hipSuccess;
  if (n <= fit) return launch(p, (unsigned)n);
  AttnParams q = p;
  q.n_dec_tiles = 0;
  const int n_groups = p.grp ? p.n_groups : 1;
  const int64_t per_group = prompt / n_groups, step = fit > per_group ? fit / std::max<int64_t>(per_group, 1) : 1;
  for (int64_t g = 0; prompt && g < n_groups; g += step) {
    q.n_groups = (int)std::min(step, n_groups - g);
    if (p.grp) q.grp = p.grp + 4 * g;
    const hipError_t e = launch(q, (unsigned)(q.n_groups * per_group));
    if (e != hipSuccess) return e;
  }
  q = p;
  q.n_ctx_tiles = 0;
  return launch_sequences(q, per_seq, threads, launch);
}

// dK/dV workgroups: of the prompt tiles (with their parts), and per sequence; fills the kernel's fields
struct KeyTiles {
  int64_t prompt, per_seq;
};
inline KeyTiles key_tiles(AttnParams& p, int key_tile) {
  p.n_ctx_tiles = (p.ctx_len + key_tile - 1) / key_tile;
  p.n_dec_tiles = (p.max_rows + key_tile - 1) / key_tile;
  if (p.n_split < 1) p.n_split = 1;
  return {(int64_t)(p.grp ? p.n_groups : 1) * p.n_ctx_tiles * p.Hk * p.n_split, (int64_t)p.n_dec_tiles * p.Hk};
}
// dK/dV kernels that know both directions of a walk (kvsched.h)
template <typename F>
inline hipError_t launch_direction(const AttnParams& p, int head_dim, F launch) {
  if (p.window > 0 || (p.ctx_len > 0 && !p.grp) || !walk_down(p.max_rows, p.G, head_dim)) return launch(std::integral_constant<int, WALK_UP>{});
  if (p.cu) return launch(std::integral_constant<int, WALK_OWN>{});
  return launch(std::integral_constant<int, WALK_DOWN>{});
}

}  // namespace dkv
