// Bandwidth-bound helper kernels: D = rowsum(dO * O) (the "dot_do_o" preprocess of Alg. 1), fp32 fill,
// fp32 -> bf16 cast of the accumulated shared-prompt gradients (Alg. 2) and the layout gathers between
// the standard packing (Eq. 1) and the single-prompt packing (Eq. 5).
#include "common.h"
#include "launch.h"
#include "rules.h"

namespace dkv {

// ---------------------------------------------------------------------------------------------
// D[h][row] = sum_d dO[row,h,d] * O[row,h,d].  One group of D/8 lanes per (row, head); each lane reads
// 16 bytes of dO and of O, so a wave reads whole contiguous rows.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void dot_do_o_kernel(TView dout, TView o, const float* __restrict__ lse,
                                                       float* __restrict__ dvec, float* __restrict__ lse2,
                                                       int total, int H) {
  // lanes per (row, head): D / 8 of them carry data, rounded up to a power of two for the butterfly (d = 96, 192)
  constexpr int LPR = D / 8 <= 8 ? 8 : D / 8 <= 16 ? 16 : D / 8 <= 32 ? 32 : 64;
  constexpr int RPB = 256 / LPR;      // (row, head) pairs per block
  const int tid = threadIdx.x;
  const int64_t pair = (int64_t)blockIdx.x * RPB + tid / LPR;
  const int sub = tid % LPR;
  float acc = 0.f;
  const bool ok = pair < (int64_t)total * H;
  const int64_t row = ok ? pair / H : 0;
  const int h = ok ? (int)(pair % H) : 0;
  if (ok && sub < D / 8) {
    const u32x4 a = *reinterpret_cast<const u32x4*>(dout.ptr + row * dout.ts + (int64_t)h * dout.hs + sub * 8);
    const u32x4 b = *reinterpret_cast<const u32x4*>(o.ptr + row * o.ts + (int64_t)h * o.hs + sub * 8);
    acc = dot8_bf16(a, b);
  }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (ok && sub == 0) {
    dvec[(int64_t)h * total + row] = acc;
    lse2[(int64_t)h * total + row] = lse[(int64_t)h * total + row] * LOG2E;   // exponent offset in base-2 units
  }
}

hipError_t launch_dot_do_o(const TView& dout, const TView& o, const float* lse, float* dvec, float* lse2, int total,
                           int H, int head_dim, hipStream_t st) {
  const int64_t pairs = (int64_t)total * H;
  if (pairs == 0) return hipSuccess;
  const int lanes = head_dim / 8, lpr = lanes <= 8 ? 8 : lanes <= 16 ? 16 : lanes <= 32 ? 32 : 64, rpb = 256 / lpr;
  const unsigned grid = (unsigned)((pairs + rpb - 1) / rpb);
  switch (head_dim) {
    case 64:  hipLaunchKernelGGL(dot_do_o_kernel<64>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    case 96:  hipLaunchKernelGGL(dot_do_o_kernel<96>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    case 128: hipLaunchKernelGGL(dot_do_o_kernel<128>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    case 192: hipLaunchKernelGGL(dot_do_o_kernel<192>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    case 256: hipLaunchKernelGGL(dot_do_o_kernel<256>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    case 512: hipLaunchKernelGGL(dot_do_o_kernel<512>, dim3(grid), dim3(256), 0, st, dout, o, lse, dvec, lse2, total, H); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Two fp32 arrays of n elements each, cleared by one launch (the dK and the dV accumulator): at small sizes a launch is
// most of the time.  With the two casts in one launch as well, the layer of 4 x (256 + 128) rows, 4 / 2 heads, d = 64 goes
// from 91.9 to 88.0 us.
__global__ __launch_bounds__(256) void clear2_f32_kernel(float* __restrict__ ptr0, float* __restrict__ ptr1, int64_t n) {
  float* ptr = blockIdx.y ? ptr1 : ptr0;
  const int64_t stride = (int64_t)gridDim.x * 256 * 4;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += stride) {
    if (i + 4 <= n) {
      *reinterpret_cast<f32x4*>(ptr + i) = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
      for (int64_t j = i; j < n; ++j) ptr[j] = 0.f;
    }
  }
}

hipError_t launch_clear2_f32(float* ptr0, float* ptr1, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 1023) / 1024;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(clear2_f32_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, st, ptr0, ptr1, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Several prompt groups in one launch: per-sequence {first prompt row, prompt length} from the group table
// {first prompt row, P_g, first sequence, end sequence}; one thread per (group, sequence slot).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void expand_groups_kernel(const int32_t* __restrict__ grp, int n_groups,
                                                            int32_t* __restrict__ seq_ctx) {
  const int g = blockIdx.y;
  if (g >= n_groups) return;
  const int s0 = grp[4 * g + 2], s1 = grp[4 * g + 3];
  for (int s = s0 + blockIdx.x * 256 + threadIdx.x; s < s1; s += gridDim.x * 256) {
    seq_ctx[2 * s] = grp[4 * g];
    seq_ctx[2 * s + 1] = grp[4 * g + 1];
  }
}

// prompt offsets (n + 1) of groups packed back to back: the groups' first rows, then the total
__global__ __launch_bounds__(256) void group_offsets_kernel(const int32_t* __restrict__ grp, int n_groups, int total_ctx,
                                                            int32_t* __restrict__ cu) {
  for (int g = blockIdx.x * 256 + threadIdx.x; g <= n_groups; g += gridDim.x * 256) cu[g] = g < n_groups ? grp[4 * g] : total_ctx;
}

hipError_t launch_group_offsets(const int32_t* grp, int n_groups, int total_ctx, int32_t* cu, hipStream_t st) {
  hipLaunchKernelGGL(group_offsets_kernel, dim3((unsigned)min(64, (n_groups + 256) / 256)), dim3(256), 0, st, grp, n_groups,
                     total_ctx, cu);
  return hipGetLastError();
}

hipError_t launch_expand_groups(const int32_t* grp, int n_groups, int n_seqs, int32_t* seq_ctx, hipStream_t st) {
  if (n_groups <= 0 || n_seqs <= 0) return hipSuccess;
  const int bx = min(64, (n_seqs + 255) / 256);
  hipLaunchKernelGGL(expand_groups_kernel, dim3((unsigned)bx, (unsigned)n_groups), dim3(256), 0, st, grp, n_groups,
                     seq_ctx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// acc (P, Hk, D) fp32 contiguous -> out (P, Hk, D) bf16 strided, the dK and the dV accumulator in one launch (blockIdx.y)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void convert2_ctx_kernel(const float* __restrict__ acc0, TViewOut out0,
                                                           const float* __restrict__ acc1, TViewOut out1, int64_t n8, int Hk,
                                                           int D) {
  const float* acc = blockIdx.y ? acc1 : acc0;
  const TViewOut out = blockIdx.y ? out1 : out0;
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int cpr = D / 8;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += stride) {
    const int ch = (int)(i % cpr);
    const int64_t rh = i / cpr;
    const int h = (int)(rh % Hk);
    const int64_t row = rh / Hk;
    const f32x4 a = *reinterpret_cast<const f32x4*>(acc + i * 8);
    const f32x4 b = *reinterpret_cast<const f32x4*>(acc + i * 8 + 4);
    u32x4 w;
    w.x = pack2_bf16(a[0], a[1]);
    w.y = pack2_bf16(a[2], a[3]);
    w.z = pack2_bf16(b[0], b[1]);
    w.w = pack2_bf16(b[2], b[3]);
    *reinterpret_cast<u32x4*>(out.ptr + row * out.ts + (int64_t)h * out.hs + ch * 8) = w;
  }
}

hipError_t launch_convert2_ctx(const float* acc0, const TViewOut& out0, const float* acc1, const TViewOut& out1, int P, int Hk,
                               int head_dim, hipStream_t st) {
  const int64_t n8 = (int64_t)P * Hk * head_dim / 8;
  if (n8 == 0) return hipSuccess;
  int64_t blocks = (n8 + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  // (a caller may let the second output overwrite the first accumulator: one after the other then)
  const uintptr_t a0 = (uintptr_t)acc0, o1 = (uintptr_t)out1.ptr;
  const uintptr_t o1_end = o1 + (uintptr_t)((int64_t)(P - 1) * out1.ts + (int64_t)(Hk - 1) * out1.hs + head_dim) * 2;
  if (o1 < a0 + (uintptr_t)n8 * 32 && a0 < o1_end) {
    hipLaunchKernelGGL(convert2_ctx_kernel, dim3((unsigned)blocks), dim3(256), 0, st, acc0, out0, acc0, out0, n8, Hk, head_dim);
    hipLaunchKernelGGL(convert2_ctx_kernel, dim3((unsigned)blocks), dim3(256), 0, st, acc1, out1, acc1, out1, n8, Hk, head_dim);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(convert2_ctx_kernel, dim3((unsigned)blocks, 2), dim3(256), 0, st, acc0, out0, acc1, out1, n8, Hk, head_dim);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Layout copies between the standard packing (Eq. 1) and the single-prompt packing (Eq. 5); rows are opaque records of 4- or
// 16-byte units.  All three kernels are bound by memory once enough of it is in flight.
//   * repack, long rows: driven by the destination rows, TPR threads a row, source row by binary search in cu_seqlens;
//   * replicate, long rows: driven by the source rows, so that a prompt row is read once and written up to 16 times from
//     registers, where a gather read it again for every copy (replicate_copies);
//   * short rows (token ids, labels): a workgroup per row spends its life in the binary search; one lane takes one unit.
// 16 x (8192 + 1024) rows of 8 KB: replicate 335 -> 260 us (5.4 TB/s, the rate of a plain copy), repack 77 -> 65 us; of 4
// bytes: replicate 118 -> 4.9 us, repack 14 -> 4.7 us.
// ---------------------------------------------------------------------------------------------
// the last sequence s with base * s + cu[s] <= x (x >= 0, cu[0] == 0)
__device__ __forceinline__ int find_seq(const int32_t* cu, int n_seqs, int64_t base, int64_t x) {
  int lo = 0, hi = n_seqs;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (base * mid + cu[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// packed row -> row of the standard packing (prompt rows: sequence 0's copy) and logical position
__device__ __forceinline__ int64_t standard_row(const int32_t* cu, int n_seqs, int P, int64_t prow, int& pos) {
  if (prow < P) {
    pos = (int)prow;
    return prow;
  }
  const int64_t x = prow - P;
  const int s = find_seq(cu, n_seqs, 0, x);
  pos = P + (int)(x - cu[s]);
  return (int64_t)(s + 1) * P + x;
}
// row of the standard packing -> packed row and logical position
__device__ __forceinline__ int64_t packed_row(const int32_t* cu, int n_seqs, int P, int64_t srow, int& pos) {
  const int s = find_seq(cu, n_seqs, P, srow);
  const int64_t off = srow - ((int64_t)s * P + cu[s]);
  pos = (int)off;
  return off < P ? off : cu[s] + off;
}

template <typename VEC>
__global__ __launch_bounds__(256) void short_rows_kernel(bool to_packed, int n_seqs, int P, int64_t drows,
                                                         const int32_t* __restrict__ cu, int row_vecs,
                                                         const VEC* __restrict__ src, VEC* __restrict__ dst,
                                                         int32_t* __restrict__ pos_ids) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, drow = i / row_vecs;
  if (drow >= drows) return;
  const int unit = (int)(i - drow * row_vecs);
  int pos;
  const int64_t srow = to_packed ? standard_row(cu, n_seqs, P, drow, pos) : packed_row(cu, n_seqs, P, drow, pos);
  dst[i] = src[srow * row_vecs + unit];
  if (pos_ids != nullptr && unit == 0) pos_ids[drow] = pos;
}

// a workgroup's or a wave's row, in a scalar register: the search in cu_seqlens takes scalar loads then (53 x 506 + 20099 rows of
// 4 KB, repack: 29.5 us with vector loads, 25.0 with scalar ones)
template <int TPR>
__device__ __forceinline__ int64_t row_index() {
  static_assert(TPR == 64 || TPR == 256);
  if constexpr (TPR == 256) return blockIdx.x;
  else return (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
}

// (four units in flight a thread: 6 x 725 + 56 rows of 64 KB, repack: 16.8 us with two, 16.4 with four)
template <bool NT, int TPR, typename VEC>
__device__ __forceinline__ void copy_row(const VEC* s, VEC* d, int64_t row_vecs, int t) {
  auto load = [](const VEC* p) { return NT ? __builtin_nontemporal_load(p) : *p; };
  auto store = [](VEC v, VEC* p) {
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
  };
  int64_t i = t;
  for (; i + 3 * TPR < row_vecs; i += 4 * TPR) {
    const VEC a = load(s + i), b = load(s + i + TPR), c = load(s + i + 2 * TPR), e = load(s + i + 3 * TPR);
    store(a, d + i);
    store(b, d + i + TPR);
    store(c, d + i + 2 * TPR);
    store(e, d + i + 3 * TPR);
  }
  for (; i + TPR < row_vecs; i += 2 * TPR) {
    const VEC a = load(s + i), b = load(s + i + TPR);
    store(a, d + i);
    store(b, d + i + TPR);
  }
  if (i < row_vecs) store(load(s + i), d + i);
}

// NT: the copy is larger than the last-level cache, nothing of it is found there again
template <typename VEC, int TPR, bool NT>
__global__ __launch_bounds__(256) void repack_rows_kernel(int n_seqs, int P, int64_t drows, const int32_t* __restrict__ cu,
                                                          int64_t row_vecs, const VEC* __restrict__ src, VEC* __restrict__ dst,
                                                          int32_t* __restrict__ pos_ids) {
  const int64_t drow = row_index<TPR>();
  if (drow >= drows) return;
  const int t = threadIdx.x % TPR;
  int pos;
  const VEC* s = src + standard_row(cu, n_seqs, P, drow, pos) * row_vecs;
  copy_row<NT, TPR>(s, dst + drow * row_vecs, row_vecs, t);
  if (pos_ids != nullptr && t == 0) pos_ids[drow] = pos;
}

template <typename VEC, int TPR>
__global__ __launch_bounds__(256) void replicate_rows_kernel(int n_seqs, int P, int total_resp, int copies, int64_t prompt_items,
                                                             const int32_t* __restrict__ cu, int64_t row_vecs,
                                                             const VEC* __restrict__ src, VEC* __restrict__ dst,
                                                             int32_t* __restrict__ pos_ids) {
  // items: the P prompt rows for every group of `copies` sequences, then the response rows
  const int64_t item = row_index<TPR>();
  const int t = threadIdx.x % TPR;
  if (item >= prompt_items) {
    const int64_t x = item - prompt_items;
    if (x >= total_resp) return;
    const int q = find_seq(cu, n_seqs, 0, x);
    const int64_t drow = (int64_t)(q + 1) * P + x;
    copy_row<false, TPR>(src + (P + x) * row_vecs, dst + drow * row_vecs, row_vecs, t);
    if (pos_ids != nullptr && t == 0) pos_ids[drow] = P + (int)(x - cu[q]);
    return;
  }
  const int pos = (int)(item % P), s0 = (int)(item / P) * copies, s1 = min(n_seqs, s0 + copies);
  const VEC* s = src + (int64_t)pos * row_vecs;
  auto row_of = [&](int q) { return (int64_t)q * P + cu[q] + pos; };
  int64_t i = t;
  for (; i + TPR < row_vecs; i += 2 * TPR) {
    const VEC a = s[i], b = s[i + TPR];
    for (int q = s0; q < s1; ++q) {
      VEC* d = dst + row_of(q) * row_vecs + i;
      d[0] = a;
      d[TPR] = b;
    }
  }
  if (i < row_vecs) {
    const VEC a = s[i];
    for (int q = s0; q < s1; ++q) dst[row_of(q) * row_vecs + i] = a;
  }
  if (pos_ids != nullptr && t == 0)
    for (int q = s0; q < s1; ++q) pos_ids[row_of(q)] = pos;
}

template <typename VEC>
static hipError_t launch_rows_copy_t(bool to_packed, int n_seqs, int P, int T, const int32_t* cu, int64_t row_vecs, const void* src,
                                     void* dst, int32_t* pos_ids, hipStream_t st) {
  const VEC* s = static_cast<const VEC*>(src);
  VEC* d = static_cast<VEC*>(dst);
  const int64_t drows = (to_packed ? (int64_t)P : (int64_t)n_seqs * P) + T;
  const bool wide = row_vecs > 128;   // (a workgroup or a wave per row: at most half of the threads idle at the end of a row)
  auto launch = [&](auto kern, int64_t items, int per_block, auto... args) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((items + per_block - 1) / per_block)), dim3(256), 0, st, args...);
    return hipGetLastError();
  };
  if (row_vecs < 32)
    return launch(short_rows_kernel<VEC>, drows * row_vecs, 256, to_packed, n_seqs, P, drows, cu, (int)row_vecs, s, d, pos_ids);
  if (to_packed) {
    const bool nt = 2 * drows * row_vecs * (int64_t)sizeof(VEC) > (int64_t)256 << 20;
    if (wide && nt) return launch(repack_rows_kernel<VEC, 256, true>, drows, 1, n_seqs, P, drows, cu, row_vecs, s, d, pos_ids);
    if (wide) return launch(repack_rows_kernel<VEC, 256, false>, drows, 1, n_seqs, P, drows, cu, row_vecs, s, d, pos_ids);
    return launch(repack_rows_kernel<VEC, 64, false>, drows, 4, n_seqs, P, drows, cu, row_vecs, s, d, pos_ids);
  }
  const int copies = rules::replicate_copies(n_seqs, P, T);
  const int64_t prompt_items = (int64_t)P * ((n_seqs + copies - 1) / copies), items = prompt_items + T;
  if (wide) return launch(replicate_rows_kernel<VEC, 256>, items, 1, n_seqs, P, T, copies, prompt_items, cu, row_vecs, s, d, pos_ids);
  return launch(replicate_rows_kernel<VEC, 64>, items, 4, n_seqs, P, T, copies, prompt_items, cu, row_vecs, s, d, pos_ids);
}

hipError_t launch_rows_copy(bool to_packed, int n_seqs, int ctx_len, int total_resp, const int32_t* cu,
                            int64_t row_bytes, const void* src, void* dst, int32_t* pos_ids, hipStream_t st) {
  if ((to_packed ? (int64_t)ctx_len : (int64_t)n_seqs * ctx_len) + total_resp == 0) return hipSuccess;
  const bool v16 = (row_bytes % 16 == 0) && (((uintptr_t)src | (uintptr_t)dst) % 16 == 0);
  return v16 ? launch_rows_copy_t<u32x4>(to_packed, n_seqs, ctx_len, total_resp, cu, row_bytes / 16, src, dst, pos_ids, st)
             : launch_rows_copy_t<uint32_t>(to_packed, n_seqs, ctx_len, total_resp, cu, row_bytes / 4, src, dst, pos_ids, st);
}

// ---------------------------------------------------------------------------------------------
// Next-token map of the single-prompt packing (Sec. 2.3 "shared prompt logits"): packed row t predicts the
// token at packed row next_index[t] (-1: nothing).  Prompt rows and response rows shift by one inside their own
// segment; the row of the last prompt token predicts the FIRST token of every response, which cannot be
// expressed per row: first_token_index[i] (row P + cu[i], or -1 for an empty response or P = 0) lists them, all
// read from row P - 1.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void label_map_kernel(int n_seqs, int P, int total_resp,
                                                        const int32_t* __restrict__ cu, int32_t* __restrict__ next_index,
                                                        int32_t* __restrict__ first_token_index) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t T = (int64_t)P + total_resp;
  if (next_index != nullptr && t < T) {
    int nxt;
    if (t < P) {
      nxt = t + 1 < P ? (int)(t + 1) : -1;
    } else {
      const int x = (int)(t - P);
      int lo = 0, hi = n_seqs;   // find i with cu[i] <= x < cu[i+1]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= x) lo = mid; else hi = mid;
      }
      nxt = x + 1 < cu[lo + 1] ? (int)(t + 1) : -1;
    }
    next_index[t] = nxt;
  }
  if (first_token_index != nullptr && t < n_seqs) {
    const int i = (int)t;
    first_token_index[i] = (P > 0 && cu[i + 1] > cu[i]) ? P + cu[i] : -1;
  }
}

hipError_t launch_label_map(int n_seqs, int ctx_len, int total_resp, const int32_t* cu, int32_t* next_index,
                            int32_t* first_token_index, hipStream_t st) {
  const int64_t n = max((int64_t)ctx_len + total_resp, (int64_t)n_seqs);
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(label_map_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n_seqs, ctx_len,
                     total_resp, cu, next_index, first_token_index);
  return hipGetLastError();
}

}  // namespace dkv
