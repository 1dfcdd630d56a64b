// Un-padded, XOR-swizzled LDS tiles for head dims 64 / 96 / 128 / 192 / 256 / 512 and the LDS transpose read.
//
// A tile is ROWS x D bf16, row-major, 2*D bytes per row, made of 16-byte chunks.  Chunk c of row r is
// stored at chunk position c ^ swz<D>(r).  The swizzle makes all three access patterns used by the
// kernels bank-conflict free on the 64-bank LDS:
//   * 16-byte staging writes (16 lanes = consecutive chunks of a row),
//   * 16-byte MFMA operand reads with the lane on the row axis (16 lanes = 16 consecutive rows, same
//     chunk),
//   * ds_read_b64_tr_b16 transpose reads with the lane on the column axis (16 lanes = 4 consecutive
//     rows x 32 contiguous bytes; the neighbouring 16 lanes read the next 32 bytes of the same rows).
//
// ds_read_b64_tr_b16: within each group of 16 lanes, lane i supplies the address of 4 consecutive
// 16-bit values; viewing the 16 x 4 values as a flat list v[0..63] (lane-major), lane i receives
// v[i], v[16+i], v[32+i], v[48+i].  With lane i pointing at row k0 + i/4, columns d0 + 4*(i%4) .. +3 of
// a row-major tile, lane i therefore receives column d0 + i of rows k0 .. k0+3: a K-indexed MFMA
// operand of the transposed tile without any transposed copy in LDS.
#pragma once
#include "common.h"

namespace dkv {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int D>
__device__ __forceinline__ int swz(int row) {
  static_assert(D == 64 || D == 96 || D == 128 || D == 192 || D == 256 || D == 512, "swizzle defined for these head dims");
  // (the 512- and 1024-byte rows of head dims 256 and 512 span several bank lines: the chunk index bits from 4 on
  // do not select a bank)
  // The 192- and 384-byte rows of head dims 96 and 192 are not powers of two, but row r starts 4 (-r mod 4) resp.
  // 8 (r mod 2) chunks into a 256-byte bank line, which separates four (two) consecutive rows by itself; the XOR of the
  // lowest two (three) chunk bits separates the others and stays inside the row's 12 = 3 x 4 (24 = 3 x 8) chunks.
  if (D == 96) return (row >> 2) & 3;
  if (D == 128 || D == 256 || D == 512) return ((row & 3) << 2) | ((row >> 2) & 3);
  return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

// Rows that do not divide the 1 KB of a global -> LDS load instruction (head dims 96 and 192): lane l of the t-th
// consecutive instruction lands at 16-byte unit 64 t + l, i.e. chunk position (64 t + l) % CPR of row (64 t + l) / CPR.
// Three instructions cover kSplitRows<D> whole rows (16 or 8), and the pattern of rows and chunk positions repeats.
template <int D>
constexpr bool kSplitRow = 1024 % (2 * D) != 0;
template <int D>
constexpr int kSplitRows = 3 * 64 / (D / 8);
template <int D>
__device__ __forceinline__ int split_row(int t, int lane) { return (64 * (t % 3) + lane) / (D / 8) + (t / 3) * kSplitRows<D>; }
template <int D>
__device__ __forceinline__ int split_pos(int t, int lane) { return (64 * (t % 3) + lane) % (D / 8); }

// byte offset of chunk `chunk` of row `row` inside a tile
template <int D>
__device__ __forceinline__ int tile_off(int row, int chunk) {
  return row * (2 * D) + ((chunk ^ swz<D>(row)) << 4);
}

// Per-lane byte offset for a transpose read of rows (row_base + (lane%16)/4), columns
// col_base + 16*((lane/16)%2) + 4*(lane%4) .. +3, where row_base is a multiple of 4 given relative to a
// 16-row aligned origin (the swizzle has period 16 rows).
template <int D>
__device__ __forceinline__ int tr_off(int lane, int row_base, int col_base) {
  const int r16 = lane & 15, g = (lane >> 4) & 1;
  const int row = row_base + (r16 >> 2);
  const int col = col_base + g * 16 + (r16 & 3) * 4;
  return tile_off<D>(row, col >> 3) + ((col >> 2) & 1) * 8;
}

// two transpose reads (rows k0..k0+3 and k0+8..k0+11 of the lane's group) -> one MFMA operand
__device__ __forceinline__ bf16x8 tr_pair(const unsigned char* a0, const unsigned char* a1) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a0));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a1));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// ---- tiles read by the 16x16x32 MFMA (head dims 64, 96, 128).  A row operand is row l % 16, 64-byte k-step ks, of which lane group
// g = l / 16 takes chunk kgrp16<D>(g) (both operands of a product alike); a transpose read takes rows 4 g .. 4 g + 3 (+ 16) and 16
// columns.  A 16-byte read is served in groups of sixteen lanes {0-3, 12-15, 20-23, 24-27}, {4-11, 16-19, 28-31}, + 32; an 8-byte
// transpose read in halves of the wave.  This swizzle and choice of chunks keeps both free of bank conflicts (all rows of eight
// consecutive ones on different pairs of chunks for the latter; checked by enumeration).
template <int D>
__device__ __forceinline__ int swz16(int row) {
  static_assert(D == 64 || D == 96 || D == 128, "");
  const int pair = D == 128 ? row & 7 : D == 64 ? (row >> 1) & 3 : (row >> 2) & 1;
  return 2 * pair | ((row >> 3) & 1);
}
template <int D>
__device__ __forceinline__ int kgrp16(int g) {
  return D == 96 ? (g == 0 ? 0 : g == 1 ? 3 : g - 1) : ((g & 1) << 1) | (g >> 1);
}
// byte offset of this lane's row operand of k-step ks, rows 0-15
template <int D>
__device__ __forceinline__ int frag16_off(int lane, int ks) {
  const int row = lane & 15;
  return row * (2 * D) + (((4 * ks + kgrp16<D>(lane >> 4)) ^ swz16<D>(row)) << 4);
}
// byte offset of this lane's transpose read of rows 0-15, columns 16 db .. 16 db + 15
template <int D>
__device__ __forceinline__ int tr16_off(int lane, int db) {
  const int row = 4 * (lane >> 4) + ((lane & 15) >> 2), col = 16 * db + (lane & 3) * 4;
  return row * (2 * D) + (((col >> 3) ^ swz16<D>(row)) << 4) + ((col >> 2) & 1) * 8;
}
// transpose reads of rows 0-15 and 16-31 -> the 32-deep operand of a 16-column block
template <int D>
__device__ __forceinline__ bf16x8 tr16_pair(const unsigned char* a) {
  return tr_pair(a, a + 16 * 2 * D);
}
// the same by LDS address: a row operand; the operand of a transpose read
__device__ __forceinline__ bf16x8 lds_frag(uint32_t a) { return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(a); }
template <int D>
__device__ __forceinline__ bf16x8 lds_tr16(uint32_t a) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)a);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(a + 16 * 2 * D));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace dkv
