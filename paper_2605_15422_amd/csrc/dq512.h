// dQ kernel for head dim 512 with producer / consumer wave specialisation:
//   dQ = scale * dS K,  dS = P * (dP - D),  P = exp(scale * Q K^T - LSE),  dP = dO V^T     (Alg. 1)
// evaluated per query block over all its visible key tiles (prompt tiles, then own-response tiles), dQ
// accumulated in registers and written once, as in the narrower kernels.
//
// What this head dim dictates.  The fp32 dQ of one row fills 2 KB and the four consumer waves can give 128 of
// their 256 registers to accumulators: a workgroup owns 64 rows (two 32-row subtiles), each consumer wave
// holding four of the sixteen 32-wide head-dim blocks of dQ^T for both.  The Q and dO fragments of 16 rows
// already fill 128 registers, so each of the four producers takes 16 rows and works with the 16x16x32 MFMA:
// per 16-key tile it forms S^T = K Q^T, dP^T - D = V dO^T - D, P and dS^T in fp32 and publishes dS^T as the
// bf16 B operand of the consumers' 32x32x16 product (32 small MFMAs per tile); the consumers, one tile behind,
// add K^T dS^T with K^T from LDS transpose reads (8 MFMAs per tile).  K / V tiles of 16 keys (16 KB + 16 KB)
// travel global -> LDS three tiles ahead into four stages, issued by the consumers, which read their K^T
// operands one interval early so that a stage is free again after one interval.  One barrier per tile.
#pragma once
#include "common.h"
#include "dma.h"
#include "qsched.h"
#include "tiles.h"

namespace dkv {
namespace dq512 {

constexpr int D = 512;
constexpr int BN = 16, NSUB = 2;                 // keys per tile, 32-row subtiles per workgroup (consumers' view)
constexpr int NDB = D / 128;                     // head-dim blocks per consumer wave
constexpr int KS = D / 32, RB = 2 * D;           // k-steps of the 16x16x32 MFMA
constexpr int TILE_BYTES = BN * RB;
constexpr int NSTAGE = 4, STAGE_BYTES = 2 * TILE_BYTES;   // K tile | V tile
constexpr int XCH_OFF = NSTAGE * STAGE_BYTES;
constexpr int XCH_BYTES = NSUB * 1024;           // [subtile][lane] x 16 B
constexpr int SMEM_BYTES = XCH_OFF + 2 * XCH_BYTES;
constexpr int IPT = TILE_BYTES / 1024 / 4;       // 1 KB load instructions per consumer wave, tile and tensor

// workgroup `bid` of `nblk`, the row statistics given
template <bool LOCAL>
__device__ __forceinline__ void workgroup(const AttnParams p, int bid, int nblk) {
  constexpr bool STATS = false;
#include "dq512_body.h"
}

}  // namespace dq512
}  // namespace dkv
