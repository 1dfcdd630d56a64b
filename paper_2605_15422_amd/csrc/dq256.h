// dQ kernel for head dims 192 and 256 with producer / consumer wave specialisation:
//   dQ = scale * dS K,  dS = P * (dP - D),  P = exp(scale * Q K^T - LSE),  dP = dO V^T     (Alg. 1)
// evaluated per query block over all its visible key tiles (prompt tiles, then own-response tiles), dQ
// accumulated in registers and written once, as in the head-dim 64 / 128 kernel.
//
// At this head dim the Q and dO fragments of a 32-row subtile (128 registers) and its dQ accumulator (128
// more) cannot live in one wave of 256 registers, so the two are given to different waves.  A workgroup owns
// four 32-row subtiles (128 rows that share the staged K / V tiles: GQA heads and / or consecutive row blocks):
//   * producer wave w (0-3) keeps Q and dO of subtile w in registers and forms, per 32-key tile,
//     S^T = K Q^T, dP^T - D = V dO^T - D, P and dS^T in fp32, and publishes dS^T as the bf16 B operand of the
//     product through a double-buffered exchange area (32 MFMAs per tile);
//   * consumer wave c (4-7) owns the head-dim blocks c and c + 4 of dQ^T for ALL four subtiles (128 accumulator
//     registers) and, one tile behind, adds K^T dS^T with K^T from LDS transpose reads of the row-major K tile
//     (16 MFMAs per tile; every transposed operand feeds four MFMAs, so the slow transpose reads stay at four
//     per tile).  The consumers also issue the global -> LDS loads of K and V, three tiles ahead, into four
//     stages, and read their K^T operands one interval early, so that a stage is free again after one interval.
// Each SIMD runs one producer and one consumer: 48 MFMAs per 32-key tile and one barrier.
// LDS: 4 x (16 KB K + 16 KB V) + 2 x 8 KB exchange = 144 KB.
// Head dim 192: consumer waves 4-6 own head-dim blocks c and c + 3, wave 7 makes all requests, as in the forward kernel.
// On N = 8, P = 4096, R ~ U(131, 2048), 12 / 4 heads: 0.61 + 0.13 ms (Call 2 + Call 1), against 1.62 + 0.35 ms for the
// register-staged kernel that served it before.
#pragma once
#include "common.h"
#include "dma.h"
#include "qsched.h"
#include "tiles.h"

namespace dkv {
namespace dq256 {

constexpr int BN = 32, NSUB = 4;                 // keys per tile, 32-row subtiles per workgroup
constexpr int NSTAGE = 4;                        // LDS stages of a K tile and a V tile
constexpr int XCH_BYTES = NSUB * 2048;           // [subtile][k-step 0,1][lane] x 16 B
template <int D>
struct Cfg {
  static constexpr bool LOADER = kSplitRow<D>;   // one consumer wave makes all requests and owns no accumulator
  static constexpr int KS = D / 16, RB = 2 * D, CPR = D / 8;
  static constexpr int TILE_BYTES = BN * RB, STAGE_BYTES = 2 * TILE_BYTES;   // K tile | V tile
  static constexpr int XCH_OFF = NSTAGE * STAGE_BYTES;
  static constexpr int SMEM_BYTES = XCH_OFF + 2 * XCH_BYTES;
  static constexpr int OUT_RS = RB + 16;         // row stride of the output tile staged in LDS (rows 4 banks apart)
  static_assert(NSUB * 32 * OUT_RS <= XCH_OFF, "the output tile fits the stages");
  static constexpr int IPT = TILE_BYTES / 1024 / (LOADER ? 1 : 4);   // 1 KB load instructions per requesting wave, tile and tensor
  static constexpr int RPI = 1024 / RB;          // rows per load instruction
  // The swizzle works on the lowest four (head dim 192: three) bits of the chunk index: NRO per-lane offsets serve all
  // k-steps, every further NRO k-steps lying NRO * 32 bytes further.
  static constexpr int NRO = LOADER ? 4 : 8;
  static constexpr int EBLK = D / 64;            // a consumer wave owns head-dim blocks jb and jb + EBLK
};

// workgroup `bid` of `nblk`, the row statistics given
template <int D, bool LOCAL>
__device__ __forceinline__ void workgroup(const AttnParams p, int bid, int nblk) {
  constexpr bool STATS = false;
#include "dq256_body.h"
}

}  // namespace dq256
}  // namespace dkv
