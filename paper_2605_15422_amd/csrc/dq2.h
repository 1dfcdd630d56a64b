// dQ kernel for head dims 64, 96 and 128, tuned variant:
//   dQ = scale * dS K,  dS = P * (dP - D),  P = exp(scale * Q K^T - LSE),  dP = dO V^T     (Alg. 1)
// evaluated per query block over all its visible key tiles (prompt tiles, then own-response tiles), so
// dQ is accumulated in registers and written once: no fp32 dQ scratch, no atomics, no convert pass.
//
// Shape: 4 waves, two workgroups a CU (three at head dim 64), or 8, two per SIMD, by the rule of row_block_waves (rules.h); each
// owns 32 rows, two halves of 16, with Q, dO fragments and the dQ^T accumulator in registers; K and
// V tiles of 64 keys travel global -> LDS directly (global_load_lds, two or three tiles ahead: no staging registers) into
// two rings of swizzled tiles.  S^T = K Q^T and dP^T = V dO^T take 16-byte row operands from LDS; dQ^T += K^T dS^T takes K^T
// through LDS transpose reads of the same row-major K tile.  A 64-key tile is consumed as two 32-key halves.
// 16x16x32 MFMAs, as in the forward kernel (fwd2.hip): more work in the card's power than with 32x32x16, and the two halves of the
// rows are two streams of work, so that softmax and products of one issue beside the chains of the other and the next half's
// operands travel under the last MFMAs.  Measured against one stream of 32x32x16: 16 x 1024 rows behind 8192, 32 / 8 heads,
// d = 128 2.83 -> 2.61 ms (1341 TFLOP/s of MFMA work); 8 x U(131, 2048) (9112 rows) behind 4096, 16 / 4 heads, d = 96 396 -> 368 us; d = 64, 32 / 8
// heads 518 -> 483 us.  Head dim 96: tiles of un-padded 192-byte rows (tiles.h).
#pragma once
#include <type_traits>
#include "common.h"
#include "dma.h"
#include "qsched.h"
#include "tiles.h"

namespace dkv {

// Ring slots of K and V: with four the K tiles travel three tiles ahead, with three two; with two slots the V tiles travel one ahead.
template <int D, int NW>
constexpr int kDq2Stages = rules::dq_ring_slots(D, NW);
template <int D, int NW>
constexpr int kDq2VStages = rules::dq_v_slots(D, NW);

// workgroup `bid` of `nblk`; STATS: it may have to form the row statistics (p.make_stats())
template <int D, int NW, bool LOCAL, bool STATS>
__device__ __forceinline__ void dq2_workgroup(const AttnParams& p, int bid, int nblk) {
  constexpr int BN = 64;
  constexpr int KS = D / 32, DB = D / 16, RB = 2 * D, CPR = D / 8;
  constexpr int T = BN * RB, HT = 32 * RB;         // bytes of a tile, of half a tile
  constexpr int NSTAGE = kDq2Stages<D, NW>, NVST = kDq2VStages<D, NW>, V_RING = NSTAGE * T;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];   // K ring | V ring (aligned: addresses are formed by XOR)

  QBlock b;
  if (!decode_qblock<BN>(p, b, bid, nblk)) return;
  make_uniform(b);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, lg = lane >> 4;
  const int P = b.P, R = b.R, W = p.window;
  const float c = p.scale_log2;

  const int head = b.hk * p.G + b.hc * p.GP + wave / p.RSH;
  const int row0 = b.blk_row0 + (wave % p.RSH) * 32;
  const bool wave_valid = row0 < R;

  // (the first tiles are requested ahead of Q and dO: one latency for both; with two slots the second V tile is requested by tile 0)
  TileLoader<D, NW> loader(p, b, wave, lane, smem, V_RING);
  constexpr int IPT = decltype(loader)::IPT;
  loader.request(0);
  if (NVST > 2 || !loader.v) loader.request(1);

  bf16x8 qf[2][KS], dof[2][KS];   // rows row0 + i16 and row0 + 16 + i16
  float lse2[2];
  f32x4 negd[2];                  // accumulator image of -D: this lane's query row in all four registers
  {
    // all loads of both halves before the first use of one (half by half, short walks took 1.2 us longer)
    const bool stats = STATS && p.make_stats();
    bf16x8 of[2][KS];
    float dvec[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t grow = b.row_begin + min(row0 + 16 * h + i16, R - 1);
      const u16* qp = p.q.ptr + grow * p.q.ts + (int64_t)head * p.q.hs + kgrp16<D>(lg) * 8;
      const u16* dop = p.dout.ptr + grow * p.dout.ts + (int64_t)head * p.dout.hs + kgrp16<D>(lg) * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        qf[h][ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 32);
        dof[h][ks] = *reinterpret_cast<const bf16x8*>(dop + ks * 32);
      }
      lse2[h] = p.lse[(int64_t)head * p.total + grow];
      if (stats) {
        const u16* op = p.o.ptr + grow * p.o.ts + (int64_t)head * p.o.hs + kgrp16<D>(lg) * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) of[h][ks] = *reinterpret_cast<const bf16x8*>(op + ks * 32);
      } else {
        dvec[h] = p.dvec[(int64_t)head * p.total + grow];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      lse2[h] *= LOG2E;
      if (stats) {
        float t[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) t[ks] = dot8_bf16(dof[h][ks], of[h][ks]);   // chunk 4 ks + kgrp16(lg)
        dvec[h] = butterfly_sum(t);
        dvec[h] += __shfl_xor(dvec[h], D == 96 ? 48 : 16);   // the chunk two further, then the next one (kgrp16)
        dvec[h] = xor32_sum(dvec[h]);
      }
      negd[h] = f32x4{-dvec[h], -dvec[h], -dvec[h], -dvec[h]};
      // consumed (and therefore waited for) here: no compiler-placed vector-memory wait inside the main loop
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : : "v"(qf[h][ks]), "v"(dof[h][ks]));
      asm volatile("" : : "v"(lse2[h]), "v"(dvec[h]));
    }
  }

  f32x4 dqacc[2][DB];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int db = 0; db < DB; ++db) dqacc[h][db] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Per-lane LDS addresses in slot 0; the loop is unrolled over the slots, so that all others are immediate offsets.  At head dim 128,
  // where the registers are full, one address of each kind: k-steps and column blocks differ in bits that the swizzle flips and not in the rows.
  constexpr bool ONE = D == 128;
  const uint32_t smem_addr = (uint32_t)reinterpret_cast<uintptr_t>(smem);
  uint32_t kadr[ONE ? 1 : KS], vadr[ONE ? 1 : KS], tadr[ONE ? 1 : DB];
#pragma unroll
  for (int ks = 0; ks < (ONE ? 1 : KS); ++ks) {
    kadr[ks] = smem_addr + frag16_off<D>(lane, ks);
    vadr[ks] = kadr[ks] + V_RING;
  }
#pragma unroll
  for (int db = 0; db < (ONE ? 1 : DB); ++db) tadr[db] = smem_addr + tr16_off<D>(lane, db);
  auto k_at = [&](int ks) __attribute__((always_inline)) { return ONE ? kadr[0] ^ (ks * 64) : kadr[ONE ? 0 : ks]; };
  auto v_at = [&](int ks) __attribute__((always_inline)) { return ONE ? vadr[0] ^ (ks * 64) : vadr[ONE ? 0 : ks]; };
  auto t_at = [&](int db) __attribute__((always_inline)) { return ONE ? tadr[0] ^ (db * 32) : tadr[ONE ? 0 : db]; };

  const int n_ctx_run = b.n_ctx - b.c0;
  wait_vm<0>();
  if (NSTAGE == 4 && !loader.v) loader.request(2);
  __syncthreads();

  // tiles that can hold an invisible (row, key) pair for this wave; the others need no test per half
  const bool never_plain = LOCAL || !wave_valid;
  const int ctx_masked = (P % BN) && n_ctx_run > 0 ? n_ctx_run - 1 : -1;   // the partial last prompt tile
  const int dec_masked = n_ctx_run - b.d0 + min(row0 + 1, R) / BN;         // response tiles from the diagonal (or the sequence end) on

  // K operand i of a half tile: keys 16 (i / KS) .., k-step i % KS
  bf16x8 ko[2 * KS];
  auto load_k = [&](int at) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) ko[i] = lds_frag(k_at(i % KS) + at + i / KS * 16 * RB);
  };
  // One half tile (32 keys) at offset `at` of the K ring and `atv` of the V ring, whose K operands are in `ko`; requests those of the next half at `next`.
  // For each half h of the rows: S^T = K Q^T, dP^T - D = V dO^T - D (accumulator initialised to -D), dS^T = P (dP^T - D),
  // dQ^T += K^T dS^T.  The exponentials of h = 0 issue beside the score MFMAs of h = 1, those of h = 1 beside the dP MFMAs of
  // h = 0, and so on.  Two sets of operand registers: V is requested under the score MFMAs, K^T under the dP MFMAs (where K was),
  // the next half's K under the dQ MFMAs (where V was).
  auto half_tile = [&](bool masked, int at, int atv, int next, bool is_ctx, int key0) __attribute__((always_inline)) {
    f32x4 s[4], dp[4];   // tile 2 h + kh: keys 16 kh .. of rows 16 h ..
    float ev[16];        // score e = 8 h + 4 kh + r: key 16 kh + 4 lg + r
    bf16x8 vo[2 * KS], kt[DB], ds[2];
    uint32_t dw[8];
    static_assert(DB == 2 * KS, "");
    constexpr int NM = 2 * KS, EPM = (8 + NM - 1) / NM;   // MFMAs of a chain pair, most scores beside one of them
    auto exps = [&](int h, int i) __attribute__((always_inline)) {   // beside MFMA i
#pragma unroll
      for (int j = 0; j < EPM; ++j) {
        const int e = 8 * h + 8 * i / NM + j;
        if (e >= 8 * h + 8 * (i + 1) / NM) continue;
        ev[e] = __builtin_amdgcn_exp2f(s[e >> 2][e & 3] * c - lse2[h]);
        asm volatile("" : "+v"(ev[e]));
      }
    };
    auto products = [&](int h, int i) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < EPM; ++j) {
        const int e = 8 * h + 8 * i / NM + j;
        if (e >= 8 * h + 8 * (i + 1) / NM) continue;
        ev[e] *= dp[e >> 2][e & 3];
        if (e & 1) {
          dw[e >> 1] = pack2_bf16(ev[e - 1], ev[e]);
          asm volatile("" : "+v"(dw[e >> 1]));
        }
      }
    };
    auto mask = [&](int h) __attribute__((always_inline)) {
      if (__builtin_expect(masked, 0)) {
        const int l = opaque(lane), row = row0 + 16 * h + (l & 15), k0 = key0 + 4 * (l >> 4);   // (formed here: no registers in between)
        const int lim = (is_ctx ? P : min(row + 1, R)) - k0, lo = (is_ctx ? P : 0) + row - W - k0;
        // bit k of a word says whether this lane's key k is visible
        uint32_t bits = 0x0fffffu >> (20 - min(max(lim, 0), 20));
        if (LOCAL) bits &= ~0u << min(max(lo + 1, 0), 31);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = 16 * (e >> 2) + (e & 3);
          const uint32_t see = (uint32_t)((int32_t)(bits << (31 - k)) >> 31);
          ev[8 * h + e] = __builtin_bit_cast(float, see & __builtin_bit_cast(uint32_t, ev[8 * h + e]));
        }
      }
    };
    if (ONE) asm volatile("" : "+v"(kadr[0]), "+v"(vadr[0]), "+v"(tadr[0]));   // (what is formed from them is not kept in registers)
#pragma unroll
    for (int i = 0; i < NM; ++i) vo[i] = lds_frag(v_at(i % KS) + atv + i / KS * 16 * RB);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        s[2 * h + i / KS] = mfma16(ko[i], qf[h][i % KS], i % KS ? s[2 * h + i / KS] : f32x4{0.f, 0.f, 0.f, 0.f});
        if (h == 1) exps(0, i);
        __builtin_amdgcn_sched_barrier(0);
      }
    // the first half of K^T; the other half where V operands have been used
#pragma unroll
    for (int db = 0; db < DB / 2; ++db) kt[db] = lds_tr16<D>(t_at(db) + at);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      mask(h);
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        dp[2 * h + i / KS] = mfma16(vo[i], dof[h][i % KS], i % KS ? dp[2 * h + i / KS] : negd[h]);
        if (h == 0) {
          exps(1, i);
        } else {
          if (i % 2 == 0) kt[DB / 2 + i / 2] = lds_tr16<D>(t_at(DB / 2 + i / 2) + at);
          products(0, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    load_k(next);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      ds[h] = __builtin_bit_cast(bf16x8, u32x4{dw[4 * h], dw[4 * h + 1], dw[4 * h + 2], dw[4 * h + 3]});
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        dqacc[h][db] = mfma16(kt[db], ds[h], dqacc[h][db]);
        if (h == 0 && db < NM) products(1, db);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  int it = 0;
  load_k(0);
  // tile `it` in slot U; false: it was the last one
  auto tile = [&](auto Uc) __attribute__((always_inline)) -> bool {
    constexpr int N = decltype(Uc)::value, U = N % NSTAGE, UN = (U + 1) % NSTAGE, UV = N % NVST;
    // the K tile requested goes into the slot that tile it-1 left at the last barrier, the V tile (two ahead, or one) into its or an older one
    const bool issued = loader.request(NVST == 2 && loader.v ? (UV + 1) % 2 : NSTAGE == 4 && loader.v ? (U + 2) % NSTAGE : (U + NSTAGE - 1) % NSTAGE);
    const bool plain = !(never_plain || it == ctx_masked || it >= dec_masked);
    const bool is_ctx = it < n_ctx_run;
    const int key0 = (is_ctx ? b.c0 + it : b.d0 + it - n_ctx_run) * BN;
    static_for<2>([&](auto Hc) __attribute__((always_inline)) {
      constexpr int H = decltype(Hc)::value, at = U * T + H * HT, atv = UV * T + H * HT, next = H ? UN * T : U * T + HT;
      const int k0 = key0 + H * 32;
      const bool active = plain || (wave_valid && tile_active<LOCAL, 32>(is_ctx, k0, row0, row0 + 31, P, W) && k0 < (is_ctx ? P : R));
      if (__builtin_expect(active, 1)) half_tile(!plain && tile_needs_mask<LOCAL, 32>(is_ctx, k0, row0, P, R, W), at, atv, next, is_ctx, k0);
      else load_k(next);
    });
    // the next tile's V and the K tile after it must have landed
    if (__builtin_expect(issued && NVST > 2 && (NSTAGE == 4 || loader.v), 1)) wait_vm<IPT>();
    else wait_vm<0>();
    __syncthreads();
    return ++it < b.n_tiles;
  };
  while (true) {
    if (!tile(std::integral_constant<int, 0>{})) break;
    if (!tile(std::integral_constant<int, 1>{})) break;
    if (!tile(std::integral_constant<int, 2>{})) break;
    if constexpr (NSTAGE > 3 || NVST == 2)
      if (!tile(std::integral_constant<int, 3>{})) break;
    if constexpr (NVST == 2) {
      if (!tile(std::integral_constant<int, 4>{})) break;
      if (!tile(std::integral_constant<int, 5>{})) break;
    }
  }

  // ---- epilogue: lane owns a query row of each half, register r the head-dim column 4 lg + r of a 16-column block.  Stored from
  // here a row would leave in 8-byte pieces, 16 rows per instruction.  The wave's scaled 32 x D tile goes through LDS
  // instead (all stages are free after the last barrier; 16-byte chunks XOR-swizzled by the row) and is read back as
  // whole rows.  Wave-private: no barrier.
  if (STATS && p.make_stats() && lg == 0) {   // (stored here: the waits of the main loop count loads only)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = row0 + 16 * h + i16;
      if (row >= R) continue;
      p.dvec[(int64_t)head * p.total + b.row_begin + row] = -negd[h][0];
      p.lse2[(int64_t)head * p.total + b.row_begin + row] = lse2[h];
    }
  }
  unsigned char* ot = smem + wave * 32 * RB;
  auto oswz = [](int r) { return D == 96 ? swz<96>(r) : r & (CPR - 1); };
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const int tr = 16 * h + i16;
      u32x2 w;
      w.x = pack2_bf16(dqacc[h][db][0] * p.scale, dqacc[h][db][1] * p.scale);
      w.y = pack2_bf16(dqacc[h][db][2] * p.scale, dqacc[h][db][3] * p.scale);
      *reinterpret_cast<u32x2*>(ot + tr * RB + (((db * 2 + (lg >> 1)) ^ oswz(tr)) << 4) + (lg & 1) * 8) = w;
    }
#pragma unroll
  for (int i = 0; i < CPR / 2; ++i) {   // 64 of the tile's 32 CPR chunks per store instruction
    const int tr = (i * 64 + lane) / CPR, chunk = (i * 64 + lane) % CPR;
    const u32x4 w = *reinterpret_cast<const u32x4*>(ot + tr * RB + ((chunk ^ oswz(tr)) << 4));
    if (row0 + tr < R) {
      u16* op = p.dq.ptr + (int64_t)(b.row_begin + row0 + tr) * p.dq.ts + (int64_t)head * p.dq.hs;
      *reinterpret_cast<u32x4*>(op + chunk * 8) = w;
    }
  }
}

template <int D, int NW>
constexpr size_t kDq2Smem = (kDq2Stages<D, NW> + kDq2VStages<D, NW>) * 64 * 2 * D;

}  // namespace dkv
