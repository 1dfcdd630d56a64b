// Forward kernel for head dims 64, 96 and 128 (Alg. 3 of the paper re-tiled for CDNA4), tuned variant.
//
// One workgroup owns BMR response rows x GP packed query heads of one KV head ("GQA packing": the staged K / V tiles
// are shared by all packed heads) and walks the two KV regions in logical order, prompt tiles then own-response tiles.
// The scores are computed transposed, S^T = K Q^T, so that a lane owns one query row and exp(S^T) is already laid out
// as the B operand of O^T += V^T P^T:
//   * 4 waves, two workgroups a CU (three at head dim 64), or 8, two per SIMD, by the rule of row_block_waves (rules.h); each owns
//     32 query rows, two halves of 16: Q fragments (B operands) and the O^T accumulator stay in registers;
//   * the 16x16x32 MFMA, each K or V operand read from LDS feeding the two halves.  These kernels run into the card's power
//     limit, not into its matrix rate: with all inputs zero the 32x32x16 form of this kernel took 16.0 ms for 16 x U(1024, 2048)
//     behind 32768, 32 / 4 heads, d = 128, and 20.5 with normal ones.  On normal values a bare loop of 16x16x32 MFMAs reaches
//     2040 TFLOP/s, one of 32x32x16 1775 (2460 both on zeros), and a loop with this kernel's operand reads and softmax
//     1466 against 1344;
//   * K and V tiles (64 keys) are staged row-major, un-padded, XOR-swizzled by row (tiles.h) so that both the 16-byte K
//     operand reads and the transposing V reads are bank-conflict free; V^T operands come from ds_read_b64_tr_b16
//     (LDS transpose read), so nothing is transposed on the way into LDS;
//   * the tiles travel global -> LDS directly (global_load_lds) into two rings, K requested by the first half of the waves and V by
//     the second: no staging registers, no LDS stores, one barrier per tile; the loop is unrolled over the slots, so that every
//     operand address is a register plus an immediate.  Eight waves have four slots each, K three tiles ahead and V two.  Four have three
//     for K, two tiles ahead, and two for V, one ahead, at d = 128 exactly half of a CU's LDS: there the second half of V tile i-1
//     is still read beside the first half of tile i, so that halves of tiles are requested, V from the middle of one tile to
//     the middle of the next.  With the start and end of one workgroup beside the tiles of the other and half the rows in the last
//     round: 32 x U(17, 256) behind 517, 32 / 8 heads 97 -> 73 us, 4 x U(789, 1163) behind 5059 403 -> 331 (eight waves -> four, d = 128);
//   * each wave runs a software pipeline over 32-key half tiles: while the VALU does the softmax of half g, the matrix pipe
//     computes the scores of half g+1 and the P V product of half g-1.  Two waves per SIMD do not hide a wave's own MFMA ->
//     softmax -> MFMA dependency chain on this chip (their phases drift together at every barrier); interleaving
//     independent work inside one instruction stream does;
//   * no row maximum per half tile: the reference of the exponentials moves when a sum of probabilities says so.
// Measured against the same kernel on 32x32x16 MFMAs with a row maximum and addresses formed per tile: 16 x 1024 rows behind 8192,
// 32 / 8 heads, d = 128 2.05 -> 1.84 ms (1271 TFLOP/s); 8 x U(131, 2048) (9112 rows) behind 4096, d = 64 440 -> 404 us, d = 96 (16 / 4 heads)
// 359 -> 303 us.
#include <type_traits>
#include "common.h"
#include "dma.h"
#include "launch.h"
#include "qsched.h"
#include "tiles.h"

namespace dkv {

template <int D, int NWAVES, bool PAIR>
struct F2Cfg {
  static constexpr int NW = NWAVES, NT = NW * 64, BN = 64;
  static constexpr int KS = D / 32, DB = D / 16;   // k-steps of a score, 16-wide head-dim blocks
  static constexpr int RB = 2 * D;                 // row bytes
  static constexpr int CPR = D / 8;                // 16-byte chunks per row
  static constexpr int TILE_BYTES = BN * RB;
  static constexpr bool HALVES = PAIR;             // halves of tiles are requested
  static constexpr int NK = HALVES ? 3 : 4, NV = HALVES ? 2 : 4;
};

template <int D, int NW, bool PAIR, bool LOCAL>
__global__ __launch_bounds__(NW * 64, PAIR && D == 64 ? 3 : 2) void fwd2_kernel(const AttnParams p) {
  using C = F2Cfg<D, NW, PAIR>;
  constexpr int BN = C::BN;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // K ring | V ring
  QBlock b;
  if (!decode_qblock<BN>(p, b, blockIdx.x, gridDim.x)) return;
  make_uniform(b);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, lg = lane >> 4;
  const int P = b.P, R = b.R, W = p.window;
  const float c = p.scale_log2;

  const int head = b.hk * p.G + b.hc * p.GP + wave / p.RSH;
  const int row0 = b.blk_row0 + (wave % p.RSH) * 32;
  const bool wave_valid = row0 < R;

  constexpr int NK = C::NK, NV = C::NV;               // ring slots: K ring, then V ring
  constexpr int V_RING = NK * C::TILE_BYTES;

  bf16x8 qf[2][C::KS];   // rows row0 + i16 and row0 + 16 + i16
  {
    const u16* qp = p.q.ptr + (int64_t)b.row_begin * p.q.ts + (int64_t)head * p.q.hs + kgrp16<D>(lg) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks)
        qf[h][ks] = *reinterpret_cast<const bf16x8*>(qp + (int64_t)min(row0 + 16 * h + i16, R - 1) * p.q.ts + ks * 32);
  }
  // (the first tiles are requested under the loads of Q, which leave first: behind 16 to 32 KB of tiles they are late)
  __builtin_amdgcn_sched_barrier(0);
  TileLoader<D, NW, C::HALVES ? 32 : 64> loader(p, b, wave, lane, smem, V_RING);
  loader.request(0);
  if (!C::HALVES || !loader.v) loader.request(1);
  if (C::HALVES && !loader.v) {   // two whole K tiles, half a V tile
    loader.request(2);
    loader.request(3);
  }
  // consumed (and therefore waited for) here: no compiler-placed vector-memory wait inside the main loop
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) asm volatile("" : : "v"(qf[h][ks]));

  f32x4 oacc[2][C::DB];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int db = 0; db < C::DB; ++db) oacc[h][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref[2] = {NEG_BIG, NEG_BIG}, l_sum[2] = {0.f, 0.f};

  // ---- per-lane LDS addresses in slot 0.  The loop is unrolled over the slots, so that all others are immediate offsets.
  const unsigned char* kadr[C::KS];   // K operand of k-step ks
#pragma unroll
  for (int ks = 0; ks < C::KS; ++ks) kadr[ks] = smem + frag16_off<D>(lane, ks);
  const unsigned char* vadr[C::DB];   // V^T operand of head-dim block db
#pragma unroll
  for (int db = 0; db < C::DB; ++db) vadr[db] = smem + V_RING + tr16_off<D>(lane, db);

  const int n_ctx_run = b.n_ctx - b.c0;

  // ---- the three pieces of work of a 32-key half tile
  // S^T half = K_half Q^T: tile 2 h + kh holds keys 16 kh .. 16 kh + 15 of rows 16 h .. 16 h + 15
  auto s_half = [&](int kh0, f32x4 (&s)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kadr[ks] + kh0 + kh * 16 * C::RB);
#pragma unroll
        for (int h = 0; h < 2; ++h) s[2 * h + kh] = mfma16(a, qf[h][ks], s[2 * h + kh]);
      }
  };
  // O^T += V_half^T P_half^T
  auto pv_half = [&](int v0, const bf16x8 (&pp)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int db = 0; db < C::DB; ++db) {
      const bf16x8 a = tr16_pair<D>(vadr[db] + v0);
#pragma unroll
      for (int h = 0; h < 2; ++h) oacc[h][db] = mfma16(a, pp[h], oacc[h][db]);
    }
  };
  // One step of the software pipeline: the softmax of half tile g (scores in `sc`) runs on the VALU while the
  // matrix pipe computes the scores of half g+1 (into `sn`) and accumulates the P V product of half g-1
  // (`pprev`); the three are independent.  A SIMD issues one VALU-class instruction (MFMA included) per ~5 cycles over all its
  // waves.  The step consists of NSLOT slots of {two MFMAs that share an operand from LDS, the softmax of 16 / NSLOT scores}
  // in groups of four.  All operand reads of a group are requested at the start of the previous group, and a group's MFMAs consume their operands
  // in the reverse of the request order, so one wait per group covers them all; the softmax of a score is spread over three slots so that no instruction of a
  // slot depends on another one of the same slot.  Fences keep the compiler from regrouping.  The operands of the first
  // group are requested by the previous step (`pre`), those of the next step's first group here.
  constexpr int NS = 2 * C::KS, NPV = C::DB, NSLOT = NS + NPV, LEAD = 4, NG = NSLOT / LEAD;
  constexpr int EPS = (16 + NSLOT - 1) / NSLOT;   // most scores per slot
  static_assert(NS == NPV && NSLOT <= 16 && NSLOT % LEAD == 0, "slot layout");
  // the sixteen scores of a lane are spread evenly over the slots: slot i finishes scores [sc0(i), sc0(i + 1))
  auto sc0 = [](int i) constexpr { return i < NSLOT ? 16 * i / NSLOT : 16; };
  // slot i < NS: scores of key half i % 2, k-step i / 2; slot NS + j: products of head-dim block j
  // (k0, v0: the half tile's offset in the ring)
  auto operand = [&](int k0, int v0, int i) __attribute__((always_inline)) {
    if (i < NS) return *reinterpret_cast<const bf16x8*>(kadr[i >> 1] + k0 + (i & 1) * 16 * C::RB);
    return tr16_pair<D>(vadr[i - NS] + v0);
  };
  // score e = 8 h + 4 kh + r of a lane: row 16 h + i16, key 16 kh + 4 lg + r
  auto mask = [&](f32x4 (&sc)[4], int it, int half) __attribute__((always_inline)) {
    const bool is_ctx = it < n_ctx_run;
    const int keyh0 = (is_ctx ? b.c0 + it : b.d0 + it - n_ctx_run) * BN + half * 32;
    // visible keys of a row: lo < key < lim (indices inside the region)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = row0 + 16 * h + i16;
      int lim, lo = -1;
      if (is_ctx) {
        lim = P;
        if (LOCAL) lo = P + row - W;
      } else {
        lim = min(row + 1, R);
        if (LOCAL) lo = row - W;
      }
      lim -= keyh0 + 4 * lg;
      if (!LOCAL) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = 16 * (e >> 2) + (e & 3);
          sc[2 * h + (e >> 2)][e & 3] = k < lim ? sc[2 * h + (e >> 2)][e & 3] : -INFINITY;
        }
        continue;
      }
      // both bounds: bit k of a word says whether this lane's key k is visible (two instructions a score instead of four: 1024 rows,
      // window 256, 32 / 8 heads, d = 128 14.6 -> 13.3 us; 8 x U(300, 900) behind 2000, window 512, 16 / 4 heads, d = 96 50.5 -> 46.0)
      lo -= keyh0 + 4 * lg;
      const uint32_t bits = (~0u << min(max(lo + 1, 0), 31)) & (0x0fffffu >> (20 - min(max(lim, 0), 20)));
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = 16 * (e >> 2) + (e & 3);
        const float x = sc[2 * h + (e >> 2)][e & 3];   // (the bits of a vector's element are taken from a copy)
        const uint32_t see = (uint32_t)((int32_t)(bits << (31 - k)) >> 31);
        sc[2 * h + (e >> 2)][e & 3] = __builtin_bit_cast(float, (see & __builtin_bit_cast(uint32_t, x)) | (~see & 0xff800000u));
      }
    }
  };
  // the maximum of half h's scores over the four lanes that hold a row
  auto row_max = [&](const f32x4 (&sc)[4], int h) __attribute__((always_inline)) {
    float mx = sc[2 * h][0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sc[2 * h + (e >> 2)][e & 3]);
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    return xor32_max(mx);
  };
  auto step = [&](bool masked, f32x4 (&sc)[4], f32x4 (&sn)[4], bf16x8 (&pprev)[2], bf16x8 (&pcur)[2], bf16x8 (&pre)[LEAD],
                  int Kn, int Vp, int Kn2, int Vn2, int it, int half) __attribute__((always_inline)) {
    if (LOCAL ? masked : __builtin_expect(masked, 0)) mask(sc, it, half);
    auto score = [&](int e) __attribute__((always_inline)) { return sc[e >> 2][e & 3]; };
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 ob[NSLOT];
#pragma unroll
    for (int i = 0; i < LEAD; ++i) ob[i] = pre[i];
    uint32_t pw[8];
    float tv[16], ev[16];
    float ls[2] = {0.f, 0.f};
#pragma unroll
    for (int e = 0; e < sc0(2); ++e) tv[e] = score(e) * c - m_ref[e >> 3];
#pragma unroll
    for (int e = 0; e < sc0(1); ++e) ev[e] = __builtin_amdgcn_exp2f(tv[e]);
    bool first_s[2] = {true, true};
#pragma unroll
    for (int g = 0; g < NG; ++g) {
#pragma unroll
      for (int q = 0; q < LEAD; ++q) {
        const int i = g * LEAD + (LEAD - 1 - q);   // reverse of the request order
        auto mm = [&](int h) __attribute__((always_inline)) {
          if (i >= NS) oacc[h][i - NS] = mfma16(ob[i], pprev[h], oacc[h][i - NS]);
          else sn[2 * h + (i & 1)] = mfma16(ob[i], qf[h][i >> 1], first_s[i & 1] ? f32x4{0.f, 0.f, 0.f, 0.f} : sn[2 * h + (i & 1)]);
        };
        const int n = g * LEAD + q;
        mm(0);
        if (q == 0) {
          // request the next group's operands (the next step's first group at the end)
#pragma unroll
          for (int n = 0; n < LEAD; ++n) {
            const int i2 = (g + 1) * LEAD + n;
            if (i2 < NSLOT) ob[i2] = operand(Kn, Vp, i2);
            else pre[n] = operand(Kn2, Vn2, n);
          }
        }
#pragma unroll
        for (int j = 0; j < EPS; ++j) {
          const int e2 = sc0(n + 2) + j, e1 = sc0(n + 1) + j;
          if (e1 < sc0(n + 2)) {
            ev[e1] = __builtin_amdgcn_exp2f(tv[e1]);
            asm volatile("" : "+v"(ev[e1]));   // (keeps this slot's softmax work inside the slot)
          }
          if (e2 < sc0(n + 3)) {
            tv[e2] = score(e2) * c - m_ref[e2 >> 3];
            asm volatile("" : "+v"(tv[e2]));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        mm(1);
        if (i < NS) first_s[i & 1] = false;
#pragma unroll
        for (int j = 0; j < EPS; ++j) {
          const int e = sc0(n) + j;
          if (e >= sc0(n + 1)) continue;
          ls[e >> 3] += ev[e];
          if (e & 1) {
            pw[e >> 1] = pack2_bf16(ev[e - 1], ev[e]);
            asm volatile("" : "+v"(pw[e >> 1]), "+v"(ls[e >> 3]));
          } else {
            asm volatile("" : "+v"(ls[e >> 3]));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // The reference of a row's exponentials moves lazily: it is kept until the probabilities of a half tile in some lane sum up
    // to more than 2^8 (or to infinity).  They are then formed again from the scores, against the row's new maximum.  The products of
    // the half before are complete and rescaled with the rest.
    if (__builtin_expect(__any(!(fmaxf(ls[0], ls[1]) < 256.0f)), 0)) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float mn = fmaxf(m_ref[h], row_max(sc, h) * c);
        const float alpha = __builtin_amdgcn_exp2f(m_ref[h] - mn);
        m_ref[h] = mn;
        l_sum[h] *= alpha;
#pragma unroll
        for (int db = 0; db < C::DB; ++db) oacc[h][db] *= alpha;
        ls[h] = 0.f;
#pragma unroll
        for (int e = 8 * h; e < 8 * h + 8; e += 2) {
          const float e0 = __builtin_amdgcn_exp2f(score(e) * c - mn), e1 = __builtin_amdgcn_exp2f(score(e + 1) * c - mn);
          ls[h] += e0 + e1;
          pw[e >> 1] = pack2_bf16(e0, e1);
        }
      }
    }
    asm volatile("" : "+v"(m_ref[0]), "+v"(m_ref[1]));
    l_sum[0] += ls[0];
    l_sum[1] += ls[1];
    u32x4 w0 = {pw[0], pw[1], pw[2], pw[3]}, w1 = {pw[4], pw[5], pw[6], pw[7]};
    pcur[0] = __builtin_bit_cast(bf16x8, w0);
    pcur[1] = __builtin_bit_cast(bf16x8, w1);
  };

  // ---- prologue: K0 V0 K1 V1 (four waves: the first half of V0) landed and published, scores of the first half, K2 requested.  The
  // first step multiplies P = 0 with the second half of the last V slot: whatever is there has to be finite.
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < 32 * C::CPR; i += C::NT)
    if (32 * C::CPR % C::NT == 0 || i + tid < 32 * C::CPR)
      *reinterpret_cast<u32x4*>(smem + V_RING + (NV - 1) * C::TILE_BYTES + 32 * C::RB + (i + tid) * 16) = zero4;
  wait_vm<0>();
  __syncthreads();

  // tiles that can hold an invisible (row, key) pair for this wave: the partial last prompt tile, response tiles from the diagonal
  // (or the end of the sequence) on; windowed runs mask every tile
  const bool always_masked = LOCAL || !wave_valid;
  const int ctx_masked = (P % BN) && n_ctx_run > 0 ? n_ctx_run - 1 : -1;
  const int dec_masked = n_ctx_run - b.d0 + min(row0 + 1, R) / BN;
  f32x4 sA[4], sB[4];
  bf16x8 pA[2], pB[2];
  pB[0] = __builtin_bit_cast(bf16x8, zero4);
  pB[1] = __builtin_bit_cast(bf16x8, zero4);
  constexpr int T = C::TILE_BYTES, HT = 32 * C::RB;
  s_half(0, sA);
  // The first reference is the maximum of the first half tile.  Left at its start value, every wave would form its first sixteen
  // probabilities twice, the second time out of line: 4 x 128 rows behind 256, 4 / 2 heads, d = 64 9.05 -> 8.73 us.
  if (always_masked || ctx_masked == 0 || dec_masked <= 0) mask(sA, 0, 0);
#pragma unroll
  for (int h = 0; h < 2; ++h) m_ref[h] = fmaxf(m_ref[h], row_max(sA, h) * c);
  bf16x8 pre[LEAD];   // operands of the first four slots of step (tile 0, half 0): K half 1 of tile 0
#pragma unroll
  for (int i = 0; i < LEAD; ++i) pre[i] = operand(HT, (NV - 1) * T + HT, i);
  if (!C::HALVES && !loader.v) loader.request(2);

  int it = 0;
  // tile `it` in slot U; false: it was the last one
  auto tile = [&](auto Uc) __attribute__((always_inline)) -> bool {
    constexpr int N = decltype(Uc)::value, U = N % NK, UN = (N + 1) % NK, V = N % NV, VP = (N + NV - 1) % NV;
    // K tile it+3 replaces K tile it-1, V tile it+2 replaces V tile it-2 (four waves: K tile it+2 replaces K tile it-1, the second half of
    // V tile it that of V tile it-2 and the first half of V tile it+1 that of V tile it-1): all were last read before the barrier that
    // ended tile it-1
    bool issued = false;
    if constexpr (C::HALVES) {
      loader.request(loader.v ? 2 * V + 1 : 2 * ((N + 2) % NK));
      loader.request(loader.v ? 2 * VP : 2 * ((N + 2) % NK) + 1);
    } else {
      issued = loader.request(loader.v ? (N + 2) % NV : (N + NK - 1) % NK);
    }
    const bool masked = always_masked || it == ctx_masked || it >= dec_masked;
    step(masked && it > 0, sA, sB, pB, pA, pre, U * T + HT, VP * T + HT, UN * T, V * T, it, 0);
    step(masked, sB, sA, pA, pB, pre, UN * T, V * T, UN * T + HT, V * T + HT, it, 1);
    // tiles it+2 (K) and it+1 (V; four waves: its first half) must have landed; the loads that eight waves requested at the top of this
    // tile may stay in flight
    if (__builtin_expect(issued, 1)) wait_vm<decltype(loader)::IPT>();
    else wait_vm<0>();
    __syncthreads();
    return ++it < b.n_tiles;
  };
  while (true) {
    if (!tile(std::integral_constant<int, 0>{})) break;
    if (!tile(std::integral_constant<int, 1>{})) break;
    if (!tile(std::integral_constant<int, 2>{})) break;
    if (!tile(std::integral_constant<int, 3>{})) break;
    if constexpr (C::HALVES) {
      if (!tile(std::integral_constant<int, 4>{})) break;
      if (!tile(std::integral_constant<int, 5>{})) break;
    }
  }
  // the product of the last half tile
  pv_half(((b.n_tiles - 1) & (NV - 1)) * T + HT, pB);

  // ---- epilogue: lane owns a query row of each half, register r the head-dim column 4 lg + r of a 16-column block.  Stored from
  // here a row would leave in 8-byte pieces, 16 rows per instruction.  The wave's normalised 32 x D tile goes through
  // LDS instead: its own 32 rows of the K ring (free since the last barrier: only V is read after it; 16-byte chunks
  // XOR-swizzled by the row), read back as whole rows.  Wave-private: no barrier.
  unsigned char* ot = smem + wave * 32 * C::RB;
  auto oswz = [](int r) { return D == 96 ? swz<96>(r) : r & (C::CPR - 1); };
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float l = l_sum[h];
    l += __shfl_xor(l, 16);
    l = xor32_sum(l);
    const float inv = 1.0f / l;
    const int tr = 16 * h + i16, row = row0 + tr;
#pragma unroll
    for (int db = 0; db < C::DB; ++db) {
      u32x2 w;
      w.x = pack2_bf16(oacc[h][db][0] * inv, oacc[h][db][1] * inv);
      w.y = pack2_bf16(oacc[h][db][2] * inv, oacc[h][db][3] * inv);
      *reinterpret_cast<u32x2*>(ot + tr * C::RB + (((db * 2 + (lg >> 1)) ^ oswz(tr)) << 4) + (lg & 1) * 8) = w;
    }
    if (lg == 0 && row < R) p.lse[(int64_t)head * p.total + b.row_begin + row] = (m_ref[h] + log2f(l)) * LN2;
  }
#pragma unroll
  for (int i = 0; i < C::CPR / 2; ++i) {   // 64 of the tile's 32 CPR chunks per store instruction
    const int tr = (i * 64 + lane) / C::CPR, chunk = (i * 64 + lane) % C::CPR;
    const u32x4 w = *reinterpret_cast<const u32x4*>(ot + tr * C::RB + ((chunk ^ oswz(tr)) << 4));
    if (row0 + tr < R) {
      u16* op = p.out_o.ptr + (int64_t)(b.row_begin + row0 + tr) * p.out_o.ts + (int64_t)head * p.out_o.hs;
      *reinterpret_cast<u32x4*>(op + chunk * 8) = w;
    }
  }
}

template <int D, int NW, bool PAIR, bool LOCAL>
static hipError_t launch_fwd2_t(AttnParams p, hipStream_t st) {
  using C = F2Cfg<D, NW, PAIR>;
  fill_packing(p, NW);
  const size_t smem = (C::NK + C::NV) * C::TILE_BYTES;
  auto kern = fwd2_kernel<D, NW, PAIR, LOCAL>;
  hipError_t e = ensure_dynamic_lds<fwd2_kernel<D, NW, PAIR, LOCAL>>(smem);
  if (e != hipSuccess) return e;
  return launch_sequences(p, (int64_t)p.MB * p.HC * p.Hk, C::NT, [&](const AttnParams& q, unsigned n) {
    hipLaunchKernelGGL(kern, dim3(n), dim3(C::NT), smem, st, q);
    return hipGetLastError();
  });
}

template <int D>
static hipError_t launch_fwd2_d(const AttnParams& p, hipStream_t st) {
  const bool local = p.window > 0;
  const rules::Waves w = choose_waves(p, D, false);
  if constexpr (D != 64)   // (which takes four always)
    if (w.n == 8) return local ? launch_fwd2_t<D, 8, false, true>(p, st) : launch_fwd2_t<D, 8, false, false>(p, st);
  if (!w.pair) return local ? launch_fwd2_t<D, 4, false, true>(p, st) : launch_fwd2_t<D, 4, false, false>(p, st);
  return local ? launch_fwd2_t<D, 4, true, true>(p, st) : launch_fwd2_t<D, 4, true, false>(p, st);
}

hipError_t launch_fwd2(const AttnParams& p, int head_dim, hipStream_t st) {
  switch (head_dim) {
    case 64:  return launch_fwd2_d<64>(p, st);
    case 96:  return launch_fwd2_d<96>(p, st);
    case 128: return launch_fwd2_d<128>(p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace dkv
