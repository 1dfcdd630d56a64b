// dK / dV of Call 2 at head dims 96 and 128, prompt gradients added to fp32 sums, where the prompt tiles fill the chip: a wave does all
// the work of its keys.
//
// One workgroup of four waves owns a 128-key tile of one KV head (ownership, parts and gradients as in dkdv4.hip), each wave 32 keys: it
// keeps K and -V operands and the fp32 dK, dV of its keys in registers and forms S, D - dP, P, -dS, dV += P^T dO and -dK += (-dS)^T Q
// itself.  P and -dS never pass through LDS, where dkdv4's roles hand them over at a barrier that ties the waves of a SIMD together: it holds
// Q, dO, the row statistics and at head dim 128 a part of -V.  Two workgroups share a CU (256 registers a wave, at most 80 KB of LDS each), so that one wave's softmax and waits
// are beside the other's MFMAs.  16x16x32 MFMAs, as in the forward kernel: more work in the card's power.
//   * A row block of 32 rows is two halves h of 16: S(0) | D - dP(0), exponentials of 0 | S(1), -dS of 0 | D - dP(1), exponentials
//     of 1 | dV, -dS of 1 | dK.  P and -dS of both halves are the 32-deep operand of dV and dK without leaving registers (common.h).
//   * An operand from LDS is requested into the registers of the one that has just been used, four (three) operands ahead: the
//     register file is full.  At head dim 128 the -V operands of the last two k-steps do not fit: LDS, read back for every half.
//   * Three stages of row blocks (global -> LDS loads, dma.h), one barrier a block; every wave walks the schedule by itself and
//     requests a quarter of a block two blocks ahead.  The loop is not unrolled and has no branch but for masks and the end of a
//     sequence: with more, the register allocator moves accumulators about (or spills) at every one.
//
// What bounds it: power.  At 16 x 1024 rows behind 8192, 32 / 8 heads, d = 128 the matrix pipes are busy for 59 % of the
// 2.03 GHz that are left of 2.4; issue slots 46 %, LDS 22 %, no bank conflict.  There dkdv4 takes 4.12 ms, this kernel 3.70
// (1262 TFLOP/s); 5 x U(85, 416) behind 25804, 4 / 2 heads 172 -> 148 us; d = 96, 8 x U(131, 2048) behind 4111, 16 / 4 heads 699 -> 590 us,
// 5 x U(22, 31) behind 11889, 32 / 8 heads 136 -> 108 us.  A workgroup alone on its CU takes 1.27 times as long as one of dkdv4 (one
// wave a SIMD has nothing to hide its latencies with): calls that do not fill the chip stay there, and Call 1, whose tiles are of
// falling length (d = 128 1.00 -> 1.22 ms).  Head dim 64 (three workgroups a CU): 1.21 -> 1.21 ms, stays there too.
// Also measured: 64 keys a wave in 512 registers, one wave a SIMD (half the LDS reads, but nothing runs beside the softmax): 4.9 ms;
// wave priorities by phase, the next block's first operands read ahead of the barrier: within 1 %.
#include <climits>
#include <type_traits>
#include "common.h"
#include "dma.h"
#include "kvsched.h"
#include "kvstore.h"
#include "launch.h"
#include "tiles.h"

namespace dkv {

constexpr int kPairStages = 3;   // row blocks in LDS: one being computed, two requested ahead

template <int V>
using IC = std::integral_constant<int, V>;

template <int D>
__global__ __launch_bounds__(256, 2) void dkdvw_kernel(const AttnParams p, int n_blocks) {
  constexpr int NKT = 2, KEYS = 16 * NKT, BN = 4 * KEYS, HB = 32;   // keys per wave and workgroup, query rows per block
  constexpr int KS = D / 32, DB = D / 16, RB = 2 * D, CPR = D / 8;
  constexpr int HT = HB * RB;                      // one Q or dO row block
  constexpr int NBUF = kPairStages, AHEAD = NBUF - 1;
  constexpr int DO_RING = NBUF * HT, STAT = 2 * NBUF * HT;   // Q ring | dO ring | NBUF x (LSE*log2e[32] | D[32])
  constexpr int V_LDS = STAT + NBUF * 256;         // head dim 128: the waves' -V operands of the last two k-steps
  constexpr int VR = D == 128 ? KS - 2 : KS;       // k-steps whose -V operands are in registers
  constexpr bool SPLIT = kSplitRow<D>;             // head dim 96: waves 0 and 1 request Q, 2 and 3 dO
  constexpr int IPB = 2 * HT / 1024 / 4;           // load instructions per wave and row block
  constexpr int RPI = 1024 / RB;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];   // (addresses are formed by XOR)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, lg = lane >> 4;

  KVBlock kb;
  if (!decode_kvblock(p, BN, HB, kb, blockIdx.x, n_blocks)) return;
  const bool is_ctx = kb.is_ctx;
  const int hk = kb.hk, key0 = kb.key0, seq_lo = kb.seq_lo, seq_hi = kb.seq_hi, P = kb.P;
  int region_len, key_row_begin;
  if (is_ctx) {
    region_len = P;
    key_row_begin = kb.ctx_off;
  } else {
    key_row_begin = p.cu ? p.cu[seq_lo] : 0;
    region_len = p.cu ? (p.cu[seq_lo + 1] - key_row_begin) : p.total;
  }
  const int wkey0 = key0 + wave * KEYS;            // this wave's first key
  const float c = p.scale_log2;

  // ---- row-block schedule and requests
  const uint32_t smem_addr = (uint32_t)own_sgpr((int)(uint32_t)reinterpret_cast<uintptr_t>(smem));
  const int q_tsb = own_sgpr((int)p.q.ts * 2), do_tsb = own_sgpr((int)p.dout.ts * 2);   // bytes per token
  const uint32_t ld_lds = smem_addr + (SPLIT ? (wave >> 1) * DO_RING + (wave & 1) * 16 * RB : wave * 1024);
  const int64_t stat_gap = (const char*)p.lse2 - (const char*)p.dvec;   // lanes 0-31 fetch LSE*log2e, lanes 32-63 D
  RowWalk<HB, true> walk(p, hk, seq_hi);
  uint32_t flags = 0;
  auto ld_row = [&](int t) __attribute__((always_inline)) { return SPLIT ? (wave & 1) * 16 + split_row<D>(t, lane) : wave * RPI + lane / CPR; };
  auto ld_col = [&](int t) __attribute__((always_inline)) {
    return ((SPLIT ? split_pos<D>(t, lane) : lane % CPR) ^ swz16<D>(ld_row(t))) * 16;
  };
  int row_step = walk.DIR, live = HDR_VALID | HDR_MASK;   // 0 past the end
  auto new_rows = [&]() __attribute__((always_inline)) {
    flags = live & (HDR_VALID | (walk.nvalid < HB || (!is_ctx && walk.row0 < wkey0 + KEYS - 1) ? HDR_MASK : 0));
  };
  const int rows_lo = kb.rb_lo * HB, rows_hi = kb.rb_hi == INT_MAX ? INT_MAX : kb.rb_hi * HB;
  auto init_seq = [&](auto first) __attribute__((always_inline)) {
    const int Rs = walk.enter_seq(p);
    int lo = 0, end = Rs;
    if (!decltype(first)::value || is_ctx) {
      if (decltype(first)::value) lo = rows_lo;
      if (walk.seq == seq_hi - 1) end = min(end, rows_hi);
    } else {
      lo = key0;
    }
    walk.enter_rows(p, lo, end);
    new_rows();
  };
  constexpr int NL = SPLIT ? IPB : 1;   // (the swizzle has a period of 16 rows)
  int l_row[NL], l_col[NL];
#pragma unroll
  for (int t = 0; t < NL; ++t) {
    l_row[t] = ld_row(t);
    l_col[t] = ld_col(t);
  }
  // load instruction t of the next row block, into the stage at `st` bytes of both rings
  auto load = [&](uint32_t st, auto Tc) __attribute__((always_inline)) {
    constexpr int t = decltype(Tc)::value;
    // rows past the end of the sequence re-read the last one (no branch for whole blocks: see above)
    const int last = walk.nvalid - 1;
    if constexpr (SPLIT) {
      const uint32_t vo = __umul24((unsigned)min(l_row[t], last), (unsigned)(wave >= 2 ? do_tsb : q_tsb)) + l_col[t];
      dma16_at<t * 1024>(reinterpret_cast<const void*>(wave >= 2 ? walk.dout : walk.q), vo, ld_lds + st);
    } else {
      constexpr int half = t % (IPB / 2), is_do = t / (IPB / 2);
      const uint32_t vo = __umul24((unsigned)min(l_row[0] + half * 16, last), (unsigned)(is_do ? do_tsb : q_tsb)) + l_col[0];
      dma16_at<is_do * DO_RING + half * 4096>(reinterpret_cast<const void*>(is_do ? walk.dout : walk.q), vo, ld_lds + st);
    }
  };
  // LSE*log2e (lanes 0-31) and D of the next row block, by the first wave (the branch in the statement: see above)
  auto load_stats = [&](uint32_t st) __attribute__((always_inline)) {
    const int l = opaque(lane);
    const char* a = reinterpret_cast<const char*>(walk.st) + (l >= 32 ? 0 : stat_gap) + (uint32_t)min(l & 31, walk.nvalid - 1) * 4u;
    asm volatile("s_cmp_lg_u32 %2, 0\n\ts_cbranch_scc1 1f\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n1:"
                 : : "s"(smem_addr + STAT + st / (HT / 256)), "v"(a), "s"(wave) : "memory", "m0", "scc");
  };
  // Flags and first row of the row blocks requested and not yet computed.
  uint32_t fl0 = 0, fl1 = 0, fl2 = 0;
  int rw0 = 0, rw1 = 0, rw2 = 0;
  // records the row block that the loads were for, on to the next one.  Past the end the last block is requested again: the
  // number of loads in flight stays the same, its data are not used
  auto advance = [&]() __attribute__((always_inline)) {
    fl2 = flags | (uint32_t)walk.nvalid << 8;
    rw2 = walk.row0;
    const bool wrap = walk.g + 1 == walk.G;
    const uint64_t q = walk.q + (wrap ? walk.q_row : walk.q_head), dout = walk.dout + (wrap ? walk.do_row : walk.do_head),
                   st = walk.st + (wrap ? walk.st_row : walk.st_head);
    const int row0 = walk.row0 + (wrap ? row_step : 0);
    if (__builtin_expect(!walk.within(row0), 0)) {
      const uint64_t lq = walk.q, ldo = walk.dout, lst = walk.st;
      const int lrow0 = walk.row0, R = walk.R;
      walk.next_seq([&]() __attribute__((always_inline)) { init_seq(std::false_type{}); });
      if (!walk.more) {
        walk.q = lq;
        walk.dout = ldo;
        walk.st = lst;
        walk.row0 = lrow0;
        walk.R = R;
        walk.q_head = walk.q_row = walk.do_head = walk.do_row = walk.st_head = walk.st_row = 0;
        walk.row_end = INT_MIN;
        live = row_step = 0;
      }
    } else {
      walk.q = q;
      walk.dout = dout;
      walk.st = st;
      walk.row0 = row0;
      walk.g = wrap ? 0 : walk.g + 1;
    }
    walk.nvalid = min(HB, walk.R - walk.row0);
    new_rows();
    asm("" : "+s"(fl2), "+s"(rw2));
  };
  auto shift = [&]() __attribute__((always_inline)) {
    fl0 = fl1;
    fl1 = fl2;
    rw0 = rw1;
    rw1 = rw2;
  };

  walk.start(seq_lo, [&]() __attribute__((always_inline)) { init_seq(std::true_type{}); },
             [&]() __attribute__((always_inline)) { init_seq(std::false_type{}); });
  const bool any = walk.more;
  if (any) {
#pragma nounroll
    for (int i = 0; i < AHEAD; ++i) {
      static_for<IPB>([&](auto Tc) __attribute__((always_inline)) { load((uint32_t)i * HT, Tc); });
      load_stats((uint32_t)i * HT);
      shift();
      advance();
    }
    shift();
  }

  // ---- K and -V (sign bits flipped: exact), rows wkey0 + 16 kt + i16
  bf16x8 kf[NKT][KS], vf[NKT][VR], vl[2][NKT];
  const uint32_t vlds = smem_addr + V_LDS + wave * NKT * 2048;
  {
    const TView kt_ = is_ctx ? p.kc : p.kd, vt_ = is_ctx ? p.vc : p.vd;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt) {
      const int64_t kr = key_row_begin + min(wkey0 + 16 * kt + i16, region_len - 1);   // gradients of padded keys are never stored
      const u16* kp = kt_.ptr + kr * kt_.ts + (int64_t)hk * kt_.hs + kgrp16<D>(lg) * 8;
      const u16* vp = vt_.ptr + kr * vt_.ts + (int64_t)hk * vt_.hs + kgrp16<D>(lg) * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kf[kt][ks] = *reinterpret_cast<const bf16x8*>(kp + ks * 32);
        u32x4 v = *reinterpret_cast<const u32x4*>(vp + ks * 32);
        v ^= u32x4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
        if (ks < VR) vf[kt][ks < VR ? ks : 0] = __builtin_bit_cast(bf16x8, v);
        else *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(vlds + ((ks - VR) * NKT + kt) * 1024 + lane * 16) = v;
      }
    }
    // consumed (and therefore waited for) here: no compiler-placed vector-memory wait inside the main loop
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        asm volatile("" : "+v"(kf[kt][ks]));
        if (ks < VR) asm volatile("" : "+v"(vf[kt][ks < VR ? ks : 0]));
      }
  }
  f32x4 dk[NKT][DB], dv[NKT][DB];
#pragma unroll
  for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      dk[kt][db] = f32x4{0.f, 0.f, 0.f, 0.f};
      dv[kt][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

  // per-lane LDS addresses in stage 0; k-steps and column blocks differ in bits that the swizzle flips (head dim 96: in the lowest
  // two chunk bits only) and not in the rows, so that each is the first one's address with a constant XORed (added)
  const uint32_t fbase = smem_addr + frag16_off<D>(lane, 0), tbase = smem_addr + tr16_off<D>(lane, 0);
  auto frag = [&](uint32_t at, auto KSc, int off) __attribute__((always_inline)) {
    constexpr int ks = decltype(KSc)::value;
    const uint32_t x = D == 96 ? at + ks * 64 : at ^ (ks * 64);
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(x + off);
  };
  auto frag_tr = [&](uint32_t at, auto DBc, int off) __attribute__((always_inline)) {
    constexpr int db = decltype(DBc)::value;
    const uint32_t x = D == 96 ? (at ^ (db % 2 * 32)) + db / 2 * 64 : at ^ (db * 32);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(x + off));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(x + off + 16 * RB));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto stat = [&](uint32_t st, int which, int h) __attribute__((always_inline)) {
    return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(smem_addr + STAT + (opaque(lane) >> 4) * 16 + st / (HT / 256) + which * 128 + h * 64);
  };

  uint32_t cur = 0, req = AHEAD * HT;   // stage of the block computed; of the block requested
  if (any) {
    wait_vm<(AHEAD - 1) * IPB>();
    __syncthreads();
  }
  while (fl0 & HDR_VALID) {
    const uint32_t next = cur == (NBUF - 1) * HT ? 0 : cur + HT;
    constexpr int NM = NKT * KS, NE = 4 * NKT;    // MFMAs of a chain group, scores per lane and half
    f32x4 s[2][NKT], dp[2][NKT];
    bf16x8 ro[KS];   // row operands (Q or dO) of the next chains
    float ev[2][NE];
    uint32_t pw[2][NE / 2], dw[2][NE / 2];
    const uint32_t vat = vlds + opaque(lane) * 16, fat = fbase + cur, tat = tbase + cur;
    auto exps = [&](int h, int i, const f32x4& l2) __attribute__((always_inline)) {   // beside MFMA i of NM
#pragma unroll
      for (int e = NE * i / NM; e < NE * (i + 1) / NM; ++e) {
        ev[h][e] = __builtin_amdgcn_exp2f(s[h][e >> 2][e & 3] * c - l2[e & 3]);
        asm volatile("" : "+v"(ev[h][e]));
      }
    };
    auto packs = [&](int h, int i, int n) __attribute__((always_inline)) {   // beside MFMA i of n
      if (i >= n) return;
#pragma unroll
      for (int e = NE / 2 * i / n; e < NE / 2 * (i + 1) / n; ++e) {
        pw[h][e] = pack2_bf16(ev[h][2 * e], ev[h][2 * e + 1]);
        asm volatile("" : "+v"(pw[h][e]));
      }
    };
    auto products = [&](int h, int i, int n) __attribute__((always_inline)) {
      if (i >= n) return;
#pragma unroll
      for (int e = NE / 2 * i / n; e < NE / 2 * (i + 1) / n; ++e) {
        dw[h][e] = pack2_bf16(ev[h][2 * e] * dp[h][e >> 1][2 * e & 3], ev[h][2 * e + 1] * dp[h][e >> 1][(2 * e + 1) & 3]);
        asm volatile("" : "+v"(dw[h][e]));
      }
    };
    auto mask = [&](int h) __attribute__((always_inline)) {
      if (__builtin_expect(fl0 & HDR_MASK, 0)) {
        // score e is that of row 16 h + 4 lg + e % 4 of the block and key 16 (e / 4) + i16 (formed here: hoisted out of the loop
        // the bounds would take registers of all blocks)
        int l = lane;
        asm volatile("" : "+v"(l));
        const int row = 4 * (l >> 4), key = l & 15;
        const int end = (int)(fl0 >> 8) - 16 * h - row, first = is_ctx ? INT_MIN / 2 : wkey0 - rw0 - 16 * h + key - row;
#pragma unroll
        for (int e = 0; e < NE; ++e)
          if (!((e & 3) < end && (e & 3) >= first + 16 * (e >> 2))) ev[h][e] = 0.f;
      }
    };
    // operands of the dV and dK MFMAs: dO^T, then Q^T; each is requested where the one RT before it has been used
    constexpr int RT = 4;
    bf16x8 tr[RT];
    auto load_tr = [&](auto Nc) __attribute__((always_inline)) {
      constexpr int n = decltype(Nc)::value;
      tr[n % RT] = frag_tr(tat, IC<n % DB>{}, n < DB ? DO_RING : 0);
    };
    auto load_vl = [&](int i) __attribute__((always_inline)) {
      vl[i / NKT][i % NKT] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(vat + i * 1024);
    };
    // S (h = 0); every row operand is requested where the one of the group before it has been used
    auto load_row = [&](auto Kc, uint32_t at, int off) __attribute__((always_inline)) { ro[decltype(Kc)::value] = frag(at, Kc, off); };
    static_for<KS>([&](auto Kc) __attribute__((always_inline)) { load_row(Kc, fat, 0); });
    f32x4 l2 = stat(cur, 0, 0), dinit = stat(cur, 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    static_for<NM>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int i = decltype(Ic)::value, kt = i % NKT, ks = i / NKT;
      s[0][kt] = mfma16(ro[ks], kf[kt][ks], ks ? s[0][kt] : f32x4{0.f, 0.f, 0.f, 0.f});
      if constexpr (kt == NKT - 1) load_row(IC<ks>{}, fat, DO_RING);
      if constexpr (i * IPB / NM != (i + 1) * IPB / NM) load(req, IC<i * IPB / NM>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    // D - dP (h = 0), its exponentials
    static_for<NM>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int i = decltype(Ic)::value, kt = i % NKT, ks = i / NKT;
      if constexpr (VR < KS && i < 2 * NKT) load_vl(i);
      dp[0][kt] = mfma16(ro[ks], ks < VR ? vf[kt][ks < VR ? ks : 0] : vl[ks < VR ? 0 : ks - VR][kt], ks ? dp[0][kt] : dinit);
      if constexpr (kt == NKT - 1) load_row(IC<ks>{}, fat, 16 * RB);
      exps(0, i, l2);
      __builtin_amdgcn_sched_barrier(0);
    });
    mask(0);
    // S (h = 1), P and -dS of h = 0
    static_for<NM>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int i = decltype(Ic)::value, kt = i % NKT, ks = i / NKT;
      s[1][kt] = mfma16(ro[ks], kf[kt][ks], ks ? s[1][kt] : f32x4{0.f, 0.f, 0.f, 0.f});
      if constexpr (kt == NKT - 1) load_row(IC<ks>{}, fat, DO_RING + 16 * RB);
      packs(0, i, NM / 2);
      products(0, i, NM / 2);
      if constexpr (i == NM / 2) {
        l2 = stat(cur, 0, 1);
        dinit = stat(cur, 1, 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // D - dP (h = 1), its exponentials
    static_for<NM>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int i = decltype(Ic)::value, kt = i % NKT, ks = i / NKT;
      if constexpr (VR < KS && i < 2 * NKT) load_vl(i);
      dp[1][kt] = mfma16(ro[ks], ks < VR ? vf[kt][ks < VR ? ks : 0] : vl[ks < VR ? 0 : ks - VR][kt], ks ? dp[1][kt] : dinit);
      exps(1, i, l2);
      if constexpr (i >= NM - RT) load_tr(IC<i - (NM - RT)>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    mask(1);
    load_stats(req);
    packs(1, 0, 1);
    // dV += P^T dO, -dS of h = 1; then -dK += (-dS)^T Q
    auto acc_part = [&](auto Fc, auto Lc) __attribute__((always_inline)) {
      constexpr int first = decltype(Fc)::value;
      static_for<(decltype(Lc)::value - first) * NKT>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int i = decltype(Ic)::value, n = first + i / NKT, kt = i % NKT, db = n % DB;
        constexpr bool K = n >= DB;
        const uint32_t(&w)[2][NE / 2] = K ? dw : pw;
        const bf16x8 a = __builtin_bit_cast(bf16x8, u32x4{w[0][2 * kt], w[0][2 * kt + 1], w[1][2 * kt], w[1][2 * kt + 1]});
        f32x4& acc = K ? dk[kt][db] : dv[kt][db];
        acc = mfma16(a, tr[n % RT], acc);
        if constexpr (kt == NKT - 1 && n + RT < 2 * DB) load_tr(IC<n + RT>{});
        if constexpr (!K && first == 0) products(1, i, NM);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    acc_part(IC<0>{}, IC<DB + DB / 2>{});
    advance();
    __builtin_amdgcn_sched_barrier(0);
    acc_part(IC<DB + DB / 2>{}, IC<2 * DB>{});
    // the next block must have landed (the first wave's bound is stricter by its loads of the statistics)
    wait_vm<(AHEAD - 1) * IPB>();
    __syncthreads();
    cur = next;
    req = req == (NBUF - 1) * HT ? 0 : req + HT;
    shift();
  }
  wait_vm<0>();   // no load may land in LDS that belongs to another workgroup by then

  // ---- epilogue: lane owns a head-dim column, register r key 4 lg + r of a tile
  // (head dim 128, whose vector registers are full: with the arguments read again the allocator spills four of them inside the loop,
  // with those already read none; 16 x 1024 behind 8192, 32 / 8 heads 3.7 ms, with spills 5.2)
  const auto args = [&]() __attribute__((always_inline)) {
    if constexpr (D == 128) return &p;
    else return args_again();
  };
  const GradStore out(args(), is_ctx, (int64_t)key_row_begin + key0, min(region_len - key0, BN), hk, D);
  auto store = [&](auto sums) __attribute__((always_inline)) {
    constexpr bool S = decltype(sums)::value;
    const int l = opaque(lane), first = wave * KEYS + 4 * (l >> 4), col = l & 15;   // (formed here: no registers across the loop)
    uint32_t at_k = first * out.row_k + col * (S ? 4 : 2), at_v = first * out.row_v + col * 2;
#pragma unroll
    for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int db = 0; db < DB; ++db) out.put<S>(at_k, at_v, 16 * db, dk[kt][db][r], dv[kt][db][r]);
        at_k += r == 3 ? 13 * out.row_k : out.row_k;
        if (!S) at_v += r == 3 ? 13 * out.row_v : out.row_v;
      }
  };
  if (out.sums) store(std::true_type{});
  else store(std::false_type{});
}

template <int D>
constexpr size_t kPairSmem = kPairStages * (2 * 32 * 2 * D + 256) + (D == 128 ? 16384 : 0);

template <int D>
static hipError_t launch_dkdvw_t(AttnParams p, hipStream_t st) {
  constexpr int tile = 128, threads = 256;
  p.n_ctx_tiles = (p.ctx_len + tile - 1) / tile;
  p.n_dec_tiles = (p.max_rows + tile - 1) / tile;
  if (p.n_split < 1) p.n_split = 1;
  auto kern = dkdvw_kernel<D>;
  const hipError_t e = ensure_dynamic_lds<dkdvw_kernel<D>>(kPairSmem<D>);
  if (e != hipSuccess) return e;
  const int64_t prompt = (int64_t)(p.grp ? p.n_groups : 1) * p.n_ctx_tiles * p.Hk * p.n_split;
  return launch_key_tiles(p, prompt, (int64_t)p.n_dec_tiles * p.Hk, threads, [&](const AttnParams& q, unsigned n) {
    hipLaunchKernelGGL(kern, dim3(n), dim3(threads), kPairSmem<D>, st, q, (int)n);
    return hipGetLastError();
  });
}
hipError_t launch_dkdvw(const AttnParams& p, int head_dim, hipStream_t st) {
  if (p.window > 0 || p.dkc_acc == nullptr || p.dvc_acc == nullptr) return hipErrorInvalidValue;
  switch (head_dim) {
    case 96: return launch_dkdvw_t<96>(p, st);
    case 128: return launch_dkdvw_t<128>(p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace dkv
