// dK / dV kernel for head dims 64, 96 and 128 with producer / consumer wave specialisation (same mathematics
// and the same ownership rule as the other dK/dV kernels: one workgroup owns a 128-key tile of one KV
// head; a shared-prompt tile sums the contributions of ALL sequences and heads of the group in fp32
// registers and is cast once -- Alg. 1 with the race of the shared prompt gradients removed by ownership).
//
// Measured on gfx950 with two waves per SIMD: a wave issues about one instruction every 4-5 cycles, a taken
// branch costs ~25 cycles, a VGPR -> SGPR round trip ~35, an LDS round trip ~130.  At 32 query rows per
// step the MFMA work of a SIMD is only ~1050 cycles, so the kernel is bound by the instruction stream of
// its busiest wave unless control flow, address arithmetic and waiting are kept out of it.  Hence:
//   * two roles share each SIMD.  A producer wave (0-3, one per 32-key subtile) keeps K and -V fragments in
//     registers and computes S = Q K^T, D - dP = D + dO (-V)^T (accumulator initialised to D),
//     P = exp2(S*scale*log2e - LSE*log2e) and -dS = P * (D - dP), publishing P and -dS as bf16 MFMA
//     operands in LDS.  A consumer wave (4-7) owns one 32-wide head-dim block of dK, dV for all 128 keys
//     and, one row block behind, accumulates dV += P^T dO and -dK += (-dS)^T Q with dO^T / Q^T from LDS
//     transpose reads.  The producers' exponentials overlap the consumers' MFMAs.
//   * the consumers also walk the row-block schedule (a few scalar operations per block) and issue the
//     global -> LDS loads (global_load_lds: Q, dO, LSE*log2e, D never pass through registers) five row
//     blocks ahead; each of them leaves the 16-byte header of one key subtile in the stage (valid / active /
//     mask flags, first row, row count), which is all a producer needs to know about the schedule.
//   * the main loop is unrolled over the LDS stages (six; eight at head dim 64), so every LDS address is an
//     immediate offset;
//     every LDS operand is read one interval before its use, across the single barrier per row block.
//
// Head dim 96 has three 32-wide head-dim blocks for the four consumer waves.  Three of them own a block each and do
// nothing but accumulate (like the producers they learn from the header whether a block exists); the fourth owns no
// accumulator and is the loader: it walks the schedule, writes the headers and makes all twelve requests of a row block.
// Of the 28 MFMAs that the busiest SIMD then has per interval 24 are the average; in return the requests and the scalar
// work, a third of a consumer's time at head dim 128, leave the accumulating waves altogether.  Measured on N = 8,
// P = 4111, R ~ U(131, 2048), 16 / 4 heads: 0.88 + 0.35 ms (Call 2 + Call 1), against 1.95 + 0.82 ms for the kernel with
// register staging, transposed copies and a barrier per phase that served this head dim before.
//
// Head dim 64 halves the MFMAs of a block but not its exponentials, and its waves need 168 registers at most: three fit on a
// SIMD.  Two groups of four producers take two row blocks per interval, the four consumers accumulate both, one after the
// other: half the barriers per block, and the softmax of one group runs beside the chains of the other.  Measured on N = 8,
// P = 4096, R ~ U(131, 2048), 32 / 8 heads: Call 2 1.43 -> 1.34 ms, Call 1 0.237 -> 0.221 ms.
//
// The compiler does not know about the global -> LDS loads: the consumers count them themselves
// (s_waitcnt vmcnt) before the barrier that publishes a row block, and no compiler-visible vector memory
// load is issued inside the main loop (a compiler-placed wait would also wait for all blocks in flight).
#include <type_traits>
#include "common.h"
#include "dma.h"
#include "dq2.h"
#include "kvsched.h"
#include "kvstore.h"
#include "launch.h"
#include "tiles.h"

namespace dkv {

// Producer groups: how many row blocks an interval takes.
template <int D>
constexpr int kGroups = D == 64 ? 2 : 1;
template <int D>
constexpr int kWaves = 4 * kGroups<D> + 4;
template <int D>
constexpr int kStages = kGroups<D> == 2 ? 8 : 6;   // LDS stages (row blocks)
template <int V>
using IC = std::integral_constant<int, V>;

constexpr int kDqWaves = 4;   // of the dQ workgroups in a launch of both

// WITH_DQ: both backward kernels in one launch, for calls that do not fill the chip: n_kv dK/dV workgroups, then dQ workgroups
// of four waves (dq2.h).  The two are independent once the row statistics are there, each is as long as its longest walk when
// a CU has no second workgroup to do, and side by side they take the longer of the two instead of the sum.  Measured (backward call,
// captured in graphs, two launches -> one with its preprocess):
//   1 x 1021 rows, 16 / 16 heads, d = 128 (128 + 128 workgroups)                     69.7 -> 43.7 us; d = 64 45.5 -> 29.0
//   1 x 1021 rows, 16 / 4 heads, d = 128 (32 + 128)                                  143.5 -> 117.8 us; d = 64 94.1 -> 77.1
//   1 x 1500 rows, 8 / 8 heads, d = 128 (96 + 96)                                    90.0 -> 53.0 us; d = 96 75.9 -> 51.5
//   1 x 512 rows, 32 / 8 heads, d = 128 (32 + 128)                                   84.3 -> 69.3 us
//   2 x <= 64 rows behind a prompt of 64, 8 / 2 heads, d = 128 (6 + 8)               31.8 -> 25.1 us; d = 64 24.5 -> 24.0
// The dQ workgroups come behind those of dK/dV, or before them where their walks are the long ones (first_kv: their number).
template <int D, bool LOCAL>
__device__ __forceinline__ void dkdv4_workgroup(const AttnParams& p, int bid, int n_kv);

template <int D, bool LOCAL, bool WITH_DQ>
__global__ __launch_bounds__(kWaves<D> * 64) void dkdv4_kernel(const AttnParams p, int n_kv, int first_kv) {
  const int bid = (int)blockIdx.x - first_kv;
  if (WITH_DQ && (unsigned)bid >= (unsigned)n_kv) {
    if (threadIdx.x >= kDqWaves * 64) return;   // (waves that have ended do not take part in barriers)
    dq2_workgroup<D, kDqWaves, LOCAL, false>(p, bid < 0 ? blockIdx.x : blockIdx.x - n_kv, gridDim.x - n_kv);
    return;
  }
  dkdv4_workgroup<D, LOCAL>(p, bid, n_kv);
}
// The same with dQ workgroups of eight waves, for causal sequences whose dQ is more than the CUs beside long walks of dK/dV can take.
template <int D>
__global__ __launch_bounds__(kWaves<D> * 64) void dkdv4_dq8_kernel(const AttnParams p, int n_kv) {
  if ((int)blockIdx.x >= n_kv) {
    if (threadIdx.x >= 512) return;
    dq2_workgroup<D, 8, false, false>(p, blockIdx.x - n_kv, gridDim.x - n_kv);
    return;
  }
  dkdv4_workgroup<D, false>(p, blockIdx.x, n_kv);
}

template <int D, bool LOCAL>
__device__ __forceinline__ void dkdv4_workgroup(const AttnParams& p, int bid, int n_kv) {
  constexpr int BN = 128, HB = 32;                 // keys per workgroup, query rows per block
  constexpr int KS = D / 16, DSUB = D / 32, RB = 2 * D, CPR = D / 8;
  constexpr int HT_BYTES = HB * RB;                // one Q or dO row block
  constexpr int STAT_OFF = 2 * HT_BYTES;           // lse2[32] | D[32]
  constexpr int HDR_OFF = STAT_OFF + 256;          // 4 x {flags, row0, nvalid, -}
  constexpr int STAGE_BYTES = HDR_OFF + 64;
  constexpr int NPG = kGroups<D>, CW = 4 * NPG;    // row blocks per interval; the first consumer wave
  constexpr int NBUF = kStages<D>, NIS = NBUF / NPG;   // stages: one row block each, NIS intervals in all
  constexpr int AHEAD = NIS - 1;                   // intervals requested ahead of the one being computed
  constexpr int IST_BYTES = NPG * STAGE_BYTES;
  constexpr int HDR_GO = NPG == 1 ? HDR_VALID : HDR_RUN;
  constexpr int XCH_OFF = NBUF * STAGE_BYTES;
  constexpr int XCH_BYTES = NPG * 16384;           // [row block][key subtile][P k-step 0,1 | dS k-step 0,1][lane] x 16 B
  constexpr int NIT = HT_BYTES / 1024;             // 1 KB load instructions per row block and tensor
  constexpr bool LOADER = kSplitRow<D>;            // one consumer wave makes all requests
  constexpr int IPB = LOADER ? 2 * NIT : 2 * NIT / 4;   // per requesting wave (Q and dO)
  constexpr int LOAD_WAVE = 7, STAT_WAVE = CW + 1;
  constexpr int RPI = 1024 / RB;                   // rows per load instruction
  extern __shared__ __attribute__((aligned(256))) unsigned char smem[];   // (as the dQ part needs it)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int kvs = wave & 3;
  const int W = p.window;

  KVBlock kb;
  if (!decode_kvblock(p, BN, HB, kb, bid, n_kv)) return;
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

  if (wave < CW) {
    // ================================= producer ==============================================
    const float c = p.scale_log2;
    const int pg = NPG == 1 ? 0 : wave >> 2;   // the row block of every interval that this wave takes
    const int my_key = key0 + kvs * 32 + l32;
    const u16 *kbase, *vbase;
    int64_t kts, vts;
    if (is_ctx) {
      kbase = p.kc.ptr + (int64_t)key_row_begin * p.kc.ts + (int64_t)hk * p.kc.hs;
      vbase = p.vc.ptr + (int64_t)key_row_begin * p.vc.ts + (int64_t)hk * p.vc.hs;
      kts = p.kc.ts;
      vts = p.vc.ts;
    } else {
      kbase = p.kd.ptr + (int64_t)key_row_begin * p.kd.ts + (int64_t)hk * p.kd.hs;
      vbase = p.vd.ptr + (int64_t)key_row_begin * p.vd.ts + (int64_t)hk * p.vd.hs;
      kts = p.kd.ts;
      vts = p.vd.ts;
    }
    bf16x8 kf[KS], vfn[KS];   // K and -V (sign bits flipped: exact)
    {
      const int kr = min(my_key, region_len - 1);   // clamp: gradients of padded keys are never stored
      const u16* kp = kbase + (int64_t)kr * kts + hi * 8;
      const u16* vp = vbase + (int64_t)kr * vts + hi * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kf[ks] = *reinterpret_cast<const bf16x8*>(kp + ks * 16);
        u32x4 v = *reinterpret_cast<const u32x4*>(vp + ks * 16);
        v.x ^= 0x80008000u;
        v.y ^= 0x80008000u;
        v.z ^= 0x80008000u;
        v.w ^= 0x80008000u;
        vfn[ks] = __builtin_bit_cast(bf16x8, v);
      }
      // the loads are consumed (and therefore waited for) here, before the main loop
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" : : "v"(kf[ks]), "v"(vfn[ks]));
    }
    // LDS addresses: two base registers per operand (stages 0-2 and 3-5) so that every access of the
    // unrolled loop is base + immediate offset (the offset field has 16 bits)
    constexpr int NLO = NPG == 2 ? NIS : NIS / 2;   // interval stages within the 16-bit offset of one base register
    constexpr int HALF = NLO * IST_BYTES;
    const unsigned char* frag_lo[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) frag_lo[ks] = smem + pg * STAGE_BYTES + tile_off<D>(l32, 2 * ks + hi);
    const unsigned char* frag_hi[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) frag_hi[ks] = frag_lo[ks] + HALF;
    const unsigned char* stat_lo = smem + pg * STAGE_BYTES + STAT_OFF + hi * 16;   // this lane's rows 8*(r/4) + 4*hi + r%4
    const unsigned char* stat_hi = stat_lo + HALF;
    const unsigned char* hdr_lo = smem + pg * STAGE_BYTES + HDR_OFF + kvs * 16;
    const unsigned char* hdr_hi = hdr_lo + HALF;
    unsigned char* xw_lane = smem + XCH_OFF + pg * 16384 + kvs * 4096 + lane * 16;

    bf16x8 qfr[KS];
    int flags, row0, nvalid;
    auto read_header = [&](auto Uc, u32x4& h) __attribute__((always_inline)) {
      constexpr int U = decltype(Uc)::value;
      h = *reinterpret_cast<const u32x4*>((U < NLO ? hdr_lo : hdr_hi) + (U % NLO) * IST_BYTES);
    };
    // which = 0: Q fragments (read one interval early), 1: dO fragments (read at the start of their interval,
    // behind the S chain: keeping both sets across the barrier does not fit next to the K / V fragments)
    auto load_frags = [&](auto Uc, auto which, bf16x8* out) __attribute__((always_inline)) {
      constexpr int U = decltype(Uc)::value;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const unsigned char* b = U >= NLO ? frag_hi[ks] : frag_lo[ks];
        out[ks] = *reinterpret_cast<const bf16x8*>(b + (U % NLO) * IST_BYTES + decltype(which)::value * HT_BYTES);
      }
    };
    // row statistics of this lane's 16 rows (register r <-> row crow(r, hi)): which = 0 LSE*log2e, 1 D
    auto load_stat = [&](auto Uc, int which, float* out) __attribute__((always_inline)) {
      constexpr int U = decltype(Uc)::value;
      const unsigned char* b = (U < NLO ? stat_lo : stat_hi) + (U % NLO) * IST_BYTES + which * 128;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(b + r4 * 32);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) out[r4 * 4 + e4] = v[e4];
      }
    };

    // one interval: block h in stage U; returns false after the end of the schedule
    auto interval = [&](auto Uc) __attribute__((always_inline)) -> bool {
      constexpr int U = decltype(Uc)::value, NU = (U + 1) % NIS, XB = U & 1;
      if (__builtin_expect(!(flags & HDR_GO), 0)) {
        __syncthreads();
        return false;
      }
      u32x4 hn;
      read_header(IC<NU>{}, hn);
      const bool act = flags & HDR_ACTIVE;
      f32x16 s, dpv;
      float l2[16];
      if (__builtin_expect(act, 1)) {
        float dinit[16];
        bf16x8 dofr[KS];
        load_stat(Uc, 1, dinit);   // their latency hides behind the S chain
        load_frags(Uc, IC<1>{}, dofr);
        __builtin_amdgcn_sched_barrier(0);   // all reads requested before the first MFMA, not trickled in between
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s = mfma32(qfr[ks], kf[ks], s);
#pragma unroll
        for (int r = 0; r < 16; ++r) dpv[r] = dinit[r];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) dpv = mfma32(dofr[ks], vfn[ks], dpv);   // D - dP
        load_stat(Uc, 0, l2);
      }
      // keep the operand reads of block h+1 behind the MFMAs of block h: issued earlier they would need a
      // second set of 64 fragment registers and push the K / V fragments out of the register file
      __builtin_amdgcn_sched_barrier(0);
      const int nflags = __builtin_amdgcn_readfirstlane((int)hn.x);
      const int nrow0 = __builtin_amdgcn_readfirstlane((int)hn.y);
      const int nnvalid = __builtin_amdgcn_readfirstlane((int)hn.z);
      // unconditional: a load that depends on the next header would make the compiler keep the old fragments in
      // a second register set (sixteen moves per block); an inactive or invalid block's fragments are never used
      load_frags(IC<NU>{}, IC<0>{}, qfr);
      __builtin_amdgcn_sched_barrier(0);
      unsigned char* xw = xw_lane + XB * XCH_BYTES;
      if (__builtin_expect(act, 1)) {
        float pv[16], dsv[16];
        auto softmax_part = [&](auto masked) __attribute__((always_inline)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float e = __builtin_amdgcn_exp2f(s[r] * c - l2[r]);
            if (decltype(masked)::value) {
              // rows past the end of the sequence hold copies of its last row: masked like invisible keys
              const int rl = crow(r, hi), rw = row0 + rl;
              bool ok = rl < nvalid;
              if (is_ctx) ok = ok && (!LOCAL || (my_key > P + rw - W));
              else ok = ok && (my_key <= rw) && (!LOCAL || (my_key > rw - W));
              if (!ok) e = 0.f;
            }
            pv[r] = e;
            dsv[r] = e * dpv[r];   // -dS
          }
        };
        if (__builtin_expect(flags & HDR_MASK, 0)) softmax_part(std::true_type{});
        else softmax_part(std::false_type{});
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          *reinterpret_cast<bf16x8*>(xw + t2 * 1024) = pack8_bf16(pv + t2 * 8);
          *reinterpret_cast<bf16x8*>(xw + (2 + t2) * 1024) = pack8_bf16(dsv + t2 * 8);
        }
      } else {
        // no visible (row, key) pair in this block: publish zero operands, the consumers do not branch
        const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < 4; ++t) *reinterpret_cast<u32x4*>(xw + t * 1024) = z;
      }
      __syncthreads();
      flags = nflags;
      row0 = nrow0;
      nvalid = nnvalid;
      return true;
    };

    __syncthreads();   // row blocks 0 and 1 and their headers are in LDS
    {
      u32x4 h0;
      read_header(IC<0>{}, h0);
      flags = __builtin_amdgcn_readfirstlane((int)h0.x);
      row0 = __builtin_amdgcn_readfirstlane((int)h0.y);
      nvalid = __builtin_amdgcn_readfirstlane((int)h0.z);
    }
    if (flags & HDR_ACTIVE) load_frags(IC<0>{}, IC<0>{}, qfr);
    while (true) {
      if (!interval(IC<0>{})) break;
      if (!interval(IC<1>{})) break;
      if (!interval(IC<2>{})) break;
      if (!interval(IC<3>{})) break;
      if constexpr (NIS > 4) {
        if (!interval(IC<4 % NIS>{})) break;
        if (!interval(IC<5 % NIS>{})) break;
      }
    }
  } else {
    // ================================= consumer ==============================================
    const int jb = wave - CW;
    const uint32_t smem_addr = (uint32_t)reinterpret_cast<uintptr_t>(smem);
    // ---- global -> LDS loads: instruction i = jb + 4 t of a row block covers RPI rows of Q (t < IPB/2) or
    // dO; lane l lands at LDS chunk position l % CPR of row (l / CPR) of the instruction, so it fetches the
    // chunk that the tile swizzle stores there (the swizzle has period 4 RPI rows: one offset serves all t).
    const int ld_row0 = jb * RPI + lane / CPR;
    const int ld_coff = ((lane % CPR) ^ swz<D>(ld_row0)) * 16;
    const uint32_t ld_lds = smem_addr + (LOADER ? 0 : jb * 1024);
    const int q_tsb = own_sgpr((int)p.q.ts * 2), do_tsb = own_sgpr((int)p.dout.ts * 2);   // bytes per token
    // per-lane global offsets of this wave's load instructions for a block of 32 valid rows (a partial last
    // block clamps its rows instead: rare, computed on the spot)
    uint32_t voff_full[IPB];
    int ld_row[IPB / 2], ld_off[IPB / 2];   // row and byte offset within the row, the same for Q and dO
#pragma unroll
    for (int t = 0; t < IPB / 2; ++t) {
      ld_row[t] = LOADER ? split_row<D>(t, lane) : ld_row0 + t * 4 * RPI;
      ld_off[t] = LOADER ? (split_pos<D>(t, lane) ^ swz<D>(ld_row[t])) * 16 : ld_coff;
    }
#pragma unroll
    for (int t = 0; t < IPB; ++t)
      voff_full[t] = (uint32_t)(ld_row[t % (IPB / 2)] * (t < IPB / 2 ? q_tsb : do_tsb) + ld_off[t % (IPB / 2)]);
    // row statistics: lanes 0-31 fetch LSE*log2e, lanes 32-63 fetch D; both arrays live in one workspace, D
    // first and LSE*log2e less than 4 GB behind it (checked by the launcher), so one scalar base plus an
    // unsigned 32-bit lane offset addresses both (the loader of head dim 96 uses 64-bit lane addresses)
    const uint32_t stat_lane_off = hi ? 0u : (uint32_t)((const char*)p.lse2 - (const char*)p.dvec);
    const int64_t stat_lane = hi ? 0 : (const char*)p.lse2 - (const char*)p.dvec;

    // ---- row-block schedule (kvsched.h); wave jb writes the headers of key subtile jb, the loader all four
    RowWalk<HB, false> walk(p, hk, seq_hi);
    const SubtileVis<LOCAL> vis(is_ctx, key0 + (LOADER ? 0 : jb * 32), P, W);
    uint32_t flags = 0;   // of the current row block (the loader: byte i those of subtile i)
    auto new_rows = [&]() __attribute__((always_inline)) {
      flags = vis.flags(walk.row0, walk.nvalid, HB);
      if constexpr (LOADER) {
#pragma unroll
        for (int i = 1; i < 4; ++i) flags |= vis.flags(walk.row0 - i * 32, walk.nvalid, HB) << (8 * i);
      }
      asm("" : "+s"(flags));
    };
    // (response tiles have one sequence: only the first call has to know them; windowed tiles are short and not cut)
    const int rows_lo = LOCAL ? 0 : kb.rb_lo * HB, rows_hi = LOCAL || kb.rb_hi == INT_MAX ? INT_MAX : kb.rb_hi * HB;
    auto init_seq = [&](auto first) __attribute__((always_inline)) {
      const int Rs = walk.enter_seq(p);
      int lo = 0, end;
      if (LOCAL ? is_ctx : !decltype(first)::value || is_ctx) {
        const int key_hi = min(P, key0 + BN) - 1;
        end = LOCAL ? min(Rs, key_hi + W - P) : Rs;
        if (!LOCAL && decltype(first)::value) lo = rows_lo;
        if (!LOCAL && walk.seq == seq_hi - 1) end = min(end, rows_hi);
      } else {
        const int key_hi = min(Rs, key0 + BN) - 1;
        end = LOCAL ? min(Rs, key_hi + W) : Rs;
        lo = key0;
      }
      walk.enter_rows(p, lo, end);
      new_rows();
    };
    uint32_t vbits = 0;   // bit i: block (request position - 1 - i) exists
    // requests the next block of the schedule (or marks the end) in stage IS (the loader: at stage_off) and advances the
    // schedule
    auto issue_block = [&](auto ISc, uint32_t stage_off = 0) __attribute__((always_inline)) {
      constexpr int IS = decltype(ISc)::value;
      unsigned char* hdr = smem + stage_off + IS * STAGE_BYTES + HDR_OFF + (LOADER ? lane : jb) * 16;
      if (__builtin_expect(!walk.more, 0)) {
        vbits <<= 1;
        // the second block of an interval runs (with nothing visible) if the first one exists
        const uint32_t run = IS % NPG != 0 && (vbits & 2u) != 0 ? HDR_RUN : 0u;
        if (lane < (LOADER ? 4 : 1)) *reinterpret_cast<u32x4*>(hdr) = u32x4{run, 0u, 0u, 0u};
        return;
      }
      vbits = (vbits << 1) | 1u;
      if (lane < (LOADER ? 4 : 1)) {
        const uint32_t fl = LOADER ? (flags >> (8 * lane)) & 0xffu : flags;
        *reinterpret_cast<u32x4*>(hdr) = u32x4{fl | HDR_RUN, (uint32_t)walk.row0, (uint32_t)walk.nvalid, 0u};
      }
      const int last = walk.nvalid - 1;   // rows past the end of the sequence re-read its last row
      const void* const q_base = reinterpret_cast<const void*>(walk.q);
      const void* const do_base = reinterpret_cast<const void*>(walk.dout);
      auto load = [&](auto Tc, uint32_t voff) __attribute__((always_inline)) {
        constexpr int t = decltype(Tc)::value;
        constexpr int off = IS * STAGE_BYTES + (LOADER ? t * 1024 : (t < IPB / 2 ? 0 : HT_BYTES) + (t % (IPB / 2)) * 4096);
        dma16_at<off>(t < IPB / 2 ? q_base : do_base, voff, ld_lds + stage_off);
      };
      // (one branch for the whole block, not one per load)
      if (__builtin_expect(walk.nvalid == HB, 1)) {
        static_for<IPB>([&](auto Tc) __attribute__((always_inline)) { load(Tc, voff_full[decltype(Tc)::value]); });
      } else {
        static_for<IPB>([&](auto Tc) __attribute__((always_inline)) {
          constexpr int t = decltype(Tc)::value;
          load(Tc, __umul24((unsigned)min(ld_row[t % (IPB / 2)], last), (unsigned)(t < IPB / 2 ? q_tsb : do_tsb)) +
                       (uint32_t)ld_off[t % (IPB / 2)]);
        });
      }
      if constexpr (LOADER)
        dma4_from<IS * STAGE_BYTES + STAT_OFF>(reinterpret_cast<const char*>(walk.st) + stat_lane + min(l32, last) * 4,
                                               smem_addr + stage_off);
      else if (wave == STAT_WAVE)
        dma4_at<IS * STAGE_BYTES + STAT_OFF>(reinterpret_cast<const void*>(walk.st), stat_lane_off + (uint32_t)min(l32, last) * 4u,
                                             smem_addr);
      if (__builtin_expect(!walk.step(new_rows), 0)) walk.next_seq([&]() __attribute__((always_inline)) { init_seq(std::false_type{}); });
    };
    // Block b is requested AHEAD blocks early and must have landed by the end of interval b - 2 (the
    // producer reads its operands one interval early): the three youngest blocks (IPB loads each per
    // wave; wave 5 issues one more, for it the bound is a little stricter) may stay in flight.  If the
    // newest request was the end mark, fewer loads are outstanding: wait for all of them.
    auto wait_loads = [&]() __attribute__((always_inline)) {
      wait_vm<(AHEAD - 2) * NPG * (IPB + (LOADER ? 1 : 0))>();
      if (__builtin_expect(!(vbits & 1u), 0)) wait_vm<0>();
    };

    if (!LOADER || wave == LOAD_WAVE) {
      walk.start(seq_lo, [&]() __attribute__((always_inline)) { init_seq(std::true_type{}); },
                 [&]() __attribute__((always_inline)) { init_seq(std::false_type{}); });
      if constexpr (!LOADER) {
        static_for<AHEAD * NPG>([&](auto Ic) __attribute__((always_inline)) { issue_block(Ic); });
        wait_loads();
      }
    }
    if (LOADER && wave == LOAD_WAVE) {
      // (not unrolled over the stages: this wave has time for a stage offset in a register, and the code stays short)
#pragma nounroll
      for (int i = 0; i < AHEAD; ++i) issue_block(IC<0>{}, i * STAGE_BYTES);
      wait_loads();
      __syncthreads();   // row blocks 0 and 1 and their headers are in LDS
      uint32_t stage_off = AHEAD * STAGE_BYTES;
      bool cur = true;
      while (cur) {
        issue_block(IC<0>{}, stage_off);
        stage_off = stage_off == AHEAD * STAGE_BYTES ? 0 : stage_off + STAGE_BYTES;
        cur = vbits & (1u << AHEAD);
        wait_loads();
        __syncthreads();
      }
      return;
    }

    // Each consumer wave owns one 32-wide head-dim block (dblk) of the gradients of NK key subtiles: the
    // transposed Q / dO operands of its head-dim block are shared by all its key subtiles, which keeps the
    // (slow) LDS transpose reads at 8 per row block.
    constexpr int NK = D == 64 ? 2 : 4;            // key subtiles per wave
    const int dblk = jb % DSUB, k0 = (jb / DSUB) * NK;
    f32x16 dk[NK], dv[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        dk[i][r] = 0.f;
        dv[i][r] = 0.f;
      }
    const unsigned char* tr0 = smem + tr_off<D>(lane, hi * 4, dblk * 32);
    const unsigned char* tr1 = smem + tr_off<D>(lane, hi * 4 + 8, dblk * 32);
    const unsigned char* xr_lane = smem + XCH_OFF + k0 * 4096 + lane * 16;
    bf16x8 tq[NPG][2], tdo[NPG][2];   // Q^T, dO^T operands of the row blocks accumulated next interval
    bool prev = false;      // (with a loader wave) block h - 1 exists

    // one interval: accumulates block h-1, reads the transposed operands of block h (stage U), requests
    // block h + AHEAD; returns false after the end of the schedule
    auto interval = [&](auto Uc) __attribute__((always_inline)) -> bool {
      constexpr int U = decltype(Uc)::value, IS = (U + AHEAD) % NIS, XB = (U + 1) & 1;
      constexpr int CUR = AHEAD * NPG + NPG - 1, PREV = CUR + NPG;   // bits of the first block of this and of the last interval
      // requests first: the producers' MFMAs run meanwhile, the consumers' follow them
      uint32_t hdr = 0;
      if constexpr (LOADER) hdr = *reinterpret_cast<const uint32_t*>(smem + HDR_OFF + U * STAGE_BYTES);
      else static_for<NPG>([&](auto Ec) __attribute__((always_inline)) { issue_block(IC<IS * NPG + decltype(Ec)::value>{}); });
#pragma unroll
      for (int e = 0; e < NPG; ++e) {
        if (LOADER ? !prev : (vbits & (1u << (PREV - e))) == 0) continue;
        const unsigned char* xr = xr_lane + XB * XCH_BYTES + e * 16384;
        // all P / -dS operands are requested before the first MFMA (left alone, the compiler reads one operand,
        // waits for it and issues one MFMA, sixteen LDS latencies in a row)
        bf16x8 pa[2][NK], dsa[2][NK];
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int i = 0; i < NK; ++i) {
            pa[t2][i] = *reinterpret_cast<const bf16x8*>(xr + i * 4096 + t2 * 1024);
            dsa[t2][i] = *reinterpret_cast<const bf16x8*>(xr + i * 4096 + (2 + t2) * 1024);
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
          for (int i = 0; i < NK; ++i) {
            dv[i] = mfma32(pa[t2][i], tdo[e][t2], dv[i]);
            dk[i] = mfma32(dsa[t2][i], tq[e][t2], dk[i]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      const bool cur = LOADER ? (__builtin_amdgcn_readfirstlane((int)hdr) & HDR_VALID) != 0 : (vbits & (1u << CUR)) != 0;
#pragma unroll
      for (int e = 0; e < NPG; ++e) {
        if (__builtin_expect(e == 0 ? !cur : (vbits & (1u << (CUR - e))) == 0, 0)) continue;
        constexpr int ST = U * IST_BYTES;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          const int at = ST + e * STAGE_BYTES + t2 * 16 * RB;
          tdo[e][t2] = tr_pair(tr0 + at + HT_BYTES, tr1 + at + HT_BYTES);
          tq[e][t2] = tr_pair(tr0 + at, tr1 + at);
        }
      }
      if constexpr (LOADER) prev = cur;
      else wait_loads();
      __syncthreads();
      return cur;
    };

    __syncthreads();   // row blocks 0 and 1 and their headers are in LDS
    while (true) {
      if (!interval(IC<0>{})) break;
      if (!interval(IC<1>{})) break;
      if (!interval(IC<2>{})) break;
      if (!interval(IC<3>{})) break;
      if constexpr (NIS > 4) {
        if (!interval(IC<4 % NIS>{})) break;
        if (!interval(IC<5 % NIS>{})) break;
      }
    }

    // ---- epilogue: C layout -> lane owns head-dim column, register r owns key crow(r)
    const GradStore out(args_again(), is_ctx, (int64_t)key_row_begin + key0, min(region_len - key0, BN), hk, D);
    auto store = [&](auto sums) __attribute__((always_inline)) {
      constexpr bool S = decltype(sums)::value;
      uint32_t at_k = (k0 * 32 + 4 * hi) * out.row_k + (dblk * 32 + l32) * (S ? 4 : 2), at_v = (k0 * 32 + 4 * hi) * out.row_v + (dblk * 32 + l32) * 2;
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const f32x16 gk = dk[i], gv = dv[i];
        out.tile32<S>(at_k, at_v, [&](int r, uint32_t ak, uint32_t av) __attribute__((always_inline)) { out.put<S>(ak, av, 0, gk[r], gv[r]); });
      }
    };
    if (out.sums) store(std::true_type{});
    else store(std::false_type{});
  }
}

template <int D>
constexpr size_t kDkdv4Smem = kStages<D> * (2 * 32 * 2 * D + 256 + 64) + 2 * kGroups<D> * 16384;

constexpr int kKeyTile = 128;
static int64_t dq_workgroups(AttnParams& p, int waves) {
  fill_packing(p, waves);
  return (int64_t)p.n_seqs * p.MB * p.HC * p.Hk;
}

// DQ_WAVES: of the dQ workgroups in the launch (0: none); dq_first: they come before those of dK/dV
template <int D, bool LOCAL, int DQ_WAVES>
static hipError_t launch_dkdv4_t(AttnParams p, bool dq_first, hipStream_t st) {
  const KeyTiles t = key_tiles(p, kKeyTile);
  // the kernel addresses LSE*log2e as D + 32-bit unsigned byte offset (the loader wave of head dim 96 does not)
  if (!kSplitRow<D> && (reinterpret_cast<uintptr_t>(p.lse2) < reinterpret_cast<uintptr_t>(p.dvec) ||
       reinterpret_cast<uintptr_t>(p.lse2) - reinterpret_cast<uintptr_t>(p.dvec) >= (1ull << 32)))
    return hipErrorInvalidValue;
  constexpr size_t dq_smem = DQ_WAVES == 0 ? 0 : kDq2Smem<D, DQ_WAVES == 8 ? 8 : kDqWaves>, smem = std::max(dq_smem, kDkdv4Smem<D>);
  constexpr auto kern = [] {
    if constexpr (DQ_WAVES == 8) return dkdv4_dq8_kernel<D>;
    else return dkdv4_kernel<D, LOCAL, DQ_WAVES != 0>;
  }();
  const hipError_t e = ensure_dynamic_lds<kern>(smem);
  if (e != hipSuccess) return e;
  constexpr int threads = kWaves<D> * 64;
  if constexpr (DQ_WAVES != 0) {   // (no more workgroups than rules::dq_beside lets share a launch)
    const unsigned n_kv = (unsigned)(t.prompt + p.n_seqs * t.per_seq), n = n_kv + (unsigned)dq_workgroups(p, DQ_WAVES);
    if (n == 0) return hipSuccess;
    if constexpr (DQ_WAVES == 8) hipLaunchKernelGGL(kern, dim3(n), dim3(threads), smem, st, p, (int)n_kv);
    else hipLaunchKernelGGL(kern, dim3(n), dim3(threads), smem, st, p, (int)n_kv, dq_first ? (int)(n - n_kv) : 0);
    return hipGetLastError();
  }
  return launch_key_tiles(p, t.prompt, t.per_seq, threads, [&](const AttnParams& q, unsigned n) {
    if constexpr (DQ_WAVES != 8) hipLaunchKernelGGL(kern, dim3(n), dim3(threads), smem, st, q, (int)n, 0);
    return hipGetLastError();
  });
}

template <int DQ_WAVES>
static hipError_t launch_dkdv4_d(const AttnParams& p, int head_dim, bool dq_first, hipStream_t st) {
  constexpr bool L = DQ_WAVES != 8;   // (which knows no window)
  const bool local = L && p.window > 0;
  switch (head_dim) {
    case 64:  return local ? launch_dkdv4_t<64, L, DQ_WAVES>(p, dq_first, st) : launch_dkdv4_t<64, false, DQ_WAVES>(p, dq_first, st);
    case 96:  return local ? launch_dkdv4_t<96, L, DQ_WAVES>(p, dq_first, st) : launch_dkdv4_t<96, false, DQ_WAVES>(p, dq_first, st);
    case 128: return local ? launch_dkdv4_t<128, L, DQ_WAVES>(p, dq_first, st) : launch_dkdv4_t<128, false, DQ_WAVES>(p, dq_first, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dkdv4(const AttnParams& p, int head_dim, hipStream_t st) { return launch_dkdv4_d<0>(p, head_dim, false, st); }
hipError_t launch_dkdv4_dq(const AttnParams& p, int head_dim, int dq_waves, bool dq_first, hipStream_t st) {
  return dq_waves == 8 ? launch_dkdv4_d<8>(p, head_dim, false, st) : launch_dkdv4_d<kDqWaves>(p, head_dim, dq_first, st);
}

}  // namespace dkv
