// Work decomposition shared by the Q-stationary kernels (forward, dQ): block decode, KV tile schedule of
// a row block across the two KV regions, and the visibility predicates of the causal / window mask in
// the logical position space (prompt positions 0..P-1, then P + r; Sec. 3.1 and App. F of the paper).
#pragma once
#include "common.h"
#include "dma.h"
#include "rules.h"
#include "tiles.h"

namespace dkv {

// ---------------------------------------------------------------------------------------------
// block decode + KV tile schedule shared by fwd and dq
// ---------------------------------------------------------------------------------------------
struct QBlock {
  int hk, hc, mb, seq, row_begin, R, blk_row0;
  int P, ctx_off;   // prompt length and first prompt row of the sequence's group
  int c0, n_ctx, d0, n_dec, n_tiles;
};

template <int BN>
__device__ __forceinline__ bool decode_qblock(const AttnParams& p, QBlock& b, int bid, int nblk) {
  int t = bid;
  if (p.window > 0) {
    // Workgroups go to the eight XCDs round-robin by index, each XCD with an L2 of its own.  With a window a row block
    // reads only the K / V tiles of the W keys before it, nearly the same ones as the neighbouring row blocks of its
    // sequence: neighbours are therefore given to the same XCD (block i takes work item (i % 8) * n / 8 + i / 8).  All
    // items carry about the same work here; without a window the work grows with the row index and the round-robin
    // order is the balanced one.
    const int chunk = nblk / 8;
    if (t < chunk * 8) t = (t % 8) * chunk + t / 8;
  }
  b.hk = t % p.Hk; t /= p.Hk;
  b.hc = t % p.HC; t /= p.HC;
  b.mb = p.MB - 1 - (t % p.MB);   // late (long-horizon) row blocks first
  b.seq = t / p.MB;
  b.row_begin = p.cu ? p.cu[b.seq] : 0;
  b.R = p.cu ? (p.cu[b.seq + 1] - b.row_begin) : p.total;
  b.blk_row0 = b.mb * p.BMR;
  if (b.blk_row0 >= b.R) return false;
  b.P = p.seq_ctx ? p.seq_ctx[2 * b.seq + 1] : p.ctx_len;
  b.ctx_off = p.seq_ctx ? p.seq_ctx[2 * b.seq] : 0;
  const int P = b.P;
  const int last_row = min(b.R, b.blk_row0 + p.BMR) - 1;
  b.n_ctx = (P + BN - 1) / BN;
  b.n_dec = last_row / BN + 1;
  b.c0 = 0;
  b.d0 = 0;
  if (p.window > 0) {
    // lowest key any row of the block may see: logical (P + blk_row0) - W + 1
    const int lo = P + b.blk_row0 - p.window + 1;
    if (lo >= P) {
      b.c0 = b.n_ctx;
      b.d0 = (lo - P) / BN;
    } else if (lo > 0) {
      b.c0 = lo / BN;
    }
  }
  b.n_tiles = (b.n_ctx - b.c0) + (b.n_dec - b.d0);
  return true;
}

// Visibility of key `key` (index inside its region) for row `row` of the sequence.
template <bool LOCAL>
__device__ __forceinline__ bool visible(bool is_ctx, int key, int row, int P, int R, int W) {
  if (is_ctx) {
    bool ok = key < P;
    if (LOCAL) ok = ok && (key > P + row - W);
    return ok;
  }
  bool ok = (key <= row) && (key < R);
  if (LOCAL) ok = ok && (key > row - W);
  return ok;
}

// Does any (row, key) pair of a 32-row subtile x BN-key tile need masking?
template <bool LOCAL, int BN>
__device__ __forceinline__ bool tile_needs_mask(bool is_ctx, int key0, int row0, int P, int R, int W) {
  if (is_ctx) {
    bool need = key0 + BN > P;
    if (LOCAL) need = need || (key0 <= P + row0 + 31 - W);
    return need;
  }
  bool need = (key0 + BN - 1 > row0) || (key0 + BN > R);
  if (LOCAL) need = need || (key0 <= row0 + 31 - W);
  return need;
}

// Is any pair of rows [rmin, rmax] x the BN-key tile visible at all?
template <bool LOCAL, int BN>
__device__ __forceinline__ bool tile_active(bool is_ctx, int key0, int rmin, int rmax, int P, int W) {
  if (is_ctx) {
    if (LOCAL) return key0 + BN - 1 > P + rmin - W;
    return true;
  }
  bool act = key0 <= rmax;
  if (LOCAL) act = act && (key0 + BN - 1 > rmin - W);
  return act;
}


// The offsets of a block are loaded through the vector path: make their uniformity explicit.
__device__ __forceinline__ void make_uniform(QBlock& b) {
  b.row_begin = __builtin_amdgcn_readfirstlane(b.row_begin);
  b.R = __builtin_amdgcn_readfirstlane(b.R);
  b.P = __builtin_amdgcn_readfirstlane(b.P);
  b.ctx_off = __builtin_amdgcn_readfirstlane(b.ctx_off);
  b.c0 = __builtin_amdgcn_readfirstlane(b.c0);
  b.n_ctx = __builtin_amdgcn_readfirstlane(b.n_ctx);
  b.d0 = __builtin_amdgcn_readfirstlane(b.d0);
  b.n_dec = __builtin_amdgcn_readfirstlane(b.n_dec);
  b.n_tiles = __builtin_amdgcn_readfirstlane(b.n_tiles);
}

// Global -> LDS loads of the 64-key tiles of a row block's schedule, in order (head dims 64, 96, 128), or of their halves (BN = 32).
// Half of the workgroup's waves request the K tiles, half the V tiles; a wave keeps the address of its next tile, the keys of the region from there on and the
// lane offsets of a full tile, so that a request is a handful of scalar instructions.  Instruction t of a wave covers 1 KB of its
// rows; lane l lands at LDS chunk position l % CPR of its row and fetches the chunk that the swizzle stores there.  Keys past the
// end of a region re-read the last key: their scores are masked like any invisible key.
template <int D, int NW, int BN = 64>
struct TileLoader {
  static constexpr int CPR = D / 8, TILE_BYTES = BN * 2 * D, PER_TILE = 64 / BN;
  static constexpr int LW = NW / 2;                            // waves per tensor
  static constexpr int IPT = TILE_BYTES / 1024 / LW;           // load instructions per wave and tile
  static constexpr int RPI = 1024 / (2 * D);                   // whole rows per instruction (not at head dim 96)
  static constexpr int STEP = kSplitRow<D> ? 1024 : LW * 1024;   // bytes from one instruction of a wave to the next
  // the lane offsets repeat after NV instructions (the swizzle after 16 rows), GROUP rows further on
  static constexpr int NV = kSplitRow<D> ? 3 : LW * RPI % 16 == 0 ? 1 : 2, GROUP = kSplitRow<D> ? 16 : NV * LW * RPI;
  static_assert(IPT % NV == 0 && GROUP % 16 == 0, "");
  static_assert(IPT >= 1 && TILE_BYTES % (1024 * LW) == 0, "tile must split evenly over the waves");
  static_assert(!kSplitRow<D> || (IPT % 3 == 0 && BN == LW * (IPT / 3) * kSplitRows<D>), "whole rows per wave");
  const int lane, lwave;
  const bool v;                // this wave requests V tiles
  uint32_t lds;
  uint64_t ptr, own_ptr;       // next tile; first one of the response
  int keys, tsb, left;         // keys of the region from the next tile on, bytes per token, tiles to request
  int own_keys, own_tsb;
  int ctx_left;                // (BN = 32) requests left in the prompt
  uint32_t voff[NV];

  // the V ring lies v_ring bytes behind the K ring at `smem`
  __device__ __forceinline__ TileLoader(const AttnParams& p, const QBlock& b, int wave, int lane_, const unsigned char* smem, int v_ring)
      : lane(lane_), lwave(wave % LW), v(wave >= LW),
        left(b.n_tiles * PER_TILE), ctx_left((b.n_ctx - b.c0) * PER_TILE) {
    lds = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(smem) + (v ? v_ring : 0) +
                                         lwave * (kSplitRow<D> ? IPT * 1024 : 1024));
    const TView own = v ? p.vd : p.kd, ctx = v ? p.vc : p.kc;
    own_ptr = first_tile(own, (int64_t)b.row_begin + b.d0 * 64, b.hk);
    own_tsb = (int)own.ts * 2;
    own_keys = b.R - b.d0 * 64;
    ptr = first_tile(ctx, (int64_t)b.ctx_off + b.c0 * 64, b.hk);
    tsb = (int)ctx.ts * 2;
    keys = b.c0 < b.n_ctx ? b.P - b.c0 * 64 : 0;
    lane_offsets();
  }
  __device__ __forceinline__ static uint64_t first_tile(const TView& x, int64_t row, int hk) {
    return reinterpret_cast<uint64_t>(uniform_ptr(x.ptr + row * x.ts + (int64_t)hk * x.hs));
  }
  __device__ __forceinline__ int row(int t, int l) const {
    // (head dim 96: a wave's three instructions are consecutive, together its sixteen rows)
    if constexpr (kSplitRow<D>) return lwave * (IPT / 3) * kSplitRows<D> + split_row<D>(t, l);
    else return lwave * RPI + l / CPR + t * LW * RPI;
  }
  __device__ __forceinline__ int col(int t, int l) const {
    return ((kSplitRow<D> ? split_pos<D>(t, l) : l % CPR) ^ swz16<D>(row(t, l))) * 16;
  }
  __device__ __forceinline__ void lane_offsets() {
#pragma unroll
    for (int t = 0; t < NV; ++t) voff[t] = (uint32_t)(__umul24((unsigned)row(t, lane), (unsigned)tsb) + col(t, lane));
  }
  // requests this wave's next tile into ring slot `slot`; false: there is none
  __device__ __forceinline__ bool request(uint32_t slot) {
    if (left == 0) return false;
    --left;
    if (__builtin_expect(BN == 64 ? keys <= 0 : ctx_left-- == 0, 0)) {
      ptr = own_ptr;
      tsb = own_tsb;
      keys = own_keys;
      lane_offsets();
    }
    // (uniform, but not always in scalar registers, which the requests need)
    const uint64_t base = reinterpret_cast<uint64_t>(uniform_ptr(reinterpret_cast<const u16*>(ptr)));
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds + slot * TILE_BYTES);
    const int step = __builtin_amdgcn_readfirstlane(GROUP * tsb);
    if (__builtin_expect(keys >= BN, 1)) {
      static_for<IPT>([&](auto Tc) __attribute__((always_inline)) {
        constexpr int t = decltype(Tc)::value;
        dma16_at<t * STEP>(reinterpret_cast<const void*>(base + (uint32_t)(t / NV * step)), voff[t % NV], dst);
      });
    } else {
      const int l = opaque(lane);   // (rows and columns formed here: no registers in between)
      // (the second half of a tile whose first half holds the region's last key: that key is behind `base`)
      const int last = __builtin_amdgcn_readfirstlane(keys - 1), back = BN == 64 ? 0 : min(last, 0);
      const uint64_t at = base + (uint64_t)((int64_t)back * __builtin_amdgcn_readfirstlane(tsb));
      static_for<IPT>([&](auto Tc) __attribute__((always_inline)) {
        constexpr int t = decltype(Tc)::value;
        dma16_at<t * STEP>(reinterpret_cast<const void*>(at), (uint32_t)(__umul24((unsigned)min(row(t, l), last - back), (unsigned)tsb) + col(t, l)), dst);
      });
    }
    ptr += (uint64_t)(uint32_t)tsb * BN;
    keys -= BN;
    return true;
  }
};

// Head packing of one workgroup that owns `nst` 32-row subtiles (rules.h)
static inline void fill_packing(AttnParams& p, int nst) {
  const rules::Packing k = rules::pack_heads(p.G, nst);
  p.GP = k.heads;
  p.RSH = k.subtiles;
  p.BMR = p.RSH * 32;
  p.HC = p.G / p.GP;
  p.MB = (p.max_rows + p.BMR - 1) / p.BMR;
}

static inline rules::Waves choose_waves(const AttnParams& p, int head_dim, bool dq, bool shared = false) {
  const rules::RowBlocks c = {p.n_seqs, p.max_rows, p.ctx_len, p.window > 0, p.G, p.Hk, p.total};
  return rules::choose_waves(c, head_dim, dq, shared);
}

}  // namespace dkv
