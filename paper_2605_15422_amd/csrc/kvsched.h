// Block decode of the KV-stationary backward kernels.  A workgroup's row blocks are those of the (sequence, row block,
// query head) steps whose rows can see at least one key of its key tile: prompt tiles are visited
// by the rows of every sequence of the group (all of them without a window); response tiles only by the
// rows of their own sequence from the diagonal on (Alg. 1, "Q-row blocks in causal support of K_n").
#pragma once
#include <climits>
#include "common.h"

namespace dkv {

// Block decode of the KV-stationary kernels: prompt tiles first (heavy), then response tiles.  With several prompt
// groups, the prompt tiles of group g are the blocks [g * n_ctx_tiles, (g + 1) * n_ctx_tiles) x Hk x n_split, where
// n_ctx_tiles covers the longest prompt; tiles past a shorter prompt have nothing to do.
struct KVBlock {
  bool is_ctx;
  int hk, key0, seq_lo, seq_hi;
  int P, ctx_off;   // prompt length and first prompt row of the block's group
  int rb_lo, rb_hi; // first row block of seq_lo; end of the row blocks of seq_hi - 1 (of HB rows; INT_MAX: all)
};

// The start of a row block that is nearest to `target` rows behind the first row of sequence s0 (sequences [s0, s1)): its
// sequence and its index there.  Nearest and not next: where a sequence is one row block, the next start after every target
// would give one part two sequences and another none.  One parallel compare per 64 sequences instead of a search.
__device__ __forceinline__ void row_block_at(const int32_t* cu, int s0, int s1, int target, int HB, int& seq, int& rb) {
  const int lane = threadIdx.x & 63;
  const int x = __builtin_amdgcn_readfirstlane(cu[s0] + target);
  seq = s0;
  for (int i = s0 + 1; i <= s1; i += 64) {
    const int at = min(i + lane, s1);
    const uint64_t le = __ballot(cu[at] <= x && i + lane <= s1);
    seq += __popcll(le);
    if (~le) break;
  }
  rb = 0;
  if (seq >= s1) return;
  const int r0 = __builtin_amdgcn_readfirstlane(cu[seq]), r1 = __builtin_amdgcn_readfirstlane(cu[seq + 1]);
  rb = (x - r0) / HB;
  const int at_row = r0 + rb * HB;
  if (2 * (x - at_row) >= min(HB, r1 - at_row)) ++rb;
  if (r0 + rb * HB >= r1) {
    ++seq;
    rb = 0;
  }
}

// false: the block owns no key (beyond its prompt or its response)
__device__ __forceinline__ bool decode_kvblock(const AttnParams& p, int BN, int HB, KVBlock& b, int bid, int nblk) {
  const int n_grp = p.grp ? p.n_groups : 1;
  const int ctx_blocks = n_grp * p.n_ctx_tiles * p.Hk * p.n_split;
  b.rb_lo = 0;
  b.rb_hi = INT_MAX;
  if (bid < ctx_blocks) {
    b.is_ctx = true;
    b.hk = bid % p.Hk;
    int t = bid / p.Hk;
    const int split = t % p.n_split;
    t /= p.n_split;
    b.key0 = (t % p.n_ctx_tiles) * BN;
    const int g = t / p.n_ctx_tiles;
    int s0 = 0, s1 = p.n_seqs;
    b.P = p.ctx_len;
    b.ctx_off = 0;
    if (p.grp) {
      b.ctx_off = p.grp[4 * g];
      b.P = p.grp[4 * g + 1];
      s0 = p.grp[4 * g + 2];
      s1 = p.grp[4 * g + 3];
    }
    if (b.key0 >= b.P) return false;
    if (HB < 32 || p.window > 0 || p.cu == nullptr) {
      // Whole sequences: with a window a tile sees few rows of each one, and the head-dim 512 kernel (HB = 16) has no scalar
      // registers left for the bounds of its first and last one.
      const int n = s1 - s0;
      b.seq_lo = s0 + (int)((int64_t)n * split / p.n_split);
      b.seq_hi = s0 + (int)((int64_t)n * (split + 1) / p.n_split);
      // a part without sequences adds nothing to the accumulators; an unsplit tile still has to write its zeros
      if (p.n_split > 1 && b.seq_lo == b.seq_hi) return false;
      return true;
    }
    b.seq_lo = s0;
    b.seq_hi = s1;
    if (p.n_split == 1) return true;
    // the rows of all sequences, cut evenly at row blocks
    const int rows = p.cu[s1] - p.cu[s0];
    int seq_end, rb_end;
    row_block_at(p.cu, s0, s1, (int)((int64_t)rows * split / p.n_split), HB, b.seq_lo, b.rb_lo);
    row_block_at(p.cu, s0, s1, (int)((int64_t)rows * (split + 1) / p.n_split), HB, seq_end, rb_end);
    if (b.seq_lo == seq_end && b.rb_lo == rb_end) return false;
    b.seq_hi = rb_end > 0 ? seq_end + 1 : seq_end;
    if (rb_end > 0) b.rb_hi = rb_end;
    return true;
  }
  bid -= ctx_blocks;
  if (p.window > 0) {
    // Workgroups go to the eight XCDs round-robin by index, each XCD with an L2 of its own.  With a window a response
    // tile reads only the W + BN rows behind its keys, rows that its neighbours read as well: neighbouring tiles are
    // therefore given to the same XCD (block i takes tile (i % 8) * n / 8 + i / 8), where one fetch from memory then
    // serves many of them.  All tiles carry about the same work here, so the XCDs stay balanced; without a window the
    // work falls with the key index and the round-robin order is the balanced one.
    const int chunk = (nblk - ctx_blocks) / 8;
    if (bid < chunk * 8) bid = (bid % 8) * chunk + bid / 8;
  }
  b.is_ctx = false;
  b.hk = bid % p.Hk;
  const int t = bid / p.Hk;
  b.key0 = (t % p.n_dec_tiles) * BN;
  b.seq_lo = t / p.n_dec_tiles;
  b.seq_hi = b.seq_lo + 1;
  b.P = p.seq_ctx ? p.seq_ctx[2 * b.seq_lo + 1] : p.ctx_len;
  b.ctx_off = 0;
  const int rb0 = p.cu ? p.cu[b.seq_lo] : 0;
  const int Rs = p.cu ? (p.cu[b.seq_lo + 1] - rb0) : p.total;
  return b.key0 < Rs;
}

// Flags in a block's header, per 32-key subtile: the block exists; some of its (row, key) pairs are visible; some are not.
// HDR_RUN: the first block of the interval exists.
enum : int { HDR_VALID = 1, HDR_ACTIVE = 2, HDR_MASK = 4, HDR_RUN = 8 };

// Visibility of a row block (first row row0, a multiple of HB <= 32) for the 32-key subtile that starts at k_lo: four
// scalar bounds, so that a block costs a handful of scalar compares.
template <bool LOCAL>
struct SubtileVis {
  int lo, act_hi, mask_lo;   // rows from lo on reach the subtile's first key; rows before act_hi still see its last one
  bool ctx;
  __device__ __forceinline__ SubtileVis(bool is_ctx, int k_lo, int P, int W) : lo(k_lo), ctx(is_ctx) {
    const int shift = is_ctx ? P : 0;   // a row's logical position minus its index
    act_hi = k_lo + 31 + W - shift;
    mask_lo = k_lo + W - 31 - shift;
  }
  // (row0 minus 32 i gives the flags of the i-th next subtile)
  __device__ __forceinline__ uint32_t flags(int row0, int nvalid, int HB) const {
    bool a = ctx || row0 + HB > lo, m = nvalid < HB || (!ctx && row0 < lo + 31);
    if (LOCAL) {
      a = a && row0 < act_hi;
      m = m || row0 >= mask_lo;
    }
    return (uint32_t)(HDR_VALID | (a ? HDR_ACTIVE : 0) | (m ? HDR_MASK : 0));
  }
};

// The key tiles of a causal sequence begin at different rows but all end at the last one: walked downwards, tiles that run side by side
// read the same rows of Q and dO at the same time, once from memory for all of an XCD.  For short sequences the caches do the same, and the
// masked diagonal blocks are better beside the start of a walk than at its end; rows behind a prompt share their time with prompt tiles, which
// read the same rows anyway.  Measured, upwards -> downwards: d = 512, 8 / 2 heads, 14336 causal rows (117 MB of Q and dO for a KV head) 5.68 ->
// 4.33 ms; d = 256, 4 / 2 heads, 4 x U(93, 270) behind 17497 (36 MB) the layer 4.02 -> 3.79 ms, 16 / 4 heads, 5383 causal rows (22 MB) 1892 -> 1816
// us; d = 512, 4 / 2 heads, 2 x U(500, 1000) behind 3000 (12 MB) 955 -> 940 us; d = 192, 12 / 4 heads, 8 x U(131, 2048) behind 4096 (9 MB) the same;
// d = 256, 4 / 2 heads, 2 x U(500, 1000) behind 3000 (6 MB) 616 -> 625.  The line lies at 16 MB.  A sequence's direction depends on its own
// length alone, so that calls for one and for several groups give the same bits.
__host__ __device__ inline bool walk_down(int rows, int G, int D) { return (int64_t)rows * G * D >= 4 << 20; }

// Direction of the walks of a kernel: up, down (one sequence whose length the host knows), or each sequence's own.  The last
// takes scalar registers that the main loops are short of (head dim 512: 5 % slower than either), so that it serves only calls
// of several sequences some of which may walk down.
enum : int { WALK_UP = 0, WALK_DOWN = 1, WALK_OWN = 2 };
template <int DIR, int D>
struct WalkDir {
  int s = DIR == WALK_DOWN ? -1 : 1;
  // row blocks [rb, end) of a sequence; downwards: from the last one, and `end` is the one before the first
  __device__ __forceinline__ void enter(int& rb, int& end, bool is_ctx, int P, int R, int G) {
    if (DIR == WALK_OWN) s = !is_ctx && P == 0 && walk_down(R, G, D) ? -1 : 1;
    if (step() < 0) {
      const int first = rb;
      rb = end - 1;
      end = first - 1;
    }
  }
  __device__ __forceinline__ int step() const { return DIR == WALK_OWN ? s : DIR == WALK_DOWN ? -1 : 1; }
  __device__ __forceinline__ bool any(int rb, int end) const { return step() < 0 ? rb > end : rb < end; }
  __device__ __forceinline__ bool next(int& rb, int end) const {
    rb += step();
    return any(rb, end);
  }
};

// Row-block schedule of a key tile (Alg. 1, "Q-row blocks in causal support of K_n"): the sequences of the tile, row blocks
// of HB rows that see at least one of its keys, query heads of the KV group innermost.  It runs beside the MFMAs in the
// waves that make the requests, so a step is straight-line scalar code: byte addresses advance by one of two precomputed
// strides, and only another row block and the end of a sequence branch.  The empty asm statements keep the state in scalar
// registers: left alone, the compiler moves row counts to vector registers, which the twelve-wave kernel does not have.
// DOWN (dkdvw): from a sequence's last row block to its first, see walk_down; the layer of 8 x U(131, 2048) behind 4111, 16 / 4 heads,
// d = 96 1760 -> 1743 us.  dkdv4 is not bound by these reads and walks up.
template <int HB, bool DOWN>
struct RowWalk {
  uint64_t q, dout, st;      // byte addresses of the block's first row of Q, dO and D (of its head)
  int row0, nvalid, R, row_end, g, seq;   // (DOWN: row_end is the first row)
  bool more;
  const int hk, seq_hi, G;
  static constexpr int DIR = DOWN ? -HB : HB;
  int64_t q_head, q_row, do_head, do_row, st_head, st_row;   // strides to the next head / from the last head to the next block
  int row_begin;

  __device__ __forceinline__ static int64_t pin(int64_t v) {
    asm("" : "+s"(v));
    return v;
  }
  __device__ __forceinline__ RowWalk(const AttnParams& p, int hk_, int seq_hi_)
      : q(0), dout(0), st(0), row0(0), nvalid(0), R(0), row_end(0), g(0), seq(0), more(false), hk(hk_), seq_hi(seq_hi_),
        G(own_sgpr(p.G)), row_begin(0) {
    q_head = pin(p.q.hs * 2);
    q_row = pin(p.q.ts * (2 * DIR) - q_head * (G - 1));
    do_head = pin(p.dout.hs * 2);
    do_row = pin(p.dout.ts * (2 * DIR) - do_head * (G - 1));
    st_head = pin((int64_t)p.total * 4);
    st_row = pin(4 * DIR - st_head * (G - 1));
  }
  __device__ __forceinline__ void keep() {
    asm("" : "+s"(q), "+s"(dout), "+s"(st), "+s"(row0), "+s"(nvalid), "+s"(R), "+s"(row_end), "+s"(g), "+s"(seq));
  }
  // the rows of sequence `seq`; returns their number
  __device__ __forceinline__ int enter_seq(const AttnParams& p) {
    // the offsets are loaded through the vector path: make their uniformity explicit
    row_begin = p.cu ? __builtin_amdgcn_readfirstlane(p.cu[seq]) : 0;
    R = p.cu ? __builtin_amdgcn_readfirstlane(p.cu[seq + 1]) - row_begin : p.total;
    return R;
  }
  // its row blocks from row `first` (a multiple of HB) to before row `end`
  __device__ __forceinline__ void enter_rows(const AttnParams& p, int first, int end) {
    row0 = DOWN ? first + ((end - 1 - first) & -HB) : first;
    row_end = DOWN ? first : end;
    nvalid = min(HB, R - row0);
    g = 0;
    const int64_t grow = (int64_t)row_begin + row0, h0 = (int64_t)hk * G;
    q = reinterpret_cast<uint64_t>(p.q.ptr) + (uint64_t)(grow * p.q.ts + h0 * p.q.hs) * 2;
    dout = reinterpret_cast<uint64_t>(p.dout.ptr) + (uint64_t)(grow * p.dout.ts + h0 * p.dout.hs) * 2;
    st = reinterpret_cast<uint64_t>(p.dvec) + (uint64_t)(h0 * p.total + grow) * 4;
    keep();
  }
  // is there a block at row `r`?
  __device__ __forceinline__ bool within(int r) const { return DOWN ? r >= row_end : r < row_end; }
  // one block on (new_rows() if that is another row block); false: past the last block of the sequence
  template <typename F>
  __device__ __forceinline__ bool step(F&& new_rows) {
    const bool wrap = g + 1 == G;
    q += wrap ? q_row : q_head;
    dout += wrap ? do_row : do_head;
    st += wrap ? st_row : st_head;
    g = wrap ? 0 : g + 1;
    row0 += wrap ? DIR : 0;
    nvalid = min(HB, R - row0);
    keep();
    if (wrap) new_rows();
    return within(row0);
  }
  template <typename F>
  __device__ __forceinline__ void next_seq(F&& init_seq) {
    more = false;
    while (++seq < seq_hi) {
      init_seq();
      if (within(row0)) {
        more = true;
        return;
      }
    }
  }
  template <typename F, typename N>
  __device__ __forceinline__ void start(int seq_lo, F&& init_first, N&& init_next) {
    seq = seq_lo;
    if (seq >= seq_hi) return;
    init_first();
    if (within(row0)) more = true;
    else next_seq(init_next);
  }
};


}  // namespace dkv
