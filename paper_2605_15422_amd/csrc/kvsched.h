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

// The row block at `target` rows behind the first row of sequence s0 (sequences [s0, s1), whole row blocks: a target inside a
// block means the next one): its sequence and its index there.  One parallel compare per 64 sequences instead of a search.
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
  rb = (x - r0 + HB - 1) / HB;
  if (r0 + rb * HB >= r1) {
    ++seq;
    rb = 0;
  }
}

// false: the block owns no key (beyond its prompt or its response)
__device__ __forceinline__ bool decode_kvblock(const AttnParams& p, int BN, int HB, KVBlock& b) {
  const int n_grp = p.grp ? p.n_groups : 1;
  const int ctx_blocks = n_grp * p.n_ctx_tiles * p.Hk * p.n_split;
  int bid = blockIdx.x;
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
    b.seq_lo = s0;
    b.seq_hi = s1;
    if (p.n_split == 1) return true;   // (an unsplit tile without rows still has to write its zeros)
    if (p.window > 0 || p.cu == nullptr) {
      // with a window a tile sees few rows of each sequence: whole sequences
      const int n = s1 - s0;
      b.seq_lo = s0 + (int)((int64_t)n * split / p.n_split);
      b.seq_hi = s0 + (int)((int64_t)n * (split + 1) / p.n_split);
      return b.seq_lo < b.seq_hi;      // a part without rows adds nothing to the accumulators
    }
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
    const int chunk = ((int)gridDim.x - ctx_blocks) / 8;
    if (bid < chunk * 8) bid = (bid % 8) * chunk + bid / 8;
  }
  b.is_ctx = false;
  b.hk = bid % p.Hk;
  int t = bid / p.Hk;
  const int part = t % p.n_row_split;
  t /= p.n_row_split;
  b.key0 = (t % p.n_dec_tiles) * BN;
  b.seq_lo = t / p.n_dec_tiles;
  b.seq_hi = b.seq_lo + 1;
  b.P = p.seq_ctx ? p.seq_ctx[2 * b.seq_lo + 1] : p.ctx_len;
  b.ctx_off = 0;
  const int rb0 = p.cu ? p.cu[b.seq_lo] : 0;
  const int Rs = p.cu ? (p.cu[b.seq_lo + 1] - rb0) : p.total;
  if (b.key0 >= Rs) return false;
  if (p.n_row_split > 1) {
    // The row blocks that see the tile (no window here), cut evenly.  Every part adds its gradient into the fp32 accumulators.
    const int lo = b.key0 / HB, n = (Rs + HB - 1) / HB - lo;
    const int parts = min(p.n_row_split, (n + p.row_split_len - 1) / p.row_split_len);
    if (part >= parts) return false;
    b.rb_lo = __builtin_amdgcn_readfirstlane(lo + n * part / parts);   // (n < 2^27, part < 16)
    b.rb_hi = __builtin_amdgcn_readfirstlane(lo + n * (part + 1) / parts);
  }
  return true;
}

}  // namespace dkv
