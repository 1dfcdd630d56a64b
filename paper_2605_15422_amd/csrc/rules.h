// Host-side rules that size a launch from the sizes of a call.  Plain C++: no device code, no HIP types.
#pragma once
#include <algorithm>
#include <cstdint>

namespace dkv {
namespace rules {

constexpr int kCus = 256;

// ---- Call 2: workgroups per prompt tile (dK/dV) ----
struct PromptTiles {
  int64_t tiles;               // prompt tiles of all groups, times the KV heads
  int n_seqs, n_groups, total_resp, max_resp;
  int G;                       // query heads per KV head
  int kv_heads;
  int key_tile, row_block;     // keys and rows that the kernel takes at a time
  bool whole_seqs;             // parts are whole sequences (else row blocks)
  int64_t shared;              // up to so many prompt workgroups dK/dV and dQ share a launch
  int ctx_len;                 // keys of the longest prompt
  int head_dim = 128;
};

constexpr int kTargetBlocks = 512;   // prompt-tile workgroups from which on no prompt tile is cut into parts

// A bound on the parts of a prompt tile that is known to the caller's workspace: above one, the fp32 accumulators exist.
inline int most_parts(const PromptTiles& c) {
  if (c.tiles == 0 || c.tiles >= kTargetBlocks) return 1;
  const int64_t want = (kTargetBlocks + c.tiles - 1) / c.tiles, per_group = (c.n_seqs + c.n_groups - 1) / c.n_groups;
  return (int)std::max<int64_t>(1, std::min(want, per_group));
}

// The number of parts to launch: the one with the shortest time in a model of 256 CUs that take workgroups in launch order,
// prompt tiles first.  Unit: one interval of the kernel (a row block of one query head); kStart of them for a workgroup's
// start and end.  Sequences count in whole row blocks.  Three bounds: all work spread evenly; full rounds of parts; the longest
// response tile, which may start behind the full rounds.  Where dK/dV and dQ would no longer share a launch, dQ's walk over the
// keys comes on top.
// Up to two parts the sum of an element has one result whatever the order (0 + a + b = 0 + b + a), and calls where most_parts
// says so keep that; more parts add in an order that varies from run to run.
// Over 900 drawn calls the backward of Call 2 takes 0.71 of its time with most_parts parts of whole sequences and two launches
// (7 of them 1.03 to 1.24 times longer); with most_parts parts 0.76; kStart 12 to 40 differ by 1 %.
constexpr int kStart = 30, kMaxParts = 32;

struct PromptWork {
  double seqs, one;     // sequences of a group; intervals of one
  double own, longest;  // all response tiles; the longest one
  double resp_tiles;    // their number
};
inline double ceil_div(double a, double b) { return (double)(int64_t)((a + b - 1) / b); }
inline PromptWork prompt_work(const PromptTiles& c) {
  PromptWork w;
  const double mean = (double)c.total_resp / c.n_seqs;
  w.seqs = ceil_div(c.n_seqs, c.n_groups);
  w.one = ceil_div(mean, c.row_block) * c.G;
  const double tiles = ceil_div(mean, c.key_tile);
  w.resp_tiles = tiles * c.n_seqs * c.kv_heads;
  // the tiles of a response see from all of its row blocks down to the last tile's
  w.own = w.resp_tiles * (w.one * (tiles + 1) / (2 * tiles) + kStart);
  w.longest = ceil_div(c.max_resp, c.row_block) * c.G + kStart;
  return w;
}
// intervals of one of n parts of a prompt tile
inline double part_work(const PromptTiles& c, const PromptWork& w, int n) {
  return (c.whole_seqs ? ceil_div(w.seqs, n) * w.one : ceil_div(w.seqs * w.one, n)) + kStart;
}
// Time of all tiles with n parts.  `pair`: the kernel of which two workgroups share a CU (pair_interval: the time of an interval of
// each of them then, kAlone: of one that has the CU to itself; in a full round a start and end lie beside the other one's work).  The
// longest response tile may start behind the full rounds.
constexpr double kAlone = 1.27;
inline double pair_interval(const PromptTiles& c) { return c.head_dim == 96 ? 1.65 : 1.78; }
inline double parts_time(const PromptTiles& c, const PromptWork& w, int n, bool pair) {
  const double part = part_work(c, w, n);
  const int64_t all = c.tiles * n;
  if (pair) {
    const int64_t full = all / (2 * kCus), rest = all % (2 * kCus);
    const double kPair = pair_interval(c);
    const double rounds = full * (kPair * (part - kStart) + kStart);
    const double last = rest == 0 ? 0 : (rest <= kCus ? kAlone : kPair) * part;
    const double late = (rest + w.resp_tiles <= kCus ? kAlone : kPair) * w.longest;
    return std::max({(all * part + w.own) * (kPair / 2) / kCus, rounds + last, rounds + late});
  }
  return std::max({(all * part + w.own) / kCus, (all + kCus - 1) / kCus * part, all / kCus * part + w.longest});
}

inline int prompt_parts(const PromptTiles& c, bool pair = false) {
  const int most = most_parts(c);
  if (most == 1 || c.total_resp == 0) return most;
  const PromptWork w = prompt_work(c);
  const double apart = 10 + ((double)c.ctx_len + c.max_resp) / 53;   // (64 keys of dQ: 1.2 intervals)
  auto time = [&](int n) {
    const double t = parts_time(c, w, n, pair);
    return c.shared >= c.tiles && c.tiles * n > c.shared ? t + apart : t;
  };
  // (a part takes at least a sequence or a row block)
  const int limit = (int)std::min<double>(most <= 2 ? most : kMaxParts, c.whole_seqs ? w.seqs : w.seqs * w.one / c.G);
  int best = 1;
  for (int n = 2; n <= limit; ++n)
    if (time(n) < 0.98 * time(best)) best = n;
  return best;
}

// dK/dV at head dims 96 and 128, no window, one prompt: two workgroups a CU (dkdvw.hip) with `pair_parts` parts, or one with `parts`?
// Two get more done on a full chip but each is slower, and a long response tile that starts behind the prompt tiles is then late.  So
// where three quarters of the work are prompt tiles and the model says that they fill their rounds.  Both measured for 583 calls behind
// prompts of 300 to 40000, d = 96 and 128: those that go here take 0.68 to 1.02 of their time (runs of equal kernels differ by
// 0.015), all 583 together 0.924.  With one pair_interval of 1.72 for both head dims (0.929) calls of 2 to 2.75 rounds of 256 long parts
// went here, too, and lost at d = 128: 16 x 1024 rows behind 10240, 32 / 8 heads 5.67 -> 5.80 ms, behind 11264 5.56 -> 5.78.
inline bool pair_tiles(const PromptTiles& c, int parts, int pair_parts) {
  if (c.total_resp == 0 || c.tiles == 0 || c.n_groups > 1 || c.tiles * parts <= c.shared) return false;
  const PromptWork w = prompt_work(c);
  const double prompt = c.tiles * pair_parts * part_work(c, w, pair_parts);
  return prompt >= 3 * w.own && parts_time(c, w, pair_parts, true) <= parts_time(c, w, parts, false);
}

// ---- Forward and dQ of head dims 64 / 96 / 128: waves in a workgroup ----
// Head packing of one workgroup that owns `nst` 32-row subtiles: `heads` query heads of the KV group share the staged K / V
// tiles, each with `subtiles` consecutive subtiles.
struct Packing {
  int heads, subtiles;
};
inline Packing pack_heads(int G, int nst) {
  int a = G, b = nst;
  while (b) {
    const int t = a % b;
    a = b;
    b = t;
  }
  return {a, nst / a};
}

struct RowBlocks {
  int n_seqs, longest;     // sequences, rows of the longest one
  int ctx_len;             // prompt keys in front of them
  bool window;
  int G, kv_heads;
  int total = 0;           // rows of all sequences
};

// Four waves or eight where one workgroup has a CU to itself?  A wave that has its SIMD to itself takes 0.7 of the time per tile, and half
// the rows make twice as many workgroups; but four waves get less done on a CU than two per SIMD.  So four
//   * where every workgroup has a CU to itself, counted with the longest sequence: row blocks that other sequences do not have are
//     dispatched, too, and displace some (22 x U(93, 135) rows behind 392, 8 / 8 heads, d = 128, 232 of 352 with rows: 26 -> 33 us);
//   * forward, where eight would not make fewer workgroups, since half of them have no rows: 0.75 of the time;
//   * for one or two causal sequences past a short prompt up to 600 workgroups: the longest walks start first and the short ones
//     fill the gaps (d = 128, 1 x 10746 rows, 336 workgroups: 248 -> 185 us; 1 x 10723, 672: 288 -> 304).  With a window all walks
//     are alike (1 x 1229 rows, window 918, 32 / 4 heads, 312 workgroups: 39 -> 50 us); with more sequences the long walks of the
//     last one start late (23 x U(73, 496) rows behind 4793, 4 / 2 heads: 147 -> 189 us).
// dQ: eight also where half of them have no rows; the other four run like four alone, and eight request the tiles (20 x 20 rows
// behind 4283, 8 / 8 heads, d = 128: 97 us with four, 94 with eight).  But a launch that dK/dV shares takes four (`shared`).
// `pair`: two workgroups of four share a CU, which beats eight (choose_waves).
inline int64_t row_block_count(const RowBlocks& c, int waves) {
  const Packing k = pack_heads(c.G, waves);
  const int64_t rows = 32 * k.subtiles;
  return c.n_seqs * ((c.longest + rows - 1) / rows) * (c.G / k.heads) * c.kv_heads;
}
inline int row_block_waves(const RowBlocks& c, bool pair, bool dq, bool shared) {
  const int64_t n = row_block_count(c, 4);
  if (n <= kCus) {
    const Packing k = pack_heads(c.G, 8);
    return dq && !shared && std::min(k.subtiles, (c.longest + 31) / 32) * k.heads <= 4 ? 8 : 4;
  }
  if (pair || (!dq && n == row_block_count(c, 8))) return 4;
  return c.n_seqs <= 2 && !c.window && 4 * (int64_t)c.ctx_len <= c.longest && n <= 600 ? 4 : 8;
}

// One causal sequence in two rounds of eight waves, a CU each: the longest walks pair up with the shortest.  Rows, heads, d: forward and
// dQ with eight -> pairs of four in us; 3900, 32 / 8, 128: 114 -> 125, 163 -> 169; 16000, 8 / 2, 128: 441 -> 477, 624 -> 654; 7400, 16 / 4, 96:
// 166 -> 179, 218 -> 237.  The other side: 13000, 8 / 8, 128 (408 workgroups of eight) 371 -> 322, 470 -> 437; 4600, 32 / 8, 128 (576) 171 -> 162,
// 242 -> 219.
inline bool two_rounds_of_eight(const RowBlocks& c) {
  const int64_t n = row_block_count(c, 8);
  return c.n_seqs == 1 && !c.window && 4 * (int64_t)c.ctx_len <= c.longest && n > 416 && n <= 2 * kCus;
}
// Forward over long walks in a dozen rounds and more: the card's power bounds it, pairs of four waves request every tile for half the rows,
// and the last round is short beside the others.  Sustained, eight -> pairs: 16 x U(1024, 2048) behind 32768, 32 / 4 heads, d = 128
// 18.6 -> 19.1 ms, d = 96 15.4 -> 15.9.  The other side: 16 x U(512, 1024) behind 32768, 32 / 8 heads, d = 128 (six rounds of eight) 6.46 -> 5.92 ms.
inline bool many_long_walks(const RowBlocks& c) {
  const Packing k = pack_heads(c.G, 8);
  const int64_t per_block = (int64_t)(c.G / k.heads) * c.kv_heads;
  return !c.window && c.ctx_len + (int64_t)c.longest / 2 >= 8192 && (c.total / (32 * k.subtiles) + c.n_seqs / 2) * per_block >= 12 * kCus;
}

// Eight waves, or four in workgroups that share a CU (`pair`: two of them, three at head dim 64) or have one each?  With two, one starts
// and ends beside the other's tiles, and the last round of a launch is half as long: over 45 drawn calls of 2 to 3000 GFLOP at d = 128 and
// 96 each (forward and dQ of both calls) pairs take 0.80 to 0.83 of the time of eight (0.55 to 1.04), over 11 long ones 0.94 (dQ of 16 x 1024
// behind 8192, 32 / 8 heads, d = 128 2.85 -> 2.67 ms, forward 1.94 and 1.94).  A CU each where all of them have one, or where the longest walks
// of one or two causal sequences start first (1 x 3000, 16 / 4 heads, d = 128, 376 workgroups: forward 60 us in pairs, 58 without, dQ 80 and 77).
struct Waves {
  int n;
  bool pair;
};
inline Waves choose_waves(const RowBlocks& c, int head_dim, bool dq, bool shared) {
  if (dq && head_dim < 128) {   // (whose rings leave room for two or three workgroups in any case)
    const bool eight = head_dim == 96 && two_rounds_of_eight(c);
    return {row_block_waves(c, !eight, dq, shared), true};
  }
  const int64_t n = row_block_count(c, 4);
  const int alone = row_block_waves(c, false, dq, shared);
  if (alone == 4 && (n <= kCus || n != row_block_count(c, 8))) return {4, false};
  if (head_dim == 64) {   // (three to a CU leave others idle where two to a CU are one round: 56 row blocks of 8 heads 1304 -> 1336 us the layer)
    const Packing k = pack_heads(c.G, 4);
    return {4, (c.total / (32 * k.subtiles) + c.n_seqs / 2) * (int64_t)(c.G / k.heads) * c.kv_heads > 2 * kCus};
  }
  if ((n <= kCus || two_rounds_of_eight(c) || (!dq && many_long_walks(c)))) return {8, false};
  return {4, true};
}

// ---- Backward of head dims 64 / 96 / 128: dK/dV and dQ in one launch ----
// Behind a preprocess that forms the row statistics the two are independent, a workgroup of either has its CU to itself, and the tails
// of both are filled.
struct Beside {
  int waves = 0;          // of the dQ workgroups
  bool first = false;     // they come before those of dK/dV
  int64_t room = -1;      // up to so many prompt workgroups share the launch
};
// One launch
//   * where every workgroup of both kernels has one of the 256 CUs to itself: all calls measured there gained (1.02 to 1.7 times);
//   * up to 960 workgroups where the responses are long for their prompt: a response's tiles carry work that falls from the first to the
//     last.  2 x U(206, 654) behind 807, 12 / 4 heads, d = 128, 103 -> 69 us; 2 x U(1601, 1891) behind 567 (500 workgroups) 209 -> 155;
//     2 x U(791, 2882) behind 185 (744) 265 -> 204; 8 x U(681, 2345) behind 733, 4 / 2 heads, d = 96 (908) 201 -> 181.  The other side: 14 x
//     U(1283, 2013) behind 2863, 4 / 2 heads, d = 96 (1390) 554 -> 576 us; short responses: 12 x U(67, 112) behind 1602, 16 / 4 heads, d = 128
//     113.5 -> 114.0, 19 x U(128, 266) behind 1291, 12 / 4 heads, d = 64 118 -> 124;
//   * few rows behind a long prompt, up to 320 dQ workgroups, whose walks are at least a third of those of the prompt tiles: dQ first, the
//     prompt tiles on the other CUs.  110 calls take 0.62 to 1.04 of their time, 0.85 together: 4 x U(50, 138) behind 12628, 32 / 4 heads, d = 96 393
//     -> 287 us, 1 x 298 behind 4336, 32 / 8 heads, d = 64 133 -> 82.  The other side: 17 x U(119, 150) behind 31574, 32 / 8 heads, d = 64
//     (680 dQ workgroups) 2459 -> 2729 us; walks of a sixth: 8 x U(91, 152) behind 1631, 32 / 4 heads, d = 96 134 -> 146;
//   * one causal sequence up to 416 key tiles: its first tile's walk is twice the mean.  With eight waves a dQ workgroup from 240 tiles on (dQ
//     is too much work for the CUs that dK/dV leaves idle), if eight make enough workgroups.  1 x 5000, 32 / 8 heads, d = 128 (320 tiles) 778 ->
//     664 us (four waves 716), 1 x 4111, 16 / 4, d = 96 (132) 434 -> 352 (359 with eight), 1 x 3000, 8 / 8, d = 128 (192) 149 -> 89.  The other
//     side: 7200, 32 / 8, d = 64 (456) 769 -> 784;
//   * several causal sequences up to as many tiles (Call 1 of several groups; counted with the longest).  The layers of eight
//     groups behind prompts of up to 517, 32 / 8 heads, d = 128 473 -> 457 us, three behind 1500, 12 / 4, 313 -> 274, eight behind 100, 32 / 8,
//     d = 64 329 -> 328.  Call 2 of several groups gains nothing (0.98 to 1.09).
inline Beside dq_beside(const RowBlocks& c, bool several_groups, int64_t prompt_tiles, int64_t resp_tiles) {
  const int64_t n4 = row_block_count(c, 4);
  if (c.ctx_len == 0 && !several_groups && !c.window) {
    if (resp_tiles + n4 <= kCus) return {4, false, 0};
    if (resp_tiles > 416) return {};
    return {row_block_count(c, 8) >= 240 && (c.n_seqs > 1 || resp_tiles >= 240) ? 8 : 4, false, 0};
  }
  const bool one_prompt = c.ctx_len > 0 && !several_groups && !c.window;
  const bool tails = one_prompt && c.total >= 0.3 * c.ctx_len * c.n_seqs;
  const int64_t room = (tails ? 960 : kCus) - resp_tiles - n4;
  // walks in intervals of dK/dV (64 keys of dQ: 1.2)
  const double dq_walk = 10 + ((double)c.ctx_len + c.longest) / 53, part = c.total / 32.0 * c.G + c.n_seqs * (c.G / 2.0);
  if (one_prompt && room < prompt_tiles && n4 <= 320 && 3 * dq_walk >= part) return {4, true, 1 << 20};
  return {4, false, room};
}

// Head dims 192 to 512, whose dQ workgroups have a CU to themselves in any case: a shared launch loses nothing but the
// pass of the preprocess.
//   * Causal sequences up to 600 key tiles: 0.56 to 0.98 of the time.  1 x 4236 rows, 8 / 2 heads, d = 192 464 -> 371 us; 1 x 1562, 8 / 8, d =
//     256 108 -> 63; 1 x 9219, 8 / 2, d = 512 (578 tiles) 3303 -> 3138; past that the tails are short: 1 x 5980, 32 / 8, d = 192 (752) 1429 -> 1372,
//     1 x 7082, 12 / 4, d = 512 (888) 2583 -> 2557.
//   * Responses up to 700 dQ workgroups, those first where their walks are at least half of those of the prompt tiles: 44 calls take 0.58
//     to 1.01 of their time, 0.81 together (one 1.03: 7 x U(96, 546) behind 1472, 16 / 4, d = 256 273 -> 281); 3 x U(48, 88) behind 7082, 12 / 4, d = 512
//     504 -> 328 us, 2 x U(902, 1069) behind 73, 16 / 4, d = 256 153 -> 119.  The other side: 12 x U(443, 946) behind 295, 32 / 8, d = 256 (2880)
//     791 -> 799.
inline Beside dq_beside_wide(const RowBlocks& c, bool several_groups, bool d512, int64_t resp_tiles) {
  if (c.window || several_groups) return {};
  if (c.ctx_len == 0) return resp_tiles <= 600 ? Beside{8, false, 0} : Beside{};
  const Packing k = pack_heads(c.G, d512 ? 2 : 4);
  const int64_t rows = 32 * k.subtiles, n = c.n_seqs * ((c.longest + rows - 1) / rows) * (c.G / k.heads) * c.kv_heads;
  if (n > 700) return {};
  // walks in intervals of dK/dV: its row block, and 32 keys of dQ (head dim 512: half of either) take 1.5
  const double dq_walk = ((double)c.ctx_len + c.longest) / (d512 ? 10.7 : 21.3), part = (double)c.total * c.G / (d512 ? 16 : 32);
  return {8, 2 * dq_walk >= part, 1 << 20};
}

// K and V tiles that a dQ workgroup has room for, head dims 64 / 96 / 128.  Three at d = 64, so that three workgroups fit the LDS
// of a CU (their registers do, too): with four and two workgroups dQ of 8 x U(131, 2048) behind 4096, 32 / 8 heads takes 730 us instead of 686.
// At d = 128 four waves have three slots for K, two tiles ahead, and two for V, one ahead: exactly half of a CU's LDS.
constexpr int dq_ring_slots(int head_dim, int waves = 8) { return head_dim == 128 && waves == 8 ? 4 : 3; }
constexpr int dq_v_slots(int head_dim, int waves) { return head_dim == 128 && waves == 4 ? 2 : dq_ring_slots(head_dim, waves); }

// Copies of a prompt row that one workgroup of the replicating copy writes.  More of them read the row less often; but one
// workgroup then writes for longer than its share of the whole copy takes, and the few that there are keep the others waiting.
// So no more than the rows that a CU has to write: 23 x 29 + 138 rows of 64 KB take 31 us with 16 copies and 13 with 2, 16 x 64 + 270
// rows 32 and 17 with 4, 12 x 2489 + 288 rows of 16 KB 141 with one and 106 with 16.  Over 250 calls from 7 us up the choice takes 1.02 of
// the time of the best of 1, 2, 4, 8 and 16, sixteen throughout 1.04 (up to 3.6).
inline int replicate_copies(int64_t n_seqs, int64_t ctx_len, int64_t total) {
  int64_t copies = 16;
  while (copies > 1 && copies * kCus > n_seqs * ctx_len + total) copies /= 2;
  return (int)copies;
}

}  // namespace rules
}  // namespace dkv
