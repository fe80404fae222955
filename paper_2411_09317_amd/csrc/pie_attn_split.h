// How the one-launch attention cuts a call into units, and the scratch that takes: arithmetic alone, for the kernel, for
// what launches it and for a test that runs it on the CPU over its whole range.
//
// A unit is one part of one sequence for one kv head, a workgroup's work.  A part is k quanta, a quantum one pass of the
// workgroup's waves over a block each; an item is a part for all kv heads.
#pragma once

#include "pie_internal.h"

namespace pie {

constexpr int kWaves = 4;
constexpr int kBlockTokens = 16;
constexpr int kQuantum = kWaves * kBlockTokens;
constexpr int kDirectSeqs = 256;                 // sequences the kernel splits: four to a lane
constexpr int kDirectRows = 16384;               // partial states (unit, head of the group) there is room for
constexpr int kDirectMaxUnits = 4096;
constexpr int kDirectMaxQuanta = 64;             // per part: a wave's list of slots has a lane for each
static_assert(kDirectMaxUnits <= kArriveWords && kDirectMaxUnits <= kClockWgs,
              "a word per (sequence, head), a pair per workgroup");

// ---- on the host: units of a call, scratch of a pool ---------------------------------------------------------

// How many units the split of a call may make; 0: they do not fit.  As few as hold every (sequence, kv head) pair and the
// longest context the table can name, in steps of the compute units.  One workgroup a compute unit streams as fast as two
// or three, and every part more has to be stored, counted and merged: one sequence of 32 749 tokens, 64 heads over 8,
// takes 33.0 us at one unit per compute unit, 37.6 at three, 44.1 at six (6 us of each an event behind the call).  Beyond
// one, three workgroups are resident per compute unit, so multiples of three (64 sequences of 500 to 2 500 tokens, 32
// heads over 8: 77.6 / 72.8 / 74.9 us at two / three / six); short contexts want few (60 of 60 to 300 tokens, 32 heads, a
// step of 8 layers: 325 us at nine, 379 at fifteen).  The host does not know the lengths, so a table far wider than its
// contexts makes more units than they need, though never a call slower than planned among those tried: 64 sequences of
// 100 to 600 tokens, 32 heads over 8, under 600, 16 384 and 131 072 tokens: 20, 25 and 34 us (planned 53 to 56); 8 of 128 to
// 4 096, a step of 16 layers, under 4 096 and 131 072: 185 and 244 us (planned 281 and 293).
inline int32_t direct_units(int32_t n_cu, int32_t n_kv_heads, int32_t group, int32_t batch, int32_t max_blocks) {
  if (batch < 1 || batch > kDirectSeqs || max_blocks < 1) return 0;
  const int64_t tokens = (int64_t)max_blocks * kBlockTokens, longest = (int64_t)kDirectMaxQuanta * kQuantum;
  const int64_t least = batch * ((tokens + longest - 1) / longest) * n_kv_heads;
  int64_t room = kDirectRows / group;
  if (room > kDirectMaxUnits) room = kDirectMaxUnits;
  if (least > room) return 0;
  for (const int per_cu : {1, 3, 6, 9, 15}) {
    const int64_t units = (int64_t)per_cu * n_cu;
    if (units >= least && units <= room) return (int32_t)units;
  }
  return (int32_t)room;
}
// Whether a call's units do not fit because of the table's width alone.
inline bool direct_too_wide(int32_t n_cu, int32_t n_kv_heads, int32_t group, int32_t batch, int32_t max_blocks) {
  return direct_units(n_cu, n_kv_heads, group, batch, max_blocks) == 0 && direct_units(n_cu, n_kv_heads, group, batch, 1) > 0;
}
// Whether a wave of a cut 16-bit context keeps two blocks in flight, or one.  Where the memory is kept busy anyway more in
// flight is less: reads of 4 KiB tiles alone reach 7.07 / 6.95 / 6.83 TB/s with 32 / 64 / 96 KB of them in flight a compute unit.
// Else a sequence is read as fast as its waves ask.  us with one and with two:
//   64 dims, blocks of half the bytes: 30 sequences of 300 to 3 000 tokens, 32 heads over 8, 37.9 and 29.7; 64 of 2 048 to
//   4 096, 16 over 2, 29.0 and 23.6; one of 16 384, 12 heads, 15.5 and 13.2; 200 of 1 024 to 2 048 155 and 152; 64 of those
//   48.8 and 49.5; one of 32 768, 16 over 2, 12.5 and 13.0.
//   128 dims, up to three workgroups a compute unit: 30 of 300 to 3 000, 32 over 8, 45.4 and 39.2; 8 of 128 to 3 000 12.6 and
//   11.7; 7 of 6 072 to 30 360, 64 over 8, 108.0 and 106.3; 24 of 100 to 1 100, 32 heads, 41.1 and 40.8.  But where a few
//   sequences are cut into sixteen equal parts or more for eight kv heads, whose tiles lie side by side, all compute units are
//   busy alike: one of 32 749, 64 over 8, 24.7 and 25.2; 2 of 20 000, 32 over 8, 27.7 and 28.4 (of four kv heads it is not so:
//   3 of 2 000 to 9 000, 28 over 4, 11.7 and 11.1).  Sequences of one length are as well: 10 of 6 554, 32 over 8, 44.1 and
//   45.4; but the host does not know the lengths, and unequal ones lose more than that.
//   128 dims, more workgroups: 32 of 32 768, 64 over 8, 649 and 654; steps: 16 layers of 256 of 128 to 4 096, 32 over 8, 3 340
//   and 3 368, 32 layers of 8 such 162 and 165.
//   Launches that start from a plan, the largest parts first, do with one where the parts are four a pair or more: monitored
//   steps of 8 of 128 to 4 096, 32 over 8, 32 layers, 357 and 371; not of 32 of 100 to 1 500 (a part each), 8 layers, 211 and
//   194.  With three workgroups a compute unit they do as well with one: layers that move, 24 of 100 to 1 100, 32 heads, 8
//   layers 346 and 345; monitored, 60 of 300 to 2 000, 32 over 8, 8 layers 416 and 421.
inline bool direct_two_blocks(int32_t head_dim, int64_t workgroups, int32_t n_cu, int64_t pairs, int32_t n_kv_heads,
                              bool from_plan) {
  if (head_dim == 64) return true;
  if (from_plan) return workgroups <= n_cu && workgroups < 4 * pairs;
  return workgroups <= 3 * (int64_t)n_cu && !(n_kv_heads >= 8 && workgroups >= 16 * pairs);
}
// Where a step's layers do not share launches: whether one ahead of them works their plan out, or the first layer of each
// staging region leaves it.  That launch costs 4 us; the first layers, for their part, take their items as they come, which is
// longer than largest first where there are more than a workgroup takes at a time.  us by the layers and ahead: layers that
// move, 8 sequences of 128 to 4 096 tokens, 32 heads over 8, 3 / 5 / 8 layers 50 / 59 / 100 and 55 / 63 / 103; 24 of 100 to
// 1 100, 32 heads, 126 / 214 / 347 and 122 / 212 / 347; 256 of the first, 8 layers 1 750 and 1 724.
inline bool direct_plan_ahead(int32_t n_cu, int64_t pairs, int32_t layers) { return layers > 2 && pairs > 2 * (int64_t)n_cu; }
// no more workgroups than the widest context the table can hold makes units
inline int32_t direct_grid(int32_t units, int32_t n_kv_heads, int32_t batch, int32_t max_blocks) {
  const int64_t most = (int64_t)batch * ((max_blocks + kWaves - 1) / kWaves) * n_kv_heads;
  return most < units ? (int32_t)most : units;
}
// Whether contexts are left whole, a workgroup of eight waves to each (sequence, kv head): where the table cannot name more
// than 256 KB of keys and values a kv head.  What a few more passes over blocks cost is less than storing, counting and
// merging parts, up to there.  us a call, cut and whole: 9 sequences, 12 heads of 64, f16, of up to 128 / 300 / 601 / 800 / 1 000
// tokens (256 KB): 6.1 / 6.4 / 6.7 / 7.6 / 7.7 and 4.4 / 4.4 / 4.7 / 5.5 / 5.7; 4 sequences, 32 heads over 8, of up to 128 /
// 256 / 400 / 512 tokens (256 KB): 6.5 / 6.5 / 6.5 / 6.6 and 4.4 / 5.0 / 5.7 / 6.5; one of 700 (358 KB) 6.6 and 8.3; 60 of up
// to 256 11.2 and 8.8, 256 of up to 512 60.7 and 56.6; 110 of up to 300, 32 heads, f16, 58.2 and 55.3.
// A few (sequence, kv head) pairs with 64 dims are cut from 769 tokens on, more than six passes of the eight waves, for which
// that many more compute units make up: 12 pairs of 768 / 896 / 1 024 tokens 6.2 / 6.3 / 6.3 and 6.1 / 6.6 / 7.0, 24 pairs 6.5 /
// 6.4 / 6.5 and 6.1 / 6.6 / 7.0, 32 of 1 024 6.5 and 7.0, 48 7.0 and 7.0, 108 9.6 and 9.4.  The layers of a step count as pairs,
// for they may share a launch: of 1 000 tokens, 12 pairs, 2 / 4 / 8 layers 14.7 / 14.9 / 19.0 and 14.5 / 15.9 / 17.0.
// In steps up to four pairs a compute unit: beyond, their plan with the longest items first is better (8 layers of 30 sequences
// of 60 to 300, 32 heads, 171 and 154; of 120, 32 over 8, 160 and 154; of 190 208 and 227; of 250 288 and 308).
// A rule on the shape alone, the same for every kind of step.  layers: of the step; 0: a call.
constexpr int kWholeWaves = 8;                   // of a workgroup that takes a whole context
constexpr size_t kWholeBytes = (size_t)256 << 10;
inline bool direct_whole(int32_t n_cu, int64_t pairs, int32_t layers, int32_t max_blocks, size_t head_block_bytes) {
  if (max_blocks * head_block_bytes > kWholeBytes) return false;
  if (max_blocks > 6 * kWholeWaves && pairs * (layers > 0 ? layers : 1) * 6 < n_cu) return false;
  return layers == 0 || pairs <= 4 * (int64_t)n_cu;
}
// Whether the layers that share a launch are read four kv heads side by side (k_attn_direct_wide), by workgroups that stay and
// take units of four heads.  With one workgroup a compute unit there have to be several for each, or the last ones to end are
// waited for: nine.  us a launch in k_attn_direct over us side by side, both in turn on one pool, 195 steps drawn over batches of
// 1 to 256, 16 to 8 192 tokens and 2 to 24 layers, by units a compute unit: 3 to 6 0.87 to 1.10, 0.97 in the mean; 6 to 9 0.94 to
// 1.07, 1.00; 9 to 12 1.00 to 1.28, 1.05; 12 and more 0.99 to 1.36, 1.08.  us a step, units in brackets:
//   32 heads over 8, 16 layers of 256 sequences of 128 to 4 096 tokens, 3 414 and 3 153 (36); 16 of 48 such, growing caches, 573
//   and 556 (12); 13 of 30 of 249 to 7 996 694 and 659 (9.8); 8 of 45 of 144 to 723, 64 over 8, 134 and 143 (6); 32 heads over 8,
//   32 of 8 of the first 162.2 and 163.2 (8).
//   32 heads, 16 of 24 of 100 to 1 100 525 and 518 (12); 14 of 9 of 50 to 1 620 224.4 and 221.6 (10.5); 9 of 11 of 255 to 1 276 227
//   and 231 (6.8); 40 heads, 10 of 9 of 413 154 and 161 (7.4); 24 over 12, 3 of 192 of 62 to 313 140 and 146 (6.8).  Many more and
//   short: 40 heads, 12 of 44 of 6 to 33 138 and 105 (20.6).
//   28 over 4, whose blocks are half as large, 8 of 100 of 300 to 3 000, 459 and 470 (6).  64 dims, whose tiles are half as
//   large, so that four waves have too little in flight: 12 heads, 8 of 60 of 200 to 1 800, 248 and 333.
//   Under a table that names far more than the contexts have the units are many and small: 16 of 8 of the first under 131 072
//   tokens 143 and 183.
constexpr int kWideHeads = 4, kPlannedWideHeads = 8;
constexpr int kWideGroup = 8;                    // query heads of a kv head: the LDS holds the states of no more
inline bool direct_wide(int32_t n_cu, int32_t n_kv_heads, int32_t group, int32_t head_dim, int32_t elem_bytes, int32_t layers,
                        int32_t places, int32_t max_blocks) {
  if (elem_bytes != 2 || head_dim != 128 || n_kv_heads % kWideHeads || n_kv_heads < 8 || group > kWideGroup) return false;
  if (max_blocks > 2 * kDirectMaxQuanta * kWaves) return false;
  return layers > 1 && (int64_t)places * (n_kv_heads / kWideHeads) * layers >= 9 * (int64_t)n_cu;
}
// And planned steps: eight heads at a time and three waves a SIMD, of which one finishes.  It takes many units a workgroup to gain
// here too, and those a launch has follow from its layers and from the items, of which the host knows that every sequence makes
// one.  us a step in k_attn_decode_mfma over us side by side, both in turn on one pool (64 sequences of 1 024 to 2 048 tokens, 32
// heads; 26 to 256 of them over other lengths, 8, 16 and 40 heads; 300 over 50 to 700, 32 heads over 8; one rule for f16, bf16
// and grouped queries, which differ by no more than 0.01): launches of 2 layers 0.94 to 0.99, of 3 0.96 to 1.00, 4 and 5 0.98 to
// 1.02, 6 and 8 1.00 to 1.03, 10 to 28 1.00 to 1.05.  The first, 4 / 8 / 16 / 24 layers, 1 048 / 2 116 / 4 147 / 6 042 us and
// 1 046 / 2 080 / 4 052 / 5 864; 12 of 300 of 50 to 700, 32 over 8, bf16, 1 100 and 1 059; 12 of 100 of 100 to 3 000 in
// launches of 2, bf16, 4 540 and 4 657.  Many and short gain most: 10 of 116 of 13 to 66, 40 heads, 631 and 364.  Below four units a
// compute unit by that count, where tables are far wider than contexts, nothing is known.
// A layer a launch it loses: 12 of the first with host blocks 3 122 and 3 430, one of 260 of 1 000 to 3 000, 32 over 8, 332 and 368.
inline bool planned_wide(int32_t n_cu, int32_t n_kv_heads, int32_t group, int32_t head_dim, int32_t layers, int32_t batch) {
  if (head_dim != 128 || n_kv_heads % kPlannedWideHeads || group > kWideGroup / 2) return false;
  return layers >= 6 && (int64_t)batch * (n_kv_heads / kPlannedWideHeads) * layers >= 4 * (int64_t)n_cu;
}
// The LDS of such a workgroup: two halves of the heads' four states, and no less than leaves a compute unit room for one alone (with
// one query head a kv head 21 KB hold the states; two workgroups beside each other would leave another compute unit idle).
inline size_t wide_lds(int32_t heads, int32_t group, int32_t head_dim) {
  const size_t states = (size_t)2 * heads * (2 * kWaves * 16 + kWaves * group * (head_dim + 4)) * sizeof(float);
  const size_t alone = (size_t)81 << 10;
  return states > alone ? states : alone;
}
// Items, partial states and arrival words a pool has room for: as many as its largest batch and widest table can make.
inline size_t direct_pool_items(const pie_config& c) {
  const size_t most = (size_t)kDirectMaxUnits / c.n_kv_heads + 1;
  const size_t pool = (size_t)c.max_batch * (((size_t)c.max_blocks_per_seq + kWaves - 1) / kWaves) + 1;
  return pool < most ? pool : most;
}
inline size_t direct_pool_rows(const pie_config& c) {
  const size_t rows = direct_pool_items(c) * c.n_q_heads;
  return rows < (size_t)kDirectRows ? rows : (size_t)kDirectRows;
}
// and for the layers of a step that share a launch: every layer's, but no more than a 64th of what the caches take or 32 MB
inline size_t direct_step_rows(const pie_config& c) {
  const size_t one = direct_pool_rows(c), all = one * (size_t)c.n_layers;
  const size_t token = (size_t)2 * c.n_kv_heads * c.head_dim * (c.dtype == PIE_DTYPE_F32 ? 4 : 2);
  const size_t share = (size_t)c.n_layers * c.n_gpu_blocks * c.block_tokens * token / 64, least = (size_t)32 << 20;
  const size_t some = (share > least ? share : least) / ((size_t)(c.head_dim + 4) * 4);
  return some <= one ? one : some < all ? some : all;
}
inline size_t direct_pool_words(const pie_config& c) {
  const size_t pairs = (size_t)c.max_batch * c.n_kv_heads;
  return pairs < (size_t)kArriveWords ? pairs : (size_t)kArriveWords;
}
// lines of them: a pair's words of kArriveStride layers share one
inline size_t direct_arrive_lines(const pie_config& c) {
  return direct_pool_words(c) * (((size_t)c.n_layers + kArriveStride - 1) / kArriveStride);
}
// How many layers of a step one launch may take: as many as there is room for parts of, at least one.
inline int32_t direct_step_layers(const pie_config& c, int32_t units, int32_t batch, int32_t max_blocks) {
  const size_t rows = (size_t)(direct_grid(units, c.n_kv_heads, batch, max_blocks) / c.n_kv_heads) * c.n_q_heads;
  const size_t n = direct_step_rows(c) / (rows ? rows : 1);
  return n < 1 ? 1 : n < (size_t)c.n_layers ? (int32_t)n : c.n_layers;
}
// The same for the planned kernels, items of `part` tokens and a workspace of so many floats.
inline int32_t planned_step_layers(const pie_config& c, size_t ws_floats, int32_t part, int32_t batch, int32_t max_blocks) {
  const size_t items = (size_t)batch * (((size_t)max_blocks * kBlockTokens + part - 1) / part);
  if (!items) return 1;
  size_t n = ws_floats / (items * c.n_q_heads * (c.head_dim + 2));
  const size_t units = (size_t)1 << 31;           // (numbered in 32 bits, the grid's tickets beyond the last among them)
  if (n > units / (items * c.n_kv_heads)) n = units / (items * c.n_kv_heads);
  return n < 1 ? 1 : n < (size_t)c.n_layers ? (int32_t)n : c.n_layers;
}

// ---- in the kernel: the split --------------------------------------------------------------------------------
// rcp: the reciprocal of a float, to within one unit in its last place.

// ceil(x / y) for 0 <= x, 1 <= y, x + y < 2^20, exactly: half a unit keeps the quotient off the integers by more than
// the reciprocal's error.
template <class Rcp>
__host__ __device__ inline int32_t div_up(int32_t x, int32_t y, Rcp rcp) {
  return (int32_t)(((float)(x + y - 1) + 0.5f) * rcp((float)y));
}

// quanta of a context, at least one
__host__ __device__ inline int32_t quanta_of(int32_t ctx) { return ctx > 0 ? (ctx + kQuantum - 1) / kQuantum : 1; }

// Quanta per part: within an eighth of the smallest number that keeps the parts of all sequences within max_items.
// total: the quanta of all sequences; items_of(k): the parts they make at k quanta each.
template <class ItemsOf>
__host__ __device__ inline int32_t quanta_per_part(int32_t total, int32_t max_items, ItemsOf items_of) {
  int32_t k = (total + max_items - 1) / max_items;
  while (k < kDirectMaxQuanta && items_of(k) > max_items) k += 1 + k / 8;
  return k < kDirectMaxQuanta ? k : kDirectMaxQuanta;
}

// A sequence of q quanta in parts of at most k, as equal as whole quanta allow: n parts of `each`, the last of what is left.
struct SeqParts { int32_t n, each; };
template <class Rcp>
__host__ __device__ inline SeqParts seq_parts(int32_t q, int32_t k, Rcp rcp) {
  const int32_t each = div_up(q, div_up(q, k, rcp), rcp);
  return {div_up(q, each, rcp), each};
}

}  // namespace pie
