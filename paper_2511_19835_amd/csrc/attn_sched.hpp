// What the attention launch and the small kernels around it share: the shape of the schedule
// (host and device agree on it), the arguments of the dealing and merging kernels, and their launchers.
#pragma once
#include "rsa_common.hpp"

namespace rsa {

// Entries of a video query block's list as every kernel here takes them: the count that
// rsa_select_blocks wrote, held to 1 .. M so that no count, whatever it is, can derail the loops.
__device__ __forceinline__ int list_length(const AttnArgs& a, const Dims& dm, size_t vrow) {
  typedef const int32_t __attribute__((address_space(4))) * const_i32_t;     // scalar loads
  const int c = ((const_i32_t)(uintptr_t)a.count)[vrow];
  return min(max(c, 1), dm.m);
}

// A schedule entry (two int32): the query block, (batch*heads index) * RSA_MAX_BLOCKS + block, and the
// span of its key blocks that the slot walks: first entry | (entries - 1) << 12 | partial << 24. A whole
// row is the span of all its entries; a partial one (a row that several slots share) leaves its
// unnormalised result in a piece buffer, and merge_kernel puts the pieces of the row together.
constexpr int kSpanPartial = 1 << 24;
__host__ __device__ __forceinline__ int make_span(int first, int len, bool partial) {
  return first | (len - 1) << 12 | (partial ? kSpanPartial : 0);
}
__host__ __device__ __forceinline__ int span_first(int span) { return span & 4095; }
__host__ __device__ __forceinline__ int span_len(int span) { return ((span >> 12) & 4095) + 1; }

// Floats of a piece buffer: the accumulators of BLK rows ([wave of 32 rows][eight channels][half of them][row][channel], the order
// in which merge_kernel reads them), then the row sums, then the softmax references (binades).
__host__ __device__ __forceinline__ size_t piece_floats(int d, int blk) { return (size_t)blk * d + 2 * (size_t)blk; }

constexpr int kQueues = 8;                     // one queue of items per XCD
constexpr int kMaxSlots = 128;                 // slots (resident groups of waves) of an XCD: 32 CUs, at most 4 groups each
constexpr int kMaxCross = kQueues - 1;         // dense rows cut over all queues: what is left when they do not divide by 8
constexpr int kMaxTurns = 64;                  // sets of heads that are worked on one after the other
constexpr int kTailDense = 128;                // dense rows of a queue that may be cut (more: dealt whole, ahead of the others)
// Rows are cut only where an uneven last round would cost something: below this many rounds of items. (At 24 rounds
// it took 1.4 % off the layer, with products of 32 x 32 x 16; at 44 the most it could take off is 1.1 % of the attention, for
// 70 MB of buffers.)
constexpr int kSplitRounds = 32;

// Whether the `left` equally long rows of `len` key blocks that a last round has for the slots of a queue are cut when the
// call has no text rows. Cut, the round is over (1 - left / slots) len key blocks earlier. But whole rows walk the keys in step
// and share tiles, also where lists differ; their pieces are spread over the key axis and over CUs that others use,
// and go through fp32 buffers. That costs the time of 9 key blocks of 128, of 15 of 64, 20 at d = 128, where a group asks the
// L2 for the most bytes per product; twice to four times that once more than half of the slots have a row, and too much above
// five eighths (at d = 128 with blocks of 64 above a third).
// The lines were drawn with products of 32 x 32 x 16, from 0.05 to 0.9 of the slots, none to twenty rounds before, 1 to 40 heads,
// lists of a tenth, a fifth and half of the blocks, smooth and random inputs (5600 pairs). With the present ones, lists of half
// the blocks, us, whole and cut, the merging launch included: d = 128, blocks of 128: 12 rows of 17 key blocks for 64 slots 55.7
// and 45.0; 13 of 39 (after a full round) 233 and 188; 20 of 14 (after one) 101.2 and 99.6; 57 of 77 242 and 268. Blocks of 64: 26 rows
// of 104 for 128 slots 172 and 80; 40 of 20 47.8 and 46.2 (left whole); 78 of 105 176 and 192. d = 64: 12 of 17 44.9 and 36.9, blocks
// of 64, 40 of 20 36.8 and 39.0.
struct CutRule {
  int most_left;            // thirty-seconds of the slots
  int least_saved;          // quarters of a key block, up to that many rows
  int least_saved_over;     // ... and for more
};
inline CutRule cut_rule(const Dims& dm) {
  if (dm.blk == 128) return {17, 35, dm.d == 64 ? 68 : 160};
  if (dm.d == 64) return {17, 60, 100};
  return {11, 80, 1 << 20};
}
__host__ __device__ __forceinline__ bool cut_pays(const CutRule& rule, int left, int slots, int len) {
  const int least = 32 * left <= rule.most_left * slots ? rule.least_saved : rule.least_saved_over;
  return 8 * left <= 5 * slots && 4LL * len * (slots - left) >= (long long)least * slots;
}

struct DealArgs {
  int2* table;              // [queues][slots][cap] entries
  int32_t* nitems;          // [queues][slots]
  int32_t* total;           // [queues][slots] key blocks of all entries of the slot
  int32_t* piece0;          // [queues][slots] first piece of the slot
  int2* piece_info;         // [queues][pieces]: query block; pieces of its row if this is the first of them, else 0
  int2* cross;              // [queues][8]: first and last piece of this queue's part of cross row j
  float* pieces;            // [queues][pieces][piece_floats]
  int cap, slots, groups;   // slots = slots per queue, groups = slots per workgroup
  int pieces_per_queue;     // 0: no row is cut
  int heads_at_once;        // heads that the queues work on at the same time
  int most_share;           // what a queue may get of the average load, in 64ths, before the rows are shared out by load
  int rows_per_bh;          // N, or M under RSA_DENSE (every row is then walked whole, no list)
  int n_dense, dense_per_bh, dense_first;      // text query blocks (none under RSA_DENSE)
  int n_cross;              // the last n_cross dense rows are cut over all queues
  int min_piece, switch_cost;                  // shortest piece and what an item costs beside its key blocks, in key blocks
  CutRule rule;
};

// Heads that the eight queues (XCDs) work on at the same time. With one, every queue has an eighth of the rows of each head and
// their lists are spread over all of its key blocks; with eight, whole heads, and four to eight times as many resident rows
// of the same head find each other's tiles in the XCD's L2. Limited by the Infinity Cache (256 MB): the tiles that miss the L2
// should come from there, and the K rows and V^T tiles of all heads at work have to share it. At d = 128 with blocks of 64,
// which ask for the most bytes per product, a little over that still pays.
// Measured, attention in us at sparsity 0.9, one head and as chosen: blocks of 128, 24 heads of 159 blocks 467 and 454, with the
// full mask rule 1454 and 1232; 40 of 591 (39 MB a head) 9549 and 9472 (eight heads: 9599); 24 of 931 (61 MB) 14 460 and 14 400
// (four: 14 560), full rule 21 640 and 21 410. Blocks of 64: 24 of 317 557 and 543, full rule 1795
// and 1292; 24 of 1182 (39 MB) at sparsity 0.7 20 610 and 19 350; 24 of 1857 (61 MB) 17 970 and 16 930 (two: 17 070). d = 64,
// bound by its softmax: 24 of 159 302 and 297, 24 of 591 3619 and 3569, blocks of 64, 24 of 317 356 and 346.
inline int heads_at_once(const Dims& dm) {
  const int bh = dm.batch * dm.heads, least = (bh + kMaxTurns - 1) / kMaxTurns;
  const long long head_bytes = 4LL * dm.t * dm.d, most = (dm.d == 128 && dm.blk == 64 ? 250LL : 200LL) * 1000000;
  int at_once = kQueues;
  while (at_once > 1 && at_once * head_bytes > most) at_once /= 2;
  return at_once > least ? at_once : least;
}

// Sizes of the schedule for `n_wg` resident workgroups of NGRP groups.
struct SchedShape {
  int heads_at_once, most_share, slots, cap, least_cap, n_items;
  int n_dense, dense_per_bh, dense_first, rows_per_bh, n_cross, pieces_per_queue, min_piece, switch_cost;
};
inline SchedShape sched_shape(const Dims& dm, int flags, int n_wg, int ngrp) {
  SchedShape s;
  const bool dense_all = (flags & RSA_DENSE) != 0;
  const int bh = dm.batch * dm.heads;
  s.heads_at_once = heads_at_once(dm);
  // A queue of a sixteenth over the average ends that much later, and still gains where tiles bound the kernel (full mask rule,
  // heads of 5 % more or less key blocks, 24 of 366 blocks: 4386 us by eighths, 4020 by whole heads, 4250 by load); at d = 64 the
  // softmax does (24 of 591: 6200, 6560 and 6190; all with products of 32 x 32 x 16).
  s.most_share = dm.d == 64 ? 65 : 68;
  s.slots = (n_wg / 8) * ngrp;
  s.rows_per_bh = dense_all ? dm.m : dm.n;
  s.dense_per_bh = dense_all ? 0 : dm.mt;
  s.dense_first = dm.n;
  s.n_dense = bh * s.dense_per_bh;
  s.n_items = s.n_dense + bh * s.rows_per_bh;
  // An item costs its key blocks and the switch from one query block to the next: about 15 000 cycles where
  // a block of 128 keys took 6 000 (two steps of both groups) and one of 64 keys 2 600, stamped with products of 32 x 32 x 16 and
  // before the query rows were requested a step ahead. (By the times of lists of 47 to 591 blocks, 24 heads of 931 and of 1182, it
  // is now 1 to 2 blocks of 128 and 6 of 64.) A piece also writes and reads its accumulators in fp32; below a few blocks it is
  // not worth either.
  s.switch_cost = dm.blk == 128 ? 3 : 6;
  s.min_piece = 4;
  const long long longest = (long long)bh * ((s.rows_per_bh + kQueues - 1) / kQueues) + (s.n_dense + kQueues - 1) / kQueues;
  s.cap = (int)(2 * ((longest + s.slots - 1) / s.slots) + 8);      // room for twice the average share of a slot
  s.least_cap = (int)((longest + s.slots - 1) / s.slots) + 1;      // ... for the average one: still enough for all rows, when none is cut
  s.pieces_per_queue = 0;
  s.n_cross = 0;
  // Under RSA_DENSE all rows are equally long and share every tile while they are in step. Cutting the rows of the last
  // round puts them out of step, and their groups on CUs that others use: worth it while few slots would have a row of
  // that round -- fewest at d = 128 with blocks of 64, where a group asks the L2 for the most bytes per product -- and,
  // where it is the only round, while the pieces are long (a slot's share of the key blocks) or very few slots have one.
  // The lines were drawn with products of 32 x 32 x 16, over last rounds of 1/16 to 9/10 of the slots, none to two rounds before, 1 to
  // 24 heads; with the present ones cutting pays further than they go ("left": whole by the rule, though slower). Us, whole and cut:
  // d = 128, blocks of 128: 3 heads of 85 blocks, 31 rows for 64 slots 205 and 169 (left); of 106, 39 rows 255 and 249 (left); 8 of
  // 28, 28 rows 76.4 and 77.3; 24 of 159, 477 rows 3853 and 3723; 24 of 33, 99 rows 193 and 203. Blocks of 64: 3 of 128, 48 rows for
  // 128 slots 184 and 116; of 149, 55 rows 214 and 183 (left); 8 of 160, 160 rows 494 and 379; 24 of 56, 168 rows 186 and 168 (left).
  // d = 64, blocks of 128: 2 of 128, 32 rows 237 and 150; 24 of 33, 99 rows 136 and 133 (left); 24 of 8, 24 rows 26 and 33; blocks of
  // 64: 8 of 64, 64 rows 79 and 65; 24 of 66, 198 rows 157 and 148 (left).
  bool whole = false;
  if (dense_all) {
    const int rows = s.n_items / kQueues, last = rows % s.slots;
    const bool only = rows < s.slots;
    const int most = dm.d == 64 ? 16 : dm.blk == 128 ? 15 : only ? 12 : 8;       // thirty-seconds of the slots
    const long long share = (long long)last * dm.m / s.slots;
    const bool long_pieces = share >= (5 * last <= s.slots ? 3 : 20) || (10 * last <= s.slots && dm.m >= 10);
    whole = 32 * last > most * s.slots || s.n_items % (kQueues * s.slots) == 0 || (only && !long_pieces);
  }
  if (s.n_items <= kSplitRounds * kQueues * s.slots && !whole) {
    if (dm.m >= kQueues * s.min_piece && s.slots >= kQueues) s.n_cross = s.n_dense % kQueues;
    // Every cut makes two pieces (S - 1 cuts), a cross part is a piece by itself; a row of M blocks cannot become more
    // than M / min_piece, and short problems not even that many in all.
    const long long blocks = dm.m < 2 * s.min_piece ? s.n_cross : (longest + s.n_cross) * (dm.m / s.min_piece);
    const long long most = 2LL * s.slots + s.n_cross;
    s.pieces_per_queue = (int)(blocks < most ? blocks : most);
  }
  return s;
}

// Launches, on stream s and in this order, the ranking of the rows (when `sort_rows`: writes a.row_order) and, in
// one launch where both are wanted, the pooled compensation (`compensate`) and the dealing of the schedule
// (`deal`; da filled by the caller).
hipError_t launch_attn_side(const Dims& dm, const AttnArgs& a, const DealArgs& da, bool sort_rows, bool compensate, bool deal,
                            hipStream_t s);
// Puts the pieces of the rows that were cut together (after the attention kernel).
hipError_t launch_attn_merge(const Dims& dm, const AttnArgs& a, const DealArgs& da, hipStream_t s);

}  // namespace rsa
