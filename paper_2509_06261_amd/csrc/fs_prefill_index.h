// Index arithmetic of the prefill kernels' work queue (internal; plain integer functions for host and device: the
// host-compiled check of tests/sanitize/fs_index_check.cpp runs them over whole queues with every result asserted).
#pragma once

#include <cstdint>

#include "fs_attention.h"

namespace fs {

// Which item ticket `ticket` of pool `pool` stands for.  The item list is cut into chunks of 2^shift consecutive
// items, chunk k belongs to XCD k % 8, and the 8 pools of an XCD (pool = 8 s + xcd) take that XCD's items s, s + 8,
// ... in order.  Growing in the ticket for every pool, and every item belongs to exactly one (pool, ticket).
__device__ __host__ inline uint32_t pool_item(uint32_t pool, uint32_t ticket, uint32_t shift) {
  const uint32_t xcd = pool & 7, u = (pool >> 3) + 8 * ticket;  // u: index among the XCD's items
  return ((((u >> shift) << 3) + xcd) << shift) + (u & ((1u << shift) - 1));
}

// item -> (sequence, KV head, tile): sequence-major, then head, tiles of a head longest first.
// tf: [n_seq + 1] first query tile of each sequence; H: KV heads.  False for an item outside every sequence.
__device__ __host__ inline bool decode_item(const uint32_t* tf, int n_seq, uint32_t item, uint32_t H, int& seq, int& head,
                                            int& qt) {
  int lo = 0, hi = n_seq - 1;
  while (lo < hi) {  // last sequence whose first item is <= item
    const int mid = (lo + hi + 1) >> 1;
    if (tf[mid] * H <= item) lo = mid;
    else hi = mid - 1;
  }
  const uint32_t nt = tf[lo + 1] - tf[lo];
  if (nt == 0) return false;  // (cannot happen: an item lies in a sequence that has tiles)
  const uint32_t li = item - tf[lo] * H;
  seq = lo;
  head = (int)(li / nt);
  qt = (int)(nt - 1 - li % nt);
  return true;
}

// The same sequences, but the tiles of all heads together, longest first, heads innermost: with H a multiple or a divisor of 8
// and items dealt to the XCDs in turn a head's tiles still meet on one XCD (two, four, eight for fewer heads).
__device__ __host__ inline bool decode_item_by_tile(const uint32_t* tf, int n_seq, uint32_t item, uint32_t H, int& seq, int& head,
                                                    int& qt) {
  if (!decode_item(tf, n_seq, item, H, seq, head, qt)) return false;
  const uint32_t nt = tf[seq + 1] - tf[seq], li = item - tf[seq] * H;
  head = (int)(li % H);
  qt = (int)(nt - 1 - li / H);
  return true;
}

// ---- Launches whose items are split (see "Split items" in fs_prefill.hip): the items' steps in a row, cut into equal ranges ----
constexpr uint32_t kSplitGroups = 256;  // most workgroups of such a launch
constexpr uint32_t kSplitLeast = 8;     // fewest steps of a range
constexpr uint32_t kItemStart = 2;      // steps that an item's start is worth
constexpr uint32_t kSplitItems = 4;     // most items per compute unit of a launch with split items
// What a step takes where only `live` of a workgroup's `waves` waves (two on each SIMD) have query tokens, in sixths of a step of all.
__device__ __host__ inline uint32_t live_sixths(uint32_t live, uint32_t waves) { return 2 * live <= waves ? 4 : 4 * live <= 3 * waves ? 5 : 6; }
// An item's steps in such time, and the step that place x of them stands for: none of a piece's two or more gets lost.
__device__ __host__ inline uint32_t weighed(uint32_t steps, uint32_t sixths) { return steps - steps * (6 - sixths) / 6; }
__device__ __host__ inline uint32_t step_at(uint32_t x, uint32_t sixths) { return x * 6 / sixths; }
// Place u of an XCD's `per` items when `turns` sequences of per / turns items each are dealt one item from each in turn.
__device__ __host__ inline uint32_t dealt(uint32_t u, uint32_t per, uint32_t turns) { return u % turns * (per / turns) + u / turns; }
// Place i of the plan's order, an XCD's items one after the other (per each): which item of the launch that is.
__device__ __host__ inline uint32_t plan_item(bool by_tile, uint32_t i, uint32_t per, uint32_t turns) {
  const uint32_t x = i / per, u = dealt(i - x * per, per, turns);
  return by_tile ? 8 * u + x : x * per + u;
}
// How many of an XCD's `per` items stand before its u-th one by their steps, most first.
__device__ __host__ inline uint32_t item_rank(const uint32_t* steps, uint32_t per, uint32_t u) {
  const uint32_t mine = steps[u];
  uint32_t rank = 0;
#pragma unroll 8
  for (uint32_t v = 0; v < per; ++v) rank += steps[v] > mine || (steps[v] == mine && v < u);
  return rank;
}
// Whole items, dealt to `slots` workgroups there and back: the place that follows from a workgroup's u-th one (u = its own
// index, then + slots).
__device__ __host__ inline uint32_t snake(uint32_t u, uint32_t slots) {
  const uint32_t round = u / slots, k = u - round * slots;
  return round & 1 ? u - k + (slots - 1 - k) : u;
}
// How many of an XCD's `slots` workgroups come before its k-th one by what they have, least first.
__device__ __host__ inline uint32_t load_rank(const uint32_t* load, uint32_t slots, uint32_t k) {
  const uint32_t mine = load[k];
  uint32_t rank = 0;
#pragma unroll 8
  for (uint32_t i = 0; i < slots; ++i) rank += load[i] < mine || (load[i] == mine && i < k);
  return rank;
}
// The last of n items that begins at or before step p: the one with that step, where p is a step of the launch.
__device__ __host__ inline uint32_t item_of_step(const uint32_t* cum, uint32_t n, uint32_t p) {
  uint32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (cum[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
// Where the range of workgroup k begins.  A cut less than two steps from an end of its item moves there; ranges of
// kSplitLeast steps keep four at least.
__device__ __host__ inline uint32_t plan_cut(const uint32_t* cum, uint32_t n, uint32_t groups, uint32_t k) {
  const uint32_t steps = cum[n], p = (uint32_t)((uint64_t)steps * k / groups);
  if (k == 0 || k >= groups) return p;
  const uint32_t i = item_of_step(cum, n, p);
  return p - cum[i] < kItemStart + 2 ? cum[i] : cum[i + 1] - p < 2 ? cum[i + 1] : p;
}
// The workgroups first .. last with a piece of the item of steps from .. to, of which workgroup `me` has one.
__device__ __host__ inline void piece_owners(const uint32_t* cut, uint32_t me, uint32_t from, uint32_t to, uint32_t& first, uint32_t& last) {
  first = last = me;
  while (cut[first] > from) --first;     // (cut[0] = 0)
  while (cut[last + 1] < to) ++last;     // (the last cut: all steps)
}
// An item's first piece is the last of its workgroup's range, the others are the first of theirs: two places a workgroup.
__device__ __host__ inline uint32_t piece_place(uint32_t first, uint32_t k) { return 2 * (first + k) + (k ? 0 : 1); }

// Runs of 8 token slots streamed per refill of a wave's block-address table (a multiple of 4, about 500 blocks),
// and the table's entries: the blocks such a segment can touch.
__device__ __host__ inline int32_t prefill_seg_runs(int R) {
  const int64_t want = (int64_t)500 * R / 4 * 4;
  return (int32_t)(want < 4 ? 4 : (want > 1024 ? 1024 : want));
}
__device__ __host__ inline int32_t prefill_table_entries(int seg_runs, int R) { return seg_runs / R + 4; }

// ---- Token-addressed walk of the workgroup kernels: 32 consecutive tokens per sub-tile, wherever the blocks end ----
// Tokens streamed per refill of the address table: whole steps of 128, about 500 blocks, at most 8192.  A segment begins
// somewhere in its first block and touches at most seg / T + 2 blocks.
__device__ __host__ inline int32_t prefill_seg_tokens(int T) {
  const int64_t want = (int64_t)500 * T / 128 * 128;
  return (int32_t)(want < 128 ? 128 : (want > 8192 ? 8192 : want));
}
// The next segment's first token; false behind the last one.  (The differences, not the sums, stay below 2^31 in contexts of
// nearly 2^31 tokens, which a table whose entries name one block many times can hold: t0 + seg < len never ended there.)
__device__ __host__ inline bool next_segment(int& t0, int len, int seg) {
  if (len - t0 <= seg) return false;
  t0 += seg;
  return true;
}
// Of the `subs` sub-tiles of 32 tokens from token ts on, those that hold one of the first `end` tokens (none: <= 0), ...
__device__ __host__ inline int live_sub_tiles(int end, int ts, int subs) {
  const int left = end - ts;
  return ((left < 32 * subs ? left : 32 * subs) + 31) >> 5;
}
// ... and whether all of the sub-tile from token tb on lies at or before token `first`.
__device__ __host__ inline bool sub_tile_interior(int tb, int first) { return first - tb >= 31; }
// rel / T for 0 <= rel < T + 8192, rel counted from a block's start.  Below 2^15 tokens a block, ceil(2^32 / T) is off by less
// than T / 2^32, and rel T < 2^32; above, a segment spans two blocks at most.
__device__ __host__ inline uint32_t token_magic(int T) { return T >= 2 && T < (1 << 15) ? (uint32_t)(((1ull << 32) + (uint64_t)T - 1) / (uint64_t)T) : 0u; }
__device__ __host__ inline int block_of(int rel, int T, uint32_t magic) {
  return magic ? (int)(((uint64_t)(uint32_t)rel * magic) >> 32) : (rel >= T ? 1 : 0);
}
// The eight tokens from `run` (a multiple of 8) on of a segment that begins `rel0` tokens into its first block and ends with
// token `last`: the first one is slot `slot` of block k (counted from the segment's first); token i is row r = min(i, most),
// slot + r of block k where r < left, else r - left of block k1.  whole (T and so rel0 multiples of 8): eight slots of block k,
// those past `last` not tokens of the segment; a run past the end is the last one again.
struct RunRows {
  int k, slot, left, most, k1;
};
__device__ __host__ inline RunRows run_rows(int rel0, int last, int T, uint32_t magic, int run, bool whole) {
  const int end = whole ? last & ~7 : last, rel = rel0 + (run < end ? run : end);
  RunRows r;
  r.k = block_of(rel, T, magic);
  r.slot = rel - r.k * T;
  r.left = T - r.slot;
  r.most = last - run > 0 ? last - run : 0;
  const int kl = block_of(rel0 + last, T, magic);
  r.k1 = r.k + 1 < kl ? r.k + 1 : kl;
  return r;
}

}  // namespace fs
