// Host arithmetic that lays a call's work out over workgroups, from the bounds
// the caller gives. Plain integers and doubles without HIP, so that it can be
// compiled and tested alone. Bounds may lie anywhere in the int32 range, so
// block counts are taken in 64 bits.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace bros {

// Blocks of the longest context a call can meet: its bound in tokens, and what a table row holds.
inline int32_t longest_blocks(int32_t max_ctx, int32_t max_blocks_per_seq) {
  const int64_t blocks = ((int64_t)max_ctx + 15) / 16;
  return (int32_t)std::max<int64_t>(1, std::min<int64_t>(blocks, max_blocks_per_seq));
}

// Blocks of a work item of the fp32 decode. The workspace is laid out for splits
// of `plan_blocks` blocks (4 to 64, chosen by the rows alone); KV heads make items
// too, and an item costs its start-up and a partial, so an item may take several
// of these splits. The usual size leaves two items per compute unit, up to 32
// blocks, and contexts of up to 20 blocks whole; another of kSizes is taken where
// it is expected to be a tenth faster.
//
// Expected time, in units of about a microsecond: a stream of an item (four per
// workgroup, two with 8 heads per KV head) takes 1.15 for a block, 0.35 more per
// head of its wave (0.8 of that with two streams), and 0.4 of that again for each
// further item on a compute unit; an item's start-up 1.7. Items beyond the resident ones wait for a free
// workgroup. What is known is the longest context alone: equal contexts count by
// 0.17, for which the items run in whole rounds, and contexts of 0.63 of the longest on average
// by 0.83, where the last of them end with up to 0.45 of an item's time alone. A call with
// splits also pays the merge, 4.2 and 0.9 per split. Steps of few rows wait for
// their host calls instead, 11.5 and for the merge's launch 3 more: 0.6 of what a
// call is below that counts too (5 rows of 93 to 301 tokens, 32 / 8 heads: a step
// of 16.2 us whole, 19.4 split).
//
// Measured on 3168 calls of 1 to 256 rows with contexts up to 40 to 2048 tokens
// (equal, within a quarter of the longest, uniform from 2/5 or 1/8 of it,
// lognormal; 64 / 8, 32 / 8, 16 / 8, 8 / 8 and 8 / 1 heads), each at all these
// sizes: 2 % above the best size of each call on average, the usual size alone 5 %,
// the plan's own splits 12 %; against the usual size 25 calls lose 5 to 19 % (lognormal
// contexts mostly). Us, the plan's own / the usual / this: 64 rows of 40 to 320
// tokens (32 / 8 heads) 33.7 / 22.4 / 22.5, one row of 320 with 8 / 1 heads 12.5 / 16.8 /
// 12.5. (Taking the size with the least expected time for contexts of 0.66 of the
// longest gains as much on average, and loses 5 to 57 % in 237 calls: 16 rows of 2048 tokens, 64 / 8
// heads, 49.5 / 69.8.)
inline int32_t f32_item_blocks(int64_t rows, int32_t num_kv_heads, int32_t group, int32_t longest, int32_t plan_blocks,
                               int32_t resident, int32_t compute_units) {
  constexpr int32_t kSizes[] = {4, 8, 12, 16, 20, 24, 32, 48, 64};
  const int32_t streams = group > 4 ? 2 : 4;
  const double block_us = (1.15 + 0.35 * std::min(group, 4)) * (group > 4 ? 0.8 : 1.0);
  const double segments = (double)rows * num_kv_heads;
  const double most = (double)resident / compute_units;   // items of a compute unit at once
  const auto expected_us = [&](int32_t per) {
    const double splits = (longest + per - 1) / per;
    const double steps = (std::min(per, longest) + streams - 1) / streams;   // blocks of a stream
    const auto item_us = [&](double items, double blocks) {
      return 1.7 + blocks * block_us * (1.0 + 0.4 * (std::min(std::max(items / compute_units, 1.0), most) - 1.0));
    };
    const double all = segments * splits;
    const double some = splits > 1.0 ? segments * std::min(0.63 * splits + 0.5, splits) : segments;
    double us = item_us(some, steps);
    if (some > resident) {
      const double mean = 0.63 * longest / streams * segments / some;
      us = item_us(some, std::min(steps, mean)) * some / resident + 0.45 * us;
    }
    us = 0.17 * std::max(1.0, std::ceil(all / resident)) * item_us(all, steps) + 0.83 * us;
    if (splits > 1.0) us += 4.2 + 0.9 * splits;
    return us + 0.6 * std::max(0.0, 11.5 + (splits > 1.0 ? 3.0 : 0.0) - us);
  };
  const int64_t want = std::max<int64_t>(1, (int64_t)std::ceil(2.0 * compute_units / segments));   // splits of the longest
  const int32_t usual = longest <= 20 ? longest : (int32_t)std::min<int64_t>((longest + want - 1) / want, 32);
  int32_t base = 0, chosen = 0;
  double best = 0.0, base_us = 0.0;
  for (const int32_t per : kSizes) {
    if (per % plan_blocks != 0) continue;
    const double us = expected_us(per);
    if (base == 0 || base < usual) {
      base = per;
      base_us = us;
    }
    if (chosen == 0 || us < best) {
      chosen = per;
      best = us;
    }
    if (per >= longest) break;
  }
  return best < 0.9 * base_us ? chosen : base;
}

// The fp32 prefill's units (`positions` positions of one chunk and KV head each)
// and how far their blocks are split over workgroups.
struct F32ChunkPlan {
  int64_t units;           // workgroups per split, all KV heads
  int32_t tiles_per_seq;   // ranks of every sequence (0: ranks by rows)
  int32_t split_blocks;
  int32_t splits;
};

// Chunks of about one length are ranked longest tile first, every sequence with
// the ranks of the longest: its bound, and no more than all the rows. Where that
// gives more than twice the ranks the rows can need (one long chunk among short
// ones), they are counted from the rows instead. One chunk of 1024 rows and 255 of
// one on 300 tokens (32 / 8 heads): 966 us, by rows 291.
//
// Units are split over their blocks while those that the rows can need leave room,
// two workgroups per compute unit, in multiples of the plan's split, whose count the
// workspace is sized for: the count with the least expected time. A block takes a
// wave 2.75 us, and 1.4 times that beside a second workgroup, since the fp32 matrix
// instructions bound it; a unit's start takes as long as 3.3 of them, a merge 5 and
// 0.6 per split. Fitted to 550 calls of 1 to 1100 rows on 0 to 4000 cached tokens,
// each at four split sizes: 0.2 % above the best of them on average, with a split more
// only where it is 2 % faster (64 rows on 600 tokens, 32 / 8 heads: two splits 19.5 us,
// four, expected to be level, 22.7). Us, split down
// to 16 blocks / to 8 / this: one row on 300 tokens (8 / 8 heads) 12.5 / 11.5 / 10.3,
// 256 rows without cached tokens (16 / 8) 12.8 / 18.8 / 12.8.
inline F32ChunkPlan plan_f32_chunks(int32_t num_rows, int32_t num_seqs, int32_t max_q_len, int32_t num_kv_heads,
                                    int32_t positions, int32_t longest, int32_t plan_blocks, int32_t compute_units) {
  const int64_t tiles = ((int64_t)std::min(max_q_len, num_rows) + positions - 1) / positions;
  const int64_t by_rows = (int64_t)num_rows / positions + num_seqs;
  F32ChunkPlan p;
  const bool compact = num_seqs * tiles > 2 * by_rows;
  p.tiles_per_seq = compact ? 0 : (int32_t)tiles;
  p.units = (compact ? by_rows : num_seqs * tiles) * num_kv_heads;
  const int64_t live = std::min(num_seqs * tiles, by_rows) * num_kv_heads;
  double best = 0.0;
  p.split_blocks = 0;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(2 * compute_units / live, longest / 4));
  for (int64_t want = 1; want <= most; ++want) {
    const int64_t per = ((longest + want - 1) / want + plan_blocks - 1) / plan_blocks * plan_blocks;
    const int64_t splits = (longest + per - 1) / per;
    const double steps = (double)((std::min<int64_t>(per, longest) + 3) / 4);   // blocks of a wave
    double us = (steps + 3.3) * 2.75 * (live * splits > compute_units ? 1.4 : 1.0);
    if (splits > 1) us += 5.0 + 0.6 * (double)splits;
    if (want > 1 && us >= 0.98 * best) continue;
    best = us;
    p.split_blocks = (int32_t)per;
    p.splits = (int32_t)splits;
  }
  return p;
}

// What longest_whole (below) never falls short of.
constexpr int32_t kWholeOnAnyShare = 32;

// Longest context, in blocks, that the bf16 decode gives whole to one workgroup per
// (row, KV head) segment, by the segments per compute unit. With few of them,
// pieces spread a context over more compute units. They are up to 2 us shorter from
// 24 blocks on, but a step of few rows waits for its host calls, of which the
// merge's launch takes 3 us (12 rows of 108 to 408 tokens, 64 / 8 heads: a step of
// 16.8 us whole, 19.5 in pieces). From two segments per compute unit on, a few long
// contexts among short ones are waited for, and the even split's partials, which
// whole segments save, are the smaller the fewer heads share a segment.
inline int32_t longest_whole(int64_t segments, int32_t group, int32_t compute_units) {
  const int64_t cus = compute_units;
  if (segments < cus / 4) return kWholeOnAnyShare;
  if (segments < cus / 2) return 56;
  if (segments < 2 * cus || group >= 8) return 64;
  if (group >= 4) return 48;
  return segments < 4 * cus ? 40 : kWholeOnAnyShare;
}

// Whether plan_short_decode (below) gives whole segments however many compute units there are.
inline bool whole_on_any_share(int64_t segments, int64_t blocks) { return segments <= 0x7fffffff && blocks <= kWholeOnAnyShare; }

// Whether the bf16 decode runs whole segments or pieces of `split_blocks` blocks
// (decode_short.hip), or else the even split (decode.hip).
//
// Pieces take the shortest size of which a context has no more than a few (a
// workgroup folds them, eight a round) and the call no more than one per compute
// unit, or two of 32 or 64 blocks; with more of them the even split's longer walks read the
// HBM better. Pieces of 64 blocks are long enough that a long context among shorter ones
// sets the end (12 rows of lognormal contexts up to 4000 tokens, 16 / 8 heads: 34 us, even
// split 29), and gain more where contexts are alike (8 rows of 8000: 44 us, even split 51).
//
// Device time over 2502 calls of 1 to 512 rows of up to 64 to 16000 tokens (equal,
// uniform and lognormal contexts; 64 / 8, 32 / 8, 16 / 8, 8 / 8 and 8 / 1 heads)
// on 256 compute units: 4 % above the best of the even split, whole segments and
// seven piece sizes for each call, the even split 42 %; without the pieces of 8 blocks
// 6 %. In 35 calls the even split is faster by more than 5 %, lognormal contexts
// mostly. Calls in us, the even split / this (32 / 8 heads unless said):
//   whole   16 rows of 64 to 256 tokens 13.2 / 7.3, 64 of 128 to 512 25.8 / 20.0, 512 of 8
//           to 64 29.1 / 26.0 (but 512 of 64 each 30.1 / 32.6: what is known here is the
//           longest)
//   pieces  one row of 8000 22.7 / 11.7, six of 90 to 2048 17.4 / 13.0
// On a part of the chip the limits scale: four rows of 1024 to 4096 tokens on 64
// compute units take 26 us in the even split, 34 with the whole chip's limits.
inline bool plan_short_decode(int64_t segments, int32_t group, int64_t blocks, int32_t compute_units, int64_t slots,
                              int32_t* split_blocks, int32_t* n_split) {
  struct Pieces {
    int32_t blocks, per_cu, splits;   // size; pieces per compute unit and of a context, at most
  };
  constexpr Pieces kPieces[] = {{8, 1, 24}, {16, 1, 64}, {32, 2, 64}, {64, 2, 64}};
  if (segments > 0x7fffffff) return false;
  if (blocks <= longest_whole(segments, group, compute_units)) {
    *split_blocks = (int32_t)blocks;
    *n_split = 1;
    return true;
  }
  for (const Pieces& p : kPieces) {
    const int64_t splits = (blocks + p.blocks - 1) / p.blocks;
    if (splits < 2 || splits > p.splits || segments * splits > (int64_t)p.per_cu * compute_units) continue;
    if (segments * splits * group > slots) continue;   // (partials)
    *split_blocks = p.blocks;
    *n_split = (int32_t)splits;
    return true;
  }
  return false;
}

}  // namespace bros
