// Which blocks the attention launch of kvp_eval_configs has.  Host arithmetic only, so that it can be checked without a GPU.
#pragma once

#include <stdint.h>

#include "kvp_math.h"

namespace kvp {

constexpr int kEvalMaxLevels = 8;
constexpr int kEvalXcds = 8;
constexpr int kEvalSlots = 512;   // blocks the chip holds

inline int64_t padded_items(int64_t items) { return ceil_div(items, kEvalXcds) * kEvalXcds; }

// A stream's tokens, in keep-level order, fall into segments: segment j ends at the j-th keep level, and one more, walked by
// the reference only, holds the tokens no level keeps.  A cell is a (layer, kv head, 128 rows).  (cells x streams below, T
// tokens, levels at equal distances unless said.)
//   by cell: a block per segment, all segments and streams of a cell in a row.  With a block per stream, a context of 8
//     layers x 4 kv heads (224 rows, ten streams, T = 5003) is 640 blocks, one and a quarter times what fits (matrix-core
//     P.V: 1.03 ms, 0.79 by segment);
//   grouped: a block per segment, by segment, the longest first, when their lengths differ by more than a quarter and there are
//     more blocks than CUs: with long and short blocks mixed the last ones run alone (256 x 2, T = 8192, levels at 0.3 and
//     1.0: 3.06 ms mixed, 2.32 grouped, a block per stream 2.49; 100 x 2, T = 3001, 400 blocks: 0.58 and 0.46).  With a CU for
//     each, the streams of a segment find its rows in the cache of their XCD only by cell (2 x 4, T = 10666: 1.25 ms, 1.34
//     grouped);
//   walk: a block takes all segments of its stream, one after the other, and what it has seen at the end of each is the
//     output of that level.  Only in the matrix-core form, whose blocks are the shortest, where segments are short, so that
//     the first loads and last stores of a block count, and streams fill the chip: segments of up to 512 tokens and 1.05 times
//     the work in whole rounds of blocks, 256 tokens and 1.2 times (256 x 10: T = 300 0.56 ms against 0.59 by cell, 1000 0.89
//     / 0.94, 2048 1.46 / 1.50, 3000 2.01 / 2.04; 320 x 10, 1.12 times: 300 0.72 / 0.76, 1000 1.15 / 1.19, 3000 2.38 / 2.35).
//     With tokens that no level keeps the reference alone would walk on: then only for one level, if nothing but the
//     reference's second segments does not fit (128 x 4, half of 2048 tokens kept: 0.225 ms, 0.256 by cell).  The default
//     form gains 2 % at most from it, and its probabilities, 16 bits relative to the largest of a block's tokens, lose a
//     little (T = 300: error of the losses 4.4e-7 -> 5.5e-7).
struct EvalBlocks {
  bool walk, grouped;
  uint8_t seg_rank[kEvalMaxLevels + 1];   // grouped: the segments by length, longest first
  int64_t blocks;
};

inline EvalBlocks choose_blocks(int64_t cells, int n_streams, int n_levels, const int32_t* level_k, int32_t T, bool matrix) {
  EvalBlocks b{};
  const int32_t top = level_k[n_levels - 1];
  const int extra = top < T ? 1 : 0, n_segs = n_levels + extra;
  const int64_t streams = cells * n_streams, rounds = ceil_div(streams, kEvalSlots) * kEvalSlots;
  const int64_t limit = 20 * rounds <= 21 * streams ? 512 : 5 * rounds <= 6 * streams ? 256 : 0;
  b.walk = matrix && (extra ? n_levels == 1 && streams <= kEvalSlots && streams + cells > kEvalSlots
                            : streams >= 2 * kEvalSlots && top <= limit * n_levels);
  if (b.walk) {
    b.blocks = padded_items(streams);
    return b;
  }
  auto length = [&](int sg) { return (sg < n_levels ? level_k[sg] : T) - (sg > 0 ? level_k[sg - 1] : 0); };
  for (int i = 0; i < n_segs; ++i) {      // insertion sort; equal lengths stay in order
    int j = i;
    for (; j > 0 && length(b.seg_rank[j - 1]) < length(i); --j) b.seg_rank[j] = b.seg_rank[j - 1];
    b.seg_rank[j] = static_cast<uint8_t>(i);
  }
  b.blocks = padded_items(streams * n_levels + extra * cells);
  b.grouped = b.blocks > kEvalSlots / 2 && 4ll * length(b.seg_rank[0]) > 5ll * length(b.seg_rank[n_segs - 1]);
  if (b.grouped) {
    b.blocks = 0;
    for (int i = 0; i < n_segs; ++i) b.blocks += padded_items(i == n_levels ? cells : streams);
  }
  return b;
}

}  // namespace kvp
