// How a call of kvp_score_tokens is shared out over the chip, and the scratch memory it needs.  Host arithmetic only, so that
// the arithmetic can be checked without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "kvp_math.h"

namespace kvp {

constexpr int kScoreWaves = 8;                     // waves per block, two per SIMD (256 registers per wave)
constexpr int kUnitTiles = 2;                      // 32-key tiles a wave of a large call works on at a time
constexpr int kSmallChunk = 32 * kScoreWaves;      // keys per block of a small call
constexpr int kFoldChunks = 16;                    // up to this many key chunks per row pass B combines their statistics itself
constexpr int kCUs = 256;                          // one block of 8 waves each

// How the keys are shared out.  Large calls: 64-key units, 8 waves per block and one block per CU of the chip, every
// block the same number of units, so that a block stages the queries of few (layer, head) rows (a chunk costs about 30 us
// besides its keys at M = 512: staging, first loads, waves that wait for the last one; two or three blocks per CU measured
// 2 and 4 % slower).  Small calls, less than one 64-key unit per wave of the chip: 256-key chunks, so that many CUs take
// part (8 heads x 4096 keys, M = 128: 15 us for both passes, 20 us with the kernel of the large calls).
struct ScorePlan {
  int32_t M, nqt, Mrows;
  bool wide, fold;
  int64_t units_lh, units_block, units, blocks;
  int64_t chunks;                                  // rows of statistics in the scratch memory
  size_t partial_bytes, bytes;
};

// Scratch of a call.  The size is part of the interface (callers keep workspaces, and the 4 MiB of
// kvp_score_tokens_static accept or refuse a shape by it), so it stays that of chunks of 256 .. 4096 keys, as few as fill
// the chip twice, and a bias per row; no plan needs more (tests/score_plan.cpp), and one that did would raise it.
inline size_t score_scratch_bytes(int64_t n_lh, int64_t T, int64_t Mrows) {
  int64_t keys = 4096;
  while (keys > 256 && n_lh * ceil_div(T, keys) < 512) keys /= 2;
  const size_t partial = static_cast<size_t>(n_lh) * ceil_div(T, keys) * Mrows * 2 * sizeof(float);
  return (partial + 255) / 256 * 256 + static_cast<size_t>(n_lh) * Mrows * sizeof(float);
}

inline ScorePlan make_score_plan(int64_t L, int64_t Hkv, int64_t Hq, int64_t W, int64_t T) {
  ScorePlan p{};
  const int64_t n_lh = L * Hkv;
  p.M = static_cast<int32_t>((Hq / Hkv) * W);
  p.nqt = (p.M + 31) / 32;              // query tiles in use (1 .. 16)
  p.Mrows = p.nqt * 32;
  p.wide = n_lh * ceil_div(T, 32 * kUnitTiles) >= kCUs * kScoreWaves;
  if (p.wide) {
    p.units_lh = ceil_div(T, 32 * kUnitTiles);
    p.units_block = ceil_div(n_lh * p.units_lh, kCUs);
  } else {
    p.units_lh = ceil_div(T, kSmallChunk);
    p.units_block = 1;
  }
  p.units = n_lh * p.units_lh;
  p.blocks = ceil_div(p.units, p.units_block);
  p.chunks = p.wide ? p.blocks + n_lh - 1 : p.blocks;
  p.fold = (p.units_lh - 1) / p.units_block + (p.wide ? 2 : 1) <= kFoldChunks;      // chunks a (layer, head) row may have
  p.partial_bytes = static_cast<size_t>(p.chunks) * p.Mrows * 2 * sizeof(float);
  p.partial_bytes = (p.partial_bytes + 255) / 256 * 256;
  const size_t need = p.partial_bytes + (p.fold ? 0 : static_cast<size_t>(n_lh) * p.Mrows * sizeof(float));
  p.bytes = std::max(score_scratch_bytes(n_lh, T, p.Mrows), need);
  return p;
}

}  // namespace kvp
