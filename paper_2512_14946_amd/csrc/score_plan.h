// How a call of kvp_score_tokens is shared out over the chip, and the scratch memory it needs.  Host arithmetic only, so that
// the arithmetic can be checked without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "kvp_math.h"

namespace kvp {

constexpr int kScoreWaves = 8;                     // waves per block, two per SIMD (256 registers per wave)
constexpr int kUnitTiles = 2;                      // 32-key tiles a wave of the throughput kernel works on at a time
constexpr int kMinChunk = 256, kMaxChunk = 4096;   // keys per block of the chunked kernel
constexpr int kFoldChunks = 16;                    // up to this many key chunks per row pass B combines their statistics itself
constexpr int kCUs = 256;                          // one block of 8 waves each

// How the keys are shared out.
//
// Chunked kernel: blocks of 256 .. 4096 keys of one (layer, head) row, as long as they leave two blocks for every CU: long
// chunks stage the queries less often, short ones fill the chip.
//
// Throughput kernel: 64-key units, 8 waves per block and one block per CU, every block the same number of units through all
// rows.  Faster inside a row, but a block goes through its parts of the rows one after the other, and each of them costs
// staging, references and four barriers, and waits for its last wave; two or three blocks per CU measured 2 and 4 % slower.
// So it needs rows of many units and many units per block, or a chunked kernel whose last round of blocks leaves much of the
// chip idle.  Both were timed over 2800 shapes (rows of 1 .. 2048 units, calls of 512 .. 163840 units, M = 8 .. 512).  Time of
// the throughput kernel over the chunked one:
//   rows of 4, 16, 32, 48, 64, 256 units, 160 units per block: M = 512 1.87, 1.27, 1.09, 0.92, 0.90, 0.80; M = 8 1.51, 1.09,
//     0.94, 0.88, 0.86, 0.92.  The line lies at 48 and 32;
//   rows of 256 units, 32, 48, 64, 96, 160 units per block: M = 128 1.05, 1.00, 0.93, 0.92, 0.86; M = 8, where the keys bound
//     both, 1.17, 1.16, 1.07, 0.96, 0.92, and 1.03 .. 1.05 for rows of 1024 units.  The line lies at 40 and 96;
//   otherwise, with 24 units per block, when the chunked kernel's rounds hold 1.2 times its work (1.6 for rows of 16 .. 31
//     units; 1.1 and 12 units for rows of 1024): 0.68 for rows of 40 units of which a call has 3.2 rounds of blocks, 0.8 at
//     118 units and 3.1 rounds, 0.78 at 1793 units and 3.5 rounds.
// With these lines the kernel taken is 0.6 % slower than the better one on average over 2600 shapes of at least 1500 units,
// and by more than 5 % for 1 in 23 (with the line at 2048 units in the call alone: 13 %, and 2 in 5).
struct ScorePlan {
  int32_t M, nqt, Mrows;
  int32_t chunk_keys;                              // keys per block (chunked kernel)
  bool wide, fold;                                 // wide: throughput kernel
  int64_t units_lh, units_block, units, blocks;    // a unit of the chunked kernel is a whole chunk
  int64_t chunks;                                  // rows of statistics in the scratch memory
  size_t partial_bytes, bytes;
};

inline int32_t score_chunk_keys(int64_t n_lh, int64_t T) {
  int32_t keys = kMaxChunk;
  while (keys > kMinChunk && n_lh * ceil_div(T, keys) < 2 * kCUs) keys /= 2;
  return keys;
}

inline bool score_wide(int64_t n_lh, int64_t T, int32_t M) {
  const int64_t row = ceil_div(T, 32 * kUnitTiles), block = ceil_div(n_lh * row, kCUs);   // units per row, per block
  if (M >= 128 ? row >= 48 && block >= 40 : row >= 32 && row < 1024 && block >= 96) return true;
  if (row < 16 || block < (row < 1024 ? 24 : 12)) return false;
  // the chunked kernel: tiles per wave of a full chunk and of a row's last one, and of all blocks together
  const int64_t keys = score_chunk_keys(n_lh, T), chunks = ceil_div(T, keys);
  const int64_t full = ceil_div(std::min(keys, T), kMinChunk), last = ceil_div(T - (chunks - 1) * keys, kMinChunk);
  const int64_t work = n_lh * ((chunks - 1) * full + last), rounds = ceil_div(n_lh * chunks, kCUs) * kCUs * full;
  return 10 * rounds >= (row >= 1024 ? 11 : row >= 32 ? 12 : 16) * work;
}

// Scratch of a call.  The size is part of the interface (callers keep workspaces, and the 4 MiB of
// kvp_score_tokens_static accept or refuse a shape by it), so it stays that of the chunked kernel and a bias per row; the
// throughput kernel never needs more (tests/score_plan.cpp), and a plan that did would raise it.
inline size_t score_scratch_bytes(int64_t n_lh, int64_t T, int64_t Mrows) {
  const size_t partial = static_cast<size_t>(n_lh) * ceil_div(T, score_chunk_keys(n_lh, T)) * Mrows * 2 * sizeof(float);
  return (partial + 255) / 256 * 256 + static_cast<size_t>(n_lh) * Mrows * sizeof(float);
}

inline ScorePlan make_score_plan(int64_t L, int64_t Hkv, int64_t Hq, int64_t W, int64_t T) {
  ScorePlan p{};
  const int64_t n_lh = L * Hkv;
  p.M = static_cast<int32_t>((Hq / Hkv) * W);
  p.nqt = (p.M + 31) / 32;              // query tiles in use (1 .. 16)
  p.Mrows = p.nqt * 32;
  p.chunk_keys = score_chunk_keys(n_lh, T);
  p.wide = score_wide(n_lh, T, p.M);
  if (p.wide) {
    p.units_lh = ceil_div(T, 32 * kUnitTiles);
    p.units_block = ceil_div(n_lh * p.units_lh, kCUs);
  } else {
    p.units_lh = ceil_div(T, p.chunk_keys);
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
