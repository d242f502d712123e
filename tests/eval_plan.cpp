// Checks the blocks of kvp_eval_configs' attention launch over their range: every (cell, stream, segment) is attended over
// by exactly one block, and no block lies beyond the launch.  With "cells streams T pv level .." as arguments: how they are
// arranged.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <random>
#include <set>
#include <vector>

#include "eval_plan.h"

using namespace kvp;

static void check(int cells, int n_streams, const std::vector<int32_t>& level, int32_t T, bool matrix) {
  const int n_levels = (int)level.size(), extra = level.back() < T ? 1 : 0;
  const EvalBlocks p = choose_blocks(cells, n_streams, n_levels, level.data(), T, matrix);
  std::vector<char> seen((size_t)cells * n_streams * (n_levels + 1), 0);
  for (int64_t i = 0; i < p.blocks; ++i) {   // as the kernel finds its work
    int64_t block = i;
    int seg0 = 0, per_cell = p.walk ? n_streams : n_streams * n_levels + extra;
    if (p.grouped)
      for (int k = 0;; ++k) {
        if (k == n_levels + extra) { printf("block beyond the groups\n"); exit(1); }
        seg0 = p.seg_rank[k];
        per_cell = seg0 == n_levels ? 1 : n_streams;
        const int64_t blocks = ceil_div((int64_t)cells * per_cell, kEvalXcds) * kEvalXcds;
        if (block < blocks) break;
        block -= blocks;
      }
    const int64_t items = (int64_t)cells * per_cell, per_xcd = ceil_div(items, kEvalXcds);
    const int64_t w = block % kEvalXcds * per_xcd + block / kEvalXcds;
    if (block / kEvalXcds >= per_xcd || w >= items) continue;
    const int index = (int)(w % per_cell), cell = (int)(w / per_cell);
    int stream = index;
    if (p.grouped) {
      if (seg0 == n_levels) stream = 0;
    } else if (!p.walk) {
      stream = index < extra ? 0 : (index - extra) % n_streams;
      seg0 = index < extra ? n_levels : (index - extra) / n_streams;
    }
    for (int sg = seg0; sg < (!p.walk ? seg0 + 1 : n_levels + (stream == 0 ? extra : 0)); ++sg) {
      char& s = seen[((size_t)cell * n_streams + stream) * (n_levels + 1) + sg];
      if (s) { printf("segment twice\n"); exit(1); }
      s = 1;
    }
  }
  size_t n = 0;
  for (char s : seen) n += s;
  if (n != (size_t)cells * (n_streams * n_levels + extra)) { printf("segments missing\n"); exit(1); }
}

int main(int argc, char** argv) {
  if (argc > 5) {
    std::vector<int32_t> level;
    for (int i = 5; i < argc; ++i) level.push_back(atoi(argv[i]));
    const EvalBlocks p = choose_blocks(atoi(argv[1]), atoi(argv[2]), (int)level.size(), level.data(), atoi(argv[3]), !strcmp(argv[4], "matrix"));
    printf("%s\n", p.walk ? "walk" : p.grouped ? "grouped" : "cell");
    return 0;
  }
  std::mt19937 rng(1);
  int n[3] = {0, 0, 0};
  for (int i = 0; i < 3000; ++i) {
    const int32_t T = 1 + (int32_t)(rng() % (i % 2 ? 3000 : 40));
    std::set<int32_t> level;
    for (int k = 1 + (int)(rng() % 8); k > 0; --k) level.insert(i % 3 ? 1 + (int32_t)(rng() % T) : (int32_t)((int64_t)T * k / 8 + 1 > T ? T : (int64_t)T * k / 8 + 1));
    if (rng() % 2) level.insert(T);
    while (level.size() > 8) level.erase(level.begin());
    const std::vector<int32_t> lv(level.begin(), level.end());
    const int cells = 1 + (int)(rng() % (i % 5 ? 40 : 700)), streams = 1 + (int)(rng() % 10);
    const bool matrix = i / 7 % 2 == 0;
    check(cells, streams, lv, T, matrix);
    const EvalBlocks p = choose_blocks(cells, streams, (int)lv.size(), lv.data(), T, matrix);
    ++n[p.walk ? 0 : p.grouped ? 1 : 2];
  }
  printf("%d %d %d\n", n[0], n[1], n[2]);
  return 0;
}
