// Checks the sharing-out of kvp_score_tokens over its range: every key unit belongs to one chunk, every chunk has a row of
// statistics of its own inside the scratch memory, a row combined in the prologue has at most kFoldChunks chunks, and the
// scratch size stays the one callers know.  Prints the number of plans walked and of sizes checked; with a shape as arguments,
// which kernel runs it.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include "score_plan.h"

using namespace kvp;

static void fail(const char* what, int64_t n_lh, int64_t M, int64_t T) {
  printf("%s: %lld rows, M = %lld, T = %lld\n", what, (long long)n_lh, (long long)M, (long long)T);
  exit(1);
}

static ScorePlan plan_of(int64_t n_lh, int64_t M, int64_t T) { return make_score_plan(n_lh, 1, M, 1, T); }   // one window row, M heads

static void check_size(int64_t n_lh, int64_t M, int64_t T) {
  const ScorePlan p = plan_of(n_lh, M, T);
  const size_t bias = p.fold ? 0 : (size_t)n_lh * p.Mrows * sizeof(float);
  if (p.partial_bytes < (size_t)p.chunks * p.Mrows * 8 || p.partial_bytes % 16) fail("statistics region", n_lh, M, T);
  if (p.partial_bytes + bias > p.bytes) fail("plan larger than the scratch size", n_lh, M, T);
  if (p.bytes != score_scratch_bytes(n_lh, T, p.Mrows)) fail("scratch size changed", n_lh, M, T);
}

// The kernels' own walk: block b takes key units [b * units_block, (b + 1) * units_block) of all rows in sequence; its part
// of row lh is a chunk whose statistics are row b (blocks never span rows) or b + lh.
static void walk(int64_t n_lh, int64_t M, int64_t T) {
  const ScorePlan p = plan_of(n_lh, M, T);
  std::vector<char> used(p.chunks, 0);
  std::vector<int64_t> first(n_lh, -1), count(n_lh, 0), units(n_lh, 0);
  for (int64_t b = 0; b < p.blocks; ++b) {
    const int64_t end = std::min(p.units, (b + 1) * p.units_block);
    for (int64_t u = b * p.units_block; u < end;) {
      const int64_t lh = u / p.units_lh, next = std::min(end, (lh + 1) * p.units_lh);
      if (!p.wide && lh != (next - 1) / p.units_lh) fail("block spans rows", n_lh, M, T);
      const int64_t row = p.wide ? b + lh : b;
      if (row < 0 || row >= p.chunks || used[row]) fail("statistics row", n_lh, M, T);
      used[row] = 1;
      if (first[lh] < 0) first[lh] = row;
      if (row != first[lh] + count[lh]) fail("statistics of a row not consecutive", n_lh, M, T);
      ++count[lh];
      units[lh] += next - u;
      u = next;
    }
  }
  for (int64_t lh = 0; lh < n_lh; ++lh) {
    if (units[lh] != p.units_lh) fail("key units of a row", n_lh, M, T);
    // the first and last chunk as the combination finds them
    const int64_t b0 = lh * p.units_lh / p.units_block, b1 = ((lh + 1) * p.units_lh - 1) / p.units_block;
    if (first[lh] != (p.wide ? b0 + lh : b0) || count[lh] != b1 - b0 + 1) fail("chunks of a row", n_lh, M, T);
    if (p.fold && count[lh] > kFoldChunks) fail("too many chunks to combine in the prologue", n_lh, M, T);
  }
}

int main(int argc, char** argv) {
  if (argc == 6) {   // L Hkv Hq W T: 1 when the call runs the throughput kernel
    int64_t v[5];
    for (int i = 0; i < 5; ++i) v[i] = atoll(argv[i + 1]);
    printf("%d\n", make_score_plan(v[0], v[1], v[2], v[3], v[4]).wide ? 1 : 0);
    return 0;
  }
  const int64_t edges[] = {1,   31,  32,   33,   63,   64,   65,   127,  128,  129,  192,  193,   255,   256,   257,    300,   448,
                           511, 512, 513, 700, 1000, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 5000, 8192, 16384, 16385,
                           32768, 65536, 131072, 131073};
  long sizes = 0, walks = 0;
  for (int64_t n = 1; n <= 1100; ++n)
    for (int64_t T : edges) { check_size(n, 32, T); ++sizes; }
  std::mt19937_64 rng(1);
  auto log_int = [&](double lo, double hi) { return (int64_t)exp2(std::uniform_real_distribution<double>(lo, hi)(rng)); };
  for (int i = 0; i < 400000; ++i) {
    check_size(log_int(0, 16), 1 + (int64_t)(rng() % 512), log_int(0, 24));
    ++sizes;
  }
  for (int64_t n : {1, 2, 8, 80, 255, 256, 257, 511, 512, 513, 640, 2048, 2049, 4096, 65535})
    for (int64_t T : edges)
      if (n * T <= (int64_t)1 << 24) { walk(n, 512, T); ++walks; }
  for (int i = 0; i < 2000; ++i) {
    const int64_t n = log_int(0, 13);
    walk(n, 1 + (int64_t)(rng() % 512), log_int(0, 23 - log2((double)n)));
    ++walks;
  }
  printf("%ld %ld\n", walks, sizes);
  return 0;
}
