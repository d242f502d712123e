// kvp_score_tokens: attention-score token importance (the paper's snapkv baseline: cross attention
// between the tokens near the query and the earlier context; Evaluation, Baselines).
//
//   scores[l][h][t] = sum over the G*W window rows r of softmax_t(q_r . k_t / sqrt(D))
//
// Two passes over K, both with the query-window x key contraction on the bf16 MFMA
// (v_mfma_f32_32x32x16_bf16, fp32 accumulate), because a softmax row must be normalized before it
// can be summed into a column:
//   pass A  row statistics: a reference exponent and the sum of exponentials per window row, per key chunk;
//   combine per-row bias b_r = max_r + log2(sum_r) over all chunks (a tiny kernel, or the prologue of pass B
//           when there are few chunks);
//   pass B  column sums: scores[t] = sum_r 2^(s_rt - b_r).
// Logits are kept in the base-2 domain (s = q.k * log2(e)/sqrt(D)) so the exponential is one
// v_exp_f32.
//
// The MFMA operand layout is the same for A and B (lane = row or column index mod 32, 8 consecutive channels per lane,
// lanes 32..63 take the upper 8 of each 16-channel step), so the same registers serve both orientations:
//   pass A computes S^T = K Q^T: a lane holds one query column and 16 keys, so the sum of a row is lane-private;
//   pass B computes S = Q K^T: a lane holds one key column and 16 rows, so the column sum of a key
//          is lane-private adds plus one exchange between half-waves, and is complete inside the wave.
// The window queries (at most 512 rows) are staged in LDS (row pitch 272 B so that the 16-byte operand reads of 8 lanes
// cover all 32 banks); keys go from global memory straight into MFMA operand registers.  Every key is owned by exactly one
// wave and every sum is formed in a fixed order: deterministic output.
//
// What bounds it (throughput kernel): the issue of matrix and vector instructions together, at the 1.9-2.0 GHz the chip holds
// under this load.  A product of 32x32x16 takes 32 cycles of the matrix pipe; the six vector instructions that go with
// it (two logits, two exponentials of 8 cycles, two sums) take 32 cycles, and 42 together measured in isolation with two
// waves per SIMD; 65 in the kernel.  Hence (80 x 8 x 16384 keys, 512 rows: 3.23 -> 2.76 ms; 28 x 4 x 131072, 224 rows:
// 2.36 -> 1.97 ms):
//   - 64 keys per wave: a query operand read from LDS serves two products;
//   - the products of one tile are interleaved with the vector instructions of the tile before in program order, across
//     query tiles and key units, so that both pipes have work whatever the other wave of the SIMD does;
//   - no running maximum in pass A (see there): 3 vector instructions per logit in both passes;
//   - the keys of the next unit (64 keys x 256 B per wave) are requested a whole unit ahead into registers of their own;
//     with one tile ahead the loads of 128K-token rows cost 25 % of the time;
//   - every block works through an equal share of the whole call, so that queries are staged once per (layer, head) row
//     and block: with 4096-key blocks the launches of 10 blocks per CU cost 30 us each.

#include <mutex>
#include <type_traits>

#include "kvp_internal.h"
#include "score_plan.h"

namespace kvp {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float floatx16;

constexpr int kWaves = kScoreWaves;
constexpr int kThreads = kWaves * kWave;
constexpr int kPitch = 136;                        // bf16 elements per LDS row (272 B)
constexpr int kMaxRows = 512;                      // G*W limit (16 query tiles)
constexpr float kLog2e = 1.4426950408889634f;

struct ScoreArgs {
  const uint16_t* q;
  int64_t q_sl, q_st, q_sh;
  const uint16_t* k;
  int64_t k_sl, k_st, k_sh;
  int32_t T, W, G, Hkv, M, Mrows, nqt;      // nqt = query tiles in use (1 .. 16); Mrows = 32 * nqt
  FastDiv div_w;                            // row r of the window queries: query head r / W, window offset r mod W
  uint32_t units_lh, units_block, units;    // key units per (layer, head), per block, in all
  FastDiv div_lh, div_block;                // by units_lh, by units_block
  int32_t chunk_keys;                       // keys per block of the chunked kernel, a multiple of 32 * kWaves
  int32_t compact_rows;                     // blocks never span two (layer, head) rows: their statistics are numbered by block
  int32_t causal, force_window;
  int32_t fold_combine;                     // pass B combines the chunk statistics itself (few chunks: saves a launch)
  float scale2;                             // log2(e) / sqrt(D)
  float2* partial;                          // [chunk][Mrows] (reference, sum) in the base-2 domain, chunks numbered by chunk_row
  float* bias;                              // [L*Hkv][Mrows]
  float* scores;                            // [L*Hkv][T]
};

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  union { uint4 u; bf16x8 b; } c;
  c.u = v;
  return c.b;
}

// row index inside a 32x32 accumulator tile held by vgpr v of this lane
__device__ __forceinline__ int acc_row(int lane, int v) { return (lane >> 5) * 4 + (v >> 2) * 8 + (v & 3); }

// A block owns units_block consecutive key units of the sequence of all (layer, head) rows.  The part of it inside one
// row is a chunk: block b's chunk of row lh keeps its statistics in this row of `partial` (b + lh grows with every chunk).
__device__ __forceinline__ int64_t chunk_row(const ScoreArgs& a, uint32_t b, uint32_t lh) { return a.compact_rows ? b : b + lh; }

// max + log2(sum) over the statistics of n chunks (uniform), a row of them every Mrows.
// FEW: n is at most kFoldChunks, the statistics in flight at once (one memory latency instead of one per chunk).
template <bool FEW>
__device__ __forceinline__ float combined_chunks(const float2* part, int n, int Mrows) {
  float m = -INFINITY, z = 0.0f;
  for (int c = 0; c < (FEW ? 1 : n); c += kFoldChunks) {
    float2 p[kFoldChunks];
#pragma unroll
    for (int i = 0; i < kFoldChunks; ++i)   // n is uniform: no lane masks, and no loads beyond the last chunk
      p[i] = c + i < n ? part[static_cast<int64_t>(c + i) * Mrows] : make_float2(-INFINITY, 0.0f);
    float m_new = m;
#pragma unroll
    for (int i = 0; i < kFoldChunks; ++i) m_new = fmaxf(m_new, p[i].x);
    if (!FEW) {
      if (m_new == -INFINITY) continue;
      z *= __builtin_amdgcn_exp2f(m - m_new);
    }
#pragma unroll
    for (int i = 0; i < kFoldChunks; ++i) z += p[i].y * __builtin_amdgcn_exp2f(p[i].x - m_new);
    m = m_new;
  }
  // v_log_f32 is log2; its error is smallest below 1
  return m + static_cast<float>(__builtin_amdgcn_frexp_expf(z)) + __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(z));
}
// bias of row r of (layer, head) lh over all its key chunks; +inf for padding rows (they then contribute 0)
template <bool FEW>
__device__ __forceinline__ float combined_bias(const ScoreArgs& a, int lh, int r) {
  if (r >= a.M) return INFINITY;
  const uint32_t b0 = __builtin_amdgcn_readfirstlane(a.div_block.quot(lh * a.units_lh));   // lh is uniform
  const int n = __builtin_amdgcn_readfirstlane(a.div_block.quot((lh + 1) * a.units_lh - 1)) - b0 + 1;
  return combined_chunks<FEW>(a.partial + chunk_row(a, b0, lh) * a.Mrows + r, n, a.Mrows);
}

template <int NQT, bool PASS_B>
__global__ __launch_bounds__(kThreads, 2) void score_kernel(const ScoreArgs a) {
  constexpr int KT = kUnitTiles;
  __shared__ __attribute__((aligned(16))) uint16_t q_s[NQT * 32 * kPitch];
  // pass A: reference exponent of every query row; pass B: its bias
  __shared__ __attribute__((aligned(16))) float row_s[NQT * 32];
  __shared__ __attribute__((aligned(16))) int32_t wpos_s[NQT * 32];   // window offset r mod W of query row r (masked tiles)
  __shared__ __attribute__((aligned(16))) float sum_s[PASS_B ? 4 : kWaves * NQT * 32];   // pass A: sums per wave and row
  __shared__ float2 merge_s[PASS_B ? 1 : kWaves * 32];
  __shared__ int32_t ticket_s;   // pass B: next key unit of the chunk that no wave has taken

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: the loops over units are scalar
  const int win0 = a.T - a.W;  // first window position
  const int nqt = a.nqt, last = nqt - 1;
  constexpr int kUnit = 32 * KT;                    // keys a wave works on at a time
  constexpr int kUnitStride = kUnit * kWaves;

  const uint32_t u_end = min(a.units, (blockIdx.x + 1) * a.units_block);
  for (uint32_t u = blockIdx.x * a.units_block; u < u_end;) {   // one chunk: this block's part of one (layer, head) row
  const int lh = __builtin_amdgcn_readfirstlane(a.div_lh.quot(u));
  const uint32_t u_lh = lh * a.units_lh;
  const int chunk0 = static_cast<int>(u - u_lh) * kUnit;                                             // this chunk's keys
  const int t_end = min(a.T, static_cast<int>(min(u_end - u_lh, a.units_lh)) * kUnit);
  u = u_lh + a.units_lh;
  const int l = lh / a.Hkv, h = lh - l * a.Hkv;
  const uint16_t* kbase = a.k + static_cast<int64_t>(l) * a.k_sl + static_cast<int64_t>(h) * a.k_sh;
  const int t_begin = chunk0 + wave * kUnit;
  uint4 kop_a[KT][8], kop_b[KT][8];   // the unit at work and the one after it
  // A 32-key tile at tk as MFMA operand: lane = key tk + lane%32, out[ks] = channels 16 ks + 8 (lane/32) .. +7.  Keys beyond
  // the row repeat its last one (and are masked).
  auto load_tile = [&](uint4 (&out)[8], int tk) {
    const int t0 = min(tk, a.T - 1);
    const uint16_t* row = kbase + t0 * a.k_st + min(lane & 31, a.T - 1 - t0) * a.k_st + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = *reinterpret_cast<const uint4*>(row + ks * 16);
  };
  // this wave's first key unit is requested before anything else, so that its latency overlaps the prologue
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) load_tile(kop_a[kt], t_begin + 32 * kt);

  // ---- stage the window queries of this (layer, kv head): row r = u * W + w, zeros beyond M.  A thread's
  //      (at most NQT) pieces are all requested before the first one is stored ----
  {
    constexpr int kRowsAtOnce = kThreads / 16, kPieces = NQT * 32 / kRowsAtOnce;
    const int part = threadIdx.x & 15;
    int r0 = threadIdx.x >> 4;
    asm volatile("" : "+v"(r0));   // the row offsets are computed here for every chunk, not kept in registers across them
    const uint16_t* qbase = a.q + static_cast<int64_t>(l) * a.q_sl + static_cast<int64_t>(h) * a.G * a.q_sh + part * 8;
    uint4 piece[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int r = min(r0 + kRowsAtOnce * i, a.M - 1);
      const int g = a.div_w.quot(r), w = r - g * a.W;
      piece[i] = *reinterpret_cast<const uint4*>(qbase + w * a.q_st + g * a.q_sh);
    }
    __syncthreads();   // the previous chunk's queries and sums are no longer read
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
      const int r = r0 + kRowsAtOnce * i;
      if (r >= a.M) piece[i] = make_uint4(0, 0, 0, 0);
      if (r < a.Mrows) *reinterpret_cast<uint4*>(q_s + r * kPitch + part * 8) = piece[i];
    }
  }
  for (int r = threadIdx.x; r < a.Mrows; r += kThreads) {
    wpos_s[r] = r - static_cast<int>(a.div_w.quot(r)) * a.W;
    // rows beyond M carry +inf: they contribute 2^-inf = 0
    if constexpr (PASS_B) row_s[r] = a.fold_combine ? combined_bias<true>(a, lh, r) : a.bias[static_cast<int64_t>(lh) * a.Mrows + r];
  }
  if (PASS_B && threadIdx.x == 0) ticket_s = 2 * kWaves;
  if constexpr (!PASS_B) {
    for (int i = threadIdx.x; i < kWaves * a.Mrows; i += kThreads) sum_s[i] = 0.0f;
  }
  __syncthreads();

  // the logit scale in a vector register: with a scalar operand the multiply-adds would issue at half their rate
  float scale2;
  asm("v_mov_b32 %0, %1" : "=v"(scale2) : "s"(a.scale2));

  auto q_piece = [&](int qt, int ks) {
    return as_bf16x8(*reinterpret_cast<const uint4*>(q_s + (qt * 32 + (lane & 31)) * kPitch + (lane >> 5) * 8 + ks * 16));
  };
  auto mfma = [&](uint4 k, bf16x8 q, floatx16 c) {
    if constexpr (PASS_B)
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(q, as_bf16x8(k), c, 0, 0, 0);   // rows = queries
    else
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(k), q, c, 0, 0, 0);   // rows = keys
  };
  auto masked = [&](int tk, int n) { return (a.causal && tk + n > win0 + 1) || tk + n > a.T; };
  // -inf where a key is beyond the row or after the query's own position
  auto mask_tile = [&](floatx16& c, int qt, int tk) {
    if constexpr (PASS_B) {   // c[v]: query row qt*32 + acc_row(v), key tk + lane%32
      const int t = tk + (lane & 31);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int4 w4 = *reinterpret_cast<const int4*>(wpos_s + qt * 32 + g * 8 + (lane >> 5) * 4);
        const int w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t >= a.T || (a.causal && t > win0 + w[i])) c[4 * g + i] = -INFINITY;
      }
    } else {                  // c[v]: key tk + acc_row(v), query row qt*32 + lane%32
      const int qpos = win0 + wpos_s[qt * 32 + (lane & 31)];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int t = tk + acc_row(lane, v);
        if (t >= a.T || (a.causal && t > qpos)) c[v] = -INFINITY;
      }
    }
  };
  auto pin = [&]() { __builtin_amdgcn_sched_barrier(0); };   // the compiler keeps the order of the groups written below

  // Row values (pass A: one per lane, pass B: one per accumulator) and the sums the exponentials go to.
  float rowv[PASS_B ? 16 : 1];
  float sum[PASS_B ? KT : 1][PASS_B ? 1 : 2];   // pass A: of the current query column; pass B: of this lane's key, per key tile
  auto row_group = [&](int qt, int g) {   // pass B: rows acc_row(lane, 4 g .. 4 g + 3) of query tile qt
    const float4 b4 = *reinterpret_cast<const float4*>(row_s + qt * 32 + g * 8 + (lane >> 5) * 4);
    rowv[(4 * g + 0) % (PASS_B ? 16 : 1)] = b4.x; rowv[(4 * g + 1) % (PASS_B ? 16 : 1)] = b4.y;
    rowv[(4 * g + 2) % (PASS_B ? 16 : 1)] = b4.z; rowv[(4 * g + 3) % (PASS_B ? 16 : 1)] = b4.w;
  };
  auto load_rows = [&](int qt) {
    if constexpr (PASS_B) {
#pragma unroll
      for (int g = 0; g < 4; ++g) row_group(qt, g);
    } else {
      rowv[0] = row_s[qt * 32 + (lane & 31)];
    }
  };
  auto expo = [&](const floatx16& c, int v) { return __builtin_amdgcn_exp2f(fmaf(c[v], scale2, -rowv[PASS_B ? v : 0])); };
  auto sink = [&](int kt, int v, float e) { sum[PASS_B ? kt : 0][PASS_B ? 0 : v & 1] += e; };
  auto consume = [&](const floatx16& c, int kt) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sink(kt, v, expo(c, v));
  };
  // pass A: the sum of a finished query tile over this unit goes to LDS (this wave's own slots)
  auto flush_rows = [&](int qt) {
    if constexpr (!PASS_B) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      const uint32_t z = __float_as_uint(sum[0][0] + sum[0][1]);
      const u32x2 halves = __builtin_amdgcn_permlane32_swap(z, z, false, false);
      if (lane < 32)   // one writer per slot, in program order: the result does not depend on timing
        __hip_atomic_fetch_add(sum_s + wave * a.Mrows + qt * 32 + lane, __uint_as_float(halves[0]) + __uint_as_float(halves[1]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      sum[0][0] = sum[0][1] = 0.0f;
    }
  };

  // Pass A: reference exponents.  2^(s - ref) may be summed with any reference that keeps the sum in range; the maximum
  // over the chunk's first key tile, rounded up, does unless a later logit exceeds it by more than 2^7, which shows as
  // an infinite sum.  The running maximum of the textbook form, and with it a third of the vector work, is not needed.
  bool slow = false;
  if constexpr (!PASS_B) {
    slow = masked(chunk0, 32);     // a row may have no key in the first tile (short rows, last few keys)
    if (!slow) {
      uint4 k0[8];
      load_tile(k0, chunk0);
      for (int qt = wave; qt < nqt; qt += kWaves) {
        floatx16 c = {0};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) c = mfma(k0[ks], q_piece(qt, ks), c);
        float m = c[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, c[v]);
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        if (lane < 32) row_s[qt * 32 + lane] = __builtin_ceilf(m * scale2);   // scale2 > 0: max commutes with it
      }
    }
    __syncthreads();
  }

  // One pipeline step: the matrix products of one 32x32 tile into acc, interleaved with the vector arithmetic of the tile
  // finished before (prev, key tile pkt): two elements per product, and three stages (logit, exponential, sum) one product
  // apart, so that neither an exponential waits for its logit, nor a sum for its exponential, nor the first logits for
  // the last product of prev.  The stages of the last elements run into the next step (of key tile pkt + 1) or drain.
  float logit[2], power[2];
  auto step = [&](auto fresh_tag, floatx16& acc, const floatx16& prev, int pkt, const uint4 (&k)[8], const bf16x8 (&q)[8], auto tail) {
    constexpr bool FRESH = decltype(fresh_tag)::value;   // nothing left of the step before
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if (ks == 0) acc = floatx16{0};
      acc = mfma(k[ks], q[ks], acc);
      pin();
      if (ks > 1 || !FRESH) {
        sink(ks > 1 ? pkt : pkt - 1, 0, power[0]);
        sink(ks > 1 ? pkt : pkt - 1, 1, power[1]);
      }
      if (ks > 0 || !FRESH) {
        power[0] = __builtin_amdgcn_exp2f(logit[0]);
        power[1] = __builtin_amdgcn_exp2f(logit[1]);
      }
      pin();
      logit[0] = fmaf(prev[2 * ks], scale2, -rowv[PASS_B ? 2 * ks : 0]);
      logit[1] = fmaf(prev[2 * ks + 1], scale2, -rowv[PASS_B ? 2 * ks + 1 : 0]);
      tail(ks);
      pin();
    }
  };
  auto drain = [&](int pkt) {
    const float p0 = __builtin_amdgcn_exp2f(logit[0]), p1 = __builtin_amdgcn_exp2f(logit[1]);
    sink(pkt, 0, power[0]);
    sink(pkt, 1, power[1]);
    sink(pkt, 0, p0);
    sink(pkt, 1, p1);
  };

  // The unit after `next`.  Pass B: the waves of a block take key units as they get to them (a column sum is complete
  // inside one wave, so the result does not depend on which wave that is); pass A: every wave its fixed share.
  auto unit_after = [&](int next) {
    if constexpr (PASS_B) {
      int u = 0;
      if (lane == 0) u = __hip_atomic_fetch_add(&ticket_s, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      return chunk0 + __builtin_amdgcn_readfirstlane(u) * kUnit;
    } else {
      return next + kUnitStride;
    }
  };
  auto clear_sums = [&]() {
#pragma unroll
    for (int i = 0; i < KT * 2; ++i) sum[PASS_B ? i / 2 : 0][PASS_B ? 0 : i % 2] = 0.0f;
  };
  auto store_column = [&](int kt, int tk) {
    if constexpr (PASS_B) {
      float col = sum[kt][0];
      col += __shfl_xor(col, 32, 64);
      const int t = tk + lane;
      if (lane < 32 && t < a.T)
        a.scores[static_cast<int64_t>(lh) * a.T + t] = (a.force_window && t >= win0) ? INFINITY : col;
      sum[kt][0] = 0.0f;
    }
  };
  // One tile by itself, without overlap: the tiles that need the mask.
  auto single_tile = [&](const uint4 (&k)[8], int tk) {
    const bool mask = masked(tk, 32);
    bf16x8 qop[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qop[ks] = q_piece(0, ks);
#pragma unroll 1
    for (int qt = 0; qt < nqt; ++qt) {
      load_rows(qt);
      floatx16 acc = {0};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) acc = mfma(k[ks], qop[ks], acc);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) qop[ks] = q_piece(min(qt + 1, last), ks);
      if (mask) mask_tile(acc, qt, tk);
      consume(acc, 0);
      flush_rows(qt);
    }
    store_column(0, tk);
  };

  // The textbook form of pass A: running maximum (an integer, so that rescaling is exact) and sum per query column.
  auto online_update = [&](floatx16& c, bool mask, int qt, int tk, float& m, float& z) {
    if (mask) mask_tile(c, qt, tk);
    float m_new = c[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m_new = fmaxf(m_new, c[v]);
    m_new = fmaxf(m, __builtin_ceilf(m_new * scale2));   // scale2 > 0: max commutes with it
    const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
    float z0 = z * __builtin_amdgcn_exp2f(m - m_safe), z1 = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      z0 += __builtin_amdgcn_exp2f(fmaf(c[v], scale2, -m_safe));
      z1 += __builtin_amdgcn_exp2f(fmaf(c[v + 1], scale2, -m_safe));
    }
    m = m_new;
    z = z0 + z1;
  };
  auto merge_halves = [&](float m, float z) {   // same query column, disjoint keys
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 mm = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    const u32x2 zz = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    const float m0 = __uint_as_float(mm[0]), m1 = __uint_as_float(mm[1]);
    const float m_new = fmaxf(m0, m1);
    const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
    return make_float2(m_new, __uint_as_float(zz[0]) * __builtin_amdgcn_exp2f(m0 - m_safe) +
                                  __uint_as_float(zz[1]) * __builtin_amdgcn_exp2f(m1 - m_safe));
  };
  auto merge_waves = [&](const float2* s, int pitch) {
    float m = -INFINITY, z = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m = fmaxf(m, s[w * pitch].x);
    const float m_safe = (m == -INFINITY) ? 0.0f : m;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float2 p = s[w * pitch];
      z += p.y * __builtin_amdgcn_exp2f(p.x - m_safe);
    }
    return make_float2(m, z);
  };

  clear_sums();
  int tk0 = slow ? t_end : t_begin, next = t_begin + kUnitStride;
  if (tk0 < t_end && !masked(tk0, kUnit)) {
    // A pipeline over the tiles in the order (unit, query tile, key tile): a tile is consumed during the products of
    // the one after it, also across units.
    bf16x8 qop[8];
    floatx16 acc[2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qop[ks] = q_piece(0, ks);
    load_rows(0);
    acc[0] = floatx16{0};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) acc[0] = mfma(kop_a[0][ks], qop[ks], acc[0]);
    pin();
    // key tiles 1 .. of the unit with the query tile at work, whose operands are replaced by those of tile qn
    auto rest_of_unit = [&](const uint4 (&kop)[KT][8], int qn) {
      step(std::true_type{}, acc[1], acc[0], 0, kop[1], qop, [&](int ks) { qop[ks] = q_piece(qn, ks); });   // each right after its last use
    };
    // key tile 0 with query tile qn, while the last tile of query tile qt is consumed
    auto first_of_next = [&](const uint4 (&k0)[8], int qt, int qn) {
      const float row_next = PASS_B ? 0.0f : row_s[qn * 32 + (lane & 31)];
      step(std::false_type{}, acc[0], acc[1], KT - 1, k0, qop, [&](int ks) {
        if constexpr (PASS_B) {
          if (ks & 1) row_group(qn, ks >> 1);   // the rows of these four accumulators are done with tile qt
        }
      });
      drain(KT - 1);
      flush_rows(qt);
      if constexpr (!PASS_B) rowv[0] = row_next;
    };
    // one unit; the rows of the next one are requested before its arithmetic
    auto unit = [&](const uint4 (&kop)[KT][8], uint4 (&knext)[KT][8]) {
      const int after = unit_after(next);
      const bool more = next < t_end && !masked(next, kUnit);
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this unit's rows, requested a unit ago, are here (no waits below)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) load_tile(knext[kt], next + 32 * kt);
      pin();
#pragma unroll 1
      for (int qt = 0; qt < last; ++qt) {
        rest_of_unit(kop, qt + 1);
        first_of_next(kop[0], qt, qt + 1);
      }
      rest_of_unit(kop, 0);
      if (more) {
        first_of_next(knext[0], last, 0);
      } else {
        drain(KT - 2);
        consume(acc[1], KT - 1);
        flush_rows(last);
      }
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) store_column(kt, tk0 + 32 * kt);
      tk0 = next;
      next = after;
      return more;
    };
    while (unit(kop_a, kop_b) && unit(kop_b, kop_a)) {
    }
  }
  while (tk0 < t_end) {
#pragma unroll 1
    for (int tk = tk0; tk < min(tk0 + kUnit, t_end); tk += 32) {
      load_tile(kop_a[0], tk);
      single_tile(kop_a[0], tk);
    }
    tk0 = next;
    next = unit_after(next);
  }

  if constexpr (!PASS_B) {
    float2* part = a.partial + chunk_row(a, blockIdx.x, lh) * a.Mrows;
    if (!slow) {
      __syncthreads();
      bool bad = false;
      for (int r = threadIdx.x; r < a.Mrows; r += kThreads) {
        float z = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) z += sum_s[w * a.Mrows + r];
        bad |= !(z < INFINITY);
        // the sum may be as large as 2^127: its exponent moves into the (integer) reference
        part[r] = make_float2(row_s[r] + static_cast<float>(__builtin_amdgcn_frexp_expf(z)), __builtin_amdgcn_frexp_mantf(z));
      }
      slow = __syncthreads_or(bad);
    }
    if (slow) {   // the textbook form, one query tile at a time
#pragma unroll 1
      for (int qt = 0; qt < nqt; ++qt) {
        float m = -INFINITY, z = 0.0f;
#pragma unroll 1
        for (int tk = chunk0 + 32 * wave; tk < t_end; tk += 32 * kWaves) {
          uint4 k0[8];
          load_tile(k0, tk);
          floatx16 c = {0};
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) c = mfma(k0[ks], q_piece(qt, ks), c);
          online_update(c, masked(tk, 32), qt, tk, m, z);
        }
        const float2 both = merge_halves(m, z);
        if (lane < 32) merge_s[wave * 32 + lane] = both;
        __syncthreads();
        if (threadIdx.x < 32) part[qt * 32 + threadIdx.x] = merge_waves(merge_s + threadIdx.x, 32);
        __syncthreads();
      }
    }
  }
  }
}

// ---- calls of few keys or of short rows: one chunk of one row per block, so that many blocks take part ----
//
// Each wave owns every eighth 32-key tile of the chunk, the first one requested before the prologue and each further one
// during the arithmetic of the one before, and walks the query tiles against it with two tiles in flight; pass A in the
// textbook form, which needs no prologue to find references (the running maximum is rounded up to an integer, so that
// rescaling is exact).
// 32 keys starting at tk0 as an MFMA operand, straight from global memory: lane holds key
// tk0 + lane%32, channels 16*ks + 8*(lane/32) .. +7.  Keys at or beyond T are zero.
__device__ __forceinline__ void load_key_tile(const ScoreArgs& a, const uint16_t* kbase, int tk0, int lane, uint4 out[8]) {
  const int t = tk0 + (lane & 31);
  if (t < a.T) {
    const uint16_t* row = kbase + static_cast<int64_t>(t) * a.k_st + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = *reinterpret_cast<const uint4*>(row + ks * 16);
  } else {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = make_uint4(0, 0, 0, 0);
  }
}

template <int NQT, bool PASS_B>
__global__ __launch_bounds__(kThreads, 2) void score_chunk_kernel(const ScoreArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t q_s[NQT * 32 * kPitch];
  __shared__ __attribute__((aligned(16))) float bias_s[PASS_B ? NQT * 32 : 4];
  __shared__ __attribute__((aligned(16))) int32_t wpos_s[NQT * 32];   // window offset r mod W of query row r (masked tiles)

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int lh = blockIdx.y;
  const int l = lh / a.Hkv, h = lh - l * a.Hkv;
  const int chunk = blockIdx.x;
  const uint16_t* kbase = a.k + static_cast<int64_t>(l) * a.k_sl + static_cast<int64_t>(h) * a.k_sh;
  const int win0 = a.T - a.W;  // first window position

  // this wave's first key tile is requested before anything else, so that its latency overlaps the prologue
  constexpr int kTileStride = 32 * kWaves;
  const int t_begin = chunk * a.chunk_keys + wave * 32;
  const int t_end = min(a.T, (chunk + 1) * a.chunk_keys);
  uint4 kop[8];
  if (t_begin < t_end) load_key_tile(a, kbase, t_begin, lane, kop);

  // ---- stage the window queries of this (layer, kv head): row r = u * W + w, zeros beyond M.  A thread's
  //      (at most NQT) pieces are all requested before the first one is stored ----
  {
    uint4 piece[NQT];
#pragma unroll
    for (int i = 0; i < NQT; ++i) {
      const int idx = static_cast<int>(threadIdx.x) + i * kThreads;
      const int r = idx >> 4, part = idx & 15;
      piece[i] = make_uint4(0, 0, 0, 0);
      if (r < a.M) {
        const int u = r / a.W, w = r - u * a.W;
        piece[i] = *reinterpret_cast<const uint4*>(a.q + static_cast<int64_t>(l) * a.q_sl + static_cast<int64_t>(w) * a.q_st +
                                                   static_cast<int64_t>(h * a.G + u) * a.q_sh + part * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < NQT; ++i) {
      const int idx = static_cast<int>(threadIdx.x) + i * kThreads;
      if (idx < a.Mrows * 16) *reinterpret_cast<uint4*>(q_s + (idx >> 4) * kPitch + (idx & 15) * 8) = piece[i];
    }
  }
  for (int r = threadIdx.x; r < a.Mrows; r += kThreads) {
    wpos_s[r] = r % a.W;
    // rows beyond M carry +inf: they contribute 2^-inf = 0
    if constexpr (PASS_B) bias_s[r] = a.fold_combine ? (r < a.M ? combined_chunks<true>(a.partial + static_cast<int64_t>(lh) * gridDim.x * a.Mrows + r, gridDim.x, a.Mrows) : INFINITY) : a.bias[static_cast<int64_t>(lh) * a.Mrows + r];
  }
  __syncthreads();

  // pass A state: running max / sum of this lane's query column (per query tile) over this lane's keys
  float run_m[PASS_B ? 1 : NQT], run_z[PASS_B ? 1 : NQT];
  if constexpr (!PASS_B) {
#pragma unroll
    for (int i = 0; i < NQT; ++i) {
      run_m[i] = -INFINITY;
      run_z[i] = 0.0f;
    }
  }

  auto q_operand = [&](int qt, bf16x8 out[8]) {
    const uint16_t* row = q_s + (qt * 32 + (lane & 31)) * kPitch + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) out[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(row + ks * 16));
  };
  auto mfma_tile = [&](const uint4 kop[8], const bf16x8 qop[8]) {
    floatx16 acc = {0};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if constexpr (PASS_B)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qop[ks], as_bf16x8(kop[ks]), acc, 0, 0, 0);  // rows = queries
      else
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kop[ks]), qop[ks], acc, 0, 0, 0);  // rows = keys
    }
    return acc;
  };

  // Vector-ALU work of one finished 32x32 tile `c` (query tile qt, keys tk0 .. tk0+31).
  auto consume = [&](auto masked_tag, floatx16& c, int qt, int tk0, float& col, float& m_run, float& z_run) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    if constexpr (!PASS_B) {
      // c[v] = raw dot product of key tk0 + acc_row(v) with query row qt*32 + lane%32
      if constexpr (MASKED) {
        const int qpos = win0 + wpos_s[qt * 32 + (lane & 31)];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int t = tk0 + acc_row(lane, v);
          if (t >= a.T || (a.causal && t > qpos)) c[v] = -INFINITY;
        }
      }
      float tmax = c[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, c[v]);
      const float m_new = fmaxf(m_run, __builtin_ceilf(tmax * a.scale2));   // scale2 > 0: max commutes with it
      const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
      float z = z_run * __builtin_amdgcn_exp2f(m_run - m_safe);
#pragma unroll
      for (int v = 0; v < 16; ++v) z += __builtin_amdgcn_exp2f(fmaf(c[v], a.scale2, -m_safe));
      m_run = m_new;
      z_run = z;
    } else {
      // c[v] = raw dot product of query row qt*32 + acc_row(v) with key tk0 + lane%32
      float bias[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 b4 = *reinterpret_cast<const float4*>(bias_s + qt * 32 + g * 8 + (lane >> 5) * 4);
        bias[4 * g + 0] = b4.x; bias[4 * g + 1] = b4.y; bias[4 * g + 2] = b4.z; bias[4 * g + 3] = b4.w;
      }
      if constexpr (MASKED) {
        const int t = tk0 + (lane & 31);
        if (a.causal) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {   // rows acc_row(lane, 4 g .. 4 g + 3), as for the bias
            const int4 w4 = *reinterpret_cast<const int4*>(wpos_s + qt * 32 + g * 8 + (lane >> 5) * 4);
            if (t > win0 + w4.x) c[4 * g + 0] = -INFINITY;
            if (t > win0 + w4.y) c[4 * g + 1] = -INFINITY;
            if (t > win0 + w4.z) c[4 * g + 2] = -INFINITY;
            if (t > win0 + w4.w) c[4 * g + 3] = -INFINITY;
          }
        }
      }
      float part = 0.0f;   // a sum of its own per tile: less rounding than adding every term to the column
#pragma unroll
      for (int v = 0; v < 16; ++v) part += __builtin_amdgcn_exp2f(fmaf(c[v], a.scale2, -bias[v]));
      col += part;
    }
  };

  // The LDS reads of a query tile's operands are issued one whole pipeline step before the MFMAs that
  // use them; a scheduling barrier keeps the compiler from sinking them back next to their use (where
  // every MFMA would wait out the LDS latency on its own).
  auto pin = [&]() { __builtin_amdgcn_sched_barrier(0); };

  // One 32-key tile against all query tiles as a software pipeline over the query tiles:
  //   step n:  LDS operand reads of tile n+2, then  MFMAs of tile n+1  |  vector-ALU work of tile n.
  // Query tiles in use.  Pass A is instantiated for the exact count (its per-tile statistics live in registers with
  // static indices), pass B for 1, 2, 4, 8 or 16 tiles of LDS with the count in use as a run-time value.
  const int nqt = PASS_B ? a.nqt : NQT;
  auto key_tile = [&](auto masked_tag, const uint4 kop[8], int tk0) {
    bf16x8 qop_a[8], qop_b[8];
    floatx16 acc_a, acc_b;
    float col = 0.0f, dummy_m = 0.0f, dummy_z = 0.0f;  // pass B: this lane's key column
    q_operand(0, qop_a);
    acc_a = mfma_tile(kop, qop_a);
    if (nqt > 1) q_operand(1, qop_b);
    // two pipeline steps: tile qt is finished in acc_a, the operands of tile qt+1 are in qop_b, tile qt+2 exists
    auto two_steps = [&](int qt, float& m0, float& z0, float& m1, float& z1) {
      q_operand(qt + 2, qop_a);
      pin();
      acc_b = mfma_tile(kop, qop_b);
      consume(masked_tag, acc_a, qt, tk0, col, m0, z0);
      pin();
      if (qt + 3 < nqt) q_operand(qt + 3, qop_b);
      pin();
      acc_a = mfma_tile(kop, qop_a);
      consume(masked_tag, acc_b, qt + 1, tk0, col, m1, z1);
      pin();
    };
    if constexpr (!PASS_B) {
      // fully unrolled: static register indices for the running statistics
#pragma unroll
      for (int qt = 0; qt + 2 < NQT; qt += 2) two_steps(qt, run_m[qt], run_z[qt], run_m[qt + 1], run_z[qt + 1]);
      if constexpr (NQT % 2 == 0) {
        acc_b = mfma_tile(kop, qop_b);
        consume(masked_tag, acc_a, NQT - 2, tk0, col, run_m[NQT - 2], run_z[NQT - 2]);
        pin();
        consume(masked_tag, acc_b, NQT - 1, tk0, col, run_m[NQT - 1], run_z[NQT - 1]);
      } else {
        consume(masked_tag, acc_a, NQT - 1, tk0, col, run_m[NQT - 1], run_z[NQT - 1]);
      }
    } else {
      // no per-tile state: a rolled loop keeps the register footprint independent of the tile count
      int qt = 0;
#pragma unroll 1
      for (; qt + 2 < nqt; qt += 2) two_steps(qt, dummy_m, dummy_z, dummy_m, dummy_z);
      if (qt + 1 < nqt) {
        acc_b = mfma_tile(kop, qop_b);
        consume(masked_tag, acc_a, qt, tk0, col, dummy_m, dummy_z);
        pin();
        consume(masked_tag, acc_b, qt + 1, tk0, col, dummy_m, dummy_z);
      } else {
        consume(masked_tag, acc_a, qt, tk0, col, dummy_m, dummy_z);
      }
      col += __shfl_xor(col, 32, 64);
      const int t = tk0 + lane;
      if (lane < 32 && t < a.T)
        a.scores[static_cast<int64_t>(lh) * a.T + t] = (a.force_window && t >= win0) ? INFINITY : col;
    }
  };

  // ---- this wave's key tiles: every kWaves-th tile of the chunk, so that the few masked tiles at the
  //      end of a row (each costs more) are spread over the waves instead of all landing on the last one ----
  if (t_begin < t_end) {
    uint4 knext[8];
    for (int tk0 = t_begin; tk0 < t_end; tk0 += kTileStride) {
      const bool more = tk0 + kTileStride < t_end;
      if (more) load_key_tile(a, kbase, tk0 + kTileStride, lane, knext);
      const bool need_mask = (a.causal && tk0 + 32 > win0 + 1) || (tk0 + 32 > a.T);
      if (need_mask)
        key_tile(std::true_type{}, kop, tk0);
      else
        key_tile(std::false_type{}, kop, tk0);
      if (more) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kop[ks] = knext[ks];
      }
    }
  }

  if constexpr (!PASS_B) {
    // merge the two half-waves (same query column, disjoint keys), then the 8 waves through LDS
    __syncthreads();                       // every wave is done reading q_s: reuse it as scratch
    float2* merge_s = reinterpret_cast<float2*>(q_s);   // [kWaves][NQT*32]
#pragma unroll
    for (int qt = 0; qt < NQT; ++qt) {
      const float m_o = __shfl_xor(run_m[qt], 32, 64);
      const float z_o = __shfl_xor(run_z[qt], 32, 64);
      const float m_new = fmaxf(run_m[qt], m_o);
      const float m_safe = (m_new == -INFINITY) ? 0.0f : m_new;
      const float z = run_z[qt] * __builtin_amdgcn_exp2f(run_m[qt] - m_safe) + z_o * __builtin_amdgcn_exp2f(m_o - m_safe);
      if (lane < 32) merge_s[wave * (NQT * 32) + qt * 32 + lane] = make_float2(m_new, z);
    }
    __syncthreads();
    for (int r = threadIdx.x; r < a.Mrows; r += kThreads) {
      float m = -INFINITY;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) m = fmaxf(m, merge_s[w * (NQT * 32) + r].x);
      const float m_safe = (m == -INFINITY) ? 0.0f : m;
      float z = 0.0f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float2 p = merge_s[w * (NQT * 32) + r];
        z += p.y * __builtin_amdgcn_exp2f(p.x - m_safe);
      }
      a.partial[(static_cast<int64_t>(lh) * gridDim.x + chunk) * a.Mrows + r] = make_float2(m, z);
    }
  }
}

// The same combination as its own launch, once per (layer, head), when there are many chunks.
__global__ void combine_kernel(const ScoreArgs a) {
  const int lh = blockIdx.x;
  for (int r = threadIdx.x; r < a.Mrows; r += blockDim.x) a.bias[static_cast<int64_t>(lh) * a.Mrows + r] = combined_bias<false>(a, lh, r);
}

// Instantiated for 1, 2, 4, 8 and 16 query tiles of LDS (M = 224 runs 7 tiles in the 8-tile instantiation); pass A of the
// chunked kernel for every tile count 1 .. 16 (its per-tile statistics live in registers with static indices).
template <bool PASS_B>
void launch_wide(int nqt, dim3 grid, hipStream_t st, const ScoreArgs& a) {
  if (nqt <= 1) score_kernel<1, PASS_B><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 2) score_kernel<2, PASS_B><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 4) score_kernel<4, PASS_B><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 8) score_kernel<8, PASS_B><<<grid, kThreads, 0, st>>>(a);
  else score_kernel<16, PASS_B><<<grid, kThreads, 0, st>>>(a);
}

template <int N>
void launch_chunked_a(int nqt, dim3 grid, hipStream_t st, const ScoreArgs& a) {
  if constexpr (N <= 16) {
    if (nqt == N) score_chunk_kernel<N, false><<<grid, kThreads, 0, st>>>(a);
    else launch_chunked_a<N + 1>(nqt, grid, st, a);
  }
}

void launch_chunked_b(int nqt, dim3 grid, hipStream_t st, const ScoreArgs& a) {
  if (nqt <= 1) score_chunk_kernel<1, true><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 2) score_chunk_kernel<2, true><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 4) score_chunk_kernel<4, true><<<grid, kThreads, 0, st>>>(a);
  else if (nqt <= 8) score_chunk_kernel<8, true><<<grid, kThreads, 0, st>>>(a);
  else score_chunk_kernel<16, true><<<grid, kThreads, 0, st>>>(a);
}

}  // namespace

// Shared with the configuration-evaluation path, which ranks tokens with the same scores.
int32_t score_tokens_impl(const kvp_view* q_win, const kvp_view* k, int32_t causal, int32_t force_window,
                          float* scores, void* ws, size_t ws_bytes, hipStream_t st) {
  int32_t rc = check_view(q_win);
  if (rc != KVP_OK) return rc;
  rc = check_view(k);
  if (rc != KVP_OK) return rc;
  if (!scores) return KVP_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(scores) & 3u) return KVP_ERR_ALIGN;
  const int64_t L = k->L, T = k->T, Hkv = k->H, Hq = q_win->H, W = q_win->T;
  if (q_win->L != L || Hq % Hkv != 0 || W > T || T >= (1ll << 30) || L * Hkv > 65535) return KVP_ERR_SHAPE;
  if ((Hq / Hkv) * W > kMaxRows) return KVP_ERR_UNSUPPORTED;
  const ScorePlan p = make_score_plan(L, Hkv, Hq, W, T);
  if (!ws || ws_bytes < p.bytes || (reinterpret_cast<uintptr_t>(ws) & 15u))
    return KVP_ERR_WORKSPACE;

  ScoreArgs a{};
  a.q = static_cast<const uint16_t*>(q_win->ptr);
  a.q_sl = q_win->stride_l; a.q_st = q_win->stride_t; a.q_sh = q_win->stride_h;
  a.k = static_cast<const uint16_t*>(k->ptr);
  a.k_sl = k->stride_l; a.k_st = k->stride_t; a.k_sh = k->stride_h;
  a.T = static_cast<int32_t>(T); a.W = static_cast<int32_t>(W); a.G = static_cast<int32_t>(Hq / Hkv);
  a.Hkv = static_cast<int32_t>(Hkv); a.M = p.M; a.Mrows = p.Mrows; a.nqt = p.nqt;
  a.div_w = FastDiv(static_cast<uint32_t>(W));
  // fewer than 2^31 units: more would need more than 2^37 scores, which no device holds
  a.units_lh = static_cast<uint32_t>(p.units_lh); a.units_block = static_cast<uint32_t>(p.units_block);
  a.units = static_cast<uint32_t>(p.units);
  a.div_lh = FastDiv(a.units_lh); a.div_block = FastDiv(a.units_block);
  a.chunk_keys = p.chunk_keys;
  a.compact_rows = p.wide ? 0 : 1;
  a.causal = causal ? 1 : 0; a.force_window = force_window ? 1 : 0;
  a.scale2 = kLog2e / sqrtf(static_cast<float>(kHeadDim));
  a.partial = static_cast<float2*>(ws);
  a.bias = reinterpret_cast<float*>(static_cast<char*>(ws) + p.partial_bytes);   // not used when pass B combines
  a.scores = scores;

  // With few chunks pass B combines the chunk statistics of its rows itself (a few KiB of reads from the cache): a call
  // is two launches, which is what counts for small, launch-bound shapes.
  a.fold_combine = p.fold ? 1 : 0;
  const dim3 rows(static_cast<unsigned>(L * Hkv));
  if (p.wide) {
    const dim3 grid(static_cast<unsigned>(p.blocks));
    launch_wide<false>(p.nqt, grid, st, a);
    if (!p.fold) combine_kernel<<<rows, 256, 0, st>>>(a);
    launch_wide<true>(p.nqt, grid, st, a);
  } else {
    const dim3 grid(static_cast<unsigned>(p.units_lh), rows.x);
    launch_chunked_a<1>(p.nqt, grid, st, a);
    if (!p.fold) combine_kernel<<<rows, 256, 0, st>>>(a);
    launch_chunked_b(p.nqt, grid, st, a);
  }
  return launch_status();
}

}  // namespace kvp

extern "C" size_t kvp_score_workspace_bytes(int64_t L, int64_t Hkv, int64_t Hq, int64_t W, int64_t T) {
  if (L <= 0 || Hkv <= 0 || Hq <= 0 || W <= 0 || T <= 0 || Hq % Hkv != 0) return 0;
  const kvp::ScorePlan p = kvp::make_score_plan(L, Hkv, Hq, W, T);
  return p.bytes;
}

extern "C" int32_t kvp_score_tokens(const kvp_view* q_win, const kvp_view* k, int32_t causal, int32_t force_window,
                                    float* scores, void* ws, size_t ws_bytes, void* stream) {
  return kvp::score_tokens_impl(q_win, k, causal, force_window, scores, ws, ws_bytes, kvp::as_stream(stream));
}

// ---- kvp_score_tokens_static: the same kernels with their scratch in a device array of the library ----
//
// `scratch` is the host-side stand-in of the device array: host code never passes it to a kernel.  Its
// device address is looked up once per device (every GPU holds its own copy at its own address) and
// only that address is used from then on.
namespace kvp {
namespace {

static __device__ __align__(256) unsigned char scratch[KVP_SCORE_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on device i, once looked up

// Device address of the current device's copy of `scratch` (nullptr + rc on failure).  Allocates nothing.
int32_t static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KVP_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return KVP_ERR_LAUNCH;
    }
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return KVP_OK;
}

}  // namespace
}  // namespace kvp

extern "C" int32_t kvp_score_tokens_static(const kvp_view* q_win, const kvp_view* k, int32_t causal,
                                           int32_t force_window, float* scores, void* stream) {
  using namespace kvp;
  // size check first (host arithmetic only), so that an oversized request fails before any lookup
  int32_t rc = check_view(q_win);
  if (rc != KVP_OK) return rc;
  rc = check_view(k);
  if (rc != KVP_OK) return rc;
  if (q_win->H % k->H != 0) return KVP_ERR_SHAPE;
  if (kvp_score_workspace_bytes(k->L, k->H, q_win->H, q_win->T, k->T) > KVP_SCORE_STATIC_SCRATCH_BYTES)
    return KVP_ERR_WORKSPACE;
  void* ptr = nullptr;
  rc = static_scratch(&ptr);
  if (rc != KVP_OK) return rc;
  // every word of the scratch that pass B and the combine step read is written earlier in the same call
  // (pass A stores the statistics of all chunks and all padded rows), so nothing has to be cleared
  return score_tokens_impl(q_win, k, causal, force_window, scores, ptr, KVP_SCORE_STATIC_SCRATCH_BYTES,
                           as_stream(stream));
}
