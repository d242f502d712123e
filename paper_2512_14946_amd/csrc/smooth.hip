// kvp_smooth_scores: 1-D average / maximum pooling of the prefix scores along the token axis, the
// smoothing step of the published snapkv method (the paper's Evaluation, Baselines) that runs
// between kvp_score_tokens and kvp_select_topk.
//
// One 256-thread block per (tile of 2048 tokens, row); the tile and its halo on each side are staged in LDS once
// (out-of-prefix taps as the pooling's neutral element).  Traffic is one read and one write of the score rows (a few tens
// of MB): the kernel is short, and what bounds it is the work per token.
//   kernels of up to 9 taps (the usual ones): a thread owns two groups of 4 consecutive tokens, reads and writes them
//     with 16-byte accesses, and needs the groups before and after each from LDS, so 2 LDS reads serve 4 outputs
//     (640 x 16384, 7 taps, 84 MB: 26.0 -> 13.6 us);
//   longer ones: 8 outputs per thread, lanes on adjacent tokens, one LDS read per tap.

#include "kvp_common.h"

namespace kvp {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 2048;
constexpr int kMaxKernel = 63;

template <bool MAXPOOL>
__global__ __launch_bounds__(kThreads) void smooth_kernel(const float* __restrict__ scores, int64_t row_stride, uint32_t T,
                                                          uint32_t P, int r, float* __restrict__ out, int64_t out_stride) {
  __shared__ float tile[kTile + kMaxKernel - 1];
  const float* in = scores + static_cast<int64_t>(blockIdx.x) * row_stride;   // x: row (up to 2^31 - 1), y: tile
  float* o = out + static_cast<int64_t>(blockIdx.x) * out_stride;
  const uint32_t t0 = blockIdx.y * kTile;
  const float neutral = MAXPOOL ? -INFINITY : 0.0f;
  const int span = kTile + 2 * r;
  for (int i = threadIdx.x; i < span; i += kThreads) {
    const int64_t u = static_cast<int64_t>(t0) - r + i;
    tile[i] = (u >= 0 && u < static_cast<int64_t>(P)) ? in[u] : neutral;
  }
  __syncthreads();
  const int taps = 2 * r + 1;
  const float divisor = static_cast<float>(taps);
  for (int j = threadIdx.x; j < kTile; j += kThreads) {
    const uint32_t t = t0 + j;
    if (t >= T) break;
    float v;
    if (t < P) {
      v = tile[j];                      // tap t - r
      for (int d = 1; d < taps; ++d) v = MAXPOOL ? fmaxf(v, tile[j + d]) : v + tile[j + d];
      if (!MAXPOOL) v = v / divisor;
    } else {
      v = in[t];                        // observation window: copied through
    }
    o[t] = v;
  }
}

// Up to 9 taps: R = kernel / 2 in 0 .. 4.  The same operations in the same order as above.
template <bool MAXPOOL, int R>
__global__ __launch_bounds__(kThreads) void smooth_short_kernel(const float* __restrict__ scores, int64_t row_stride,
                                                                uint32_t T, uint32_t P, float* __restrict__ out,
                                                                int64_t out_stride) {
  constexpr int kGroups = kTile / 4, kOwn = kGroups / kThreads;
  __shared__ float4 tile[kGroups + 2];   // one group of halo on each side
  const float* in = scores + static_cast<int64_t>(blockIdx.x) * row_stride;
  float* o = out + static_cast<int64_t>(blockIdx.x) * out_stride;
  const bool vec_in = (reinterpret_cast<uintptr_t>(in) & 15u) == 0, vec_out = (reinterpret_cast<uintptr_t>(o) & 15u) == 0;
  const uint32_t t0 = blockIdx.y * kTile;   // T < 2^31: t0 + kTile does not wrap
  const float neutral = MAXPOOL ? -INFINITY : 0.0f;
  auto load = [&](uint32_t t) {             // tokens t .. t + 3, zeros beyond the row
    if (vec_in && t + 4 <= T) return *reinterpret_cast<const float4*>(in + t);
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (t < T) v.x = in[t];
    if (t + 1 < T) v.y = in[t + 1];
    if (t + 2 < T) v.z = in[t + 2];
    if (t + 3 < T) v.w = in[t + 3];
    return v;
  };
  auto taps = [&](float4 v, uint32_t t) {   // as taps: neutral beyond the prefix
    return make_float4(t < P ? v.x : neutral, t + 1 < P ? v.y : neutral, t + 2 < P ? v.z : neutral, t + 3 < P ? v.w : neutral);
  };
  float4 raw[kOwn];
#pragma unroll
  for (int i = 0; i < kOwn; ++i) raw[i] = load(t0 + 4 * (threadIdx.x + i * kThreads));
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const uint32_t g = threadIdx.x + i * kThreads;
    tile[g + 1] = taps(raw[i], t0 + 4 * g);
  }
  if (threadIdx.x == 0)
    tile[0] = t0 == 0 ? make_float4(neutral, neutral, neutral, neutral) : taps(load(t0 - 4), t0 - 4);
  if (threadIdx.x == kWave) tile[kGroups + 1] = taps(load(t0 + kTile), t0 + kTile);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const uint32_t g = threadIdx.x + i * kThreads, t = t0 + 4 * g;
    if (t >= T) break;
    const float4 b = tile[g], c = tile[g + 1], d = tile[g + 2];
    const float x[12] = {b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w, d.x, d.y, d.z, d.w};
    const float own[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = x[4 + e - R];
#pragma unroll
      for (int k = 1; k <= 2 * R; ++k) v = MAXPOOL ? fmaxf(v, x[4 + e - R + k]) : v + x[4 + e - R + k];
      if (!MAXPOOL) v = v / static_cast<float>(2 * R + 1);
      y[e] = t + e < P ? v : own[e];        // observation window: copied through
    }
    if (vec_out && t + 4 <= T) {
      *reinterpret_cast<float4*>(o + t) = make_float4(y[0], y[1], y[2], y[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e < T) o[t + e] = y[e];
    }
  }
}

template <bool MAXPOOL>
void launch(dim3 grid, hipStream_t st, const float* scores, int64_t row_stride, uint32_t T, uint32_t P, int r, float* out,
            int64_t out_stride) {
  switch (r) {
    case 0: smooth_short_kernel<MAXPOOL, 0><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, out, out_stride); break;
    case 1: smooth_short_kernel<MAXPOOL, 1><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, out, out_stride); break;
    case 2: smooth_short_kernel<MAXPOOL, 2><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, out, out_stride); break;
    case 3: smooth_short_kernel<MAXPOOL, 3><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, out, out_stride); break;
    case 4: smooth_short_kernel<MAXPOOL, 4><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, out, out_stride); break;
    default: smooth_kernel<MAXPOOL><<<grid, kThreads, 0, st>>>(scores, row_stride, T, P, r, out, out_stride); break;
  }
}

}  // namespace
}  // namespace kvp

extern "C" int32_t kvp_smooth_scores(const float* scores, int64_t n_rows, int64_t T, int64_t row_stride, int64_t window,
                                     int32_t kernel, int32_t mode, float* out, int64_t out_stride, void* stream) {
  using namespace kvp;
  if (!scores || !out) return KVP_ERR_NULL;
  if (n_rows < 0 || T <= 0 || T >= (1ll << 31) || row_stride < T || out_stride < T || window < 0 || window > T)
    return KVP_ERR_SHAPE;
  if (n_rows >= (1ll << 31) || ceil_div(T, kTile) > 65535) return KVP_ERR_SHAPE;
  if (kernel < 1 || kernel > kMaxKernel || kernel % 2 == 0) return KVP_ERR_UNSUPPORTED;
  if (mode != KVP_SMOOTH_AVG && mode != KVP_SMOOTH_MAX) return KVP_ERR_UNSUPPORTED;
  if ((reinterpret_cast<uintptr_t>(scores) & 3u) || (reinterpret_cast<uintptr_t>(out) & 3u)) return KVP_ERR_ALIGN;
  if (n_rows == 0) return KVP_OK;
  {  // the two row sets must not overlap (a block reads its halo after neighbours may have written)
    const char* a0 = reinterpret_cast<const char*>(scores);
    const char* a1 = a0 + ((n_rows - 1) * row_stride + T) * 4;
    const char* b0 = reinterpret_cast<const char*>(out);
    const char* b1 = b0 + ((n_rows - 1) * out_stride + T) * 4;
    if (a0 < b1 && b0 < a1) return KVP_ERR_SHAPE;
  }
  const dim3 grid(static_cast<unsigned>(n_rows), static_cast<unsigned>(ceil_div(T, kTile)));
  const hipStream_t st = as_stream(stream);
  const uint32_t P = static_cast<uint32_t>(T - window);
  if (mode == KVP_SMOOTH_MAX)
    launch<true>(grid, st, scores, row_stride, static_cast<uint32_t>(T), P, kernel / 2, out, out_stride);
  else
    launch<false>(grid, st, scores, row_stride, static_cast<uint32_t>(T), P, kernel / 2, out, out_stride);
  return launch_status();
}
