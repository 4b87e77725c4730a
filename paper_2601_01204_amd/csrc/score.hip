// Token-importance scoring (paper Sec. 3.2, Eq. 2-6).
//
// Eq. 5-6 average the rows of Qbar Kbar^T, which by linearity equals q~ . Kbar_j with
// q~ the mean of the pooled, head-averaged query rows.  Every value here feeds top-k,
// so each kernel evaluates in fp32 with one rounding per operation and the fixed order
// of additions stated at the kernel (compiled without FMA contraction).
#include "score_select.h"

#include <algorithm>
#include <type_traits>

namespace kvx {

// Eq. 2-3: one block per pooled row, sixteen lanes per head, four channels per lane.  Per
// (head, channel): add the row's tokens in ascending order starting from the first, divide
// by the group size; then per channel add heads 0..H-1 in order starting from zero, divide
// by H.  A group's tokens are requested sixteen at a time before any is added, so a row
// costs one memory round trip.  Bound by latency, of which fetching the kernel's code is a
// good part: rows are addressed from one uniform pointer, the input type is a template
// argument, and four channels a lane (not eight) halve the code and double the waves.
// Against eight unrolled channels a lane with 64-bit addresses per token: one cache of 782 or
// 1041 tokens 11 -> 4.5 us, 24 caches 24 -> 14 us, 48 caches of 1374 tokens 39 -> 26 us.
constexpr int kPoolBatch = 16;
template <bool F32IN, int N>
__global__ __launch_bounds__(1024) void pool_rows_kernel(const KvxBatchT<N> b) {
  const Geometry& g = b.g;
  const Item it = b.items[blockIdx.y];
  if (!it.prune) return;
  // pooled row -> (frame of the call, row within the frame): every frame is pooled by itself
  const int row = blockIdx.x;
  const int fr = row / g.n_pooled, rr = row - fr * g.n_pooled;
  int a, e;
  if (rr < g.n_special) {
    a = fr * g.n + rr;
    e = a + 1;
  } else {
    a = fr * g.n + g.n_special + (rr - g.n_special) * g.pool_group;
    e = min(a + g.pool_group, (fr + 1) * g.n);
  }
  __shared__ __attribute__((aligned(16))) float pooled[64][kHeadDim];     // up to 64 heads
  typedef typename std::conditional<F32IN, float4, uint2>::type Raw;      // four channels as they come
  constexpr int kElt = F32IN ? 4 : 2;
  const int h = threadIdx.x >> 4, c0 = (threadIdx.x & 15) * 4;
  if (h < g.H) {
    const int64_t lane_off = ((int64_t)h * g.head_stride + c0) * kElt, step = g.tok_stride * kElt;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t0 = a; t0 < e; t0 += kPoolBatch) {
      Raw v[kPoolBatch];
      const uint8_t* p = reinterpret_cast<const uint8_t*>(it.q) + t0 * step;
#pragma unroll
      for (int k = 0; k < kPoolBatch; ++k) {
        v[k] = *reinterpret_cast<const Raw*>(p + lane_off);
        if (t0 + k + 1 < e) p += step;                     // a repeated token is loaded but not added
      }
#pragma unroll
      for (int k = 0; k < kPoolBatch; ++k) {
        if (t0 + k < e) {
          float x[4];
          if constexpr (F32IN) {
            x[0] = v[k].x; x[1] = v[k].y; x[2] = v[k].z; x[3] = v[k].w;
          } else {
            x[0] = __uint_as_float(v[k].x << 16); x[1] = __uint_as_float(v[k].x & 0xFFFF0000u);
            x[2] = __uint_as_float(v[k].y << 16); x[3] = __uint_as_float(v[k].y & 0xFFFF0000u);
          }
          const bool first = k == 0 && t0 == a;
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = first ? x[j] : acc[j] + x[j];
        }
      }
    }
    const float cnt = (float)(e - a);
    *reinterpret_cast<float4*>(&pooled[h][c0]) = make_float4(acc[0] / cnt, acc[1] / cnt, acc[2] / cnt, acc[3] / cnt);
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int c = threadIdx.x;
    float acc = 0.f;
#pragma unroll 4
    for (int hh = 0; hh < g.H; ++hh) acc = acc + pooled[hh][c];
    reinterpret_cast<float*>(cache_scratch(g, it.cache) + g.sl.qbar)[row * kHeadDim + c] = acc / (float)g.H;
  }
}

// The row mean of Eq. 6 pulled inside the product: q~ = (pooled rows added in ascending
// order from zero) / N_pooled.  A kernel of its own, so that the pooled rows reach it
// through the kernel boundary and no block has to fence.  The rows are brought into LDS
// 128 at a time by the whole block (one memory round trip per 128 rows), then one thread
// per channel adds them in order.
template <int N>
__global__ __launch_bounds__(1024) void pool_mean_kernel(const KvxBatchT<N> b) {
  const Geometry& g = b.g;
  const Item it = b.items[blockIdx.x];
  if (!it.prune) return;
  uint8_t* sc = cache_scratch(g, it.cache);
  const float4* qbar = reinterpret_cast<const float4*>(sc + g.sl.qbar);
  __shared__ __attribute__((aligned(16))) float rows[kMeanRows][kHeadDim];
  const int tid = threadIdx.x;
  float acc = 0.f;
  const int n_rows = g.n_pooled * (g.n_new / g.n);          // the pooled rows of all the call's frames, in frame order
  for (int r0 = 0; r0 < n_rows; r0 += kMeanRows) {
    const int cnt = min(kMeanRows, n_rows - r0);
    // 16 float4 per row: threads 0..1023 cover 64 rows per step
#pragma unroll
    for (int k = 0; k < kMeanRows / 64; ++k) {
      const int r = k * 64 + (tid >> 4);
      if (r < cnt) *reinterpret_cast<float4*>(&rows[r][(tid & 15) * 4]) = qbar[(int64_t)(r0 + r) * 16 + (tid & 15)];
    }
    __syncthreads();
    if (tid < kHeadDim) {
      for (int r = 0; r < cnt; ++r) acc = acc + rows[r][tid];
    }
    __syncthreads();
  }
  if (tid < kHeadDim) reinterpret_cast<float*>(sc + g.sl.qt)[tid] = acc / (float)n_rows;
}

// MEAN: every block forms q~ itself, in pool_mean_kernel's order, from the pooled rows (at most 128, one LDS load).
template <int B, bool MEAN, int N>
__global__ __launch_bounds__(kScoreWaves * 64) void score_kernel(const KvxBatchT<N> b) {
  const Geometry& g = b.g;
  const Item it = b.items[blockIdx.y];
  if (!it.prune) return;
  const int j0 = (g.n / 64 + (int)blockIdx.x) * 64;
  if (j0 >= it.t_c) return;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  if constexpr (MEAN) {
    __shared__ __attribute__((aligned(16))) float rows[kMeanRows * kHeadDim];
    __shared__ float s_qt[kHeadDim];
    score_block<B>(g, it, j0, lds, [&]() { return pooled_mean(g, it, rows, s_qt); });
  } else {
    score_block<B>(g, it, j0, lds, [&]() { return reinterpret_cast<const float*>(cache_scratch(g, it.cache) + g.sl.qt)[threadIdx.x & 63]; });
  }
}

void launch_pool(const KvxBatch& b, int max_tc, hipStream_t st) {
  const dim3 rows(b.g.n_pooled * (b.g.n_new / b.g.n), b.n_items), block(std::max(64, 16 * b.g.H));
  if (b.g.in_f32) with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((pool_rows_kernel<true, KVX_ITEMS(bb)>), rows, block, 0, st, bb); });
  else with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((pool_rows_kernel<false, KVX_ITEMS(bb)>), rows, block, 0, st, bb); });
  // (scoring blocks inside the attention launch form the mean themselves)
  if (!b.g.side_blocks && !mean_in_score(b, max_tc)) with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((pool_mean_kernel<KVX_ITEMS(bb)>), dim3(b.n_items), dim3(1024), 0, st, bb); });
}

// Scoring and selection together, on several caches (selects_in_score).
template <int B>
__global__ __launch_bounds__(kScoreWaves * 64) void score_select_kernel(const KvxBatch b) {
  const Geometry& g = b.g;
  const Item it = b.items[blockIdx.y];
  if (!it.prune) return;
  const int blocks = (it.t_c + 63) / 64 - g.n / 64;
  if ((int)blockIdx.x >= blocks) return;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  score_and_select<B, kScoreWaves * 64>(g, it, blockIdx.x, blocks, lds);
}

template <int B>
static void launch_score_t(const KvxBatch& b, int max_tc, hipStream_t st) {
  if (b.g.score_selects) {
    const size_t lds = score_select_lds_bytes(b.g.H, kScoreWaves, max_tc - b.g.n);
    hipLaunchKernelGGL((score_select_kernel<B>), dim3(score_blocks(b, max_tc), b.n_items), dim3(kScoreWaves * 64), lds, st, b);
    return;
  }
  const int blocks = score_blocks(b, max_tc), waves = score_waves(b.g.H, B, blocks * b.n_items, b.g.n_cus);
  const dim3 grid(blocks, b.n_items), block(64 * waves);
  const size_t lds = score_lds_bytes(b.g.H, waves);
  if (mean_in_score(b, max_tc)) with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((score_kernel<B, true, KVX_ITEMS(bb)>), grid, block, lds, st, bb); });
  else with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((score_kernel<B, false, KVX_ITEMS(bb)>), grid, block, lds, st, bb); });
}

void launch_score(const KvxBatch& b, int max_tc, hipStream_t st) {
  switch (b.g.k_bits) {
    case 2: launch_score_t<2>(b, max_tc, st); break;
    case 4: launch_score_t<4>(b, max_tc, st); break;
    default: launch_score_t<8>(b, max_tc, st); break;
  }
}

}  // namespace kvx
