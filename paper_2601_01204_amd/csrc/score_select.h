// Scoring and selection in one launch, of their own (score_select_kernel) or in front of the attention of a small call
// (attn_tile_kernel).  n_blocks workgroups share a cache's positions; the one that finishes last selects.  Nobody waits for
// anybody: a block that is not the last one leaves.  A block's scores are released once, by its first thread, so that an XCD's
// cache is written back no more often than there are blocks.
#pragma once
#include "score_block.h"
#include "select_block.h"

namespace kvx {

constexpr size_t kMeanLdsBytes = (size_t)(kMeanRows + 1) * kHeadDim * 4;
inline size_t score_select_lds_bytes(int H, int waves, int middle) {
  const size_t a = kMeanLdsBytes + score_lds_bytes(H, waves), b = select_lds_bytes(middle);
  return a > b ? a : b;
}

template <int KB, int THREADS>
__device__ __forceinline__ void score_and_select(const Geometry& g, const Item& it, int block, int n_blocks, void* lds) {
  float* rows = reinterpret_cast<float*>(lds);
  float* mean = rows + kMeanRows * kHeadDim;
  const float qc = pooled_mean(g, it, rows, mean);
  const int first = g.n / 64, total = (it.t_c + 63) / 64 - first;
  for (int x = block; x < total; x += n_blocks) {
    __syncthreads();                          // the dots of the positions before have been read
    score_block<KB>(g, it, (first + x) * 64, mean + kHeadDim, [&]() { return qc; });
  }
  int32_t* done = reinterpret_cast<int32_t*>(cache_scratch(g, it.cache) + g.sl.sel) + 7;
  __shared__ int ticket;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // every wave's scores have left it before the first thread releases them
  __syncthreads();
  if (threadIdx.x == 0) ticket = __hip_atomic_fetch_add(done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (ticket != n_blocks - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (threadIdx.x == 0) __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  select_cache<THREADS>(g, it, reinterpret_cast<int*>(lds));
}

}  // namespace kvx
