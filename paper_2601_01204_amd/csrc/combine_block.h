// Merging the split-KV partials of attention, by blocks of 256 threads: out = sum_s w_s O_s / sum_s w_s l_s, w_s = 2^(m_s - max m).
#pragma once
#include "kvx_dev.h"

namespace kvx {

constexpr int kCombineRows = 16;      // query rows a block merges, sixteen lanes each

// BATCH: partial rows requested before any is used (a register each per lane and channel).
template <int BATCH>
__device__ __forceinline__ void combine_block(const Geometry& g, const Item& it, int item, int h, int block) {
  const int qi = block * kCombineRows + (threadIdx.x >> 4);
  const int c = (threadIdx.x & 15) * 4;
  if (qi >= g.n_new) return;
  const int64_t row0 = ((int64_t)item * g.n_splits * g.H + h) * g.n_pad + qi;
  const int64_t row_step = (int64_t)g.H * g.n_pad;
  float2 ml[kMaxSplits];
  float4 po[BATCH];
#pragma unroll
  for (int s = 0; s < kMaxSplits; ++s) {
    if (s < g.n_splits) {
      const int64_t row = row0 + s * row_step;
      ml[s] = *reinterpret_cast<const float2*>(g.part_ml + row * 2);
      if (s < BATCH) po[s] = *reinterpret_cast<const float4*>(g.part_o + row * kHeadDim + c);
    }
  }
  float m_max = -1.0e30f;               // what a range without a key leaves
#pragma unroll
  for (int s = 0; s < kMaxSplits; ++s)
    if (s < g.n_splits) m_max = fmaxf(m_max, ml[s].x);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  float l = 0.f;
#pragma unroll
  for (int s = 0; s < kMaxSplits; ++s) {
    if (s < g.n_splits) {
      const float w = __builtin_amdgcn_exp2f(ml[s].x - m_max);
      const float4 p = po[s % BATCH];
      acc.x += w * p.x; acc.y += w * p.y; acc.z += w * p.z; acc.w += w * p.w;
      l += w * ml[s].y;
      if constexpr (BATCH < kMaxSplits)
        if (s + BATCH < kMaxSplits && s + BATCH < g.n_splits)
          po[s % BATCH] = *reinterpret_cast<const float4*>(g.part_o + (row0 + (s + BATCH) * row_step) * kHeadDim + c);
    }
  }
  const float inv = 1.0f / l;
  const int64_t off = (int64_t)qi * g.out_tok_stride + (int64_t)h * g.out_head_stride + c;
  if (g.out_f32) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(it.out) + off) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  } else {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 lo = {acc.x * inv, acc.y * inv}, hi = {acc.z * inv, acc.w * inv};
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(it.out) + off) =
        make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2)), __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2)));
  }
}

}  // namespace kvx
