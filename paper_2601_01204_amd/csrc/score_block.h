// Scoring of 64 cache positions by a workgroup (paper Sec. 3.2, Eq. 5-6 and the row mean of Eq. 6): the body of score_kernel and
// of the scoring blocks that ride in the attention launch of a small call.  fp32, one rounding per operation, fixed order of additions
// (compiled without FMA contraction).
#pragma once
#include "kvx_dev.h"

namespace kvx {

__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The mean of the pooled rows (added in ascending order from zero, divided by their number), this lane's channel of it.
// rows: LDS of kMeanRows rows, mean: 64 floats behind.
__device__ __forceinline__ float pooled_mean(const Geometry& g, const Item& it, float* rows, float* mean) {
  const float4* qbar = reinterpret_cast<const float4*>(cache_scratch(g, it.cache) + g.sl.qbar);
  const int lane = threadIdx.x & 63;
  const int n_rows = g.n_pooled * (g.n_new / g.n);
  float acc = 0.f;
  for (int r0 = 0; r0 < n_rows; r0 += kMeanRows) {
    const int cnt = min(kMeanRows, n_rows - r0);
    if (r0) __syncthreads();
    for (int i = threadIdx.x; i < cnt * 16; i += blockDim.x) reinterpret_cast<float4*>(rows)[i] = qbar[(int64_t)r0 * 16 + i];
    __syncthreads();
    if (threadIdx.x < 64) {
#pragma unroll 8
      for (int r = 0; r < cnt; ++r) acc = acc + rows[r * kHeadDim + lane];
    }
  }
  if (threadIdx.x < 64) mean[lane] = acc / (float)n_rows;
  __syncthreads();
  return mean[lane];
}

// One row's codes as floats; 2-bit codes are spread into the bytes of four words.
// f[0..7] = codes of channels 8 o .. 8 o + 7 of a row whose words are w
template <int B>
__device__ __forceinline__ void octet_as_floats(const uint32_t* w, int o, float (&f)[8]) {
  if constexpr (B == 8) {
    bytes_to_floats(w[2 * o], w[2 * o + 1], f);
  } else if constexpr (B == 4) {
    nibbles_to_floats(w[o], f);
  } else {
    const uint32_t x = (w[o >> 1] >> (16 * (o & 1))) & 0xFFFFu;          // eight 2-bit codes
    const uint32_t t = x | (x << 16);                                     // codes 0..3 in bits 0..7, codes 4..7 in bits 24..31
    const uint32_t lo = t & 0x03000003u, m1 = (t >> 2) & 0x03000003u, m2 = (t >> 4) & 0x03000003u, m3 = (t >> 6) & 0x03000003u;
    // byte 0 of each word holds code k, byte 3 holds code k + 4
    f[0] = byte_to_float<0>(lo); f[4] = byte_to_float<3>(lo);
    f[1] = byte_to_float<0>(m1); f[5] = byte_to_float<3>(m1);
    f[2] = byte_to_float<0>(m2); f[6] = byte_to_float<3>(m2);
    f[3] = byte_to_float<0>(m3); f[7] = byte_to_float<3>(m3);
  }
}

// Per head and middle token: D[h, j] = sum over channels of q~[c] K~[h, j, c], K~ = s (code - z) (Eq. 10), evaluated
// with the per-group factors pulled out of the per-token work: a = q~[c] * s[c] and b = -float(z[c]) * a once per
// (head, key group, channel), p[c] = fma(float(code[c]), a[c], b[c]) per token, then the stride-halving pairwise tree
// p[c] += p[c + m] for m = 32, 16, ..., 1.  Then S_j = (D[0, j] + D[1, j] + ... + D[H-1, j]) / H, heads added in order
// (Eq. 4-6), and the order-preserving key of the score.
// A block covers 64 consecutive cache positions of all heads, one token per lane; its waves take turns over the heads (see
// score_waves) and the dots of a token meet in LDS, so they never travel through memory.  Blocks start at a multiple of 64
// positions, so a wave needs the factors of one key group (two of 32 tokens), which it stages for itself.  Bound by vector
// instructions; the code row and the factors of a wave's next head are requested before the arithmetic of this one, and the
// block holds the LDS its waves and heads need and no more, so that six to seven waves a SIMD cover what is left.
// us at 48 caches of 16384 tokens, 4-bit codes, against blocks of one shape for all head counts (32 KB of LDS, eight waves,
// nothing requested ahead): 1 head 27 -> 12, 4 heads 41 -> 30, 9 heads 78 -> 56, 16 heads 112 -> 89; and with the selection
// behind it, against dots through memory and a launch of its own for the head sum: 41 -> 32, 62 -> 50, 86 -> 76, 130 -> 109.
// 24 layers of 782 tokens at a budget of 2048, one call each, 1852 -> 1766 us a frame for the launch saved.
// j0: the block's first position; lds: score_lds_bytes of the heads and waves; mean(): this lane's channel of q~ (a call that
// every thread of the block makes).  Ends without a barrier behind the last use of lds.
template <int B, typename Mean>
__device__ __forceinline__ void score_block(const Geometry& g, const Item& it, int j0, float* lds, Mean&& mean) {
  const uint8_t* half = cache_half(g, it.cache, it.cur);
  uint8_t* sc = cache_scratch(g, it.cache);
  constexpr int kRowWords = 2 * B;                 // 64 channels * B bits / 32
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
  float* s_a = lds + wave * (4 * kHeadDim);        // [2 groups][64] of this wave, b behind a
  float* s_b = s_a + 2 * kHeadDim;
  float* dots = lds + n_waves * (4 * kHeadDim);    // [H][64]

  const int j = j0 + lane;
  const int jl = min(j, it.t_c - 1);
  const int k_shift = g.k_group == 64 ? 6 : 5;      // groups of 64 or 32 tokens
  const int gi = k_shift == 6 ? 0 : lane >> 5;      // the lane's token's group within the block
  // (a group past the cache's end lies inside the buffer; its factors are not used)
  const int grp = j0 >> k_shift;
  uint32_t w[kRowWords];                            // a head's code row of the lane's token
  uint32_t rs[2], rz[2];                            // scale and zero-point of this lane's channel as they are stored
  auto load_head = [&](int h, uint32_t (&w)[kRowWords], uint32_t (&rs)[2], uint32_t (&rz)[2]) __attribute__((always_inline)) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(half + g.lay.k_codes + (int64_t)h * g.t_cap * (8 * B) + (uint32_t)(jl * (8 * B)));
#pragma unroll
    for (int i = 0; i < kRowWords; ++i) w[i] = src[i];
    const int64_t moff = ((int64_t)h * g.g_cap + grp) * kHeadDim;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == 1 && k_shift == 6) break;
      if (g.meta16) {
        rs[q] = (reinterpret_cast<const uint16_t*>(half + g.lay.k_scale) + moff + q * kHeadDim)[meta16_pos(lane)];
        rz[q] = (reinterpret_cast<const uint16_t*>(half + g.lay.k_zero) + moff + q * kHeadDim)[meta16_pos(lane)];
      } else {
        rs[q] = (reinterpret_cast<const uint32_t*>(half + g.lay.k_scale) + moff + q * kHeadDim)[lane];
        rz[q] = (reinterpret_cast<const uint32_t*>(half + g.lay.k_zero) + moff + q * kHeadDim)[lane];
      }
    }
  };
  load_head(min(wave, g.H - 1), w, rs, rz);      // requested first: its latency runs beside the row mean (no branch around it)
  const float qc = mean();
  for (int h = wave; h < g.H; h += n_waves) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == 1 && k_shift == 6) break;
      float sv, zf;
      if (g.meta16) {
        // halves: logit-domain scale a16 (s = a16 * fp32(1 / scale_log2)) and 1024 + z, channels of an octet in the order 0 4 1 5 2 6 3 7
        sv = (float)__builtin_bit_cast(_Float16, (uint16_t)rs[q]) * g.inv_scale_log2;
        zf = (float)__builtin_bit_cast(_Float16, (uint16_t)rz[q]) - 1024.0f;
      } else {
        sv = __uint_as_float(rs[q]);
        zf = (float)(int32_t)rz[q];
      }
      const float a = qc * sv;
      s_a[q * kHeadDim + lane] = a;
      s_b[q * kHeadDim + lane] = (-zf) * a;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");    // the factors cross lanes of this wave only
    __builtin_amdgcn_wave_barrier();

    uint32_t wn[kRowWords], rsn[2], rzn[2];         // of the next head this wave takes
    const bool more = h + n_waves < g.H;
    if (more) load_head(h + n_waves, wn, rsn, rzn);
    // The tree's upper levels octet by octet: m = 32 adds octet o + 4 to octet o, m = 16 octet 2 to 0 and 3 to 1, m = 8
    // octet 1 to 0.  The same additions in an order that keeps few octets at a time in registers.
    auto octet = [&](int o, float (&x)[8]) __attribute__((always_inline)) {
      float f[8];
      octet_as_floats<B>(w, o, f);
      const float* pa = s_a + gi * kHeadDim + 8 * o;
      const float* pb = s_b + gi * kHeadDim + 8 * o;
      const float4 a0 = *reinterpret_cast<const float4*>(pa), a1 = *reinterpret_cast<const float4*>(pa + 4);
      const float4 b0 = *reinterpret_cast<const float4*>(pb), b1 = *reinterpret_cast<const float4*>(pb + 4);
      const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w}, c[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(f[e], a[e], c[e]);
    };
    float p[8], p1[8];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const int lo = ((o & 1) << 1) | (o >> 1);      // octets 0, 2, 1, 3
      float x[8], y[8];
      octet(lo, x);
      octet(lo + 4, y);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float v = x[e] + y[e];
        if (o == 0) p[e] = v;
        else if (o == 1) p[e] = p[e] + v;
        else if (o == 2) p1[e] = v;
        else p1[e] = p1[e] + v;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = p[e] + p1[e];
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) {
#pragma unroll
      for (int c = 0; c < m; ++c) p[c] = p[c] + p[c + m];
    }
    dots[h * 64 + lane] = p[0];
    __builtin_amdgcn_wave_barrier();
    if (!more) break;
#pragma unroll
    for (int i = 0; i < kRowWords; ++i) w[i] = wn[i];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == 1 && k_shift == 6) break;
      rs[q] = rsn[q];
      rz[q] = rzn[q];
    }
  }
  __syncthreads();
  if (wave == 0 && j >= g.n && j < it.t_c) {
    float acc = dots[lane];
#pragma unroll 4
    for (int h = 1; h < g.H; ++h) acc = acc + dots[h * 64 + lane];
    const float s = acc / (float)g.H;
    reinterpret_cast<float*>(sc + g.sl.scores)[j - g.n] = s;
    reinterpret_cast<uint32_t*>(sc + g.sl.keys)[j - g.n] = order_key(s);
  }
}

}  // namespace kvx
