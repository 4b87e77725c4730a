// Top-k selection and keep list (paper Sec. 3.2): keep the first frame, the k best
// middle tokens (k = L_max - T_first - T_current) and the current frame, in ascending
// position order.  Integer work throughout: scores are compared through an
// order-preserving uint32 image of their fp32 bits, equal scores keep the lower
// position, so the result is unique and bit-exact.
//
// One workgroup per cache, bound by latency: the number of block barriers
// and the instructions fetched for the first time, not the work per key.  The keys go to
// LDS once (their first digit is counted on the way) and every later pass is a short loop
// over them, so the code stays small whatever the cache's length.  A 3-pass
// most-significant-digit-first radix select (12, 10 and 10 bits, a histogram each, all
// cleared up front) finds the key of the last token to drop; the first digit takes sign,
// exponent and three mantissa bits, so scores of one magnitude still spread over several
// bins and the LDS atomics of a wave rarely pile onto one address.  Then every wave takes a
// contiguous run of positions, counts its kept and its equal-to-threshold keys by ballots,
// and after one barrier writes its survivors in position order at the offset the earlier
// waves' counts give.
#pragma once
#include "kvx_dev.h"

namespace kvx {

constexpr int kSelWaves = 16;                          // at most
constexpr int kSelBins0 = 4096, kSelBins = 1024;       // bins of the first and of the two later digits

// Of PER consecutive bins per thread, find the bin that holds the sh[1]-th smallest candidate (counting from 1):
// that bin is added to the prefix sh[0], sh[1] becomes the rank within it and sh[2] its count.  Ends with a barrier.
template <int PER>
__device__ __forceinline__ void find_bin(const int* hist, int shift, int* wave_sums, volatile int* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int c[PER], cnt = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) { c[j] = hist[threadIdx.x * PER + j]; cnt += c[j]; }
  int inc = cnt;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(inc, d);
    if (lane >= d) inc += t;
  }
  if (lane == 63) wave_sums[wave] = inc;
  const int rem = sh[1];
  const uint32_t prefix = (uint32_t)sh[0];
  __syncthreads();
  int before = inc - cnt;
  for (int w = 0; w < wave; ++w) before += wave_sums[w];
  if (before < rem && before + cnt >= rem) {            // exactly one thread
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (before < rem && before + c[j] >= rem) {
        sh[0] = (int)(prefix | ((uint32_t)(threadIdx.x * PER + j) << shift));
        sh[1] = rem - before;
        sh[2] = c[j];
        before = rem;                                   // no later bin matches
      } else {
        before += c[j];
      }
    }
  }
  __syncthreads();
}

// LDS: histograms, then the keys: at most 24 KB + 128 KB
constexpr int kSelLdsInts = kSelBins0 + 2 * kSelBins;
constexpr size_t select_lds_bytes(int middle) { return (size_t)(kSelLdsInts + (middle > 0 ? middle : 0)) * 4; }

// The selection of one cache by a workgroup of THREADS threads; lds: select_lds_bytes of its middle tokens.
template <int THREADS>
__device__ __forceinline__ void select_cache(const Geometry& g, const Item& it, int* lds) {
  constexpr int kSelThreads = THREADS, kWaves = THREADS / 64;
  const int n = g.n, t_c = it.t_c;
  const int n_cur = g.n_new;             // the call's tokens: always kept
  const int M = t_c - n;                 // middle tokens: cache positions n .. t_c - 1
  const int T = t_c + n_cur;
  const int n_drop = T - g.budget;       // >= 1
  const int k_keep = M - n_drop;         // = budget - n - n_cur
  uint8_t* sc = cache_scratch(g, it.cache);
  const uint32_t* keys = reinterpret_cast<const uint32_t*>(sc + g.sl.keys);
  int32_t* keep = reinterpret_cast<int32_t*>(sc + g.sl.keep);
  int32_t* sel = reinterpret_cast<int32_t*>(sc + g.sl.sel);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  int* hist0 = lds;
  int* hist1 = lds + kSelBins0;
  int* hist2 = hist1 + kSelBins;
  uint32_t* key = reinterpret_cast<uint32_t*>(lds + kSelLdsInts);
  __shared__ int wave_sums[3][kSelWaves];
  __shared__ int wave_gt[kSelWaves], wave_eq[kSelWaves];
  __shared__ int sh[3];                  // prefix (as bits), rank wanted, count of the found bin
  __shared__ int sh_p0;

  for (int i = tid; i < kSelLdsInts; i += kSelThreads) lds[i] = 0;
  if (tid == 0) {
    sh[0] = 0;
    sh[1] = n_drop;
    sh_p0 = T;
  }
  __syncthreads();
  // Key of the n_drop-th smallest element, digit by digit.
  constexpr int kBatch = 8;                              // keys requested before any is counted
  for (int b0 = tid; b0 < M; b0 += kBatch * kSelThreads) {
    uint32_t k[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) k[u] = keys[min(b0 + u * kSelThreads, M - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = b0 + u * kSelThreads;
      if (i < M) {
        key[i] = k[u];
        atomicAdd(&hist0[k[u] >> 20], 1);
      }
    }
  }
  __syncthreads();
  find_bin<kSelBins0 / kSelThreads>(hist0, 20, wave_sums[0], sh);
  const uint32_t top = (uint32_t)sh[0] >> 20;
  for (int b0 = tid; b0 < M; b0 += kBatch * kSelThreads) {
    uint32_t k[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) k[u] = key[min(b0 + u * kSelThreads, M - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (b0 + u * kSelThreads < M && k[u] >> 20 == top) atomicAdd(&hist1[(k[u] >> 10) & (kSelBins - 1)], 1);
  }
  __syncthreads();
  find_bin<kSelBins / kSelThreads>(hist1, 10, wave_sums[1], sh);
  const uint32_t top2 = (uint32_t)sh[0] >> 10;
  for (int b0 = tid; b0 < M; b0 += kBatch * kSelThreads) {
    uint32_t k[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) k[u] = key[min(b0 + u * kSelThreads, M - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (b0 + u * kSelThreads < M && k[u] >> 10 == top2) atomicAdd(&hist2[k[u] & (kSelBins - 1)], 1);
  }
  __syncthreads();
  find_bin<kSelBins / kSelThreads>(hist2, 0, wave_sums[2], sh);
  const uint32_t thr = (uint32_t)sh[0];
  const int eq_keep = sh[2] - sh[1];             // equal-keyed tokens kept: the eq_keep lowest positions

  // This wave's run of positions, 64 at a time.
  const int run = ((M + kSelThreads - 1) / kSelThreads) * 64;
  const int i0 = min(wave * run, M), i1 = min(i0 + run, M);
  int gt = 0, eq = 0;
  for (int b0 = i0 + lane; b0 - lane < i1; b0 += kBatch * 64) {
    uint32_t k[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) k[u] = key[min(b0 + u * 64, M - 1)];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const bool in = b0 + u * 64 < i1;
      gt += __popcll(__ballot(in && k[u] > thr));
      eq += __popcll(__ballot(in && k[u] == thr));
    }
  }
  if (lane == 0) {
    wave_gt[wave] = gt;
    wave_eq[wave] = eq;
  }
  // the first frame and the call's own tokens are always kept
  for (int i = tid; i < n; i += kSelThreads) keep[i] = i;
  for (int i = tid; i < n_cur; i += kSelThreads) keep[n + k_keep + i] = t_c + i;
  // slot layout: the freed slots in ascending order, then the never-used tail, take the call's tokens in order
  int32_t* newtok = reinterpret_cast<int32_t*>(sc + g.sl.newtok);
  int32_t* assign = reinterpret_cast<int32_t*>(sc + g.sl.assign);
  if (g.slots) {
    for (int i = tid; i < n; i += kSelThreads) newtok[i] = -1;
    for (int sl = t_c + tid; sl < g.budget; sl += kSelThreads) {
      const int d = n_drop + (sl - t_c);
      assign[d] = sl;
      newtok[sl] = d;
    }
  }
  __syncthreads();
  int gt_before = 0, eq_before = 0, tot_gt = 0;
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) { gt_before += wave_gt[w]; eq_before += wave_eq[w]; }
    tot_gt += wave_gt[w];
  }
  int out = gt_before + min(eq_before, eq_keep);   // survivors in front of this wave's run
  const uint64_t below = (1ull << lane) - 1ull;
  int first_drop = T;
  for (int i = i0 + lane; i - lane < i1; i += 64) {
    const bool in = i < i1;
    const uint32_t k = in ? key[i] : 0u;
    const uint64_t is_eq = __ballot(in && k == thr);
    const bool kept = in && (k > thr || (k == thr && eq_before + __popcll(is_eq & below) < eq_keep));
    const uint64_t is_kept = __ballot(kept);
    const int pos = out + __popcll(is_kept & below);
    if (kept) {
      keep[n + pos] = n + i;
      if (g.slots) newtok[n + i] = -1;
    } else if (in) {
      first_drop = min(first_drop, n + i);
      if (g.slots) {
        const int d = i - pos;             // dropped tokens before this one
        assign[d] = n + i;
        newtok[n + i] = d;
      }
    }
    out += __popcll(is_kept);
    eq_before += __popcll(is_eq);
  }
  if (first_drop < T) atomicMin(&sh_p0, first_drop);
  __syncthreads();
  if (tid == 0) {
    sel[0] = sh_p0;
    sel[1] = sh_p0 / g.k_group;
    sel[3] = tot_gt + eq_keep;                    // survivors among the middle tokens (= k)
  }
}

}  // namespace kvx
