// Attention of one frame's queries over [de-quantised cache ; the frame's own K/V] (paper Sec. 3.1 Eq. 1 with the
// de-quantisation of Sec. 3.3 Eq. 10 fused in), bf16 inputs; fp32 inputs have a kernel of their own (attn.hip).
//
// Work decomposition.  A workgroup of eight waves, two per SIMD at 256 registers, owns up to twelve 32-row query blocks of one
// head (wave w block w, waves 0-3 also block 8 + w) and a contiguous range of 64-key tiles (split-KV, merged by combine_kernel).
// Waves 4-7 stage: each decodes a quarter of the codes of a K and of a V tile into LDS (K row-major, V transposed), two tiles
// and one tile ahead of their use, three tiles of each in LDS, one barrier per tile.  The staging waves own at most one block,
// their SIMD's other wave up to two, and run at raised priority: what they produce everybody waits for.
//
// Products.  S^T = K Q^T and O^T += V^T P^T on the matrix cores (32 x 32 x 16).  The transposed products put a query in a lane
// and its keys in that lane's registers, so the probabilities feed the second product straight from registers; the key order
// inside a 16-key step is a permutation shared by V^T's LDS layout.  Queries stay in registers.
//   16-bit metadata (per key group and channel the logit-domain scale a = s * softmax scale * log2(e) with 7 significant bits
//     and 1024 + z, halves): a de-quantised key times the logit factor, a (code - z), is exact in a half and so are bf16
//     queries: one f16 instruction per step.  The code word is spread into halves 1024 + code by masks, 1024 + z is subtracted
//     exactly, the difference multiplied by a.  Octets of channels lie in the order 0 4 1 5 2 6 3 7 the masks produce.
//   fp32 metadata: s (code - z) is an fp32 value; rounded to 8 bits it would perturb the logits of the dominant channels by
//     1e-2, so a cached key is staged as a bf16 pair hi + lo (16 significand bits) and takes two bf16 instructions per step.
//   The frame's own keys and an uncompressed cache: bf16 as they are, one instruction per step from a zero accumulator, the
//     logit factor applied to the logits by the fused operation that subtracts the softmax reference.
// P and V go through the f16 instruction in every format.
//
// Softmax.  p = 2^(s - m) with m the largest logit of the range's first tile, without a prior maximum: cached logits leave the
// matrix core as s - m, because the first instruction takes a block of 16 copies of -m as its accumulator.  f16 holds p up to 2^16;
// a key further above m makes p and the unit's row sum infinite, and only then (rare, wave-uniform) is m raised, O and l rescaled
// and the probabilities formed again.  (m from the first 32 keys instead: in a small cache one row in ten has its largest key,
// whose p of 1 does not round, among the others; the error of 230 tokens at a budget of 1200 was 5 % higher.)
//
// Schedule.  The unit of work is 32 keys x one query block.  A step runs three units at once, the first product of one, the
// softmax of the unit before and the second product of the one before that: nothing in it depends on anything else in it, and
// the source interleaves each matrix instruction (32 cycles) with two or three vector instructions that run under it.  Row sums
// are matrix instructions too (below): v_dot2_f32_f16 shares the matrix core's operand path, and one of them per matrix
// instruction costs 16 cycles (8 matrix instructions 258 cycles, with a dot product behind each 388, with 24 exponentials 266).
// What bounds it, in cycles per tile of a SIMD with three blocks (six units): vector issue (96 exponentials of 8, 48 conversions of
// 4, the staging's 75 instructions of 4, 60 matrix instructions of about 9: 1800, addresses, checks and LDS operations on top) and
// matrix work (1730, 2500 with key pairs) against some 2800 measured (3700 with key pairs), at a clock that power holds to 1.87 GHz
// (2.11 for the kernel before, which idled more).
// Against one block a wave, twelve waves, product - softmax - product one after the other and all waves staging, us a launch:
// 24 caches of 16384 tokens, 1041 queries, 4-bit codes: 16-bit metadata 2030 -> 1783, fp32 2735 -> 2452; 48 caches of 24576,
// 1374 queries, 2-bit keys 7718 -> 6690; four frames of 1041 on one cache of 8192 284 -> 250; one frame on it, fp32 metadata
// 82.6 -> 74.4.  Staging by all eight waves, K first and V last, took 1885 where the four staging waves take 1783; without
// their raised priority they take 1877.
//
// Domain: finite inputs, |v| below 65504 (the half range); 16-bit metadata: also |q|, |k| of the call's own tokens as they are, and
// |k * softmax scale * log2 e| of those in the cache.  A query row outside it spoils its own output row only.
#pragma once
#include "score_select.h"

#include <hip/hip_ext.h>

#include <type_traits>
#include <utility>

namespace kvx {
namespace tile {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kLdsRow = 72;                       // halves per LDS row: 64 + 8 pad (144 B)
constexpr int kTileElems = kTileK * kLdsRow;      // one K or V^T tile
constexpr float kNegBig = -1.0e30f;
constexpr float kRescaleGap = 8.0f;               // log2 units
constexpr int kThreads = 512;                     // eight waves, two per SIMD, of one or two 32-row query blocks each
constexpr int kBufs = 3;                          // tiles of K and of V in LDS
constexpr float kSumLimit = 1.0e37f;              // a row sum at or above this (or NaN) saw a half overflow
constexpr uint32_t kBias = 0x64006400u;           // two halves of 1024

__device__ __forceinline__ int swap23(int x) { return (x & ~0xC) | ((x & 4) << 1) | ((x & 8) >> 1); }

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2 x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  const f32x2 x = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, f16x2));
}
__device__ __forceinline__ f16x2 as_h2(uint32_t w) { return __builtin_bit_cast(f16x2, w); }
__device__ __forceinline__ uint32_t as_u(f16x2 h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ float bf16lo_to_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi_to_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Eight bf16 values (channels 0..7 of an octet, two per word) as four half pairs in the octet order
// (0,4) (1,5) (2,6) (3,7).  bf16 -> half is exact inside the half range.
__device__ __forceinline__ uint4 bf16_octet_to_half_pairs(const uint4& r) {
  return make_uint4(pack_f16(bf16lo_to_f32(r.x), bf16lo_to_f32(r.z)), pack_f16(bf16hi_to_f32(r.x), bf16hi_to_f32(r.z)),
                    pack_f16(bf16lo_to_f32(r.y), bf16lo_to_f32(r.w)), pack_f16(bf16hi_to_f32(r.y), bf16hi_to_f32(r.w)));
}

// Code words as they are loaded: four bytes (8-bit value codes in the launch: eight) with the codes of eight consecutive
// channels of a row somewhere in them; 2-bit codes take half a word, `sel` says which (a v_perm selector).
typedef uint32_t u32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool WIDE> struct CodeWord { uint32_t x; };
template <> struct CodeWord<true> { uint32_t x, y; };

// Eight key codes as four pairs of halves 1024 + code: channels (0,4) (1,5) (2,6) (3,7).
template <int B>
__device__ __forceinline__ void key_pairs(uint32_t w, uint32_t sel, uint32_t bias, uint32_t (&p)[4]) {
  if constexpr (B == 2) w = __builtin_amdgcn_perm(w, w, sel);      // codes 0-3 in byte 0, 4-7 in byte 2
  constexpr uint32_t mask = B == 4 ? 0x000F000Fu : 0x00030003u;
#pragma unroll
  for (int j = 0; j < 4; ++j) p[j] = ((w >> (B * j)) & mask) | bias;
}
// Eight channels' codes of two value rows a, b as eight pairs of halves 1024 + code, row a's in the low half and row b's in
// the high one: the form in which they are stored, so that nothing is permuted afterwards.
template <int B, typename W>
__device__ __forceinline__ void val_pairs(const W& a, const W& b, uint32_t sel, uint32_t bias, uint32_t (&p)[8]) {
  if constexpr (B == 8) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      p[e] = __builtin_amdgcn_perm(e < 4 ? b.x : b.y, e < 4 ? a.x : a.y, 0x0C040C00u + 0x00010001u * (uint32_t)(e & 3)) | bias;
  } else if constexpr (B == 4) {
    const uint32_t lo = __builtin_amdgcn_perm(b.x, a.x, 0x05040100u), hi = __builtin_amdgcn_perm(b.x, a.x, 0x07060302u);
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = (((e < 4 ? lo : hi) >> (4 * (e & 3))) & 0x000F000Fu) | bias;
  } else {
    const uint32_t w = __builtin_amdgcn_perm(b.x, a.x, sel);
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = ((w >> (2 * e)) & 0x00030003u) | bias;
  }
}

// The codes of eight channels as floats.  half_shift: 16 where the eight 2-bit codes are in the word's upper half.
template <int B, typename W>
__device__ __forceinline__ void code_floats(const W& w, uint32_t half_shift, float (&f)[8]) {
  if constexpr (B == 8) {
    bytes_to_floats(w.x, w.y, f);
  } else if constexpr (B == 4) {
    nibbles_to_floats(w.x, f);
  } else {
    const uint32_t x = w.x >> half_shift;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = (float)((x >> (2 * e)) & 0x3u);
  }
}
// Two fp32 values -> packed bf16 truncations (hi) and packed bf16 truncated remainders (lo).
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t& hi, uint32_t& lo) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  hi = __builtin_amdgcn_perm(ub, ua, 0x07060302u);          // the upper halves of a (low) and b (high)
  const float ra = a - __uint_as_float(ua & 0xFFFF0000u), rb = b - __uint_as_float(ub & 0xFFFF0000u);
  lo = __builtin_amdgcn_perm(__float_as_uint(rb), __float_as_uint(ra), 0x07060302u);
}

// The larger, and the sum, of a lane's value and that of the lane 32 away.
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float add_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// What the cache holds.
enum Format {
  kMeta16,    // codes with 16-bit metadata: keys staged as exact halves that carry the logit factor
  kMeta32,    // codes with fp32 scales and zero-points: keys staged as bf16 pairs hi + lo that carry the logit factor
  kBf16,      // uncompressed bf16 rows: keys as they are, the logit factor is applied to their logits
};

// Linear block id -> (column, query tile), column = (item, split, head).  Workgroups go to the 8 XCDs round-robin by
// id and each XCD has its own L2, so the query tiles of one column, which read the same K/V codes, get ids that are
// multiples of 8 apart and next to each other in dispatch order: they run on one XCD at about the same time and the
// second and third read of a tile is served by that XCD's L2 instead of HBM.  Columns are taken in groups of 8 (the
// last group may be smaller): id = group * 8 * n_qtiles + qt * group_size + (column within the group).
__device__ __forceinline__ void decode_block(int bid, int n_cols, int n_qtiles, int& col, int& qt) {
  const int per_group = 8 * n_qtiles;
  const int grp = bid / per_group;
  const int rest = bid - grp * per_group;
  const int gsize = min(8, n_cols - grp * 8);
  qt = rest / gsize;
  col = grp * 8 + (rest - qt * gsize);
}

template <int I> using Int = std::integral_constant<int, I>;
#define KVX_PIN() __builtin_amdgcn_sched_barrier(0)

template <Format FMT, int KB, int VB, int N>
__global__ __launch_bounds__(kThreads) void attn_tile_kernel(const KvxBatchT<N> b) {
  const Geometry& g = b.g;
  constexpr int kParts = FMT == kMeta32 ? 2 : 1;          // operands a cached key is staged as
  constexpr int kLdsV = kParts * kBufs * kTileElems;      // the tiles of V lie behind those of K: one lane offset addresses both
  constexpr bool kSide = FMT != kBf16;                    // the launch may carry scoring blocks
  constexpr int kLdsElems = kLdsV + kBufs * kTileElems, kSideElems = (int)select_lds_bytes(32768) / 2;
  __shared__ __attribute__((aligned(16))) uint16_t lds[kSide && kSideElems > kLdsElems ? kSideElems : kLdsElems];
  int side = 0;
  if constexpr (kSide) {
    side = g.side_blocks * b.n_items;
    if ((int)blockIdx.x < side) {
      const Item it = b.items[blockIdx.x / g.side_blocks];
      if (it.prune) score_and_select<KB, kThreads>(g, it, blockIdx.x % g.side_blocks, g.side_blocks, lds);
      return;
    }
  }
  int bid, qt;
  decode_block((int)blockIdx.x - side, g.H * g.n_splits * b.n_items, g.n_qtiles, bid, qt);
  const int h = bid % g.H; bid /= g.H;
  const int split = bid % g.n_splits; bid /= g.n_splits;
  const int item_idx = bid;
  const Item it = b.items[item_idx];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;
  const int hf = lane >> 5;

  const int n = g.n_new;                                  // query rows = the call's own keys: one frame, or a chunk of frames
  const int t_c = it.t_c;
  const int ntc = (t_c + kTileK - 1) / kTileK;            // cache tiles
  const int nto = g.own_tiles ? (n + kTileK - 1) / kTileK : 0;   // tiles of the call's own keys (none when they are in the cache already)
  const int nt = ntc + nto;
  const int tile_begin = (int)(((int64_t)nt * split) / g.n_splits);
  const int tile_end = (int)(((int64_t)nt * (split + 1)) / g.n_splits);

  const uint8_t* half = cache_half(g, it.cache, it.cur);
  // The frame's own keys (and those of an uncompressed cache) enter the product as they are and the logit factor is applied to
  // their logits.  bf16 products could then leave fp32's range where the logit does not, so that a factor below one is taken
  // in two parts: its power of two with the queries (exact, once per workgroup), the rest with the logits or the cached keys.
  const int sc_exp = FMT != kMeta16 ? max(min((int)(__float_as_uint(g.scale_log2) >> 23) - 127, 0), -126) : 0;
  const float q_factor = __uint_as_float((uint32_t)(127 + sc_exp) << 23), sc = FMT != kMeta16 ? ldexpf(g.scale_log2, -sc_exp) : g.scale_log2;

  // ---- the wave's query blocks: block `wave`, and block 8 + wave where the tile has that many ----
  auto run = [&](auto nbc, auto stagec) __attribute__((always_inline)) {
    constexpr int NB = decltype(nbc)::value;
    constexpr bool STAGER = decltype(stagec)::value;
    constexpr int NA = NB > 0 ? NB : 1;      // array bounds
    constexpr int U = 2 * NB;                // units per tile: (key half, block), blocks innermost
    // LDS buffers (element offsets) of tiles t, t + 1 and t + 2 (which is that of tile t - 1 too)
    int r0 = 0, r1 = kTileElems, r2 = 2 * kTileElems;
    if constexpr (STAGER) __builtin_amdgcn_s_setprio(1);
    f32x16 o[NA][2];                         // O^T, [channel block]
    f32x16 negm[NA];                         // 16 copies of -m, the accumulator input of a cached unit's first MFMA
    uint4 qf[NA][4];                         // query fragments (B operand of S^T = K Q^T): halves, octets permuted, or bf16
    float l[NA];                             // row sums
    bool started[NA];                        // the block has a reference (its first tile sets m)
    int row0[NA];
    // own keys a query may see (frame-wise causal mask, Sec. 3.1): the smallest and the largest number over the wave's rows
    int limit_lo = 1 << 30, limit_hi = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      row0[i] = (qt * g.q_blocks + wave + 8 * i) * 32;
      limit_lo = min(limit_lo, (min(row0[i], n - 1) / g.n + 1) * g.n);
      limit_hi = max(limit_hi, (min(row0[i] + 31, n - 1) / g.n + 1) * g.n);
      const int qi = min(row0[i] + l32, n - 1);
      const uint8_t* qrow = reinterpret_cast<const uint8_t*>(it.q) + ((int64_t)qi * g.tok_stride + (int64_t)h * g.head_stride + hf * 8) * 2;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint4 x = *reinterpret_cast<const uint4*>(qrow + 32 * ks);
        if constexpr (FMT == kMeta16) {
          qf[i][ks] = bf16_octet_to_half_pairs(x);
        } else {
          // (a word's lower half rides along in the upper one's significand and is cut off again)
          auto scaled = [&](uint32_t w) __attribute__((always_inline)) {
            return __builtin_amdgcn_perm(__float_as_uint(__uint_as_float(w) * q_factor), __float_as_uint(__uint_as_float(w << 16) * q_factor), 0x07060302u);
          };
          qf[i][ks] = make_uint4(scaled(x.x), scaled(x.y), scaled(x.z), scaled(x.w));
        }
      }
      started[i] = false;
#pragma unroll
      for (int r = 0; r < 16; ++r) { negm[i][r] = 0.f; o[i][0][r] = 0.f; o[i][1][r] = 0.f; }
      l[i] = 0.f;
    }
    // A operand of the row sums.  v_mfma_f32_16x16x32_f16 (16 cycles) reads a fragment of probabilities (32 queries x 16 keys)
    // as 16 columns of 32, column c holding the keys of queries c and 16 + c in alternating octets; rows 0-3 and 8-11 of this
    // matrix pick the first, rows 4-7 and 12-15 the second, which is where the results of lanes 0-15 and 32-47 and of the
    // others come from: every lane receives its query's sum over both halves' keys.
    const _Float16 pick = ((lane >> 2) & 1) == ((lane >> 4) & 1) ? (_Float16)1.0f : (_Float16)0.0f;
    const f16x8 ones = {pick, pick, pick, pick, pick, pick, pick, pick};

    uint4 kf[4];
    f16x8 vf[2][2];
    const int lane_off = l32 * kLdsRow + hf * 8;
    auto read_k = [&](int part, int i, int buf, int kh) __attribute__((always_inline)) {
      return *reinterpret_cast<const uint4*>(lds + (lane_off + buf) + (part * (kBufs * kTileElems) + kh * 32 * kLdsRow + i * 16));
    };
    auto mma_k = [&](const uint4& k, const uint4& q, const f32x16& acc) __attribute__((always_inline)) {
      if constexpr (FMT == kMeta16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, k), __builtin_bit_cast(f16x8, q), acc, 0, 0, 0);
      else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, q), acc, 0, 0, 0);
    };
    // the first product of one key half and one block, from operands fetched for it (what is not pipelined)
    auto logits = [&](auto partsc, int i, int buf, int kh) __attribute__((always_inline)) {
      constexpr int P = decltype(partsc)::value;
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int part = 0; part < P; ++part) s = mma_k(read_k(part, ks, buf, kh), qf[i][ks], s);
      return s;
    };
    auto read_v = [&](int kk, int cb, int buf, int kh) __attribute__((always_inline)) {
      vf[kk][cb] = *reinterpret_cast<const f16x8*>(lds + (lane_off + buf) + (kLdsV + cb * 32 * kLdsRow + (2 * kh + kk) * 16));
    };
    auto frag = [](const uint32_t (&w)[8], int kk) __attribute__((always_inline)) { return __builtin_bit_cast(f16x8, make_uint4(w[4 * kk], w[4 * kk + 1], w[4 * kk + 2], w[4 * kk + 3])); };
    const f32x4 no_sum = {0.f, 0.f, 0.f, 0.f};
    auto sums = [&](const uint32_t (&w)[8]) __attribute__((always_inline)) {
      const f32x4 x = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, frag(w, 0), no_sum, 0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, frag(w, 1), x, 0, 0, 0)[0];
    };
    // The same sum lane by lane, for units in which some row saw infinities or NaNs: there the ones matrix's zeros times that
    // row's probabilities would spoil the sum of the row it shares a column with (slower, and rare).
    auto lane_sums = [&](const uint32_t (&w)[8]) __attribute__((always_inline)) {
      const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
      float x = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) x = __builtin_amdgcn_fdot2(as_h2(w[e]), one, x, false);
      return add_halves(x);
    };
    auto probabilities = [&](const f32x16& s, uint32_t (&w)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = pack_f16(__builtin_amdgcn_exp2f(s[2 * e]), __builtin_amdgcn_exp2f(s[2 * e + 1]));
    };
    // Sets m of a block: to the largest logit of its first tile (`a`: over this lane's keys, before the factor f).
    auto set_reference = [&](int i, float a, float f) __attribute__((always_inline)) {
      const float mq = max_halves(a);                              // both halves of a query agree
      // rounded down, so that the largest key's fused logit below is not negative: near the top of fp32 the rounding error of m is
      // more than the exponent's range, and that key would be lost (above the range it raises m).  A sum that starts from -m
      // is rounded elsewhere than one from zero: the margin where that could be as much.
      float m0 = mq * f;
      const uint32_t u = __float_as_uint(m0);
      if (__builtin_fmaf(mq, f, -m0) < 0.f && (u << 1) != 0) m0 = __uint_as_float((int32_t)u < 0 ? u + 1 : u - 1);
      if (FMT != kBf16 && fabsf(m0) >= 0x1p20f) m0 = __builtin_fmaf(fabsf(m0), -0x1p-16f, m0);
      // a query that sees none of the tile's keys (all masked) keeps zero
      m0 = mq > -__builtin_inff() ? m0 : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) negm[i][r] = -m0;
      asm volatile("" : "+v"(negm[i]));     // opaque: the block stays in its registers
      started[i] = true;
    };
    // Raises m of the rows whose logits exceed it by more than the gap, rescales what has been accumulated and forms the unit's
    // probabilities again.  Returns the raise.
    auto raise = [&](int i, f32x16& s, uint32_t (&w)[8]) __attribute__((always_inline)) {
      float a = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) a = fmaxf(a, s[r]);
      const float mq = max_halves(a);
      const float delta = mq > kRescaleGap ? mq : 0.f;
      const float alpha = __builtin_amdgcn_exp2f(-delta);
      const float nm = negm[i][0] - delta;
      l[i] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o[i][0][r] *= alpha;
        o[i][1][r] *= alpha;
        s[r] -= delta;
        negm[i][r] = nm;
      }
      asm volatile("" : "+v"(negm[i]));
      probabilities(s, w);
      return delta;
    };

    // ---- staging: 256 threads (waves 4-7), each two rows x eight channels of K and of V ----
    constexpr int kKRow = 8 * KB;     // bytes per cached key row (codes of KB bits; KB = 16: bf16)
    constexpr int kVRow = 8 * VB;
    const int st = tid & 255;
    // K: consecutive lanes read consecutive words; the two rows, 16 apart, are of one key group.  V: two adjacent keys,
    // consecutive lanes write consecutive words.
    const int k_oct = st & 7, v_oct = st >> 5;
    const int k_row = ((st >> 3) & 15) | ((st >> 2) & 32), v_row = swap23(2 * (st & 31));
    const int ngv = kHeadDim / g.v_group;
    const int k_shift = g.k_group == 64 ? 6 : 5;
    const int v_shift = g.v_group == 64 ? 6 : 5;
    uint32_t bias = kBias;
    asm volatile("" : "+v"(bias));                          // in a register, so that mask and bias are one instruction
    // which half of a word holds the thread's eight 2-bit codes
    const uint32_t k_sel = (k_oct & 1) ? 0x0C030C02u : 0x0C010C00u, v_sel = (v_oct & 1) ? 0x07060302u : 0x05040100u;
    const uint32_t k_half = (k_oct & 1) * 16, v_half = (v_oct & 1) * 16;

    // A tile's raw data stays in registers for one tile's time before it is decoded.  Whatever the tile holds, the same four
    // loads a tensor fill the same registers (only the addresses differ), so that nothing waits for them before they are used.
    //   cached K: c, d = the rows' codes, a = the eight channels' scales, b = their zero-points (16-bit metadata: halves, 1024 + z;
    //             fp32 and int32 metadata: a2, b2 the second four channels)
    //   cached V: c, d = the rows' codes, a, b begin with their scales and zero-points; the rest is what lies behind
    //   bf16 rows (own K, V, uncompressed cache): a, b = the two rows; c, d, a2, b2 are loaded from the same place and not used
    constexpr bool kWide = KB == 8 || VB == 8;
    typedef CodeWord<kWide> Code;
    struct Feed {
      Code c, d;
      u32x4_a4 a, b, a2, b2;
      // where the next tile to be requested lies (uniform pointers) and the thread's part of it (offsets); tiles are
      // requested in order, so the pointers only advance
      const uint8_t *p_c, *p_d, *p_a, *p_b;
      int64_t code_step, meta_step;
      uint32_t off_code, off_a, off_b;
      int next, hi;                       // hi: bytes from a to a2
    } fk, fv;
    auto seek_own = [&](Feed& f, const void* base, int row, int row_step, int oct, int trow) __attribute__((always_inline)) {
      f.p_a = reinterpret_cast<const uint8_t*>(base) + ((int64_t)trow * g.tok_stride + (int64_t)h * g.head_stride) * 2;
      f.p_b = f.p_a + (int64_t)row_step * g.tok_stride * 2;
      f.off_a = ((uint32_t)row * (uint32_t)g.tok_stride + oct * 8) * 2;
      f.off_b = f.off_a;
      f.meta_step = (int64_t)kTileK * g.tok_stride * 2;
      f.code_step = f.meta_step;
      f.p_c = f.p_a;
      f.p_d = f.p_a;
      f.off_code = 0;
      f.hi = 0;
      const int left = n - trow;
      if (left < kTileK) {      // the call's last tile: rows past its end repeat the last one (they are zeroed when decoded)
        f.p_b = f.p_a;
        f.off_a = ((uint32_t)min(row, left - 1) * (uint32_t)g.tok_stride + oct * 8) * 2;
        f.off_b = ((uint32_t)min(row + row_step, left - 1) * (uint32_t)g.tok_stride + oct * 8) * 2;
      }
    };
    auto load_code = [&](const uint8_t* p) __attribute__((always_inline)) {
      Code c;
      if constexpr (kWide) {
        const u32x2_a4 x = *reinterpret_cast<const u32x2_a4*>(p);
        c.x = x.x;
        c.y = x.y;
      } else {
        c.x = *reinterpret_cast<const uint32_t*>(p);
      }
      return c;
    };
    auto request = [&](auto second, Feed& f, const void* base, int row, int row_step, int oct) __attribute__((always_inline)) {
      if constexpr (FMT != kBf16) {
        f.c = load_code(f.p_c + f.off_code);
        f.d = load_code(f.p_d + f.off_code);
      }
      if constexpr (decltype(second)::value) {
        f.a2 = *reinterpret_cast<const u32x4_a4*>(f.p_a + f.hi + f.off_a);
        f.b2 = *reinterpret_cast<const u32x4_a4*>(f.p_b + f.hi + f.off_b);
      }
      f.a = *reinterpret_cast<const u32x4_a4*>(f.p_a + f.off_a);
      f.b = *reinterpret_cast<const u32x4_a4*>(f.p_b + f.off_b);
      if (f.next + 1 < tile_end) {                         // (past the range's end the last tile is requested again)
        f.next += 1;
        f.p_c += f.code_step;
        f.p_d += f.code_step;
        f.p_a += f.meta_step;
        f.p_b += f.meta_step;
        // the first of the call's own tiles, and a ragged last one
        const int trow = (f.next - ntc) * kTileK;
        if (f.next == ntc || (f.next > ntc && n - trow < kTileK)) seek_own(f, base, row, row_step, oct, trow);
      }
    };
    auto request_k = [&]() __attribute__((always_inline)) { request(std::bool_constant<kParts == 2>{}, fk, it.k, k_row, 16, k_oct); };
    auto request_v = [&]() __attribute__((always_inline)) { request(std::false_type{}, fv, it.v, v_row, 1, v_oct); };
    auto seek = [&]() __attribute__((always_inline)) {
      fk.next = fv.next = tile_begin;
      fk.hi = fv.hi = 0;
      if (FMT == kBf16 && tile_begin < ntc) {
        // (the row after a tile's last valid one is inside the buffer)
        const int64_t row0t = (int64_t)h * g.t_cap + tile_begin * kTileK;
        fk.p_a = half + g.lay.k_codes + row0t * (kHeadDim * 2);
        fk.p_b = fk.p_a + 16 * (kHeadDim * 2);
        fv.p_a = half + g.lay.v_codes + row0t * (kHeadDim * 2);
        fv.p_b = fv.p_a + kHeadDim * 2;
        fk.meta_step = fv.meta_step = kTileK * kHeadDim * 2;
        fk.off_a = fk.off_b = (uint32_t)((k_row * kHeadDim + k_oct * 8) * 2);
        fv.off_a = fv.off_b = (uint32_t)((v_row * kHeadDim + v_oct * 8) * 2);
        fk.p_c = fk.p_d = fk.p_a;
        fv.p_c = fv.p_d = fv.p_a;
        fk.code_step = fv.code_step = 0;
        fk.off_code = fv.off_code = 0;
      } else if (tile_begin < ntc) {
        constexpr int kKElt = FMT == kMeta16 ? 2 : 4, kVElt = FMT == kMeta16 ? 4 : (int)sizeof(VMeta);
        const int64_t row0t = (int64_t)h * g.t_cap + tile_begin * kTileK;
        const int64_t moff = ((int64_t)h * g.g_cap + ((tile_begin * kTileK) >> k_shift)) * (kHeadDim * kKElt);
        fk.hi = 16;
        fk.p_c = half + g.lay.k_codes + row0t * kKRow;
        fk.p_d = fk.p_c + 16 * kKRow;
        fk.p_a = half + g.lay.k_scale + moff;
        fk.p_b = half + g.lay.k_zero + moff;
        fk.code_step = kTileK * kKRow;
        fk.meta_step = (kTileK >> k_shift) * (kHeadDim * kKElt);
        fk.off_code = (uint32_t)(k_row * kKRow + ((k_oct * KB) & ~3));
        fk.off_a = (uint32_t)(((k_row >> k_shift) * kHeadDim + k_oct * 8) * kKElt);
        fk.off_b = fk.off_a;
        fv.p_c = half + g.lay.v_codes + row0t * kVRow;
        fv.p_d = fv.p_c + kVRow;
        fv.p_a = half + g.lay.v_meta + row0t * ngv * kVElt;
        fv.p_b = fv.p_a + ngv * kVElt;
        fv.code_step = kTileK * kVRow;
        fv.meta_step = kTileK * ngv * kVElt;
        fv.off_code = (uint32_t)(v_row * kVRow + ((v_oct * VB) & ~3));
        fv.off_a = (uint32_t)((v_row * ngv + ((v_oct * 8) >> v_shift)) * kVElt);
        fv.off_b = fv.off_a;
      } else {
        seek_own(fk, it.k, k_row, 16, k_oct, (tile_begin - ntc) * kTileK);
        seek_own(fv, it.v, v_row, 1, v_oct, (tile_begin - ntc) * kTileK);
      }
    };
    // Decodes the requested rows of `tile` into LDS at element offset buf.
    auto store_k = [&](int tile, int buf) __attribute__((always_inline)) {
      uint16_t* kdst = lds + buf + k_row * kLdsRow + k_oct * 8;
      if constexpr (FMT == kMeta32) if (tile < ntc) {
        // s (code - z) evaluated as fma(code, s, -z s): it differs from Eq. 10's form by a rounding of z s, far below what the
        // bf16 pair keeps
        float sk[8], nz[8], f[8], x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          sk[e] = __uint_as_float(e < 4 ? fk.a[e & 3] : fk.a2[e & 3]) * sc;
          nz[e] = -(float)(int32_t)(e < 4 ? fk.b[e & 3] : fk.b2[e & 3]) * sk[e];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          code_floats<KB>(i == 0 ? fk.c : fk.d, k_half, f);
          uint32_t hi[4], lo[4];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(f[e], sk[e], nz[e]);
#pragma unroll
          for (int e = 0; e < 4; ++e) split_bf16(x[2 * e], x[2 * e + 1], hi[e], lo[e]);
          *reinterpret_cast<uint4*>(kdst + i * 16 * kLdsRow) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
          *reinterpret_cast<uint4*>(kdst + kBufs * kTileElems + i * 16 * kLdsRow) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
        return;
      }
      if constexpr (FMT == kMeta16) if (tile < ntc) {
        // (1024 + code) - (1024 + z) is exact; times a: exact up to |code - z| = 16.  Rows past the cache's end hold
        // finite stale values; their logits are masked.
        uint32_t p[4], q[4];
        key_pairs<KB>(fk.c.x, k_sel, bias, p);
        key_pairs<KB>(fk.d.x, k_sel, bias, q);
  #pragma unroll
        for (int j = 0; j < 4; ++j) {
          p[j] = as_u((as_h2(p[j]) - as_h2(fk.b[j])) * as_h2(fk.a[j]));
          q[j] = as_u((as_h2(q[j]) - as_h2(fk.b[j])) * as_h2(fk.a[j]));
        }
        *reinterpret_cast<uint4*>(kdst) = make_uint4(p[0], p[1], p[2], p[3]);
        *reinterpret_cast<uint4*>(kdst + 16 * kLdsRow) = make_uint4(q[0], q[1], q[2], q[3]);
        return;
      }
      {
        const int left = tile < ntc ? t_c - tile * kTileK : n - (tile - ntc) * kTileK;
        uint4 ra = make_uint4(fk.a.x, fk.a.y, fk.a.z, fk.a.w), rb = make_uint4(fk.b.x, fk.b.y, fk.b.z, fk.b.w);
        if (left < kTileK) {
          if (k_row >= left) ra = make_uint4(0, 0, 0, 0);
          if (k_row + 16 >= left) rb = make_uint4(0, 0, 0, 0);
        }
        *reinterpret_cast<uint4*>(kdst) = FMT == kMeta16 ? bf16_octet_to_half_pairs(ra) : ra;
        *reinterpret_cast<uint4*>(kdst + 16 * kLdsRow) = FMT == kMeta16 ? bf16_octet_to_half_pairs(rb) : rb;
      }
    };
    // V: rows of the tile in LDS are channels; the two keys of a thread land side by side as one 4-byte store per channel,
    // column 2 (st & 31) (the key order inside a 16-key step is the permutation swap23, which the probabilities' register order shares).
    auto store_v = [&](int tile, int buf) __attribute__((always_inline)) {
      uint32_t* vdst = reinterpret_cast<uint32_t*>(lds + kLdsV + buf + v_oct * 8 * kLdsRow + 2 * (st & 31));
      if constexpr (FMT == kMeta32) if (tile < ntc) {
        // rows past the cache's end become zeros (scale and offset zero): their probabilities are zero too
        const int left = t_c - tile * kTileK;
        const bool ok0 = left >= kTileK || v_row < left, ok1 = left >= kTileK || v_row + 1 < left;
        const float s0 = ok0 ? __uint_as_float(fv.a.x) : 0.f, s1 = ok1 ? __uint_as_float(fv.b.x) : 0.f;
        const float nz0 = -(float)(int32_t)fv.a.y * s0, nz1 = -(float)(int32_t)fv.b.y * s1;
        float fa[8], fb[8];
        code_floats<VB>(fv.c, v_half, fa);
        code_floats<VB>(fv.d, v_half, fb);
#pragma unroll
        for (int e = 0; e < 8; ++e) vdst[e * (kLdsRow / 2)] = pack_f16(__builtin_fmaf(fa[e], s0, nz0), __builtin_fmaf(fb[e], s1, nz1));
        return;
      }
      if constexpr (FMT == kMeta16) if (tile < ntc) {
        // rows past the cache's end become zeros (scale zero): their probabilities are zero too
        uint32_t m0 = fv.a.x, m1 = fv.b.x;
        if ((tile + 1) * kTileK > t_c) {       // uniform; only a cache's last tile can be ragged
          const int ja = tile * kTileK + v_row;
          m0 = ja < t_c ? m0 : 0x64000000u;
          m1 = ja + 1 < t_c ? m1 : 0x64000000u;
        }
        const uint32_t s = __builtin_amdgcn_perm(m1, m0, 0x05040100u), z = __builtin_amdgcn_perm(m1, m0, 0x07060302u);
        uint32_t p[8];
        val_pairs<VB>(fv.c, fv.d, v_sel, bias, p);
  #pragma unroll
        for (int e = 0; e < 8; ++e) vdst[e * (kLdsRow / 2)] = as_u((as_h2(p[e]) - as_h2(z)) * as_h2(s));
        return;
      }
      {
        const int left = tile < ntc ? t_c - tile * kTileK : n - (tile - ntc) * kTileK;
        u32x4_a4 ra = fv.a, rb = fv.b;
        if (left < kTileK) {
  #pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (v_row >= left) ra[e] = 0u;
            if (v_row + 1 >= left) rb[e] = 0u;
          }
        }
  #pragma unroll
        for (int e = 0; e < 4; ++e) {
          vdst[2 * e * (kLdsRow / 2)] = pack_f16(bf16lo_to_f32(ra[e]), bf16lo_to_f32(rb[e]));
          vdst[(2 * e + 1) * (kLdsRow / 2)] = pack_f16(bf16hi_to_f32(ra[e]), bf16hi_to_f32(rb[e]));
        }
      }
    };

    // While tile t is computed, the staging waves decode K of tile t + 2 and V of tile t + 1 and request the tiles behind them.
    auto stage_k = [&](int t) __attribute__((always_inline)) {
      if constexpr (STAGER) {
        if (t + 2 < tile_end) store_k(t + 2, r2);
        request_k();
      }
    };
    auto stage_v = [&](int t) __attribute__((always_inline)) {
      if constexpr (STAGER) {
        if (t + 1 < tile_end) store_v(t + 1, r1);
        request_v();
      }
    };

    // ---- tiles whose keys every query of the wave sees, pipelined over units ----
    f32x16 s_cur;              // the logits of the last step's unit
    uint32_t w_prev[8];        // the probabilities of the unit before, packed
    // step u of tile t; rv: the buffer that holds V of the tile before
    auto step = [&](auto uc, auto ownc, int rv) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;
      constexpr bool OWN = decltype(ownc)::value;
      constexpr int bq = u % NA, bs = (u + U - 1) % NA, pu = (u + U - 2) % (U > 0 ? U : 1), bp = pu % NA;
      constexpr bool prev_tile = u < 2;                                  // the second product's unit is of the tile before
      f32x16 s_nxt;
      uint32_t w[8];
      float p[16];
      f32x4 sum;
      auto ex = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (r >= from && r < to) {
            if constexpr (OWN) s_cur[r] = __builtin_fmaf(s_cur[r], sc, negm[bs][0]);
            p[r] = __builtin_amdgcn_exp2f(s_cur[r]);
            asm volatile("" : "+v"(p[r]));               // stays in its place between the matrix instructions
          }
      };
      auto cv = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e >= from && e < to) w[e] = pack_f16(p[2 * e], p[2 * e + 1]);
      };
      constexpr int P = OWN ? 1 : kParts;
      constexpr int NQ = 4 * P;                                          // matrix instructions of the first product
      // Operand i is part i % P of channel slice i / P.  Where they all fit in four fragments, both blocks of a wave use
      // them and the last one's instructions replace them by the next half's; otherwise four slots run ahead of the use.
      auto qk = [&](int i) __attribute__((always_inline)) {
        if (i == 0) {
          if constexpr (OWN) {
            f32x16 zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
            s_nxt = mma_k(kf[0], qf[bq][0], zero);
          } else {
            s_nxt = mma_k(kf[0], qf[bq][0], negm[bq]);
          }
        } else {
          s_nxt = mma_k(kf[i & 3], qf[bq][i / P], s_nxt);
        }
        constexpr bool next_half = bq == NB - 1;
        if constexpr (P == 1) {
          if constexpr (next_half) kf[i] = read_k(0, i, u / NA == 0 ? r0 : r1, u / NA == 0 ? 1 : 0);
        } else {
          const int x = (i + 4) % NQ;
          if (i + 4 < NQ || !next_half) kf[i & 3] = read_k(x % P, x / P, r0, u / NA);
          else kf[i & 3] = read_k(x % P, x / P, u / NA == 0 ? r0 : r1, u / NA == 0 ? 1 : 0);
        }
      };
      auto pv = [&](int j) __attribute__((always_inline)) {
        const int kk = j >> 1, cb = j & 1;
        o[bp][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[kk][cb], frag(w_prev, kk), o[bp][cb], 0, 0, 0);
        if constexpr (bp == NB - 1) {
          if constexpr (pu / NA == 0) read_v(kk, cb, prev_tile ? rv : r0, 1);
          else read_v(kk, cb, r0, 0);
        }
      };
      KVX_PIN();
      if constexpr (NQ == 4) {
        qk(0); KVX_PIN(); ex(0, 3); KVX_PIN();
        qk(1); KVX_PIN(); ex(3, 6); cv(0, 1); KVX_PIN();
        qk(2); KVX_PIN(); ex(6, 9); cv(1, 3); KVX_PIN();
        qk(3); KVX_PIN(); ex(9, 12); cv(3, 4); KVX_PIN();
        pv(0); KVX_PIN(); ex(12, 15); cv(4, 6); KVX_PIN();
        sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, frag(w, 0), no_sum, 0, 0, 0); KVX_PIN();
        pv(1); KVX_PIN(); ex(15, 16); cv(6, 8); KVX_PIN();
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) { qk(i); KVX_PIN(); ex(2 * i, 2 * i + 2); if (i > 0) cv(i - 1, i); KVX_PIN(); }
        sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, frag(w, 0), no_sum, 0, 0, 0); KVX_PIN();
        pv(0); KVX_PIN(); cv(7, 8); KVX_PIN();
        pv(1); KVX_PIN();
      }
      sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, frag(w, 1), sum, 0, 0, 0); KVX_PIN();
      pv(2); KVX_PIN();
      // an overflow of the half range shows in the row sum; asked for one matrix instruction before it is branched on
      float unit_sum = sum[0];
      const uint64_t over = __ballot(!(unit_sum < kSumLimit)); KVX_PIN();
      pv(3); KVX_PIN();
      if (__builtin_expect(over != 0, 0)) {
        const float delta = raise(bs, s_cur, w);
        unit_sum = lane_sums(w);
        if constexpr (NB == 1 && !OWN) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s_nxt[r] -= delta;       // the next unit's logits were formed with the old reference
        }
      }
      l[bs] += unit_sum;
      s_cur = s_nxt;
#pragma unroll
      for (int e = 0; e < 8; ++e) w_prev[e] = w[e];
    };
    auto plain_tiles = [&](auto ownc, int& t, int end) __attribute__((always_inline)) {
      constexpr bool OWN = decltype(ownc)::value;
      constexpr int P = OWN ? 1 : kParts;
      if (t >= end) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) { kf[i] = read_k(i % P, i / P, r0, 0); read_v(i >> 1, i & 1, r0, 0); }
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (started[i]) continue;
        float a = -__builtin_inff();
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
          const f32x16 s = logits(Int<P>{}, i, r0, kh);
#pragma unroll
          for (int r = 0; r < 16; ++r) a = fmaxf(a, s[r]);
        }
        set_reference(i, a, OWN ? sc : 1.0f);
      }
      // the pipeline starts with units of no weight: infinitely far below any reference, also after a small logit factor
#pragma unroll
      for (int r = 0; r < 16; ++r) s_cur[r] = -__builtin_inff();
#pragma unroll
      for (int e = 0; e < 8; ++e) w_prev[e] = 0;
      int rv = r0;
      for (; t < end; ++t) {
        step(Int<0>{}, ownc, rv);
        stage_k(t);
        step(Int<1>{}, ownc, rv);
        if constexpr (NB == 2) {
          step(Int<2>{}, ownc, rv);
          step(Int<3>{}, ownc, rv);
        }
        stage_v(t);
        __syncthreads();
        const int x = r0; r0 = r1; r1 = r2; r2 = x;
        rv = r2;
      }
      // the last unit's softmax and the last two units' second products
      uint32_t w[8];
      constexpr int bs = NB - 1;
      if constexpr (OWN) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s_cur[r] = __builtin_fmaf(s_cur[r], sc, negm[bs][0]);
      }
      constexpr int bp = (U - 2) % NA;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kk = j >> 1, cb = j & 1;
        o[bp][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[kk][cb], frag(w_prev, kk), o[bp][cb], 0, 0, 0);
        if constexpr (NB == 1) read_v(kk, cb, r2, 1);
      }
      probabilities(s_cur, w);
      float unit_sum = sums(w);
      if (__any(!(unit_sum < kSumLimit))) {
        raise(bs, s_cur, w);
        unit_sum = lane_sums(w);
      }
      l[bs] += unit_sum;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kk = j >> 1, cb = j & 1;
        o[bs][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[kk][cb], frag(w, kk), o[bs][cb], 0, 0, 0);
      }
    };

    // ---- tiles with a ragged end or a mask that crosses the wave's queries, unit by unit ----
    auto masked_tiles = [&](int& t, int end) __attribute__((always_inline)) {
      for (; t < end; ++t) {
        stage_k(t);
        const bool own = t >= ntc;
        // keys past the end of the wave's frames are skipped (uniform)
        if (NB > 0 && !(own && (t - ntc) * kTileK >= limit_hi)) {
          for (int kh = 0; kh < 2; ++kh) {
#pragma unroll
            for (int i = 0; i < 4; ++i) read_v(i >> 1, i & 1, r0, kh);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              auto product = [&](int x) __attribute__((always_inline)) {
                return kParts == 2 && !own ? logits(Int<kParts>{}, i, r0, x) : logits(Int<1>{}, i, r0, x);
              };
              const float f = own || FMT == kBf16 ? sc : 1.0f;         // cached keys in codes carry the logit factor
              // keys this lane's query may see in the tile: valid rows of the cache's last tile, or own keys up to the end
              // of the query's frame (also covers the ragged end of the call's rows)
              const int own_limit = n == g.n ? n : (min(row0[i] + l32, n - 1) / g.n + 1) * g.n;
              const int valid = own ? own_limit - (t - ntc) * kTileK : t_c - t * kTileK;
              const int lane_key = 4 * hf;                              // register r: key lane_key + 8 (r / 4) + r % 4 of a unit
              if (!started[i]) {
                float a = -__builtin_inff();
#pragma unroll 1
                for (int x = 0; x < 2; ++x) {
                  const f32x16 s = product(x);
#pragma unroll
                  for (int r = 0; r < 16; ++r) a = lane_key + 8 * (r >> 2) + (r & 3) < valid - 32 * x ? fmaxf(a, s[r]) : a;
                }
                set_reference(i, a, f);
              }
              f32x16 s = product(kh);
#pragma unroll
              for (int r = 0; r < 16; ++r) s[r] = lane_key + 8 * (r >> 2) + (r & 3) < valid - 32 * kh ? __builtin_fmaf(s[r], f, negm[i][0]) : kNegBig;
              uint32_t w[8];
              probabilities(s, w);
              float unit_sum = sums(w);
              if (__any(!(unit_sum < kSumLimit))) {
                raise(i, s, w);
                unit_sum = lane_sums(w);
              }
              l[i] += unit_sum;
#pragma unroll
              for (int j = 0; j < 4; ++j) o[i][j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[j >> 1][j & 1], frag(w, j >> 1), o[i][j & 1], 0, 0, 0);
            }
          }
        }
        stage_v(t);
        __syncthreads();
        const int x = r0; r0 = r1; r1 = r2; r2 = x;
      }
    };

    // ---- the tile range ----
    if (tile_begin < tile_end) {
      if constexpr (STAGER) {
        seek();
        request_k();
        request_v();
        store_k(tile_begin, 0);
        request_k();
        store_v(tile_begin, 0);
        request_v();
        if (tile_begin + 1 < tile_end) store_k(tile_begin + 1, r1);
        request_k();
      }
      __syncthreads();
      int t = tile_begin;
      if constexpr (NB > 0) {
        plain_tiles(std::bool_constant<FMT == kBf16>{}, t, min(tile_end, t_c / kTileK));
        masked_tiles(t, min(tile_end, ntc));
        plain_tiles(std::true_type{}, t, min(tile_end, ntc + min(limit_lo, n) / kTileK));
      }
      masked_tiles(t, tile_end);
    }

    // ---- epilogue -------------------------------------------------------------------
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int qi = row0[i] + l32;
      if (qi >= n) continue;
      const float l_tot = l[i];
      if (g.n_splits == 1) {
        const float inv = 1.0f / l_tot;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const int c = cb * 32 + 8 * r4 + 4 * hf;
            const float x0 = o[i][cb][4 * r4 + 0] * inv, x1 = o[i][cb][4 * r4 + 1] * inv;
            const float x2 = o[i][cb][4 * r4 + 2] * inv, x3 = o[i][cb][4 * r4 + 3] * inv;
            const int64_t off = (int64_t)qi * g.out_tok_stride + (int64_t)h * g.out_head_stride + c;
            if (g.out_f32) {
              *reinterpret_cast<float4*>(reinterpret_cast<float*>(it.out) + off) = make_float4(x0, x1, x2, x3);
            } else {
              *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(it.out) + off) = make_uint2(pack_bf16(x0, x1), pack_bf16(x2, x3));
            }
          }
      } else {
        const int slot = item_idx * g.n_splits + split;
        const int64_t row = ((int64_t)slot * g.H + h) * g.n_pad + qi;
        float* po = g.part_o + row * kHeadDim;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const int c = cb * 32 + 8 * r4 + 4 * hf;
            *reinterpret_cast<float4*>(po + c) = make_float4(o[i][cb][4 * r4 + 0], o[i][cb][4 * r4 + 1], o[i][cb][4 * r4 + 2], o[i][cb][4 * r4 + 3]);
          }
        // an empty key range, or one of which the query saw no key (all masked), has l = 0: it weighs nothing in the merge
        if (hf == 0) *reinterpret_cast<float2*>(g.part_ml + row * 2) = make_float2(l_tot > 0.f ? -negm[i][0] : kNegBig, l_tot);
      }
    }
  };
  // blocks of this wave inside the tile and the call's rows
  const int first_row = qt * g.q_blocks * 32;
  int nb = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (wave + 8 * i < g.q_blocks && first_row + (wave + 8 * i) * 32 < n) nb = i + 1;
  if (wave >= 4) {
    if (nb) run(Int<1>{}, std::true_type{});
    else run(Int<0>{}, std::true_type{});
  } else {
    if (nb == 2) run(Int<2>{}, std::false_type{});
    else if (nb) run(Int<1>{}, std::false_type{});
    else run(Int<0>{}, std::false_type{});
  }
}

template <Format FMT, int KB, int VB>
void launch_tile(const KvxBatch& b, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const Geometry& g = b.g;
  const dim3 grid(g.side_blocks * b.n_items + g.n_qtiles * g.H * b.n_items * g.n_splits), block(kThreads);
  // with events: the runtime stamps them at the kernel's own start and end (what a kernel trace reports)
  if (ev_start) with_batch(b, [&](const auto& bb) { hipExtLaunchKernelGGL((attn_tile_kernel<FMT, KB, VB, KVX_ITEMS(bb)>), grid, block, 0, st, ev_start, ev_stop, 0, bb); });
  else with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((attn_tile_kernel<FMT, KB, VB, KVX_ITEMS(bb)>), grid, block, 0, st, bb); });
}

}  // namespace tile
}  // namespace kvx
