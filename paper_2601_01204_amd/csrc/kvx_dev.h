// Shared declarations between the host side of libkvx and its HIP kernels.
// Everything a kernel needs arrives by value in one KvxBatch kernel argument:
// the common geometry plus one small record per cache being stepped.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace kvx {

constexpr int kHeadDim = 64;        // d; the kernels are written for 64 channels per head
constexpr int kTileK = 64;          // keys per attention tile / tokens per rebuild block
constexpr int kMaxItems = 48;       // caches per launch (bounded by the kernel-argument size)
constexpr int kMaxSplits = 16;      // key-range splits per attention workgroup column

struct VMeta {                      // per (head, token, channel group) value metadata, fp32 metadata format
  float s;
  int32_t z;
};
// 16-bit metadata format.  Keys: two arrays of halfs, the logit-domain scale a = s * scale_log2 (7 significant
// bits) and zz = 1024 + z; within every eight channels the halfs are stored in the order 0 4 1 5 2 6 3 7 (the
// order in which the attention kernel's packed unpacking of a code word produces channel pairs).  Values: one
// 32-bit word per (head, token, channel group), low half the scale s, high half zz = 1024 + z.
constexpr float kMeta16ScaleMin = 0x1p-14f;   // smallest normal half
constexpr float kMeta16ScaleMax = 2048.0f;
constexpr int kMeta16ZMin = -1024, kMeta16ZMax = 1023;
__host__ __device__ __forceinline__ int meta16_pos(int c) { return (c & ~7) | ((c & 3) << 1) | ((c >> 2) & 1); }

// Byte offsets of the parts of one half of a cache's double buffer.
struct CacheLayout {
  int64_t k_codes;    // [H][t_cap][d * k_bits / 8]
  int64_t k_scale;    // [H][g_cap][d] float (16-bit metadata: half, logit-domain scale)
  int64_t k_zero;     // [H][g_cap][d] int32 (16-bit metadata: half, 1024 + z)
  int64_t v_codes;    // [H][t_cap][d * v_bits / 8]
  int64_t v_meta;     // [H][t_cap][d / v_group] VMeta (16-bit metadata: uint32)
  int64_t ids;        // [t_cap] int32
  int64_t half_bytes; // size of one half
  int64_t cache_bytes;// both halves
};

// Byte offsets inside one cache's private scratch.
struct ScratchLayout {
  int64_t qbar;       // [n_pooled][64] float: head-mean pooled query rows
  int64_t qt;         // [64] float: mean of the pooled rows
  int64_t scores;     // [t_cap] float: importance score of middle tokens (index = cache position - n)
  int64_t keys;       // [t_cap] uint32: order-preserving image of the scores
  int64_t keep;       // [t_cap] int32: kept positions, ascending
  int64_t newtok;     // [t_cap] int32, slot layout: index of the call's token a slot receives, -1 for a slot whose token stays
  int64_t assign;     // [tokens of the largest call] int32, slot layout: slot of the call's i-th token
  int64_t sel;        // [16] int32: [0] first dropped position, [1] first rebuilt key group, [2] groups rebuilt (running), [3] kept middle tokens, [5] groups quantised with a zero-point beyond +-2^20 (running), [6] non-finite input seen (debug checks), [7] scoring blocks of the running launch that have finished, where the last one selects (0 between launches)
  int64_t bytes;
};

struct Geometry {
  uint8_t* arena;         // caches: arena + cache * lay.cache_bytes + half * lay.half_bytes + offset
  uint8_t* scratch;       // per-cache scratch: scratch + cache * sl.bytes + offset
  float* part_o;          // attention partials [slot][H][n_pad][64], slot = item * n_splits + split
  float* part_ml;         // [slot][H][n_pad][2]: running max (log2 units) and sum
  CacheLayout lay;
  ScratchLayout sl;
  int64_t tok_stride;     // q/k/v strides in elements
  int64_t head_stride;
  int64_t out_tok_stride; // out strides in elements of the output dtype
  int64_t out_head_stride;
  int32_t H;
  int32_t n;              // tokens per frame
  int32_t n_new;          // tokens this call brings: n_frames * n (query rows, own keys, appended tokens)
  int32_t own_tiles;      // 1: attention reads the call's K/V from the inputs behind the cache; 0: they are in the cache already
                          //    (update-first order: items then name the updated half and its length)
  int32_t n_special;
  int32_t pool_group;
  int32_t n_pooled;
  int32_t budget;
  int32_t t_cap;          // token capacity of a cache half (multiple of 64)
  int32_t g_cap;          // key-group capacity
  int32_t k_bits, k_group, v_bits, v_group;
  int32_t in_f32;         // 1: q/k/v are fp32, 0: bf16
  int32_t out_f32;        // 1: out is fp32, 0: bf16
  int32_t uncompressed;   // 1: bf16 cache without pruning or quantisation
  int32_t n_splits;
  int32_t n_pad;          // query rows of this call padded to n_qtiles * q_blocks * 32
  int32_t n_qtiles;       // query tiles (attention workgroups per head and key split)
  int32_t q_blocks;       // 32-row query blocks per tile (<= 12; fp32 inputs: a wave each, bf16: eight waves of up to two)
  float scale_log2;       // softmax scale * log2(e)
  float inv_scale_log2;   // fp32(1 / scale_log2): s = a * inv_scale_log2 in the 16-bit metadata format
  int32_t meta16;         // 1: 16-bit scales and zero-points
  int32_t slots;          // 1: slot-stable layout (one buffer, tokens never move), 0: compacting double buffer
  int32_t n_cus;          // compute units of the device
  int32_t merge;          // 1: the launch that rewrites the cache merges the attention partials too (it follows attention)
  int32_t score_selects;  // 1: the scoring launch selects too
  int32_t side_blocks;    // workgroups per cache in front of an attention launch that score and select (0: launches of their own)
};

struct Item {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  int32_t cache;     // cache index = stream * n_layers + layer
  int32_t t_c;       // cache length before this step
  int32_t cur;       // which half holds the cache now (the step writes the other)
  int32_t prune;     // 1 if t_c + n > budget
  int32_t frame;     // index of this frame within its stream (for token ids)
  int32_t g0_host;   // first key group to rebuild when not pruning
  int32_t pad0, pad1;
};

// Kernel argument of a launch over up to N caches.  A launch copies its whole argument into the queue's argument
// memory, so a call on one cache passes room for one (0.4 KB) instead of the 3.4 KB of a full batch.
template <int N>
struct KvxBatchT {
  static constexpr int kItems = N;
  Geometry g;
  int32_t n_items;
  int32_t pad;
  Item items[N];
};
typedef KvxBatchT<kMaxItems> KvxBatch;

// Calls f with the smallest argument that holds the batch: f(const KvxBatchT<N>&).
template <typename F>
inline void with_batch(const KvxBatch& b, F&& f) {
  if (b.n_items == 1) {
    KvxBatchT<1> one;
    one.g = b.g;
    one.n_items = 1;
    one.pad = 0;
    one.items[0] = b.items[0];
    f(one);
  } else {
    f(b);
  }
}
// inside f: the number of caches its argument holds, as a constant
#define KVX_ITEMS(bb) (std::remove_reference_t<decltype(bb)>::kItems)

// ---- launch shape of the cache rewrite -------------------------------------------
// Copy blocks (a lane moves 16 bytes of a survivor's value codes; none in the slot layout, which never moves one), and all
// blocks of a launch.  Keys and values share a launch of up to kMergedBlocks blocks (see rebuild_kernel).
constexpr int kMergedBlocks = 32768;
inline int rebuild_copy_blocks(const Geometry& g, int max_tnew) {
  const int rows_per_block = 256 / (g.v_bits / 2), carried = max_tnew > g.n_new ? max_tnew - g.n_new : 0;
  return g.slots ? 0 : (carried + rows_per_block - 1) / rows_per_block;
}
inline int64_t rebuild_blocks(const KvxBatch& b, int max_tnew) {
  return (int64_t)((max_tnew + kTileK - 1) / kTileK + rebuild_copy_blocks(b.g, max_tnew) + (b.g.n_new + kTileK - 1) / kTileK) * b.g.H * b.n_items;
}

// ---- launch shape of the scoring kernel ------------------------------------------
// Blocks of 64 positions per cache that hold middle tokens: behind the first frame.
inline int score_blocks(const KvxBatch& b, int max_tc) {
  const int blocks = (max_tc + 63) / 64 - b.g.n / 64;
  return blocks > 1 ? blocks : 1;
}
// A launch of up to a score block per compute unit is bound by its chain of dependent launches: there every score block
// forms the row mean for itself (about 1 us) and the mean's launch (4.3 us) falls away.
constexpr int kMeanRows = 128;      // pooled rows brought into LDS at a time
inline bool mean_in_score(const KvxBatch& b, int max_tc) {
  return score_blocks(b, max_tc) * b.n_items <= b.g.n_cus && b.g.n_pooled * (b.g.n_new / b.g.n) <= kMeanRows;
}

// The last block of a short scoring launch over several caches selects, which saves the issue of a launch with its 3.4 KB
// argument.  us a step, update first, 69 tokens, 4 heads: two caches of 512 37 against 39 with two launches, four of 256 47 and 50,
// eight of 256 70 and 72.  The device takes the longer: the block that selects waits for the others' scores to be written back and has
// come last (17 us for the two against 6 and 10).  So not on one cache, whose step is bound by the device (69 tokens at 256 32.5 and
// 30.8, 64 at 990 38.9 and 37.9), nor on two with more than a few blocks (128 tokens at 900, fp32, 26 blocks, 40.9 and 39.1), nor with
// many: three caches of 5001 tokens (210 blocks) take 5 us more.
inline bool selects_in_score(const KvxBatch& b, int max_tc) {
  const int blocks = score_blocks(b, max_tc) * b.n_items;
  return b.n_items > 1 && mean_in_score(b, max_tc) && blocks <= (b.n_items == 2 ? 16 : 32);
}

// Scoring workgroups per cache inside an attention launch (0: the launch cannot carry them: many caches, fp32 inputs, or scoring
// that would outlast attention).  Each takes 64 positions after 64, up to 5 us each for 16 heads and in proportion for more, and
// holds a compute unit meanwhile, and the selection takes another 20 us: so few that both are done in about 0.6 of attention's
// estimate (tile steps of 1.5 us), no more than kSideBlocks per cache and kSideBlocksMax in all.  Sixteen in all whatever the
// lengths: six caches of 4096 (523 tokens) 113 -> 124 us a step.
// Where sixteen are not enough the launch waits for them.  What they take then, from steps bound by it (17 to 64 heads, 69 to 780
// tokens, budgets of 512 to 16384): per 64 positions 0.18 us a head (8-bit codes 0.26) and 0.3, the selection 8 us and 0.08 per 64
// positions.  Up to 44 us (20 more with every further cache: launches in order take the longer, and so does their issue) that is
// still the shortest step whatever attention takes: 64 heads, 130 tokens, budget 2048, 50 us against 58 in order and 67 on the
// second stream; 32 heads at 4096 51, 52 and 66; two caches of 64 heads at 4096 87, 94 and 96.  Beyond, it has to fit
// into attention's estimate: 64 heads of 130 tokens at 8192 take 127 us inside, 97 in order and 86 on the second stream, 32 heads
// of 300 at 16384 141, 117 and 100, but 17 heads of 780 at 16384 114, 126 and 120.
constexpr int kSideBlocks = 16, kSideBlocksMax = 64;
inline int side_blocks_of(const KvxBatch& b, int max_tc, double steps) {
  if (b.g.in_f32 || b.g.uncompressed) return 0;
  const int blocks = score_blocks(b, max_tc), H = b.g.H;
  const bool wide = b.g.k_bits == 8;
  const double each = (0.9 * steps - 20.0) / (5.0 * (H > 16 ? H / 16.0 : 1.0) * (wide ? 1.4 : 1.0));
  int n = each <= 1.0 ? blocks : (int)((double)blocks / each) + 1;
  n = n < kSideBlocks ? n : kSideBlocks;
  n = n < blocks ? n : blocks;
  const double us = (double)((blocks + n - 1) / n) * (0.3 + (wide ? 0.26 : 0.18) * H) + 8.0 + 0.08 * blocks;
  if (steps > 0.0 && us > 24.0 + 20.0 * b.n_items && us > 1.35 * steps) return 0;      // (an explicit split count leaves no estimate)
  return n * b.n_items <= kSideBlocksMax ? n : 0;
}

// Waves of a scoring block, which take turns over the heads.  Up to a block per compute unit latency counts: all of 16 heads
// at once.  Beyond, no more than eight, since a unit holds one block of 16 waves but three of eight, and of those as many as
// put six waves on every SIMD, at least four: a wave requests its next head's codes before it works on this one's, so two
// turns are better than one.  us at 48 caches of 16384 tokens, 4-bit codes: 9 heads 85 with 16 waves, 59 with eight, 54 with
// four; 16 heads 140, 92 and 89.5; two waves are no better than four.  Rows of 8-bit codes take four loads and gain from
// eight waves once each still has two turns: 8 heads 92 with eight and 81 with four, 12 heads 115 and 117, 16 heads 148
// and 152.  Then no more than keep the number of turns, so that nine heads take three turns of three waves and not of four.
constexpr int kScoreWaves = 16;
inline int score_waves(int H, int k_bits, int blocks, int n_cus) {
  int waves = kScoreWaves;
  if (blocks > n_cus) {
    waves = k_bits == 8 && H > 8 ? 8 : (24 * n_cus + blocks - 1) / blocks;
    waves = waves < 4 ? 4 : (waves > 8 ? 8 : waves);
  }
  const int turns = (H + waves - 1) / waves;
  return (H + turns - 1) / turns;
}
// LDS of a scoring block: two groups' factors a and b of each wave, then the dots of every head.
inline size_t score_lds_bytes(int H, int waves) { return (size_t)(waves * 4 * kHeadDim + H * 64) * 4; }

// ---- codes as floats ---------------------------------------------------------------
// Byte K of a word as a float (v_cvt_f32_ubyteK; written out because the compiler would merge the masks of 4-bit codes into one
// bit-field extract per value).
template <int K>
__device__ __forceinline__ float byte_to_float(uint32_t w) {
  float f;
  if constexpr (K == 0) asm("v_cvt_f32_ubyte0 %0, %1" : "=v"(f) : "v"(w));
  else if constexpr (K == 1) asm("v_cvt_f32_ubyte1 %0, %1" : "=v"(f) : "v"(w));
  else if constexpr (K == 2) asm("v_cvt_f32_ubyte2 %0, %1" : "=v"(f) : "v"(w));
  else asm("v_cvt_f32_ubyte3 %0, %1" : "=v"(f) : "v"(w));
  return f;
}
// Eight 8-bit codes (two words), and eight 4-bit codes (one), which are first spread into the bytes of two words (even and odd
// channels).
__device__ __forceinline__ void bytes_to_floats(uint32_t x, uint32_t y, float (&f)[8]) {
  f[0] = byte_to_float<0>(x); f[1] = byte_to_float<1>(x); f[2] = byte_to_float<2>(x); f[3] = byte_to_float<3>(x);
  f[4] = byte_to_float<0>(y); f[5] = byte_to_float<1>(y); f[6] = byte_to_float<2>(y); f[7] = byte_to_float<3>(y);
}
__device__ __forceinline__ void nibbles_to_floats(uint32_t x, float (&f)[8]) {
  const uint32_t ev = x & 0x0F0F0F0Fu, od = (x >> 4) & 0x0F0F0F0Fu;
  f[0] = byte_to_float<0>(ev); f[2] = byte_to_float<1>(ev); f[4] = byte_to_float<2>(ev); f[6] = byte_to_float<3>(ev);
  f[1] = byte_to_float<0>(od); f[3] = byte_to_float<1>(od); f[5] = byte_to_float<2>(od); f[7] = byte_to_float<3>(od);
}

// ---- device-side address helpers ------------------------------------------------
__device__ __forceinline__ uint8_t* cache_half(const Geometry& g, int cache, int half) {
  return g.arena + (int64_t)cache * g.lay.cache_bytes + (int64_t)half * g.lay.half_bytes;
}
__device__ __forceinline__ uint8_t* cache_scratch(const Geometry& g, int cache) {
  return g.scratch + (int64_t)cache * g.sl.bytes;
}

// ---- launchers (each enqueues on `st`, never synchronises) ----------------------
void launch_attention(const KvxBatch& b, hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void launch_attention16(const KvxBatch& b, hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
void launch_combine(const KvxBatch& b, hipStream_t st);
void launch_pool(const KvxBatch& b, int max_tc, hipStream_t st);
void launch_score(const KvxBatch& b, int max_tc, hipStream_t st);
void launch_select(const KvxBatch& b, int max_tc, hipStream_t st);
void launch_rebuild(const KvxBatch& b, int max_tnew, bool keys, bool values, hipStream_t st);
void launch_append_bf16(const KvxBatch& b, hipStream_t st);
void launch_check_finite(const KvxBatch& b, hipStream_t st);

constexpr int32_t kZeroPointWarn = 1 << 20;   // |z| beyond this is counted by kv_stats (zp_range_warnings)

}  // namespace kvx
