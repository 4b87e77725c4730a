// Driver of the sanitizer build: walks the host code of the library (no kernel runs; see hip/hip_runtime.h here).
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include <hip/hip_runtime.h>

#include "../../include/kvx.h"
#include "kvx_dev.h"

#define CHECK(cond)                                                                   \
  do {                                                                                \
    if (!(cond)) {                                                                    \
      std::fprintf(stderr, "host_check: line %d: %s failed\n", __LINE__, #cond);      \
      std::exit(1);                                                                   \
    }                                                                                 \
  } while (0)

namespace {

struct Bufs {
  std::vector<int32_t> ids, kz, vz, keep;
  std::vector<uint8_t> kc, vc;
  std::vector<float> ks, vs, scores;
  kv_export_t x;
  Bufs(int H, int cap, int kg, int vg) {
    const int G = (cap + kg - 1) / kg, ngv = 64 / vg;
    ids.assign(cap, -1); kc.assign((size_t)H * cap * 64, 0xEE); vc.assign((size_t)H * cap * 64, 0xEE);
    ks.assign((size_t)H * G * 64, -1.f); kz.assign((size_t)H * G * 64, -1);
    vs.assign((size_t)H * cap * ngv, -1.f); vz.assign((size_t)H * cap * ngv, -1);
    keep.assign(cap, -1); scores.assign(cap, -1.f);
    std::memset(&x, 0, sizeof x);
    x.ids = ids.data(); x.k_codes = kc.data(); x.k_scale = ks.data(); x.k_zero = kz.data();
    x.v_codes = vc.data(); x.v_scale = vs.data(); x.v_zero = vz.data();
    x.last_keep = keep.data(); x.last_scores = scores.data(); x.capacity_tokens = cap;
  }
};

kv_config base_config(int meta, int layout, int kb, int kg, int vb, int vg) {
  kv_config c;
  std::memset(&c, 0, sizeof c);
  c.n_streams = 2; c.n_layers = 2; c.n_heads = 3; c.head_dim = 64;
  c.tokens_per_frame = 37; c.n_special = 5; c.pool_group = 16; c.budget_tokens = 160;
  c.k_bits = kb; c.k_group = kg; c.v_bits = vb; c.v_group = vg;
  c.in_dtype = KV_BF16; c.out_dtype = KV_BF16; c.mode = KV_COMPRESSED; c.max_frames = 0;
  c.softmax_scale = 0.f; c.meta_format = meta; c.max_frames_per_step = 2; c.order = KV_ATTEND_THEN_PRUNE; c.layout = layout;
  return c;
}

// A cache state that is a value of the format: codes below 2^bits, metadata representable.
void fill_state(Bufs& b, const kv_config& c, int frames, std::mt19937& rng) {
  const int T = std::min(frames * c.tokens_per_frame, c.budget_tokens), H = c.n_heads;
  const int G = (T + c.k_group - 1) / c.k_group, ngv = 64 / c.v_group;
  b.x.cache_len = T; b.x.frames_seen = frames;
  for (int i = 0; i < T; ++i) b.ids[i] = i;
  for (size_t i = 0; i < (size_t)H * T * 64; ++i) { b.kc[i] = rng() % (1u << c.k_bits); b.vc[i] = rng() % (1u << c.v_bits); }
  const float c_log2 = 0.125f * 1.4426950408889634f, inv = 1.0f / c_log2;
  for (size_t i = 0; i < (size_t)H * G * 64; ++i) {
    if (c.meta_format == KV_META_F16) {
      const float a = std::ldexp((float)(64 + rng() % 64) / 128.f, (int)(rng() % 12) - 8);      // 7 significant bits
      b.ks[i] = a * inv;
      b.kz[i] = (int)(rng() % 2048) - 1024;
    } else {
      b.ks[i] = std::ldexp(1.0f + (float)(rng() % 4096) / 4096.f, (int)(rng() % 20) - 10);
      b.kz[i] = (int)(rng() % 200001) - 100000;
    }
  }
  for (size_t i = 0; i < (size_t)H * T * ngv; ++i) {
    if (c.meta_format == KV_META_F16) {
      b.vs[i] = std::ldexp((float)(1024 + rng() % 1024) / 2048.f, (int)(rng() % 12) - 8);       // 11 significant bits
      b.vz[i] = (int)(rng() % 2048) - 1024;
    } else {
      b.vs[i] = std::ldexp(1.0f + (float)(rng() % 4096) / 4096.f, (int)(rng() % 20) - 10);
      b.vz[i] = (int)(rng() % 200001) - 100000;
    }
  }
}

void same_state(const Bufs& a, const Bufs& b, const kv_config& c) {
  const int T = a.x.cache_len, H = c.n_heads, G = (T + c.k_group - 1) / c.k_group, ngv = 64 / c.v_group;
  CHECK(a.x.cache_len == b.x.cache_len && a.x.frames_seen == b.x.frames_seen);
  CHECK(!std::memcmp(a.ids.data(), b.ids.data(), (size_t)T * 4));
  CHECK(!std::memcmp(a.kc.data(), b.kc.data(), (size_t)H * T * 64));
  CHECK(!std::memcmp(a.vc.data(), b.vc.data(), (size_t)H * T * 64));
  CHECK(!std::memcmp(a.ks.data(), b.ks.data(), (size_t)H * G * 64 * 4));
  CHECK(!std::memcmp(a.kz.data(), b.kz.data(), (size_t)H * G * 64 * 4));
  CHECK(!std::memcmp(a.vs.data(), b.vs.data(), (size_t)H * T * ngv * 4));
  CHECK(!std::memcmp(a.vz.data(), b.vz.data(), (size_t)H * T * ngv * 4));
}

void one_format(int meta, int layout, int kb, int kg, int vb, int vg) {
  std::mt19937 rng(17 + meta * 2 + layout + kb * 10 + vg);
  const kv_config c = base_config(meta, layout, kb, kg, vb, vg);
  kv_handle *h = nullptr, *h2 = nullptr;
  CHECK(kv_init(&c, &h) == KV_OK && h);
  CHECK(kv_init(&c, &h2) == KV_OK && h2);
  const int n = c.tokens_per_frame, H = c.n_heads;
  // frame buffers stand in for device memory (nothing reads them here), two frames' worth for the chunk call
  std::vector<uint16_t> q((size_t)2 * n * H * 64), k(q.size()), v(q.size()), o(q.size());
  const int64_t ts = (int64_t)H * 64, hs = 64;

  // bookkeeping over a stream that crosses the budget: lengths, drops, flat allocation
  kv_stats_t st0, st;
  CHECK(kv_stats(h, &st0) == KV_OK);
  for (int f = 0; f < 7; ++f) {
    CHECK(kv_step(h, 0, 0, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);
    CHECK(kv_stats(h, &st) == KV_OK);
    CHECK(st.cache_len_max == std::min((f + 1) * n, c.budget_tokens));
    CHECK(st.bytes_allocated == st0.bytes_allocated);
  }
  CHECK(st.tokens_dropped_total == 7 * n - c.budget_tokens);
  CHECK(kv_step_frames(h, 0, 1, 2, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);
  CHECK(kv_step_frames(h, 0, 1, 3, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_E_RANGE);
  CHECK(kv_step_static(h, 1, 0, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);
  {
    kv_step_item items[4];
    for (int i = 0; i < 4; ++i) { items[i].stream = i / 2; items[i].layer = i % 2; items[i].q = q.data(); items[i].k = k.data(); items[i].v = v.data(); items[i].out = o.data(); }
    CHECK(kv_set_timing(h, 0x7F) == KV_OK);
    CHECK(kv_step_batched(h, 4, items, ts, hs, nullptr) == KV_OK);
    float ms[16]; int32_t cnt[16];
    CHECK(kv_read_timing(h, ms, cnt) == KV_OK);
    CHECK(kv_set_timing(h, 0) == KV_OK);
    items[3] = items[0];
    CHECK(kv_step_batched(h, 4, items, ts, hs, nullptr) == KV_E_INVAL);      // one cache twice
    items[3].layer = 9;
    CHECK(kv_step_batched(h, 4, items, ts, hs, nullptr) == KV_E_RANGE);
  }
  // error paths leave the handle usable
  CHECK(kv_step(h, 0, 0, nullptr, k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_E_INVAL);
  CHECK(kv_step(h, 0, 0, (const char*)q.data() + 2, k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_E_INVAL);
  CHECK(kv_step(h, 0, 0, q.data(), k.data(), v.data(), 32, hs, o.data(), nullptr) == KV_E_INVAL);
  CHECK(kv_step(h, 2, 0, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_E_RANGE);
  CHECK(std::strlen(kv_last_error(h)) > 0);
  CHECK(kv_set_stream_tokens(h, 0, 21) == KV_E_STATE);                       // caches of stream 0 are not empty
  CHECK(kv_set_option(h, "no_such_option", 1) == KV_E_INVAL);
  CHECK(kv_set_option(h, "overlap_update", 0) == KV_OK && kv_set_option(h, "attention_splits", 3) == KV_OK);
  CHECK(kv_step(h, 0, 0, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);

  // export of whatever the arena holds (no kernel wrote it: zeros) stays inside the caller's buffers
  Bufs e0(H, c.budget_tokens, c.k_group, c.v_group);
  CHECK(kv_export(h, 0, 0, &e0.x) == KV_OK);
  CHECK(e0.x.cache_len == c.budget_tokens);
  Bufs small(H, 64, c.k_group, c.v_group);
  CHECK(kv_export(h, 0, 0, &small.x) == KV_E_RANGE);                          // capacity below the cache length

  // import -> export -> import into a second handle -> export: the packing and its inverse, every part of the state
  for (int frames : {1, 3, 9}) {
    Bufs a(H, c.budget_tokens, c.k_group, c.v_group), b(H, c.budget_tokens, c.k_group, c.v_group), d(H, c.budget_tokens, c.k_group, c.v_group);
    fill_state(a, c, frames, rng);
    CHECK(kv_import(h, 1, 1, &a.x) == KV_OK);
    CHECK(kv_export(h, 1, 1, &b.x) == KV_OK);
    same_state(a, b, c);
    CHECK(kv_import(h2, 0, 1, &b.x) == KV_OK);
    CHECK(kv_export(h2, 0, 1, &d.x) == KV_OK);
    same_state(a, d, c);
    CHECK(kv_step(h2, 0, 1, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);    // the stream goes on
    // inconsistent buffers are refused and leave the cache as it was
    a.kc[5] = (uint8_t)(1u << c.k_bits);
    if (c.k_bits < 8) CHECK(kv_import(h, 1, 1, &a.x) < 0);
    a.kc[5] = 0;
    a.x.cache_len -= 1;
    CHECK(kv_import(h, 1, 1, &a.x) < 0);
    a.x.cache_len += 1;
    if (c.meta_format == KV_META_F16) {
      a.kz[0] = 5000;
      CHECK(kv_import(h, 1, 1, &a.x) == KV_E_INVAL);
    }
    CHECK(kv_export(h, 1, 1, &d.x) == KV_OK);
    same_state(b, d, c);
  }
  CHECK(kv_reset(h, -1, -1) == KV_OK);
  CHECK(kv_set_stream_tokens(h, 0, 21) == KV_OK);
  CHECK(kv_set_stream_tokens(h, 0, 38) == KV_E_RANGE);
  CHECK(kv_step(h, 0, 0, q.data(), k.data(), v.data(), ts, hs, o.data(), nullptr) == KV_OK);
  CHECK(kv_stats(h, &st) == KV_OK && st.cache_len_max == 21);
  kv_destroy(h);
  kv_destroy(h2);
}

// The update chain goes to the second stream where attention is long, which the longest cache of a call decides.
void second_stream_by_the_longest_cache() {
  kv_config c = base_config(KV_META_F32, KV_LAYOUT_COMPACT, 4, 64, 4, 64);
  c.n_streams = 2; c.n_layers = 1; c.n_heads = 2; c.tokens_per_frame = 64; c.budget_tokens = 8192; c.max_frames_per_step = 1;
  kv_handle* h = nullptr;
  CHECK(kv_init(&c, &h) == KV_OK && h);
  const int64_t ts = (int64_t)c.n_heads * 64, hs = 64;
  std::vector<uint16_t> q((size_t)c.tokens_per_frame * ts), o(q.size());
  kv_step_item items[2];
  for (int i = 0; i < 2; ++i) { items[i].stream = i; items[i].layer = 0; items[i].q = items[i].k = items[i].v = q.data(); items[i].out = o.data(); }
  auto waits = [&](int n, const kv_step_item* it) {
    const int before = stub_stream_waits;
    CHECK(kv_step_batched(h, n, it, ts, hs, nullptr) == KV_OK);
    return stub_stream_waits - before;
  };
  CHECK(waits(2, items) == 0);                                               // two short caches: in order
  for (int f = 0; f < 200; ++f) waits(1, items);                             // stream 0 fills up
  CHECK(waits(1, items) == 2);
  CHECK(kv_reset(h, 1, 0) == KV_OK);
  CHECK(waits(2, items) == 2);                                               // a stream that starts beside a full cache
  CHECK(waits(1, items + 1) == 0);
  CHECK(kv_set_option(h, "overlap_update", 0) == KV_OK && waits(2, items) == 0);
  CHECK(kv_set_option(h, "overlap_update", 2) == KV_OK && waits(1, items + 1) == 2);
  kv_destroy(h);
}

// "A block per compute unit" means the units the device has: 63 score blocks on 64 of them and on 48.
void launch_rules_by_the_device(int cus, bool inside) {
  stub_cus = cus;
  kv_config c = base_config(KV_META_F32, KV_LAYOUT_COMPACT, 4, 64, 4, 64);
  c.n_streams = c.n_layers = 1; c.tokens_per_frame = 64; c.budget_tokens = 4096; c.max_frames_per_step = 1;
  kv_handle* h = nullptr;
  CHECK(kv_init(&c, &h) == KV_OK && h);
  const int64_t ts = (int64_t)c.n_heads * 64, hs = 64;
  std::vector<uint16_t> q((size_t)c.tokens_per_frame * ts), o(q.size());
  for (int f = 0; f < 66; ++f) CHECK(kv_step(h, 0, 0, q.data(), q.data(), q.data(), ts, hs, o.data(), nullptr) == KV_OK);
  CHECK(stub_mean_in_score == inside);
  kv_destroy(h);
  stub_cus = 256;
}

// Scoring blocks: every head has a wave's turn and no turn is nearly empty; in a launch of more than a block per compute
// unit the blocks leave LDS for six waves on each of a unit's four SIMDs, whatever the head count.
void score_block_shapes() {
  for (int i = 0; i < 128; ++i)
    for (int blocks : {1, 60, 256, 257, 300, 800, 1600, 6000, 18000}) {
      const int H = 1 + i % 64, waves = kvx::score_waves(H, i < 64 ? 4 : 8, blocks, 256), turns = (H + waves - 1) / waves;
      CHECK(waves >= 1 && waves <= H && waves <= kvx::kScoreWaves);
      CHECK(waves * turns - H < turns);
      if (blocks <= 256) continue;
      CHECK(waves <= 8);
      CHECK(kvx::score_lds_bytes(H, waves) * ((24 + waves - 1) / waves) <= 160 * 1024);
    }
}

// A handle of `caches` streams of H heads and n tokens a frame, one layer each, full at budget L.
struct Full {
  kv_handle* h = nullptr;
  kv_config c;
  std::vector<uint16_t> q;
  std::vector<kv_step_item> items;
  Full(int caches, int H, int n, int L, int k_bits = 4, int frames = 1, int dtype = KV_BF16, int order = KV_ATTEND_THEN_PRUNE) : c(base_config(KV_META_F32, KV_LAYOUT_COMPACT, k_bits, 64, 4, 64)), items(caches) {
    c.n_streams = caches; c.n_layers = 1; c.n_heads = H; c.tokens_per_frame = n; c.budget_tokens = L; c.max_frames_per_step = frames; c.in_dtype = dtype; c.order = order;
    c.n_special = std::min(c.n_special, n);
    CHECK(kv_init(&c, &h) == KV_OK && h);
    q.resize((size_t)frames * n * H * 64 * (dtype == KV_F32 ? 2 : 1));
    for (int i = 0; i < caches; ++i) { items[i].stream = i; items[i].layer = 0; items[i].q = items[i].k = items[i].v = items[i].out = q.data(); }
    for (int t = 0; t < L; t += n) step();
  }
  void step() { CHECK(kv_step_batched(h, (int)items.size(), items.data(), (int64_t)c.n_heads * 64, 64, nullptr) == KV_OK); }
  ~Full() { kv_destroy(h); }
};

// Scoring blocks inside the attention launch: as many as finish under it, none where scoring would outlast it.
void scoring_blocks_inside_attention() {
  struct { int caches, H, n, L, k_bits, blocks; } cases[] = {
    {1, 16, 1041, 8192, 4, 16},  {1, 16, 782, 2048, 4, 16},  {1, 64, 130, 2048, 4, 16},  {1, 32, 130, 4096, 4, 16},    // short, or under attention
    {2, 64, 130, 4096, 4, 16},   {1, 40, 130, 4096, 4, 16},
    {1, 17, 780, 16384, 4, 16},  {2, 12, 200, 8192, 4, 16},  {3, 6, 300, 4096, 4, 16},   {1, 24, 1041, 16384, 8, 16},
    {1, 32, 130, 8192, 4, 0},    {1, 32, 300, 16384, 4, 0},  {1, 48, 200, 8192, 4, 0},   {1, 64, 130, 24576, 4, 0},    // outlast it
    {1, 64, 300, 8192, 4, 0},    {1, 16, 400, 16384, 8, 0},  {1, 32, 400, 16384, 8, 0},
    {1, 16, 384, 4096, 4, 0},    {6, 16, 300, 4096, 4, 0},                                                            // few columns; many caches
  };
  for (const auto& x : cases) {
    Full f(x.caches, x.H, x.n, x.L, x.k_bits);
    f.step();
    if (stub_side_blocks != x.blocks) std::fprintf(stderr, "%d caches, %d heads, %d tokens, budget %d: %d blocks\n", x.caches, x.H, x.n, x.L, stub_side_blocks);
    CHECK(stub_side_blocks == x.blocks);
  }
}

// The calls by which the GPU tests check scoring and selection inside the attention launch do have them there; a static call too.
void the_tested_calls_take_the_tested_launch() {
  struct { int caches, H, n, L, k_bits, splits, blocks; } cases[] = {
    {1, 17, 3, 40, 4, 0, 1},      {1, 20, 60, 130, 2, 0, 3},     {1, 64, 40, 200, 4, 0, 4},      {1, 17, 129, 1100, 8, 0, 16},
    {1, 18, 130, 1230, 4, 0, 16}, {1, 17, 64, 2304, 2, 0, 16},   {1, 17, 900, 32768, 4, 4, 16},  {3, 8, 70, 1100, 4, 1, 16},
    {1, 20, 133, 700, 4, 3, 9},
  };
  for (const auto& x : cases) {
    Full f(x.caches, x.H, x.n, x.L, x.k_bits);
    CHECK(kv_set_option(f.h, "attention_splits", x.splits) == KV_OK);
    for (int is_static = 0; is_static < (x.caches == 1 && x.n < 900 ? 2 : 1); ++is_static) {
      const kv_step_item& it = f.items[0];
      if (is_static) CHECK(kv_step_static(f.h, 0, 0, it.q, it.k, it.v, (int64_t)x.H * 64, 64, it.out, nullptr) == KV_OK);
      else f.step();
      if (stub_side_blocks != x.blocks) std::fprintf(stderr, "%d caches, %d heads, %d tokens, budget %d: %d blocks\n", x.caches, x.H, x.n, x.L, stub_side_blocks);
      CHECK(stub_side_blocks == x.blocks && stub_merge == 1);
    }
    CHECK(kv_set_option(f.h, "overlap_update", 0) == KV_OK);
    f.step();
    CHECK(stub_side_blocks == 0);
  }
}

// A scoring launch of up to 16 blocks on two caches, or 32 on more, selects; a rewrite in order of up to 32768 blocks takes the
// merge along.
void shared_launches() {
  struct { int caches, H, n, L, selects, merge; } cases[] = {
    {1, 4, 64, 256, 0, 1}, {2, 4, 64, 576, 1, 1}, {2, 4, 64, 577, 0, 1}, {4, 4, 64, 576, 1, 1}, {4, 4, 64, 577, 0, 1},
    {1, 64, 64, 21632, 0, 1}, {1, 64, 64, 22016, 0, 0},
  };
  for (const auto& x : cases) {
    Full f(x.caches, x.H, x.n, x.L);
    CHECK(kv_set_option(f.h, "overlap_update", 0) == KV_OK);
    f.step();
    CHECK(stub_score_selects == x.selects && stub_merge == x.merge);
  }
}

// The merge does not count towards an attention launch that is long enough for the second stream; fp32 inputs are sooner.
void second_stream_by_attention_alone() {
  struct { int L; bool f32, beside; } cases[] = {{3000, false, false}, {4096, false, false}, {6000, false, false}, {8192, false, true},
                                                 {3000, true, false}, {4096, true, false}, {6000, true, true}, {8192, true, true}};
  for (const auto& x : cases) {
    Full f(1, 16, 384, x.L, 4, 1, x.f32 ? KV_F32 : KV_BF16);
    const int waits = stub_stream_waits;
    f.step();
    CHECK(stub_stream_waits - waits == (x.beside ? 2 : 0));
  }
}

// A timed call keeps the schedule of an untimed one but for the parts that are timed.
void timing_parts_only_what_it_times() {
  struct { int caches, H, n, L, timed, side, merge, selects; } cases[] = {
    {1, 16, 1041, 8192, -1, 16, 1, 0},            {1, 16, 1041, 8192, KV_K_ATTENTION, 16, 1, 0}, {1, 16, 1041, 8192, KV_K_POOL, 16, 1, 0},
    {1, 16, 1041, 8192, KV_K_SCORE, 0, 1, 0},     {1, 16, 1041, 8192, KV_K_SELECT, 0, 1, 0},     {1, 16, 1041, 8192, KV_K_COMBINE, 16, 0, 0},
    {1, 16, 1041, 8192, KV_K_REBUILD_K, 16, 0, 0}, {1, 16, 1041, 8192, KV_K_REBUILD_V, 16, 0, 0},
    {3, 4, 69, 256, -1, 0, 1, 1},                 {3, 4, 69, 256, KV_K_ATTENTION, 0, 1, 1},      {3, 4, 69, 256, KV_K_SCORE, 0, 1, 0},
    {3, 4, 69, 256, KV_K_SELECT, 0, 1, 0},        {3, 4, 69, 256, KV_K_COMBINE, 0, 0, 1},
  };
  for (const auto& x : cases) {
    Full f(x.caches, x.H, x.n, x.L);
    CHECK(kv_set_timing(f.h, x.timed < 0 ? 0u : 1u << x.timed) == KV_OK);
    const int waits = stub_stream_waits;
    f.step();
    CHECK(stub_side_blocks == x.side && stub_merge == x.merge && stub_score_selects == x.selects && stub_stream_waits == waits);
    float ms[KV_K_COUNT];
    int32_t launches[KV_K_COUNT];
    CHECK(kv_read_timing(f.h, ms, launches) == KV_OK);
    for (int k = 0; k < KV_K_COUNT; ++k) CHECK(launches[k] == (k == x.timed ? 1 : 0));
  }
}

// Several caches with scoring blocks beside them: the buffers hold the split count that the launch's rounds ask for (rounds of
// the units the blocks leave x (key tiles per range + 5), the merge on top), which a cut count misses by half.
void split_counts_fit_the_buffers() {
  struct { int caches, H, n, L; } cases[] = {{2, 6, 1174, 24050}, {2, 12, 425, 24454}, {2, 8, 821, 24218}, {3, 4, 900, 20000}, {4, 4, 300, 16384}, {2, 16, 523, 16384}};
  for (const auto& x : cases) {
    Full f(x.caches, x.H, x.n, x.L);
    CHECK(kv_set_option(f.h, "overlap_update", 1) == KV_OK);
    const int waits = stub_stream_waits;
    f.step();
    const int target = stub_stream_waits > waits ? 192 : 256 - stub_side_blocks * x.caches;
    const int blocks = (x.n + 31) / 32, qtiles = (blocks + 11) / 12, pad = qtiles * ((blocks + qtiles - 1) / qtiles) * 32, cols = x.caches * x.H * qtiles;
    const int tiles = (x.L + 63) / 64 + (x.n + 63) / 64;
    auto cost = [&](int c) { return (cols * c + target - 1) / target * ((tiles + c - 1) / c + 5.0) + (c > 1 ? 1.0 + 4e-5 * c * x.caches * x.H * pad : 0.0); };
    double best = cost(1);
    for (int c = 2; c <= std::min(16, std::max(4, 2 * target / cols)); ++c) best = std::min(best, cost(c));
    if (cost(stub_splits) > 1.05 * best) std::fprintf(stderr, "%d caches, %d heads, %d tokens, budget %d: %d splits\n", x.caches, x.H, x.n, x.L, stub_splits);
    CHECK(cost(stub_splits) <= 1.05 * best);
  }
}

// A workgroup has whole tiles: 32 key tiles go to 16 ranges of two (not to 15, of which two have three) or to 11 of up to three, 19 to ten.
void ranges_of_whole_tiles() {
  struct { int n, L, splits; } cases[] = {{144, 2000, 16}, {300, 2000, 11}, {300, 1200, 10}};
  for (const auto& x : cases) {
    Full f(1, 16, x.n, x.L, 4, 1, KV_BF16, KV_PRUNE_THEN_ATTEND);
    f.step();
    if (stub_splits != x.splits) std::fprintf(stderr, "%d tokens, budget %d: %d splits\n", x.n, x.L, stub_splits);
    CHECK(stub_splits == x.splits);
  }
}

}  // namespace

int main() {
  ranges_of_whole_tiles();
  the_tested_calls_take_the_tested_launch();
  shared_launches();
  timing_parts_only_what_it_times();
  second_stream_by_attention_alone();
  split_counts_fit_the_buffers();
  scoring_blocks_inside_attention();
  score_block_shapes();
  launch_rules_by_the_device(64, true);
  launch_rules_by_the_device(48, false);
  second_stream_by_the_longest_cache();
  for (int meta : {KV_META_F32, KV_META_F16})
    for (int layout : {KV_LAYOUT_COMPACT, KV_LAYOUT_SLOTS}) {
      one_format(meta, layout, 4, 64, 4, 64);
      one_format(meta, layout, 2, 32, 4, 32);
      if (meta == KV_META_F32) one_format(meta, layout, 8, 32, 8, 64);
    }
  // configurations that kv_init must refuse
  {
    kv_handle* h = nullptr;
    kv_config c = base_config(KV_META_F32, KV_LAYOUT_COMPACT, 4, 64, 4, 64);
    c.budget_tokens = 2 * c.tokens_per_frame - 1;
    CHECK(kv_init(&c, &h) < 0 && !h && std::strlen(kv_last_error(nullptr)) > 0);
    c = base_config(KV_META_F16, KV_LAYOUT_COMPACT, 8, 64, 4, 64);
    CHECK(kv_init(&c, &h) < 0 && !h);                                        // 8-bit codes have no 16-bit metadata format
    c = base_config(KV_META_F32, KV_LAYOUT_COMPACT, 3, 64, 4, 64);
    CHECK(kv_init(&c, &h) < 0 && !h);
    c = base_config(KV_META_F32, KV_LAYOUT_COMPACT, 4, 64, 4, 64);
    c.mode = KV_UNCOMPRESSED_BF16; c.max_frames = 4;
    CHECK(kv_init(&c, &h) == KV_OK && h);
    std::vector<uint16_t> q((size_t)c.tokens_per_frame * c.n_heads * 64), o(q.size());
    for (int f = 0; f < 4; ++f) CHECK(kv_step(h, 0, 0, q.data(), q.data(), q.data(), c.n_heads * 64, 64, o.data(), nullptr) == KV_OK);
    CHECK(kv_step(h, 0, 0, q.data(), q.data(), q.data(), c.n_heads * 64, 64, o.data(), nullptr) == KV_E_STATE);
    Bufs e(c.n_heads, 160, 64, 64);
    CHECK(kv_import(h, 0, 0, &e.x) == KV_E_STATE);
    kv_destroy(h);
    kv_destroy(nullptr);
  }
  std::printf("host checks passed\n");
  return 0;
}
