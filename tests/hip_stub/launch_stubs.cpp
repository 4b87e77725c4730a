// No-op replacements for the kernel launchers: the sanitizer build exercises the host code around them.
#include "kvx_dev.h"
namespace kvx {
static void noted(const Geometry& g) {
  stub_splits = g.n_splits;
  stub_side_blocks = g.side_blocks;
  stub_merge = g.merge;
  stub_score_selects = g.score_selects;
}
void launch_attention(const KvxBatch& b, hipStream_t, hipEvent_t, hipEvent_t) { noted(b.g); }
void launch_attention16(const KvxBatch& b, hipStream_t, hipEvent_t, hipEvent_t) { noted(b.g); }
void launch_combine(const KvxBatch&, hipStream_t) {}
void launch_pool(const KvxBatch&, int, hipStream_t) {}
void launch_score(const KvxBatch& b, int max_tc, hipStream_t) { stub_mean_in_score = mean_in_score(b, max_tc); }
void launch_select(const KvxBatch&, int, hipStream_t) {}
void launch_rebuild(const KvxBatch&, int, bool, bool, hipStream_t) {}
void launch_append_bf16(const KvxBatch&, hipStream_t) {}
void launch_check_finite(const KvxBatch&, hipStream_t) {}
}  // namespace kvx
