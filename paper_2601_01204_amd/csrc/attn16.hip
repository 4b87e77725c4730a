// Attention over caches with 16-bit metadata: the kernel of attn_tile.h.
#include "attn_tile.h"

namespace kvx {

void launch_attention16(const KvxBatch& b, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int kb = b.g.k_bits, vb = b.g.v_bits;
#define KVX_CASE(K, V) if (kb == K && vb == V) { tile::launch_tile<tile::kMeta16, K, V>(b, st, ev_start, ev_stop); return; }
  KVX_CASE(4, 4) KVX_CASE(2, 4) KVX_CASE(4, 2) KVX_CASE(2, 2) KVX_CASE(4, 8) KVX_CASE(2, 8)
#undef KVX_CASE
}

}  // namespace kvx
