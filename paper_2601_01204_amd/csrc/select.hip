// Selection launches: one workgroup per cache.
#include "select_block.h"

#include <algorithm>

namespace kvx {

constexpr int kSelectThreads = 1024;
template <int N>
__global__ __launch_bounds__(kSelectThreads) void select_kernel(const KvxBatchT<N> b) {
  const Item it = b.items[blockIdx.x];
  if (!it.prune) return;
  extern __shared__ int lds[];
  select_cache<kSelectThreads>(b.g, it, lds);
}

void launch_select(const KvxBatch& b, int max_tc, hipStream_t st) {
  if (b.g.score_selects) return;
  const size_t lds = select_lds_bytes(max_tc - b.g.n);
  with_batch(b, [&](const auto& bb) { hipLaunchKernelGGL((select_kernel<KVX_ITEMS(bb)>), dim3(b.n_items), dim3(kSelectThreads), lds, st, bb); });
}

}  // namespace kvx
