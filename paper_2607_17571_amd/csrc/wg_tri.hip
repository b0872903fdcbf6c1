// Launchers of triangle counting on the renumbered graph (kernels in wg_tri_kernels.h).
#include <hip/hip_ext.h>

#include <algorithm>

#include "wg_tri_kernels.h"

namespace wg {

namespace {
uint32_t blocks_for(uint64_t n, uint32_t threads, int most) {
  return (uint32_t)std::min<uint64_t>(std::max<uint64_t>((n + threads - 1) / threads, 1), (uint64_t)std::max(1, most));
}
}  // namespace

template <typename K>
void launch_tri_edges(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const TriArgs& a, K* up) {
  hipLaunchKernelGGL(k_tri_edges<K>, dim3(blocks_for(m, kTriEdgeThreads, g.stream / 4)), dim3(kTriEdgeThreads), 0, s, ctrl,
                     E, a, up);
}

template <typename K>
void launch_tri_count(hipStream_t s, const Grid& g, uint64_t m, const TriArgs& a, const K* up, bool wide) {
  const int cu = std::max(1, g.stream / 8);
  hipLaunchKernelGGL(k_tri_starts<K>, dim3(blocks_for(m, kBlock, g.stream)), dim3(kBlock), 0, s, a, up);
  hipLaunchKernelGGL(k_tri_pairs<K>, dim3(blocks_for(m, kTriPairThreads, cu)), dim3(kTriPairThreads), 0, s, a, up);
  if (wide)
    hipLaunchKernelGGL((k_tri_bits<K, kTriWordsWide>), dim3(cu), dim3(kTriThreads), 0, s, a, up);
  else
    hipLaunchKernelGGL((k_tri_bits<K, kTriWords>), dim3(4 * cu), dim3(kTriThreads), 0, s, a, up);
}

#define WG_TRI_INSTANTIATE(K)                                                                                   \
  template void launch_tri_edges<K>(hipStream_t, const Grid&, const Ctrl*, const K*, uint64_t, const TriArgs&, K*); \
  template void launch_tri_count<K>(hipStream_t, const Grid&, uint64_t, const TriArgs&, const K*, bool);
WG_TRI_INSTANTIATE(uint32_t)
WG_TRI_INSTANTIATE(uint64_t)

}  // namespace wg
