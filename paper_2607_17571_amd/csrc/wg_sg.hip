// Launchers of same-generation on the renumbered graph (kernels in wg_sg_kernels.h).
#include <hip/hip_ext.h>

#include <algorithm>

#include "wg_sg_kernels.h"

namespace wg {

namespace {
uint32_t blocks_for(const Grid& g, uint64_t n, uint32_t threads = kBlock) {
  return (uint32_t)std::min<uint64_t>(std::max<uint64_t>((n + threads - 1) / threads, 1), (uint64_t)g.stream);
}
}  // namespace

template <typename K>
void launch_sg_edges(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const SgArgs& a) {
  hipLaunchKernelGGL(k_sg_edges<K>, dim3(std::min<uint32_t>(blocks_for(g, m, kSgEdgeThreads), std::max(1, g.stream / 4))), dim3(kSgEdgeThreads), 0, s, ctrl, E, a);
}

void launch_sg_pairs_base(hipStream_t s, const Grid& g, const Ctrl* ctrl, uint64_t m, const SgArgs& a) {
  hipLaunchKernelGGL(k_sg_pairs_base, dim3(std::min<uint32_t>(blocks_for(g, m, kSgThreads), std::max(1, g.stream / 4))), dim3(kSgThreads), 0, s, ctrl, a);
}

void launch_sg_pairs_round(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t j) {
  hipLaunchKernelGGL(k_sg_pairs_round, dim3(std::max(1, g.stream / 8)), dim3(kSgThreads), 0, s, a, j);
}

void launch_sg_pairs_tail(hipStream_t s, const SgArgs& a, uint32_t j) {
  hipLaunchKernelGGL(k_sg_pairs_tail, dim3(1), dim3(kSgThreads), 0, s, a, j);
}

template <typename K>
void launch_sg_emit(hipStream_t s, const Grid& g, const SgArgs& a, uint64_t n, int diagonal, K* out) {
  hipLaunchKernelGGL(k_sg_emit<K>, dim3(blocks_for(g, (n + kSgEmitItems - 1) / kSgEmitItems)), dim3(kBlock), 0, s,
                     a, n, diagonal, out);
}

template <typename K>
void launch_sg_matrix_base(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const SgArgs& a,
                           uint32_t slabs) {
  const int cu = std::max(1, g.stream / 8);
  hipLaunchKernelGGL(k_sg_matrix_edges<K>, dim3(blocks_for(g, m + kSlabThreads)), dim3(kBlock), 0, s, ctrl, E, a);
  hipLaunchKernelGGL(k_sg_matrix_base, dim3(std::min<uint32_t>(slabs, cu)), dim3(kSlabThreads), 0, s, a, slabs);
}

void launch_sg_matrix_round(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t j, uint32_t slabs) {
  const uint32_t b = std::min<uint32_t>(slabs, std::max(1, g.stream / 8));
  hipLaunchKernelGGL(k_sg_matrix_half, dim3(b), dim3(kSlabThreads), 0, s, a, j, slabs);
  hipLaunchKernelGGL(k_sg_matrix_rest, dim3(b), dim3(kSlabThreads), 0, s, a, j, slabs);
}

void launch_sg_matrix_diagonal(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t cols) {
  hipLaunchKernelGGL(k_sg_matrix_diagonal, dim3(blocks_for(g, cols)), dim3(kBlock), 0, s, a, cols);
}

#define WG_SG_INSTANTIATE(K)                                                                                   \
  template void launch_sg_edges<K>(hipStream_t, const Grid&, const Ctrl*, const K*, uint64_t, const SgArgs&);  \
  template void launch_sg_emit<K>(hipStream_t, const Grid&, const SgArgs&, uint64_t, int, K*);                 \
  template void launch_sg_matrix_base<K>(hipStream_t, const Grid&, const Ctrl*, const K*, uint64_t, const SgArgs&, \
                                         uint32_t);
WG_SG_INSTANTIATE(uint32_t)
WG_SG_INSTANTIATE(uint64_t)

}  // namespace wg
