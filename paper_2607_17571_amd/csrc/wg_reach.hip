// Launchers of the row-at-a-time closure (kernels in wg_reach_kernels.h).
#include <hip/hip_ext.h>

#include <algorithm>

#include "wg_launch.h"
#include "wg_reach_kernels.h"

namespace wg {

namespace {

// Rows of the queue tier by id width: one wave per row up to 16 bits (bitmaps of at most 8 KB, as
// many rows per CU as their LDS allows), wider blocks above, where one bitmap takes a CU's LDS.
void launch_queue(hipStream_t s, int cu, const ReachArgs& a) {
  if (a.w <= 13) hipLaunchKernelGGL((k_reach_queue<1, 256, 1024, uint16_t>), dim3(cu * 24), dim3(kWave), 0, s, a);
  else if (a.w == 14)
    hipLaunchKernelGGL((k_reach_queue<1, 512, 1024, uint16_t>), dim3(cu * 20), dim3(kWave), 0, s, a);
  else if (a.w == 15)
    hipLaunchKernelGGL((k_reach_queue<1, 1024, 1024, uint16_t>), dim3(cu * 16), dim3(kWave), 0, s, a);
  else if (a.w == 16)
    hipLaunchKernelGGL((k_reach_queue<1, 2048, 1024, uint16_t>), dim3(cu * 12), dim3(kWave), 0, s, a);
  else if (a.w <= 18)
    hipLaunchKernelGGL((k_reach_queue<4, 8192, 3072, uint32_t>), dim3(cu * 2), dim3(4 * kWave), 0, s, a);
  else
    hipLaunchKernelGGL((k_reach_queue<16, 32768, 3072, uint32_t>), dim3(cu), dim3(16 * kWave), 0, s, a);
}

void launch_bits(hipStream_t s, int cu, const ReachArgs& a) {
  const dim3 B(kReachBitsWaves * kWave);
  if (a.w <= 13) hipLaunchKernelGGL((k_reach_bits<256, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else if (a.w == 14) hipLaunchKernelGGL((k_reach_bits<512, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else if (a.w == 15) hipLaunchKernelGGL((k_reach_bits<1024, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else if (a.w == 16) hipLaunchKernelGGL((k_reach_bits<2048, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else hipLaunchKernelGGL((k_reach_bits<8192, uint32_t>), dim3(cu), B, 0, s, a);
}

uint32_t list_blocks(const Grid& g, uint64_t m) {
  return (uint32_t)std::min<uint64_t>(std::max<uint64_t>((m + kBlock - 1) / kBlock, 1), (uint64_t)g.stream);
}

}  // namespace

template <typename K>
void launch_reach(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const ReachArgs& a,
                  uint64_t* part, uint32_t* off) {
  const int cu = std::max(1, g.stream / 8);
  hipLaunchKernelGGL(k_reach_thread<K>, dim3(list_blocks(g, m)), dim3(kBlock), 0, s, ctrl, E, a);
  hipLaunchKernelGGL(k_reach_group, dim3(cu * 6), dim3(kBlock), 0, s, a);
  launch_queue(s, cu, a);
  if (a.tier_after[2] >= 0 || a.hub_tier == 2) launch_bits(s, cu, a);
  hipLaunchKernelGGL(k_reach_sum, dim3(g.scan), dim3(kBlock), 0, s, ctrl, a, part);
  hipLaunchKernelGGL((k_reach_offsets<kScanBlocksMax>), dim3(g.scan), dim3(kBlock), 0, s, ctrl, a,
                     (const uint64_t*)part, off);
}

template <typename K>
void launch_reach_unpack(hipStream_t s, const Grid& g, const ReachResult& r, const K* E, uint32_t* src,
                         uint32_t* dst) {
  const uint32_t lb = list_blocks(g, r.m), bb = std::min<uint32_t>(r.n_bits, (uint32_t)g.stream);
  hipLaunchKernelGGL(k_reach_unpack<K>, dim3(lb + bb), dim3(kBlock), 0, s, r, E, lb, src, dst);
}

template <typename K>
void launch_reach_keys(hipStream_t s, const Grid& g, const ReachResult& r, const K* E, K* keys) {
  const uint32_t lb = list_blocks(g, r.m), bb = std::min<uint32_t>(r.n_bits, (uint32_t)g.stream);
  hipLaunchKernelGGL(k_reach_keys<K>, dim3(lb + bb), dim3(kBlock), 0, s, r, E, lb, keys);
}

void launch_reach_instances(hipStream_t s, const Grid& g, const ReachResult& r, uint32_t num, uint64_t* out) {
  const uint64_t need = ((uint64_t)num + kBlock) / kBlock;
  hipLaunchKernelGGL(k_reach_instances, dim3((uint32_t)std::min<uint64_t>(need, (uint64_t)g.stream)), dim3(kBlock), 0,
                     s, r, num, out);
}

#define WG_REACH_INSTANTIATE(K)                                                                          \
  template void launch_reach<K>(hipStream_t, const Grid&, const Ctrl*, const K*, uint64_t, const ReachArgs&, \
                                uint64_t*, uint32_t*);                                                    \
  template void launch_reach_unpack<K>(hipStream_t, const Grid&, const ReachResult&, const K*, uint32_t*, \
                                       uint32_t*);                                                        \
  template void launch_reach_keys<K>(hipStream_t, const Grid&, const ReachResult&, const K*, K*);
WG_REACH_INSTANTIATE(uint32_t)
WG_REACH_INSTANTIATE(uint64_t)

}  // namespace wg
