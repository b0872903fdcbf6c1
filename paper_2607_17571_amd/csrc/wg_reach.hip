// Launchers of the row-at-a-time closure (kernels in wg_reach_kernels.h).
#include <hip/hip_ext.h>

#include <algorithm>

#include "wg_launch.h"
#include "wg_reach_kernels.h"

namespace wg {

namespace {

// Blocks of the queue tier past kThinWords.
uint32_t wide_queue_blocks(int cu, uint32_t words) { return (uint32_t)cu * (words <= 8192 ? 2 : 1); }

// Rows of the queue tier by the widest instance's columns: one wave per row up to 65,536 (bitmaps
// of at most 8 KB, as many rows per CU as their LDS allows), wider blocks above, where one bitmap
// takes much of a CU's LDS.
void launch_queue(hipStream_t s, int cu, const ReachArgs& a) {
  const dim3 B(kWave);
  if (a.words <= 256) hipLaunchKernelGGL((k_reach_queue<1, 256, 512>), dim3(cu * 24), B, 0, s, a);
  else if (a.words <= 512) hipLaunchKernelGGL((k_reach_queue<1, 512, 512>), dim3(cu * 20), B, 0, s, a);
  else if (a.words <= 1024) hipLaunchKernelGGL((k_reach_queue<1, 1024, 512>), dim3(cu * 16), B, 0, s, a);
  else if (a.words <= 2048) hipLaunchKernelGGL((k_reach_queue<1, 2048, 512>), dim3(cu * 12), B, 0, s, a);
  else if (a.words <= 4096) hipLaunchKernelGGL((k_reach_queue<1, 4096, 1024>), dim3(cu * 5), B, 0, s, a);
  else if (a.words <= 8192) hipLaunchKernelGGL((k_reach_queue<4, 8192, 3072>), dim3(wide_queue_blocks(cu, a.words)), dim3(4 * kWave), 0, s, a);
  else hipLaunchKernelGGL((k_reach_queue<16, 32768, 3072>), dim3(wide_queue_blocks(cu, a.words)), dim3(16 * kWave), 0, s, a);
}

constexpr int kThinPerCu = 24;  // (waves; 23 KB of LDS for four)

void launch_bits(hipStream_t s, int cu, const ReachArgs& a) {
  const dim3 B(kReachBitsWaves * kWave);
  if (a.words <= 512) hipLaunchKernelGGL((k_reach_bits<512, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else if (a.words <= 2048) hipLaunchKernelGGL((k_reach_bits<2048, uint16_t>), dim3(cu * 8), B, 0, s, a);
  else hipLaunchKernelGGL((k_reach_bits<8192, uint32_t>), dim3(cu), B, 0, s, a);
}

uint32_t blocks_for(const Grid& g, uint64_t n) {
  return (uint32_t)std::min<uint64_t>(std::max<uint64_t>((n + kBlock - 1) / kBlock, 1), (uint64_t)g.stream);
}

template <typename Put>
void unpack(hipStream_t s, const Grid& g, const ReachResult& r, uint64_t n, Put put) {
  if (r.slab) {
    const uint32_t b = (r.rows + kSlabOutWaves - 1) / kSlabOutWaves;
    hipLaunchKernelGGL(k_slab_unpack<Put>, dim3(b), dim3(kSlabOutWaves * kWave), 0, s, r, put);
    return;
  }
  const uint32_t lb = (uint32_t)std::min<uint64_t>((n + kReachOutTile - 1) / kReachOutTile, (uint64_t)g.stream);
  const uint32_t bb = std::min<uint32_t>(r.n_bits, (uint32_t)g.stream);
  hipLaunchKernelGGL(k_reach_unpack<Put>, dim3(lb + bb), dim3(kBlock), 0, s, r, lb, put);
}

// id ranges of up to this many words are ranked by one block, without a launch for the totals (one
// block against two launches, us: 1,024 words 12 / 9, 2,048 27 / 9)
constexpr uint64_t kRankOneBlock = 512;
constexpr uint64_t kOffsetsOneBlock = 16384;

void offsets(hipStream_t s, const Grid& g, uint64_t m, const ReachArgs& a, uint64_t* part, uint32_t* off) {
  if (m <= kOffsetsOneBlock) {
    hipLaunchKernelGGL((k_reach_offsets<kScanBlocksMax>), dim3(1), dim3(kBlock), 0, s, a, (const uint64_t*)nullptr,
                       off);
  } else {
    hipLaunchKernelGGL(k_reach_sum, dim3(g.scan), dim3(kBlock), 0, s, a, part);
    hipLaunchKernelGGL((k_reach_offsets<kScanBlocksMax>), dim3(g.scan), dim3(kBlock), 0, s, a,
                       (const uint64_t*)part, off);
  }
}


}  // namespace

template <typename K>
void launch_count_rows(hipStream_t s, const Grid& g, Ctrl* ctrl, const K* E, uint64_t m, int w) {
  // (few blocks: one same-address atomic each)
  hipLaunchKernelGGL(k_count_rows<K>, dim3(std::min<uint32_t>(blocks_for(g, m), std::max(1, g.stream / 8))), dim3(kBlock), 0, s,
                     ctrl, E, w);
}

template <typename K>
void launch_reach_graph(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const ReachArgs& a,
                        uint64_t* part) {
  const uint32_t b = blocks_for(g, m);
  hipLaunchKernelGGL(k_reach_mark<K>, dim3(b), dim3(kBlock), 0, s, ctrl, E, a.g);
  if (a.g.span / 32 <= kRankOneBlock) {
    hipLaunchKernelGGL(k_reach_rank, dim3(1), dim3(kBlock), 0, s, ctrl, a.g,
                       (const uint64_t*)nullptr, a.rc);
  } else {
    hipLaunchKernelGGL(k_reach_rank_sum, dim3(g.scan), dim3(kBlock), 0, s, a.g, part);
    hipLaunchKernelGGL(k_reach_rank, dim3(g.scan), dim3(kBlock), 0, s, ctrl, a.g,
                       (const uint64_t*)part, a.rc);
  }
  hipLaunchKernelGGL(k_reach_rows<K>, dim3(b), dim3(kBlock), 0, s, ctrl, E, a.g, (const ReachCtl*)a.rc);
  hipLaunchKernelGGL(k_reach_edges<K>, dim3(b), dim3(kBlock), 0, s, ctrl, E, a.g, a.rc, a.slab_mode);
}

uint32_t thin_waves(const Grid& g, uint32_t words) {
  const uint64_t cu = (uint64_t)std::max(1, g.stream / 8);
  return (uint32_t)std::min<uint64_t>(cu * kThinPerCu, kThinBytes / 4 / words) / (kReachXcds * kThinWaves) * (kReachXcds * kThinWaves);
}

uint32_t thin_rows(const Grid& g, uint32_t words) {
  return kThinRounds * wide_queue_blocks(std::max(1, g.stream / 8), words);
}

void launch_reach(hipStream_t s, const Grid& g, uint64_t m, const ReachArgs& a, uint64_t* part, uint32_t* off) {
  const int cu = std::max(1, g.stream / 8);
  if (a.slab_mode != 1) hipLaunchKernelGGL(k_reach_thread, dim3(blocks_for(g, m)), dim3(kBlock), 0, s, a);
  if (a.slab_mode != 0) {
    if (m > kSlabRows32) hipLaunchKernelGGL(k_slab<true>, dim3(cu), dim3(kSlabThreads), 0, s, a);
    else hipLaunchKernelGGL(k_slab<false>, dim3(cu), dim3(kSlabThreads), 0, s, a);
    hipLaunchKernelGGL(k_slab_count, dim3(std::max<uint32_t>(1, blocks_for(g, 4 * m))), dim3(kBlock), 0, s, a);
  }
  if (a.slab_mode != 1) {
    hipLaunchKernelGGL((k_reach_group<0, 4, 64, 128, 32, 32, 2>), dim3(cu * 6), dim3(2 * kWave), 0, s, a);
    hipLaunchKernelGGL((k_reach_group<1, 8, 256, 512, 128, 64, 1>), dim3(cu * 6), dim3(kWave), 0, s, a);
    if (a.after_groups == kThinTier)
      hipLaunchKernelGGL((k_reach_thin<kThinQueue, kThinGroups>), dim3(thin_waves(g, a.vis_words) / kThinWaves),
                         dim3(kThinWaves * kWave), 0, s, a);
    launch_queue(s, cu, a);
    if (a.bits_tier) launch_bits(s, cu, a);
  }
  offsets(s, g, m, a, part, off);
}

void launch_slab_offsets(hipStream_t s, const Grid& g, uint64_t m, const ReachArgs& a, uint64_t* part, uint32_t* off) {
  hipLaunchKernelGGL(k_slab_count, dim3(std::max<uint32_t>(1, blocks_for(g, 4 * m))), dim3(kBlock), 0, s, a);
  offsets(s, g, m, a, part, off);
}

void launch_reach_unpack(hipStream_t s, const Grid& g, const ReachResult& r, uint64_t n, uint32_t* src,
                         uint32_t* dst) {
  unpack(s, g, r, n, PutPairs{src, dst, id_mask(r.w)});
}

template <typename K>
void launch_reach_keys(hipStream_t s, const Grid& g, const ReachResult& r, uint64_t n, K* keys) {
  unpack(s, g, r, n, PutKeys<K>{keys, r.w, id_mask(r.w)});
}

void launch_reach_instances(hipStream_t s, const Grid& g, const ReachResult& r, uint32_t num, uint64_t* out) {
  hipLaunchKernelGGL(k_reach_instances, dim3(blocks_for(g, (uint64_t)num + 1)), dim3(kBlock), 0, s, r, num, out);
}

void launch_ids_gather(hipStream_t s, const Grid& g, const uint32_t* src, const uint32_t* dst, uint64_t m, uint32_t* keys) {
  hipLaunchKernelGGL(k_ids_gather, dim3(blocks_for(g, m)), dim3(kBlock), 0, s, src, dst, m, keys);
}

void launch_ids(hipStream_t s, const Grid& g, const uint32_t* sorted, const uint32_t* src, const uint32_t* dst, uint64_t m,
                uint64_t* part, uint32_t* ids, uint32_t* n_ids, uint32_t* src_out, uint32_t* dst_out) {
  hipLaunchKernelGGL(k_ids_count, dim3(g.scan), dim3(kBlock), 0, s, sorted, 2 * m, part);
  hipLaunchKernelGGL(k_ids_write, dim3(g.scan), dim3(kBlock), 0, s, sorted, 2 * m, (const uint64_t*)part, ids, n_ids);
  hipLaunchKernelGGL(k_ids_map, dim3(blocks_for(g, m)), dim3(kBlock), 0, s, (const uint32_t*)ids, (const uint32_t*)n_ids, src,
                     dst, m, src_out, dst_out);
}

void launch_ids_back(hipStream_t s, const Grid& g, const uint32_t* ids, uint32_t* ranks, uint64_t n) {
  hipLaunchKernelGGL(k_ids_back, dim3(blocks_for(g, n)), dim3(kBlock), 0, s, ids, ranks, n);
}

template <typename K>
void launch_ids_keys(hipStream_t s, const Grid& g, const uint32_t* ids, const K* keys, uint64_t n, int w, int out_w,
                     uint64_t* out) {
  hipLaunchKernelGGL(k_ids_keys<K>, dim3(blocks_for(g, n)), dim3(kBlock), 0, s, ids, keys, n, w, out_w, out);
}

#define WG_REACH_INSTANTIATE(K)                                                                              \
  template void launch_reach_graph<K>(hipStream_t, const Grid&, const Ctrl*, const K*, uint64_t, const ReachArgs&, \
                                      uint64_t*);                                                            \
  template void launch_count_rows<K>(hipStream_t, const Grid&, Ctrl*, const K*, uint64_t, int);             \
  template void launch_reach_keys<K>(hipStream_t, const Grid&, const ReachResult&, uint64_t, K*);            \
  template void launch_ids_keys<K>(hipStream_t, const Grid&, const uint32_t*, const K*, uint64_t, int, int, uint64_t*);
WG_REACH_INSTANTIATE(uint32_t)
WG_REACH_INSTANTIATE(uint64_t)

}  // namespace wg
