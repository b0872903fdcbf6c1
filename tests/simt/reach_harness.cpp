// The row-at-a-time closure (the kernels of wg_reach_kernels.h, current text) on the CPU SIMT shim:
// the renumbering, every tier or the slabs, the row offsets and the unpacking, over one graph.
//   reach_harness <in> <out> <grid> <workers> <pool entries> <bits words> <slab mode> <rows> <degree> <thin>
// The first <rows> rows get <degree> further edges each as far as the slabs' sums of degrees can tell
// (the starts of the rows after them move on; no edge is there).
// in:  u64 header (w, key bytes, instances, |E|, level capacity, span), then the sorted distinct
//      keys of E (u64).
// thin: not 0: with the thin tier, for more than thin - 1 rows.
// out: u64 stop bits, pool entries used, rows queued for the groups, the queue and the bits tier, columns
//      per slab, rows queued for the thin tier; unless
//      the stop bits are set: levels L, then (tuples, degrees) of each, the tuples (src << 32 |
//      dst, from the unpacked pairs), the keys as the key form writes them and the instances'
//      offsets.
// Odd grids take the ranking and the offsets through one block and the queue tier with one wave;
// even ones through several blocks and four waves.
#include <hip/hip_runtime.h>
struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
template <typename T> inline T atomicCAS(T* p, T c, T v) {
  __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return c;
}
#define __builtin_amdgcn_s_barrier __syncthreads
#define WG_OPAQUE(x) (void)0
#define __builtin_amdgcn_wave_barrier simt::wave_sync
#define __builtin_amdgcn_fence(...) (void)0
#define __hip_atomic_load(p, ...) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, ...) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_or(p, v, ...) __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST)
#include "wg_launch.h"
#include "wg_reach_kernels.h"
#include <fstream>
#include <memory>
using namespace wg;

template <typename T>
static void put(std::ofstream& f, const T& v) {
  const uint64_t x = (uint64_t)v;
  f.write((const char*)&x, 8);
}

template <typename K>
int run(const std::vector<uint64_t>& E64, const uint64_t* h, uint32_t G, unsigned workers, uint64_t pool_cap,
        uint64_t bits_words, int slab_mode, uint32_t more_rows, uint32_t more, uint32_t thin, const char* out_path) {
  const int w = (int)h[0];
  const uint64_t m = E64.size(), num = h[2], span = h[5];
  std::vector<K> E(E64.begin(), E64.end());
  std::unique_ptr<Ctrl> ctrl(new Ctrl);
  std::memset(ctrl.get(), 0, sizeof(Ctrl));
  ctrl->m_unique = m;
  // control block, levels and flags laid out as the engine's buffer is (with levels to spare)
  const uint64_t levels = std::max<uint64_t>(h[4], kReachThreadCap), flags_at = reach_flags_at(sizeof(ReachCtl) + levels * sizeof(ReachLevel));
  std::vector<uint8_t> ctl_mem(flags_at + 2 * span + 256, 0);
  uint8_t* const ctl = (uint8_t*)(((uintptr_t)ctl_mem.data() + 255) & ~(uintptr_t)255);
  ReachCtl* const rc = (ReachCtl*)ctl;
  ReachLevel* const lev = (ReachLevel*)(ctl + sizeof(ReachCtl));
  std::vector<uint32_t> cnt(m, 0xDEADu), seg(m, 0xBEEFu), off(m + 1), pool(std::max<uint64_t>(pool_cap, 1), 0x5A5A5A5Au);
  std::vector<uint32_t> queue[kReachTiers];
  for (auto& q : queue) q.assign(m, 0x77777777u);
  std::vector<uint32_t> rowkey(m), rstart(m + 1), colkey(m), cstart(m), se(m + kSlabThreads), sc(m + kSlabThreads);
  std::vector<uint2> edge(m + kReachEdgePad);
  std::vector<RankWord> rank(span / 32 + 1);
  ReachArgs a{};
  a.g.rowkey = rowkey.data();
  a.g.rstart = rstart.data();
  a.g.colkey = colkey.data();
  a.g.cstart = cstart.data();
  a.g.edge = edge.data();
  a.g.slab_edge = se.data();
  a.g.slab_col = sc.data();
  a.g.rank = rank.data();
  a.g.flags = ctl + flags_at;
  a.g.span = span;
  a.g.instances = (uint32_t)num;
  a.g.w = w;
  a.bits_tier = 1;
  a.slab_mode = slab_mode;
  a.min_rows = 1;
  a.cnt = cnt.data();
  a.seg = seg.data();
  for (int t = 0; t < kReachTiers; ++t) a.queue[t] = queue[t].data();
  a.pool = pool.data();
  a.pool_cap = pool_cap;
  a.words = 32;
  a.after_groups = thin ? kThinTier : kQueueTier;
  a.thin_rows = thin ? thin - 1 : 0;
  a.vis_words = (((uint32_t)m + 31u) / 32u + 31u) & ~31u;
  std::vector<uint32_t> vis(G * kThinWaves * a.vis_words, 0u);
  a.vis = vis.data();
  std::vector<uint32_t> bits(std::max<uint64_t>(bits_words, 1), 0x33333333u);
  a.bits = bits.data();
  a.bits_words = bits_words;
  a.slots = bits_words / a.words;
  a.rc = rc;
  a.lev = lev;
  a.lev_cap = (uint32_t)h[4];
  std::vector<uint64_t> part(G);
  const bool one = G % 2;
  simt::launch(G, kBlock, [&] { k_reach_mark<K>(ctrl.get(), E.data(), a.g); }, workers);
  if (one) {
    simt::launch(1, kBlock, [&] { k_reach_rank(ctrl.get(), a.g, nullptr, a.rc); }, workers);
  } else {
    simt::launch(G, kBlock, [&] { k_reach_rank_sum(a.g, part.data()); }, workers);
    simt::launch(G, kBlock, [&] { k_reach_rank(ctrl.get(), a.g, part.data(), a.rc); }, workers);
  }
  simt::launch(G, kBlock, [&] { k_reach_rows<K>(ctrl.get(), E.data(), a.g, a.rc); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_edges<K>(ctrl.get(), E.data(), a.g, a.rc, a.slab_mode); }, workers);
  if (slab_mode != 1) simt::launch(G, kBlock, [&] { k_reach_thread(a); }, workers);
  if (more) {
    std::vector<uint32_t> start(rstart.begin(), rstart.begin() + rc->rows + 1);
    for (uint32_t c = 0; c < rc->cols; ++c)
      if (cstart[c] != kReachNone) {
        const uint32_t r = (uint32_t)(std::lower_bound(start.begin(), start.end(), cstart[c]) - start.begin());
        cstart[c] += std::min(r, more_rows) * more;
      }
    for (uint32_t r = 0; r <= rc->rows; ++r) rstart[r] += std::min(r, more_rows) * more;
  }
  if (slab_mode != 0) {
    if (m > kSlabRows32) simt::launch(G, kSlabThreads, [&] { k_slab<true>(a); }, workers);
    else simt::launch(G, kSlabThreads, [&] { k_slab<false>(a); }, workers);
    simt::launch(G, kBlock, [&] { k_slab_count(a); }, workers);
  }
  if (slab_mode != 1) {
    simt::launch(G, 2 * kWave, [&] { k_reach_group<0, 4, 64, 128, 32, 32, 2>(a); }, workers);
    simt::launch(G, kWave, [&] { k_reach_group<1, 8, 256, 512, 128, 64, 1>(a); }, workers);
    if (thin) simt::launch(G, kThinWaves * kWave, [&] { k_reach_thin<96, 32>(a); }, workers);
    for (uint32_t x : vis)
      if (x) return 3;  // (all zeros between launches)
    // (a queue of 96 rows, so that wide levels outgrow it)
    if (one) simt::launch(G, kWave, [&] { k_reach_queue<1, 32, 96>(a); }, workers);
    else simt::launch(G, 4 * kWave, [&] { k_reach_queue<4, 32, 96>(a); }, workers);
    simt::launch(G, kReachBitsWaves * kWave, [&] { k_reach_bits<32, uint16_t>(a); }, workers);
  }
  if (one) {
    simt::launch(1, kBlock, [&] { k_reach_offsets<kScanBlocksMax>(a, nullptr, off.data()); }, workers);
  } else {
    simt::launch(G, kBlock, [&] { k_reach_sum(a, part.data()); }, workers);
    simt::launch(G, kBlock, [&] { k_reach_offsets<kScanBlocksMax>(a, part.data(), off.data()); }, workers);
  }
  std::ofstream f(out_path, std::ios::binary);
  put(f, rc->stop);
  put(f, rc->cursor);
  for (int t : {0, 1, kQueueTier, kBitsTier}) put(f, rc->queued[t]);
  put(f, rc->slab);
  put(f, rc->queued[kThinTier]);
  if (rc->stop) return 0;
  const int form = rc->slab ? 1 : 0;
  uint64_t L = 0;
  while (L < levels && lev[L].n[form]) ++L;
  put(f, L);
  for (uint64_t i = 0; i < L; ++i) {
    put(f, lev[i].n[form]);
    put(f, lev[i].d[form]);
  }
  const uint64_t F = off[rc->rows];
  put(f, F);
  ReachResult r{};
  r.cnt = cnt.data();
  r.seg = seg.data();
  r.off = off.data();
  r.rowkey = rowkey.data();
  r.colkey = colkey.data();
  r.pool = pool.data();
  r.bits = bits.data();
  r.bit_rows = queue[kBitsTier].data();
  r.rank = rank.data();
  r.n_bits = rc->slab ? 0 : rc->queued[kBitsTier];
  r.words = a.words;
  r.rows = rc->rows;
  r.cols = rc->cols;
  r.slab = rc->slab;
  r.w = w;
  std::vector<uint32_t> src(F, 0x11111111u), dst(F, 0x22222222u);
  std::vector<K> keys(F, (K)0x44444444u);
  const PutPairs pp{src.data(), dst.data(), id_mask(w)};
  const PutKeys<K> pk{keys.data(), w, id_mask(w)};
  const uint32_t lb = 3, bb = r.n_bits ? 2 : 0;
  if (r.slab) {
    simt::launch(2, kSlabOutWaves * kWave, [&] { k_slab_unpack(r, pp); }, workers);
    simt::launch(2, kSlabOutWaves * kWave, [&] { k_slab_unpack(r, pk); }, workers);
  } else {
    simt::launch(lb + bb, kBlock, [&] { k_reach_unpack(r, lb, pp); }, workers);
    simt::launch(lb + bb, kBlock, [&] { k_reach_unpack(r, lb, pk); }, workers);
  }
  std::vector<uint64_t> inst(num + 1);
  simt::launch(2, kBlock, [&] { k_reach_instances(r, (uint32_t)num, inst.data()); }, workers);
  for (uint64_t i = 0; i < F; ++i) put(f, ((uint64_t)src[i] << 32) | dst[i]);
  for (uint64_t i = 0; i < F; ++i) put(f, keys[i]);
  for (uint64_t i = 0; i <= num; ++i) put(f, inst[i]);
  return 0;
}

// The tiles' order over the blocks: every tile once, no block much past an even share, and
// at least half of the blocks that an even share would keep busy.
int tiles() {
  for (uint32_t most : {16u, 64u})
    for (uint32_t grid : {1u, 7u, 8u, 32u, 98u, 104u, 256u, 1536u, 2048u})
      for (uint32_t n : {0u, 1u, 7u, 8u, 9u, 20u, 63u, 64u, 65u, 100u, 128u, 129u, 511u, 512u, 513u, 600u, 1025u, 6450u, 70000u}) {
        std::vector<uint32_t> seen(n, 0);
        uint32_t busiest = 0, busy = 0;
        gridDim = {grid, 1, 1};
        const uint32_t C = xcd_stretch(n, most);
        if (C > most) return 5;
        for (uint32_t b = 0; b < grid; ++b) {
          blockIdx = {b, 0, 0};
          uint32_t mine = 0;
          for (uint32_t i = 0;; ++i, ++mine) {
            const uint32_t t = xcd_tile(i, C);
            if (t >= n) break;
            ++seen[t];
          }
          busiest = std::max(busiest, mine);
          busy += mine ? 1 : 0;
        }
        for (uint32_t x : seen)
          if (x != 1) return 6;
        const uint32_t even = (n + grid - 1) / grid;
        if (busiest > even + 1 + even / 16 || 2 * busy < std::min(n, grid)) {
          std::printf("grid %u tiles %u stretch %u: busiest %u busy %u\n", grid, n, C, busiest, busy);
          return 7;
        }
      }
  return 0;
}

int main(int argc, char** argv) {
  if (argc == 1) return tiles();
  std::ifstream f(argv[1], std::ios::binary);
  uint64_t h[6];
  f.read((char*)h, sizeof(h));
  std::vector<uint64_t> E(h[3]);
  f.read((char*)E.data(), 8 * E.size());
  const uint32_t G = (uint32_t)atoi(argv[3]);
  const unsigned workers = (unsigned)atoi(argv[4]);
  const uint64_t pool = strtoull(argv[5], nullptr, 10), bits = strtoull(argv[6], nullptr, 10);
  const int mode = atoi(argv[7]);
  const uint32_t rows = (uint32_t)strtoul(argv[8], nullptr, 10), more = (uint32_t)strtoul(argv[9], nullptr, 10);
  const uint32_t thin = (uint32_t)atoi(argv[10]);
  if (h[1] == 4) return run<uint32_t>(E, h, G, workers, pool, bits, mode, rows, more, thin, argv[2]);
  return run<uint64_t>(E, h, G, workers, pool, bits, mode, rows, more, thin, argv[2]);
}
