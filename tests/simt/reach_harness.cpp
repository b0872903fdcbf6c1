// The row-at-a-time closure (the kernels of wg_reach_kernels.h, current text) on the CPU SIMT shim: every
// tier, the row offsets and the unpacking, over one graph.
//   reach_harness <in> <out> <grid> <workers> <pool entries> <bitmap slots> <start tier>
// in:  u64 header (w, key bytes, instances, |E|, hub degree, level capacity), then the sorted
//      distinct keys of E (u64).
// out: u64 stop bits, pool entries used, rows queued for the three tiers; unless the stop bits
//      are set: levels L, then (tuples, degrees) of each, the tuples' keys (u64, from the unpacked
//      pairs), the keys as k_reach_keys writes them (u64) and the instances' offsets.
// start tier 0: the thread tier first (its rows go on to the group tier); 1, 2: the thread tier
//      sends every row it cannot hold to the queue or the bits tier directly.
#include <hip/hip_runtime.h>
template <typename T> inline T atomicCAS(T* p, T c, T v) {
  __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return c;
}
#define __builtin_amdgcn_wave_barrier simt::wave_sync
#define __builtin_amdgcn_fence(...) (void)0
#define __hip_atomic_load(p, ...) __atomic_load_n(p, __ATOMIC_SEQ_CST)
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
        uint64_t slots, int start, const char* out_path) {
  const int w = (int)h[0];
  const uint64_t m = E64.size(), num = h[2];
  const K mask = (K)((K(1) << w) - 1);
  std::vector<K> E(E64.begin(), E64.end());
  const uint64_t dense = num << w;
  std::vector<uint32_t> R(dense + 1), Edst(std::max<uint64_t>(m, 1));
  for (uint64_t v = 0, i = 0; v <= dense; ++v) {
    while (i < m && (uint64_t)(E[i] >> w) < v) ++i;
    R[v] = (uint32_t)i;
  }
  for (uint64_t i = 0; i < m; ++i) Edst[i] = (uint32_t)(E[i] & mask);
  std::unique_ptr<Ctrl> ctrl(new Ctrl);
  std::memset(ctrl.get(), 0, sizeof(Ctrl));
  ctrl->m_unique = m;
  std::unique_ptr<ReachCtl> rc(new ReachCtl);
  std::memset(rc.get(), 0, sizeof(ReachCtl));
  std::vector<ReachLevel> lev(h[5], ReachLevel{0, 0});
  std::vector<uint32_t> cnt(m, 0xDEADu), seg(m, 0xBEEFu), off(m + 1), pool(std::max<uint64_t>(pool_cap, 1), 0x5A5A5A5Au);
  std::vector<uint32_t> queue[3];
  for (auto& q : queue) q.assign(m, 0x77777777u);
  ReachArgs a;
  a.R = R.data();
  a.Edst = Edst.data();
  a.w = w;
  a.tier_after[0] = start;
  a.tier_after[1] = 1;
  a.tier_after[2] = w <= 18 ? 2 : -1;
  a.hub = (uint32_t)h[4];
  a.hub_tier = w <= 18 ? 2 : 1;
  a.cnt = cnt.data();
  a.seg = seg.data();
  for (int t = 0; t < 3; ++t) a.queue[t] = queue[t].data();
  a.pool = pool.data();
  a.pool_cap = pool_cap;
  a.words = w > 5 ? 1u << (w - 5) : 1u;
  std::vector<uint32_t> bits(std::max<uint64_t>(slots * a.words, 1), 0x33333333u);
  a.bits = bits.data();
  a.slots = slots;
  a.rc = rc.get();
  a.lev = lev.data();
  a.lev_cap = (uint32_t)h[5];
  std::vector<uint64_t> part(G);
  if (w > 10) return 3;
  simt::launch(G, kBlock, [&] { k_reach_thread<K>(ctrl.get(), E.data(), a); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_group(a); }, workers);
  // (a queue of 96 ids, so that wide levels outgrow it; one wave, then the wide form)
  if (G % 2) simt::launch(G, kWave, [&] { k_reach_queue<1, 32, 96, uint16_t>(a); }, workers);
  else simt::launch(G, 4 * kWave, [&] { k_reach_queue<4, 32, 96, uint32_t>(a); }, workers);
  simt::launch(G, kReachBitsWaves * kWave, [&] { k_reach_bits<32, uint16_t>(a); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_sum(ctrl.get(), a, part.data()); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_offsets<kScanBlocksMax>(ctrl.get(), a, part.data(), off.data()); }, workers);
  std::ofstream f(out_path, std::ios::binary);
  put(f, rc->stop);
  put(f, rc->cursor);
  for (int t = 0; t < 3; ++t) put(f, rc->queued[t]);
  if (rc->stop) return 0;
  uint64_t L = 0;
  while (L < lev.size() && lev[L].n) ++L;
  put(f, L);
  for (uint64_t i = 0; i < L; ++i) {
    put(f, lev[i].n);
    put(f, lev[i].d);
  }
  const uint64_t F = off[m];
  put(f, F);
  ReachResult r;
  r.cnt = cnt.data();
  r.seg = seg.data();
  r.off = off.data();
  r.R = R.data();
  r.pool = pool.data();
  r.bits = bits.data();
  r.bit_rows = queue[2].data();
  r.n_bits = rc->queued[2];
  r.words = a.words;
  r.m = m;
  r.w = w;
  std::vector<uint32_t> src(F, 0x11111111u), dst(F, 0x22222222u);
  std::vector<K> keys(F, (K)0x44444444u);
  const uint32_t lb = 3, bb = r.n_bits ? 2 : 0;
  simt::launch(lb + bb, kBlock, [&] { k_reach_unpack<K>(r, E.data(), lb, src.data(), dst.data()); }, workers);
  simt::launch(lb + bb, kBlock, [&] { k_reach_keys<K>(r, E.data(), lb, keys.data()); }, workers);
  std::vector<uint64_t> inst(num + 1);
  simt::launch(2, kBlock, [&] { k_reach_instances(r, (uint32_t)num, inst.data()); }, workers);
  for (uint64_t i = 0; i < F; ++i) put(f, ((uint64_t)src[i] << 32) | dst[i]);
  for (uint64_t i = 0; i < F; ++i) put(f, keys[i]);
  for (uint64_t i = 0; i <= num; ++i) put(f, inst[i]);
  return 0;
}

int main(int argc, char** argv) {
  std::ifstream f(argv[1], std::ios::binary);
  uint64_t h[6];
  f.read((char*)h, sizeof(h));
  std::vector<uint64_t> E(h[3]);
  f.read((char*)E.data(), 8 * E.size());
  const uint32_t G = (uint32_t)atoi(argv[3]);
  const unsigned workers = (unsigned)atoi(argv[4]);
  const uint64_t pool = strtoull(argv[5], nullptr, 10), slots = strtoull(argv[6], nullptr, 10);
  const int start = atoi(argv[7]);
  if (h[1] == 4) return run<uint32_t>(E, h, G, workers, pool, slots, start, argv[2]);
  return run<uint64_t>(E, h, G, workers, pool, slots, start, argv[2]);
}
