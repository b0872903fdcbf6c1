// Triangle counting on the renumbered graph (the kernels of wg_tri_kernels.h, current text) on the
// CPU SIMT shim.
//   tri_harness <in> <grid> <workers>
// in: u64 header (w, key bytes, |E|, span), then the sorted distinct keys of E (u64).
// Prints the count, the two-paths and the pieces of rows counted with bits.
#include <hip/hip_runtime.h>
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
template <typename T> inline T atomicCAS(T* p, T c, T v) {
  __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return c;
}
#define WG_OPAQUE(x) (void)0
#define __builtin_amdgcn_wave_barrier simt::wave_sync
#define __builtin_amdgcn_s_barrier __syncthreads
#define __builtin_amdgcn_fence(...) (void)0
#define __hip_atomic_load(p, ...) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, ...) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_or(p, v, ...) __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST)
#include "wg_launch.h"
#include "wg_reach_kernels.h"
#include "wg_tri_kernels.h"
#include <algorithm>
#include <fstream>
#include <memory>
using namespace wg;

template <typename K>
int run(const std::vector<uint64_t>& E64, const uint64_t* h, uint32_t G, unsigned workers) {
  const uint64_t m = E64.size(), span = h[3];
  std::vector<K> E(E64.begin(), E64.end()), up(m, (K)~0ull);
  std::unique_ptr<Ctrl> ctrl(new Ctrl);
  std::memset(ctrl.get(), 0, sizeof(Ctrl));
  ctrl->m_unique = m;
  std::unique_ptr<ReachCtl> rc(new ReachCtl);
  std::memset(rc.get(), 0, sizeof(ReachCtl));
  TriCtl tc;
  std::memset(&tc, 0, sizeof(tc));
  std::vector<uint32_t> rowkey(m), rstart(m + 1), colkey(m), cstart(m), col(m), us(m, 0), ue(m, 0);
  std::vector<uint2> edge(m + kReachEdgePad), piece(2 * m);
  std::vector<uint4> edge4(m);
  std::vector<RankWord> rank(span / 32 + 1);
  std::unique_ptr<uint8_t, void (*)(void*)> flags((uint8_t*)std::aligned_alloc(16, 2 * span), std::free);
  std::memset(flags.get(), 0, 2 * span);
  TriArgs a{};
  a.g.rowkey = rowkey.data();
  a.g.rstart = rstart.data();
  a.g.colkey = colkey.data();
  a.g.cstart = cstart.data();
  a.g.edge = edge.data();
  a.g.rank = rank.data();
  a.g.flags = flags.get();
  a.g.span = span;
  a.g.instances = 1;
  a.g.w = (int)h[0];
  a.rc = rc.get();
  a.tc = &tc;
  a.edge = edge4.data();
  a.col = col.data();
  a.ustart = us.data();
  a.uend = ue.data();
  a.piece = piece.data();
  a.w = 1;
  while ((1ull << a.w) < std::min(m, span)) ++a.w;
  simt::launch(G, kBlock, [&] { k_reach_mark<K>(ctrl.get(), E.data(), a.g); }, workers);
  simt::launch(1, kBlock, [&] { k_reach_rank(ctrl.get(), a.g, nullptr, a.rc); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_rows<K>(ctrl.get(), E.data(), a.g, a.rc); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_edges<K>(ctrl.get(), E.data(), a.g, a.rc, 0); }, workers);
  simt::launch(G, kTriEdgeThreads, [&] { k_tri_edges<K>(ctrl.get(), E.data(), a, up.data()); }, workers);
  std::stable_sort(up.begin(), up.begin() + (ptrdiff_t)tc.up,
                   [&](K x, K y) { return x >> a.w < y >> a.w; });
  simt::launch(G, kBlock, [&] { k_tri_starts<K>(a, up.data()); }, workers);
  simt::launch(G, kTriPairThreads, [&] { k_tri_pairs<K>(a, up.data()); }, workers);
  if (tc.pieces > 2 * m) return 4;
  simt::launch(G, kTriThreads, [&] { k_tri_bits<K, kTriWords>(a, up.data()); }, workers);
  printf("%llu %llu %u\n", 3 * tc.hits + tc.loops, tc.two_paths, tc.pieces);
  return 0;
}

int main(int argc, char** argv) {
  std::ifstream f(argv[1], std::ios::binary);
  uint64_t h[4];
  f.read((char*)h, sizeof(h));
  std::vector<uint64_t> E(h[2]);
  f.read((char*)E.data(), 8 * E.size());
  const uint32_t G = (uint32_t)atoi(argv[2]);
  const unsigned workers = (unsigned)atoi(argv[3]);
  return h[1] == 4 ? run<uint32_t>(E, h, G, workers) : run<uint64_t>(E, h, G, workers);
}
