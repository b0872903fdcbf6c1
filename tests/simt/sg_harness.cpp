// Same-generation on the renumbered graph (the kernels of wg_sg_kernels.h, current text) on the CPU
// SIMT shim: both forms over one graph, to the fixpoint.
//   sg_harness <in> <out> <grid> <workers> <form: 0 pairs by rounds, 1 pairs with the tail, 2 matrices>
//     <hash slots> <diagonal>
// in:  u64 header (w, key bytes, instances, |E|, level capacity, span), then the sorted distinct
//      keys of E (u64).
// out: u64 stop bits, base candidates, whether a degree is large; unless the stop bits are set: rounds R
//      (levels 0 .. R, the last one empty), then (tuples, candidates) of each, |SG|, its sorted keys.
#include <hip/hip_runtime.h>
struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
template <typename T> inline T atomicCAS(T* p, T c, T v) {
  __atomic_compare_exchange_n(p, &c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
  return c;
}
#define __hip_atomic_compare_exchange_strong(p, c, v, ...) \
  __atomic_compare_exchange_n(p, c, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)
#define __builtin_amdgcn_s_barrier __syncthreads
#define WG_OPAQUE(x) (void)0
#define __builtin_amdgcn_wave_barrier simt::wave_sync
#define __builtin_amdgcn_fence(...) (void)0
#define __hip_atomic_load(p, ...) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, ...) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_or(p, v, ...) __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST)
#include "wg_launch.h"
#include "wg_reach_kernels.h"
#include "wg_sg_kernels.h"
#include <fstream>
#include <memory>
using namespace wg;

template <typename T>
static void put(std::ofstream& f, const T& v) {
  const uint64_t x = (uint64_t)v;
  f.write((const char*)&x, 8);
}

template <typename K>
int run(const std::vector<uint64_t>& E64, const uint64_t* h, uint32_t G, unsigned workers, int form, uint64_t slots,
        int diagonal, const char* out_path) {
  const int w = (int)h[0];
  const uint64_t m = E64.size(), span = h[5];
  std::vector<K> E(E64.begin(), E64.end());
  std::unique_ptr<Ctrl> ctrl(new Ctrl);
  std::memset(ctrl.get(), 0, sizeof(Ctrl));
  ctrl->m_unique = m;
  // control blocks, levels and flags laid out as the engine's buffer is
  const uint64_t head = sizeof(ReachCtl) + sizeof(SgCtl), flags_at = reach_flags_at(head + h[4] * sizeof(SgLevel));
  std::vector<uint8_t> ctl_mem(flags_at + 2 * span + 256, 0);
  uint8_t* const base = (uint8_t*)(((uintptr_t)ctl_mem.data() + 255) & ~(uintptr_t)255);
  ReachCtl* const rc = (ReachCtl*)base;
  std::vector<uint32_t> rowkey(m), rstart(m + 1), colkey(m), cstart(m), se(m + kSlabThreads), sc_(m + kSlabThreads), cdeg(m);
  std::vector<uint2> edge(m + kReachEdgePad);
  std::vector<RankWord> rank(span / 32 + 1);
  SgArgs a{};
  a.g.rowkey = rowkey.data();
  a.g.rstart = rstart.data();
  a.g.colkey = colkey.data();
  a.g.cstart = cstart.data();
  a.g.edge = edge.data();
  a.g.slab_edge = se.data();
  a.g.slab_col = sc_.data();
  a.g.rank = rank.data();
  a.g.flags = base + flags_at;
  a.g.span = span;
  a.g.instances = (uint32_t)h[2];
  a.g.w = w;
  a.rc = rc;
  SgCtl& ctl = *(SgCtl*)(base + sizeof(ReachCtl));
  a.sc = &ctl;
  SgLevel* const lev = (SgLevel*)(base + head);
  a.lev = lev;
  a.lev_cap = (uint32_t)h[4];
  simt::launch(G, kBlock, [&] { k_reach_mark<K>(ctrl.get(), E.data(), a.g); }, workers);
  simt::launch(1, kBlock, [&] { k_reach_rank(ctrl.get(), a.g, nullptr, a.rc); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_rows<K>(ctrl.get(), E.data(), a.g, a.rc); }, workers);
  simt::launch(G, kBlock, [&] { k_reach_edges<K>(ctrl.get(), E.data(), a.g, a.rc, 0); }, workers);
  std::vector<uint4> edge4(m);
  a.edge = edge4.data();
  simt::launch(G, kSgEdgeThreads, [&] { k_sg_edges<K>(ctrl.get(), E.data(), a); }, workers);
  const uint64_t cols = rc->cols;
  const uint32_t slabs = (uint32_t)((cols + 31) / 32);
  std::ofstream f(out_path, std::ios::binary);
  uint64_t rounds = 0;
  std::vector<K> result;
  std::vector<SgBucket> tab;
  std::vector<unsigned long long> keys;
  std::vector<uint4> front;
  std::vector<uint32_t> S, D, M;
  if (form == 2) {
    S.assign((uint64_t)slabs * cols, 0x5A5A5A5Au);
    D = M = S;
    a.S = S.data();
    a.D = D.data();
    a.M = M.data();
    a.base_edge = se.data();
    a.step_edge = sc_.data();
    a.cdeg = cdeg.data();
    simt::launch(G, kBlock, [&] { k_sg_matrix_edges<K>(ctrl.get(), E.data(), a); }, workers);
    simt::launch(G, kSlabThreads, [&] { k_sg_matrix_base(a, slabs); }, workers);
    // (rounds past the fixpoint are no-ops)
    for (uint32_t j = 1; lev[rounds].n || j % 4 != 1; ++j) {
      simt::launch(G, kSlabThreads, [&] { k_sg_matrix_half(a, j, slabs); }, workers);
      simt::launch(G, kSlabThreads, [&] { k_sg_matrix_rest(a, j, slabs); }, workers);
      if (lev[rounds].n) rounds = j;
    }
    while (rounds > 0 && lev[rounds - 1].n == 0) --rounds;
    if (!diagonal) simt::launch(G, kBlock, [&] { k_sg_matrix_diagonal(a, (uint32_t)cols); }, workers);
    uint64_t dropped = 0;
    for (uint64_t y = 0; y < cols; ++y)
      for (uint64_t x = 0; x < cols; ++x)
        if ((S[(x / 32) * cols + y] >> (x % 32)) & 1u)
          result.push_back(((K)colkey[y] << w) | (K)(colkey[x] & id_mask(w)));
    if (!diagonal) {
      for (uint64_t i = 0; i <= rounds; ++i) dropped += lev[i].n;
      if (dropped - result.size() != ctl.diagonal) return 4;
    }
  } else {
    tab.assign(slots / 4, SgBucket{{kSgEmpty, kSgEmpty, kSgEmpty, kSgEmpty}});
    keys.assign(std::max<uint64_t>(slots / 2, 1), 0);
    front.assign(std::max<uint64_t>(slots / 2, 1), uint4{0, 0, 0, 0});
    a.tab = tab.data()->s;
    a.mask = slots - 1;
    a.keys = keys.data();
    a.key_cap = slots / 2;
    a.front = front.data();
    a.front_cap = slots / 2;
    simt::launch(G, kSgThreads, [&] { k_sg_pairs_base(ctrl.get(), a); }, workers);
    uint32_t j = 1;
    while (!ctl.stop && lev[rounds].found) {
      simt::launch(G, kSgThreads, [&] { k_sg_pairs_round(a, j); }, workers);
      rounds = j++;
      if (form == 1) {
        simt::launch(1, kSgThreads, [&] { k_sg_pairs_tail(a, j); }, workers);
        if (ctl.next > j) rounds = ctl.next - 1;
        j = ctl.next;
      }
    }
    if (!ctl.stop) {
      uint64_t n = 0, both = 0, diag = 0;
      for (uint64_t i = 0; i <= rounds; ++i) {
        lev[i].n = 2ull * (uint32_t)lev[i].found - lev[i].diag;
        n += (uint32_t)lev[i].found;
        both += lev[i].n;
        diag += lev[i].diag;
      }
      result.assign(both - (diagonal ? 0 : diag), (K)0x77777777u);
      simt::launch(G, kBlock, [&] { k_sg_emit<K>(a, n, diagonal, result.data()); }, workers);
      if (ctl.out != result.size()) return 5;
    }
  }
  put(f, ctl.stop);
  put(f, ctl.base);
  put(f, ctl.wide);
  if (ctl.stop) return 0;
  put(f, rounds);
  for (uint64_t i = 0; i <= rounds; ++i) {
    put(f, lev[i].n);
    put(f, lev[i].c);
  }
  std::sort(result.begin(), result.end());
  put(f, result.size());
  for (const K& k : result) put(f, k);
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
  const int form = atoi(argv[5]), diagonal = atoi(argv[7]);
  const uint64_t slots = strtoull(argv[6], nullptr, 10);
  if (h[1] == 4) return run<uint32_t>(E, h, G, workers, form, slots, diagonal, argv[2]);
  return run<uint64_t>(E, h, G, workers, form, slots, diagonal, argv[2]);
}
