// Kernels of same-generation on the renumbered graph (see wg_sg.h).
#pragma once

#include "wg_reach_device.h"
#include "wg_sg.h"

namespace wg {

// The edges with what a round needs of them in one load, and the counts that choose the form.
// (large blocks: one same-address atomic each)
template <typename K>
__global__ __launch_bounds__(kSgEdgeThreads) void k_sg_edges(const Ctrl* ctrl, const K* __restrict__ E, SgArgs a) {
  __shared__ uint64_t s_wave[kSgEdgeThreads / kWave];
  const uint64_t n = ctrl->m_unique;
  uint64_t sum = 0;
  bool wide = false;
  for (uint64_t i = (uint64_t)blockIdx.x * kSgEdgeThreads + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kSgEdgeThreads) {
    const uint32_t row = head_row<K>(E[i], a.g.w);
    const uint2 x = a.g.edge[i];
    const RankWord q = a.g.rank[row >> 5];
    const uint32_t key = a.g.colkey[x.x & ~kReachLast];
    const uint32_t r = q.rowpre + bits_below(q.rowbits, row);
    const uint32_t first = a.g.rstart[r], end = a.g.rstart[r + 1];
    uint4 e;
    e.x = x.x & ~kReachLast;
    e.y = x.y;
    e.z = 0;
    if (x.y != kReachNone) {
      const RankWord t = a.g.rank[key >> 5];
      e.z = a.g.rstart[t.rowpre + bits_below(t.rowbits, key) + 1] - x.y;
    }
    e.w = end - (uint32_t)i;
    a.edge[i] = e;
    sum += end - first - 1;
    wide |= end - first > kSgPairDegree;
  }
  uint64_t total;
  (void)block_excl_scan<uint64_t, kSgEdgeThreads / kWave>(sum, s_wave, total);
  if (threadIdx.x == 0 && total) atomicAdd(&a.sc->base, (unsigned long long)total);
  if (wide) a.sc->wide = 1;
}

// ---------------------------------------------------------------------------
// Pairs.
// ---------------------------------------------------------------------------
constexpr unsigned long long kSgEmpty = ~0ull;  // (columns have 31 bits)

struct alignas(32) SgBucket {
  unsigned long long s[4];
};

// Inserts the pair {x, y}; true if it was not in the table.  A bucket is read whole before the
// compare-and-swap on its first empty slot: two latencies, whatever the load (slot by slot, the
// longest probe of a wave's 64 lanes took 5).  A slot is written once, so a stale read shows at
// worst an empty one.  Solo: the caller's workgroup is the only one at the table (the swap stays in
// its XCD's L2).
template <bool Solo>
__device__ __forceinline__ bool sg_insert(const SgArgs& a, uint32_t x, uint32_t y, unsigned long long& key) {
  key = x < y ? ((unsigned long long)x << 32) | y : ((unsigned long long)y << 32) | x;
  unsigned long long h = key;
  h ^= h >> 29;
  h *= 0x9E3779B97F4A7C15ull;  // (a multiplicative hash: 2^64 over the golden ratio)
  h ^= h >> 32;
  uint64_t at = h & a.mask & ~3ull;
  for (uint32_t p = 0; p < kSgProbes; ++p) {
    SgBucket b = *(const SgBucket*)(a.tab + at);
    for (;;) {
      uint32_t q = 4;
#pragma unroll
      for (int i = 3; i >= 0; --i)
        if (b.s[i] == kSgEmpty) q = i;
      if (b.s[0] == key || b.s[1] == key || b.s[2] == key || b.s[3] == key) return false;
      if (q == 4) break;
      unsigned long long old = kSgEmpty;
      if (__hip_atomic_compare_exchange_strong(&a.tab[at + q], &old, key, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               Solo ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT))
        return true;
      if (old == key) return false;
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i)
        if (i == q) b.s[i] = old;
    }
    at = (at + 4) & a.mask;
  }
  atomicOr(&a.sc->stop, (uint32_t)kSgTableFull);
  return false;
}

__device__ __forceinline__ void sg_put_key(const SgArgs& a, uint64_t p, unsigned long long key) {
  if (p < a.key_cap) a.keys[p] = key;
  else atomicOr(&a.sc->stop, (uint32_t)kSgListFull);
}
__device__ __forceinline__ void sg_put_front(const SgArgs& a, uint64_t p, uint4 f) {
  if (p < a.front_cap) a.front[p] = f;
  else atomicOr(&a.sc->stop, (uint32_t)kSgListFull);
}

// A wave's pairs, whose children's pairs its lanes take one candidate each, whatever the degrees.
struct SgWave {
  uint4 front[kWave];   // the pairs that have candidates
  uint32_t pre[kWave];  // ... candidates before each
  uint32_t mark[kWave];
};

// Expands the lanes' pairs f, 64 candidates a step until over(): step(true if the lane's is new, its key,
// its entry of the next round's list), by whole waves.  Returns the candidates.  The pair of
// candidate k is the one whose start is the last at or below k: its rank is counted from the
// starts' bits (a bisection took ten LDS round trips, 4,000 cycles with 16 waves at it).
template <bool Solo, typename Step, typename Over>
__device__ __forceinline__ uint32_t sg_expand(const SgArgs& a, SgWave& w, uint4 f, Step step, Over over) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t n = f.z * f.w, incl = wave_incl_scan<uint32_t>(n), pre = incl - n;
  const uint32_t total = __shfl(incl, kWave - 1, kWave);
  const uint64_t some = __builtin_amdgcn_ballot_w64(n != 0);
  wave_lds_sync();
  if (n) {
    const uint32_t at = (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
    w.front[at] = f;
    w.pre[at] = pre;
  }
  uint32_t pairs = 0;  // with a start before this step
  for (uint32_t k0 = 0; k0 < total && !over(); k0 += kWave) {
    wave_lds_sync();
    w.mark[lane] = 0;
    wave_lds_sync();
    if (n && pre >= k0 && pre < k0 + kWave) w.mark[pre - k0] = 1;
    wave_lds_sync();
    const uint64_t starts = __builtin_amdgcn_ballot_w64(w.mark[lane] != 0);
    const uint32_t k = k0 + lane;
    bool is_new = false;
    unsigned long long key = 0;
    uint4 next;
    next.x = next.y = next.z = next.w = 0;
    if (k < total) {
      const uint32_t p = pairs + (uint32_t)__popcll(starts & ((2ull << lane) - 1ull)) - 1u;
      const uint4 g = w.front[p];
      // (r < 4,096, g.w <= 64: half past a whole number never rounds over to the next)
      const uint32_t r = k - w.pre[p], i = (uint32_t)(((float)r + 0.5f) / (float)g.w), j = r - i * g.w;
      // (a, a): its children's unordered pairs, (x, x) included
      if (g.x != g.y || j >= i) {
        const uint4 x = a.edge[g.x + i], y = a.edge[g.y + j];
        is_new = sg_insert<Solo>(a, x.x, y.x, key);
        next.x = x.y;
        next.y = y.y;
        next.z = x.z;
        next.w = y.z;
      }
    }
    pairs += (uint32_t)__popcll(starts);
    step(is_new, key, next);
  }
  return total;
}

// Adds the candidates of the wave's pairs f to an LDS counter: both orders of all but (a, a)'s.
__device__ __forceinline__ void sg_count(unsigned long long* cand, uint4 f, uint32_t total) {
  if (lane_id() == 0 && total) atomicAdd(cand, 2ull * total);
  if (f.x == f.y && f.z) atomicAdd(cand, 0ull - (unsigned long long)(f.z * f.w));
}

// Which of a wave's lanes found a pair, and places for them by one atomic on `found` (keys in the
// low half, fronts in the high half).
struct SgPlace {
  uint32_t key, front;    // the lane's places
  uint32_t first, keys;   // the wave's first key's and how many
  bool expand, diag;
};
__device__ __forceinline__ SgPlace sg_place(bool is_new, unsigned long long key, uint4 next, unsigned long long* found) {
  SgPlace p;
  p.expand = is_new && next.z != 0 && next.w != 0;
  p.diag = is_new && (uint32_t)(key >> 32) == (uint32_t)key;
  const uint64_t nb = __builtin_amdgcn_ballot_w64(is_new), fb = __builtin_amdgcn_ballot_w64(p.expand);
  p.keys = (uint32_t)__popcll(nb);
  p.first = p.key = p.front = 0;
  if (p.keys) {
    const uint64_t below = (1ull << lane_id()) - 1ull;
    unsigned long long at = 0;
    if (lane_id() == 0) at = atomicAdd(found, ((unsigned long long)__popcll(fb) << 32) | p.keys);
    p.first = wave_uniform((uint32_t)at);
    p.key = p.first + (uint32_t)__popcll(nb & below);
    p.front = wave_uniform((uint32_t)(at >> 32)) + (uint32_t)__popcll(fb & below);
  }
  return p;
}

// Pairs found by a block, buffered in LDS and appended to their round's stretches of the lists a
// buffer at a time: one atomic takes the places of both (same-address atomics of all blocks
// serialise at 12 ns).
struct SgOut {
  unsigned long long keys[kSgBuf];
  uint4 front[kSgBuf];
  unsigned long long found, at;  // keys (low half), fronts (high half)
  unsigned long long valid;      // ... that are in the buffers, once they were too small
  unsigned long long cand;
  uint32_t diag;
  volatile uint32_t full;  // the list of keys is
};

__device__ __forceinline__ void sg_found(const SgArgs& a, SgOut& o, bool is_new, unsigned long long key, uint4 next,
                                         uint32_t kstart, uint32_t fstart, SgLevel* out) {
  SgPlace p = sg_place(is_new, key, next, &o.found);
  if (p.diag) atomicAdd(&o.diag, 1u);
  if (p.first + p.keys <= kSgBuf) {
    if (is_new) o.keys[p.key] = key;
    if (p.expand) o.front[p.front] = next;
  } else {
    // full: straight to the lists (the first wave past the end notes where the buffers end)
    if (p.first <= kSgBuf && lane_id() == 0) o.valid = ((unsigned long long)p.front << 32) | p.first;
    p = sg_place(is_new, key, next, &out->found);
    if ((uint64_t)kstart + p.first + p.keys > a.key_cap) o.full = 1;
    if (is_new) sg_put_key(a, (uint64_t)kstart + p.key, key);
    if (p.expand) sg_put_front(a, (uint64_t)fstart + p.front, next);
  }
}

// (the whole block) empties the buffers into the lists; true if that of the keys is full: the round is
// over then
__device__ __forceinline__ bool sg_flush(const SgArgs& a, SgOut& o, uint32_t kstart, uint32_t fstart, SgLevel* out) {
  block_lds_sync();
  const unsigned long long found = (uint32_t)o.found <= kSgBuf ? o.found : o.valid;
  const uint32_t nk = (uint32_t)found, nf = (uint32_t)(found >> 32);
  if (threadIdx.x == 0) {
    o.full = 0;
    if (nk) {
      o.at = atomicAdd(&out->found, found);
      o.full = (uint64_t)kstart + (uint32_t)o.at + nk > a.key_cap ? 1u : 0u;
    }
    if (o.diag) atomicAdd(&out->diag, o.diag);
    if (o.cand) atomicAdd(&out->c, o.cand);
  }
  block_lds_sync();
  const uint64_t at_k = (uint64_t)kstart + (uint32_t)o.at, at_f = (uint64_t)fstart + (uint32_t)(o.at >> 32);
  for (uint32_t t = threadIdx.x; t < nk; t += kSgThreads) sg_put_key(a, at_k + t, o.keys[t]);
  for (uint32_t t = threadIdx.x; t < nf; t += kSgThreads) sg_put_front(a, at_f + t, o.front[t]);
  const bool full = o.full != 0;
  block_lds_sync();
  if (threadIdx.x == 0) {
    o.found = o.cand = 0;
    o.diag = 0;
  }
  block_lds_sync();
  return full;
}

// The base pairs: every edge with the later edges of its row.
__global__ __launch_bounds__(kSgThreads) void k_sg_pairs_base(const Ctrl* ctrl, SgArgs a) {
  constexpr uint32_t T = kSgThreads;
  __shared__ SgOut o;
  __shared__ SgWave s_wave[T / kWave];
  const uint64_t n = ctrl->m_unique;
  const uint32_t tid = threadIdx.x;
  if (tid == 0) {
    o.found = o.cand = 0;
    o.diag = o.full = 0;
  }
  block_lds_sync();
  for (uint64_t base = (uint64_t)blockIdx.x * T; base < n; base += (uint64_t)gridDim.x * T) {
    const uint64_t i = base + tid;
    uint4 f;
    f.x = (uint32_t)i;
    f.y = (uint32_t)i + 1;
    f.z = 1;
    f.w = i < n ? a.edge[i].w - 1 : 0;
    sg_expand<false>(a, s_wave[tid / kWave], f, [&](bool is_new, unsigned long long key, uint4 next) {
      sg_found(a, o, is_new, key, next, 0, 0, &a.lev[0]);
    }, [&] { return wave_uniform(o.full) != 0; });
    if (sg_flush(a, o, 0, 0, &a.lev[0])) break;
  }
}

// Round j: expands the pairs found in round j - 1.  (Its stretches of the lists start where those of
// round j - 1 end; block 0 notes them for the next round.)
__global__ __launch_bounds__(kSgThreads) void k_sg_pairs_round(SgArgs a, uint32_t j) {
  constexpr uint32_t kWaves = kSgThreads / kWave;
  __shared__ SgOut o;
  __shared__ SgWave s_wave[kWaves];
  const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id(), wid = tid / kWave;
  const SgLevel prev = a.lev[j - 1];
  if (j >= a.lev_cap) {  // (enqueued behind the last round counted; nothing to do after the fixpoint)
    if (tid == 0 && blockIdx.x == 0 && prev.found != 0) atomicOr(&a.sc->stop, (uint32_t)kSgDeep);
    return;
  }
  if (block_stop(a.sc->stop != 0)) return;
  const uint32_t fn = (uint32_t)(prev.found >> 32);
  const uint32_t kstart = prev.kstart + (uint32_t)prev.found, fstart = prev.fstart + fn;
  SgLevel* const out = &a.lev[j];
  if (blockIdx.x == 0 && tid == 0) {
    out->kstart = kstart;
    out->fstart = fstart;
  }
  // pairs per wave: over all the waves of the grid, but no block for less than 256
  const uint32_t waves = gridDim.x * kWaves;
  const uint32_t per = min(max((fn + waves - 1) / waves, 256u / kWaves), (uint32_t)kWave);
  if ((uint64_t)blockIdx.x * kWaves * per >= fn) return;
  if (tid == 0) {
    o.found = o.cand = 0;
    o.diag = o.full = 0;
  }
  block_lds_sync();
  for (uint64_t base = (uint64_t)blockIdx.x * kWaves * per; base < fn; base += (uint64_t)waves * per) {
    const uint64_t i = base + (uint64_t)wid * per + lane;
    uint4 f;
    f.x = f.y = f.z = f.w = 0;
    if (lane < per && i < fn) f = a.front[prev.fstart + i];
    const uint32_t total = sg_expand<false>(a, s_wave[wid], f, [&](bool is_new, unsigned long long key, uint4 next) {
      sg_found(a, o, is_new, key, next, kstart, fstart, out);
    }, [&] { return wave_uniform(o.full) != 0; });
    sg_count(&o.cand, f, total);
    if (sg_flush(a, o, kstart, fstart, out)) break;
  }
}

// Rounds j, j + 1, ... in one workgroup, while each has at most kSgTail pairs to expand; the pairs of
// the next round stay in LDS.  sc->next: the round it leaves to the host.  (A full table or list
// drops pairs, so that the rounds end then too.)
__global__ __launch_bounds__(kSgThreads) void k_sg_pairs_tail(SgArgs a, uint32_t j) {
  constexpr uint32_t kWaves = kSgThreads / kWave;
  struct Counts {
    unsigned long long found, cand;
    uint32_t diag;
  };
  __shared__ uint4 s_front[2][kSgTail];
  __shared__ SgWave s_wave[kWaves];
  __shared__ Counts s_cnt[3];  // (this round's; the next one's, cleared; the last one's, being read)
  __shared__ uint32_t s_stop;
  const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id(), wid = tid / kWave;
  const SgLevel first = a.lev[j - 1];
  uint32_t fn = (uint32_t)(first.found >> 32);
  if (block_stop(a.sc->stop != 0) || fn > kSgTail || first.found == 0) {
    if (tid == 0) a.sc->next = j;
    return;
  }
  uint32_t kstart = first.kstart + (uint32_t)first.found, fstart = first.fstart + fn;
  for (uint32_t t = tid; t < fn; t += kSgThreads) s_front[(j - 1) & 1u][t] = a.front[first.fstart + t];
  if (tid == 0) {
    s_cnt[j % 3] = Counts{0, 0, 0};
    s_stop = 0;
  }
  block_lds_sync();
  for (;; ++j) {
    if (j >= a.lev_cap) {
      if (tid == 0) atomicOr(&a.sc->stop, (uint32_t)kSgDeep);
      break;
    }
    if (tid == 0) {
      s_cnt[(j + 1) % 3] = Counts{0, 0, 0};
      if (j % kStopLevels == 0) s_stop = cancelled(a.cancel, &a.sc->stop);
    }
    Counts& cnt = s_cnt[j % 3];
    const uint32_t per = min(max((fn + kWaves - 1) / kWaves, 1u), (uint32_t)kWave);
    for (uint32_t base = wid * per; base < fn; base += kWaves * per) {
      uint4 f;
      f.x = f.y = f.z = f.w = 0;
      if (lane < per && base + lane < fn) f = s_front[(j - 1) & 1u][base + lane];
      const uint32_t total = sg_expand<true>(a, s_wave[wid], f, [&](bool is_new, unsigned long long key, uint4 next) {
        const SgPlace p = sg_place(is_new, key, next, &cnt.found);
        if (is_new) sg_put_key(a, (uint64_t)kstart + p.key, key);
        if (p.diag) atomicAdd(&cnt.diag, 1u);
        if (p.expand) {
          if (p.front < kSgTail) s_front[j & 1u][p.front] = next;
          else sg_put_front(a, (uint64_t)fstart + p.front, next);  // (for a round that goes back to the host)
        }
      }, [] { return false; });
      sg_count(&cnt.cand, f, total);
    }
    block_lds_sync();
    const uint32_t nk = (uint32_t)cnt.found, nf = (uint32_t)(cnt.found >> 32);
    if (tid == 0) {
      SgLevel l;
      l.n = 0;
      l.c = cnt.cand;
      l.found = cnt.found;
      l.diag = cnt.diag;
      l.kstart = kstart;
      l.fstart = fstart;
      l.pad = 0;
      a.lev[j] = l;
    }
    if (nf > kSgTail)
      for (uint32_t t = tid; t < kSgTail; t += kSgThreads) sg_put_front(a, (uint64_t)fstart + t, s_front[j & 1u][t]);
    kstart += nk;
    fstart += nf;
    fn = nf;
    if (nk == 0 || nf > kSgTail || s_stop || kstart > a.key_cap) {
      ++j;
      break;
    }
  }
  if (tid == 0) a.sc->next = j;
}

constexpr int kSgEmitItems = 8;

template <typename K>
__global__ __launch_bounds__(kBlock) void k_sg_emit(SgArgs a, uint64_t n, int diagonal, K* __restrict__ out) {
  constexpr uint32_t T = kBlock * kSgEmitItems;
  __shared__ uint32_t s_wave[kWavesPerBlock];
  __shared__ unsigned long long s_at;
  const uint32_t idm = id_mask(a.g.w);
  for (uint64_t base = (uint64_t)blockIdx.x * T; base < n; base += (uint64_t)gridDim.x * T) {
    uint32_t kx[kSgEmitItems], ky[kSgEmitItems], c[kSgEmitItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kSgEmitItems; ++k) {
      const uint64_t i = base + (uint64_t)k * kBlock + threadIdx.x;
      c[k] = 0;
      if (i < n) {
        const unsigned long long key = a.keys[i];
        kx[k] = a.g.colkey[(uint32_t)(key >> 32)];
        ky[k] = a.g.colkey[(uint32_t)key];
        c[k] = kx[k] != ky[k] ? 2u : (diagonal ? 1u : 0u);
      }
      sum += c[k];
    }
    uint32_t total;
    uint32_t at = block_excl_scan<uint32_t>(sum, s_wave, total);
    if (threadIdx.x == 0) s_at = atomicAdd(&a.sc->out, (unsigned long long)total);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSgEmitItems; ++k) {
      const uint64_t p = s_at + at;
      if (c[k]) out[p] = ((K)kx[k] << a.g.w) | (K)(ky[k] & idm);
      if (c[k] > 1) out[p + 1] = ((K)ky[k] << a.g.w) | (K)(kx[k] & idm);
      at += c[k];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Matrices.
// ---------------------------------------------------------------------------
template <typename K>
__global__ __launch_bounds__(kBlock) void k_sg_matrix_edges(const Ctrl* ctrl, const K* __restrict__ E, SgArgs a) {
  const uint64_t n = ctrl->m_unique;
  const uint32_t rows = a.rc->rows, cols = a.rc->cols;
  const uint32_t per = slab_per((uint32_t)n);
  const uint64_t end = (uint64_t)per * kSlabThreads;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < end; i += (uint64_t)gridDim.x * kBlock) {
    uint32_t p = rows, src = cols, c = cols;  // (past the edges: idle)
    if (i < n) {
      const uint32_t row = head_row<K>(E[i], a.g.w);
      const RankWord q = a.g.rank[row >> 5];
      p = q.rowpre + bits_below(q.rowbits, row);
      if ((q.colbits >> (row & 31u)) & 1u) src = q.colpre + bits_below(q.colbits, row);
      const uint4 e = a.edge[i];
      c = e.x;
      a.cdeg[c] = e.z;  // (every edge into c writes the same)
    }
    const uint64_t at = (i % per) * kSlabThreads + i / per;
    a.base_edge[at] = (p << 16) | c;
    a.step_edge[at] = (src << 16) | c;
  }
}

// acc[x] |= D[p] for every edge p << 16 | x of the thread's stretch.
__device__ __forceinline__ void sg_gather(const uint32_t* __restrict__ ed, uint32_t per, const uint32_t* D, uint32_t* acc) {
  constexpr uint32_t TH = kSlabThreads;
  for (uint32_t k = 0; k < per; k += 8) {
    uint32_t u[8], d[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = k + q < per ? ed[(k + q) * TH + threadIdx.x] : kReachNone;
#pragma unroll
    for (int q = 0; q < 8; ++q) d[q] = u[q] != kReachNone ? D[u[q] >> 16] : 0u;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (d[q]) atomicOr(&acc[u[q] & 0xFFFFu], d[q]);
  }
}

// Word l of a 32 x 32 bit block (lane l of each half wave) becomes column l.
__device__ __forceinline__ uint32_t transpose32(uint32_t v) {
  const uint32_t lane = (uint32_t)lane_id() & 31u;
  uint32_t m = 0x0000FFFFu;
#pragma unroll
  for (uint32_t s = 16; s >= 1; s >>= 1, m ^= m << s) {
    const uint32_t o = __shfl_xor(v, (int)s, kWave);
    // lanes with bit s clear keep their low parts and take the partner's low parts as high ones
    v = (lane & s) ? ((v & ~m) | ((o & ~m) >> s)) : ((v & m) | ((o & m) << s));
  }
  return v;
}

// A round's new pairs: the difference with Full and the counts.
__device__ __forceinline__ void sg_take_new(const SgArgs& a, uint32_t slab, uint32_t cols, bool base, const uint32_t* acc,
                                            const uint32_t* s_tab, unsigned long long* s_sum) {
  uint64_t found = 0, cand = 0;
  for (uint32_t y = threadIdx.x; y < cols; y += kSlabThreads) {
    const uint64_t at = (uint64_t)slab * cols + y;
    uint32_t nw = acc[y];
    if (base) {
      if (y / 32 == slab) nw &= ~(1u << (y % 32));  // x != y in the base rule
      a.S[at] = nw;
    } else if (nw) {
      const uint32_t full = a.S[at];
      nw &= ~full;
      if (nw) a.S[at] = full | nw;
    }
    a.D[at] = nw;
    if (nw) {
      found += (uint32_t)__popc(nw);
      uint32_t deg = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) deg += s_tab[256 * q + ((nw >> (8 * q)) & 255u)];
      cand += (uint64_t)deg * a.cdeg[y];
    }
  }
  found = wave_sum<uint64_t>(found);
  cand = wave_sum<uint64_t>(cand);
  if (lane_id() == 0 && found) {
    atomicAdd(&s_sum[0], (unsigned long long)found);
    if (cand) atomicAdd(&s_sum[1], (unsigned long long)cand);
  }
}

__device__ __forceinline__ void sg_byte_tables(const SgArgs& a, uint32_t slab, uint32_t cols, uint32_t* s_tab) {
  for (uint32_t x = threadIdx.x; x < 1024; x += kSlabThreads) {
    uint32_t sum = 0;
    for (uint32_t v = x & 255u; v; v &= v - 1) {
      const uint32_t c = slab * 32u + (x >> 8) * 8u + (uint32_t)__ffs(v) - 1u;
      if (c < cols) sum += a.cdeg[c];
    }
    s_tab[x] = sum;
  }
}

// The base rule: for each slab of columns x, the bits of every parent's children in the slab, ORed
// into every child's row.
__global__ __launch_bounds__(kSlabThreads) void k_sg_matrix_base(SgArgs a, uint32_t slabs) {
  __shared__ uint32_t s_mem[kSlabLdsWords];
  __shared__ uint32_t s_tab[1024];
  __shared__ unsigned long long s_sum[2];
  constexpr uint32_t TH = kSlabThreads;
  const uint32_t tid = threadIdx.x;
  const uint32_t rows = wave_uniform(a.rc->rows), cols = wave_uniform(a.rc->cols);
  const uint32_t per = slab_per(wave_uniform(a.rc->edges));
  if (tid == 0 && blockIdx.x == 0) a.rc->slab = 32;  // (for the launches that count and read the rows)
  uint32_t* const D = s_mem;             // by row (and an idle one)
  uint32_t* const acc = s_mem + rows + 1;  // by column (and an idle one)
  for (uint32_t slab = blockIdx.x; slab < slabs; slab += gridDim.x) {
    for (uint32_t x = tid; x < rows + cols + 2; x += TH) s_mem[x] = 0;
    if (tid < 2) s_sum[tid] = 0;
    sg_byte_tables(a, slab, cols, s_tab);
    __syncthreads();
    for (uint32_t k = 0; k < per; ++k) {
      const uint32_t u = a.base_edge[k * TH + tid], c = u & 0xFFFFu;
      if (c < cols && c / 32 == slab) atomicOr(&D[u >> 16], 1u << (c % 32));
    }
    __syncthreads();
    sg_gather(a.base_edge, per, D, acc);
    __syncthreads();
    sg_take_new(a, slab, cols, true, acc, s_tab, s_sum);
    __syncthreads();
    if (tid == 0 && s_sum[0]) {
      atomicAdd(&a.lev[0].n, s_sum[0]);
      if (s_sum[1]) atomicAdd(&a.lev[1].c, s_sum[1]);
    }
    __syncthreads();
  }
}

// First half of round j: slab s of Delta's columns, ORed from every row into its children's rows;
// written transposed, so that the second half finds the product's rows as columns.
__global__ __launch_bounds__(kSlabThreads) void k_sg_matrix_half(SgArgs a, uint32_t j, uint32_t slabs) {
  __shared__ uint32_t s_mem[kSlabLdsWords];
  constexpr uint32_t TH = kSlabThreads;
  if (block_stop(a.lev[j - 1].n == 0)) return;
  const uint32_t tid = threadIdx.x;
  const uint32_t cols = wave_uniform(a.rc->cols);
  const uint32_t per = slab_per(wave_uniform(a.rc->edges));
  uint32_t* const D = s_mem;
  uint32_t* const acc = s_mem + cols + 1;
  for (uint32_t slab = blockIdx.x; slab < slabs; slab += gridDim.x) {
    for (uint32_t x = tid; x <= cols; x += TH) {
      D[x] = x < cols ? a.D[(uint64_t)slab * cols + x] : 0u;
      acc[x] = 0;
    }
    __syncthreads();
    sg_gather(a.step_edge, per, D, acc);
    __syncthreads();
    for (uint32_t x0 = 0; x0 < cols; x0 += TH) {
      const uint32_t x = x0 + tid;
      const uint32_t t = transpose32(x < cols ? acc[x] : 0u);
      const uint32_t b = slab * 32u + (tid & 31u), xs = x / 32u;
      if (b < cols && xs < slabs) a.M[(uint64_t)xs * cols + b] = t;
    }
    __syncthreads();
  }
}

// Second half: the same over the product, then the difference with Full.
__global__ __launch_bounds__(kSlabThreads) void k_sg_matrix_rest(SgArgs a, uint32_t j, uint32_t slabs) {
  __shared__ uint32_t s_mem[kSlabLdsWords];
  __shared__ uint32_t s_tab[1024];
  __shared__ unsigned long long s_sum[2];
  constexpr uint32_t TH = kSlabThreads;
  if (block_stop(a.lev[j - 1].n == 0)) return;
  const uint32_t tid = threadIdx.x;
  const uint32_t cols = wave_uniform(a.rc->cols);
  const uint32_t per = slab_per(wave_uniform(a.rc->edges));
  uint32_t* const D = s_mem;
  uint32_t* const acc = s_mem + cols + 1;
  for (uint32_t slab = blockIdx.x; slab < slabs; slab += gridDim.x) {
    for (uint32_t x = tid; x <= cols; x += TH) {
      D[x] = x < cols ? a.M[(uint64_t)slab * cols + x] : 0u;
      acc[x] = 0;
    }
    if (tid < 2) s_sum[tid] = 0;
    sg_byte_tables(a, slab, cols, s_tab);
    __syncthreads();
    sg_gather(a.step_edge, per, D, acc);
    __syncthreads();
    sg_take_new(a, slab, cols, false, acc, s_tab, s_sum);
    __syncthreads();
    if (tid == 0 && s_sum[0]) {
      atomicAdd(&a.lev[j].n, s_sum[0]);
      if (s_sum[1]) atomicAdd(&a.lev[j + 1].c, s_sum[1]);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void k_sg_matrix_diagonal(SgArgs a, uint32_t cols) {
  for (uint32_t y = blockIdx.x * kBlock + threadIdx.x; y < cols; y += gridDim.x * kBlock) {
    const uint64_t at = (uint64_t)(y / 32) * cols + y;
    const uint32_t v = a.S[at], bit = 1u << (y % 32);
    if (v & bit) {
      a.S[at] = v & ~bit;
      atomicAdd(&a.sc->diagonal, 1u);
    }
  }
}

}  // namespace wg
