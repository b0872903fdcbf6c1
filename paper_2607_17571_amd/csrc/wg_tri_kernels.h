// Kernels of triangle counting on the renumbered graph (see wg_tri.h).
#pragma once

#include "wg_reach_device.h"
#include "wg_tri.h"

namespace wg {

constexpr uint32_t kTriEdgeThreads = 1024;
constexpr uint32_t kTriPairThreads = 1024;
constexpr uint32_t kTriPairWaves = kTriPairThreads / kWave;

// (large blocks: a few same-address atomics each)
template <typename K>
__global__ __launch_bounds__(kTriEdgeThreads) void k_tri_edges(const Ctrl* ctrl, const K* __restrict__ E, TriArgs a,
                                                              K* __restrict__ up) {
  constexpr uint32_t T = kTriEdgeThreads;
  __shared__ uint32_t s_wave[T / kWave];
  __shared__ unsigned long long s_two;
  __shared__ uint32_t s_loops;
  __shared__ unsigned long long s_at;
  const uint64_t n = ctrl->m_unique;
  if (threadIdx.x == 0) {
    s_two = 0;
    s_loops = 0;
  }
  __syncthreads();
  uint64_t two = 0;
  for (uint64_t base = (uint64_t)blockIdx.x * T; base < n; base += (uint64_t)gridDim.x * T) {
    const uint64_t i = base + threadIdx.x;
    bool is_up = false;
    K key = 0;
    if (i < n) {
      const uint32_t row = head_row<K>(E[i], a.g.w);
      const uint2 x = a.g.edge[i];
      const RankWord q = a.g.rank[row >> 5];
      const uint32_t c = x.x & ~kReachLast, bkey = a.g.colkey[c];
      const uint32_t r = q.rowpre + bits_below(q.rowbits, row);
      const uint32_t first = a.g.rstart[r], deg = a.g.rstart[r + 1] - first;
      uint4 e;
      e.x = c;
      e.y = x.y;
      e.z = e.w = 0;
      if (bkey == row) atomicAdd(&s_loops, 1u);
      if (x.y != kReachNone) {
        const RankWord t = a.g.rank[bkey >> 5];
        const uint32_t rb = t.rowpre + bits_below(t.rowbits, bkey);
        e.z = a.g.rstart[rb + 1] - x.y;
        // (rows' first edges order like their numbers)
        const bool before = e.z < deg || (e.z == deg && x.y <= first);  // b is not after a
        e.w = before ? 1 : 0;
        is_up = !before && ((q.colbits >> (row & 31u)) & 1u);
        key = ((K)rb << a.w) | (K)(q.colpre + bits_below(q.colbits, row));
        two += e.z;
      }
      a.edge[i] = e;
      a.col[i] = c;
    }
    uint32_t total;
    const uint32_t at = block_excl_scan<uint32_t, T / kWave>(is_up ? 1u : 0u, s_wave, total);
    if (threadIdx.x == 0 && total) s_at = atomicAdd(&a.tc->up, (unsigned long long)total);
    __syncthreads();
    if (is_up) up[s_at + at] = key;
    __syncthreads();
  }
  two = wave_sum<uint64_t>(two);
  if (lane_id() == 0 && two) atomicAdd(&s_two, (unsigned long long)two);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_two) atomicAdd(&a.tc->two_paths, s_two);
    if (s_loops) atomicAdd(&a.tc->loops, s_loops);
  }
}

// Where each row's up edges are (rows without any: both zero already).
template <typename K>
__global__ __launch_bounds__(kBlock) void k_tri_starts(TriArgs a, const K* __restrict__ up) {
  const uint64_t n = a.tc->up;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) {
    const uint32_t r = (uint32_t)(up[i] >> a.w);
    if (i == 0 || (uint32_t)(up[i - 1] >> a.w) != r) a.ustart[r] = (uint32_t)i;
    if (i + 1 == n || (uint32_t)(up[i + 1] >> a.w) != r) a.uend[r] = (uint32_t)i + 1;
  }
}

// The lanes' counts n flattened: U x 64 units a step, each with its lane and its index there.  All of
// a step's load(lane, index) come before its use(loaded): U loads in flight.
template <int U>
struct TriWave {
  uint32_t lane[kWave];  // the lanes that have units
  uint32_t pre[kWave];   // ... units before each
  uint32_t mark[U * kWave];
};
template <int U, typename Load, typename Use>
__device__ __forceinline__ void tri_flat(TriWave<U>& w, uint32_t n, Load load, Use use) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t incl = wave_incl_scan<uint32_t>(n), pre = incl - n;
  const uint32_t total = __shfl(incl, kWave - 1, kWave);
  const uint64_t some = __builtin_amdgcn_ballot_w64(n != 0);
  wave_lds_sync();
  if (n) {
    const uint32_t at = (uint32_t)__popcll(some & ((1ull << lane) - 1ull));
    w.lane[at] = lane;
    w.pre[at] = pre;
  }
  uint32_t before = 0;  // starts before this step
  for (uint32_t k0 = 0; k0 < total; k0 += U * kWave) {
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) w.mark[u * kWave + lane] = 0;
    wave_lds_sync();
    if (n && pre >= k0 && pre < k0 + U * kWave) w.mark[pre - k0] = 1;
    wave_lds_sync();
    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t starts = __builtin_amdgcn_ballot_w64(w.mark[u * kWave + lane] != 0);
      const uint32_t k = k0 + u * kWave + lane;
      v[u] = 0;
      if (k < total) {
        const uint32_t p = before + (uint32_t)__popcll(starts & ((2ull << lane) - 1ull)) - 1u;
        v[u] = load(w.lane[p], k - w.pre[p]);
      }
      before += (uint32_t)__popcll(starts);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k0 + u * kWave + lane < total) use(v[u]);
  }
  wave_lds_sync();
}

// Adds the lanes' counts to the total.
__device__ __forceinline__ void tri_add(const TriArgs& a, uint64_t hits, unsigned long long* s_hits) {
  hits = wave_sum<uint64_t>(hits);
  if (lane_id() == 0 && hits) atomicAdd(s_hits, (unsigned long long)hits);
  __syncthreads();
  if (threadIdx.x == 0 && *s_hits) atomicAdd(&a.tc->hits, *s_hits);
}

// Every row, a lane each: its pairs (b, c) flattened over the wave, c looked up in b's out-edges;
// rows with more pairs are queued in pieces for k_tri_bits.
template <typename K>
__global__ __launch_bounds__(kTriPairThreads) void k_tri_pairs(TriArgs a, const K* __restrict__ up) {
  struct Row {
    uint32_t first, ustart, u;
  };
  __shared__ TriWave<1> s_flat[kTriPairWaves];
  __shared__ Row s_row[kTriPairWaves][kWave];
  __shared__ uint32_t s_pieces, s_piece0;
  __shared__ unsigned long long s_hits;
  const uint32_t rows = a.rc->rows, lane = (uint32_t)lane_id(), wid = threadIdx.x / kWave;
  if (threadIdx.x == 0) s_hits = 0;
  __syncthreads();
  uint32_t hits = 0;
  // (a wave's rows are far apart: the rows of hubs may be next to each other)
  const uint32_t waves = gridDim.x * kTriPairWaves;
  for (uint32_t base = blockIdx.x * kTriPairWaves; base < rows; base += waves * kWave) {
    const uint32_t r = base + wid + lane * waves;
    uint32_t n = 0, pieces = 0, at = 0, first = 0;
    if (threadIdx.x == 0) s_pieces = 0;
    __syncthreads();
    if (r < rows) {
      Row q;
      q.first = a.g.rstart[r];
      q.ustart = a.ustart[r];
      q.u = a.uend[r] - q.ustart;
      const uint32_t deg = a.g.rstart[r + 1] - q.first;
      if (q.u && (uint64_t)q.u * deg > kTriPairs) {
        pieces = (deg + kTriPiece - 1) / kTriPiece;
        first = q.first;
        at = atomicAdd(&s_pieces, pieces);
      } else {
        n = q.u * deg;
        s_row[wid][lane] = q;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_pieces) s_piece0 = atomicAdd(&a.tc->pieces, s_pieces);
    __syncthreads();
    for (uint32_t k = 0; k < pieces; ++k) {
      uint2 p;
      p.x = r;
      p.y = first + k * kTriPiece;
      a.piece[s_piece0 + at + k] = p;
    }
    tri_flat<1>(s_flat[wid], n, [&](uint32_t from, uint32_t k) {
      const Row q = s_row[wid][from];
      const uint32_t i = k / q.u, j = k - i * q.u;
      const uint4 e = a.edge[q.first + i];
      if (e.w == 0) return 0u;
      const uint32_t c = (uint32_t)up[q.ustart + j] & id_mask(a.w);
      uint32_t lo = e.y, len = e.z;
      while (len > 1) {
        const uint32_t half = len / 2;
        if (a.col[lo + half] <= c) lo += half;
        len -= half;
      }
      return a.col[lo] == c ? 1u : 0u;
    }, [&](uint32_t v) { hits += v; });
    __syncthreads();
  }
  tri_add(a, hits, &s_hits);
}

// A piece of a row's out-edges per workgroup: the row's c as bits, tested by the out-edges of its b,
// 64 a step of a wave whatever their degrees.
template <typename K, uint32_t WORDS>
__global__ __launch_bounds__(kTriThreads) void k_tri_bits(TriArgs a, const K* __restrict__ up) {
  constexpr uint32_t kWaves = kTriThreads / kWave;
  __shared__ uint32_t s_bits[WORDS];
  __shared__ TriWave<4> s_flat[kWaves];
  __shared__ uint32_t s_first[kWaves][kWave];
  __shared__ unsigned long long s_hits;
  const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id(), wid = tid / kWave;
  const uint32_t pieces = a.tc->pieces;
  if (tid == 0) s_hits = 0;
  for (uint32_t x = tid; x < WORDS; x += kTriThreads) s_bits[x] = 0;
  __syncthreads();
  uint64_t hits = 0;
  for (uint32_t p = blockIdx.x; p < pieces; p += gridDim.x) {
    const uint2 q = a.piece[p];
    const uint32_t u0 = a.ustart[q.x], u1 = a.uend[q.x], end = min(a.g.rstart[q.x + 1], q.y + kTriPiece);
    for (uint32_t u = u0 + tid; u < u1; u += 4 * kTriThreads) {
      uint32_t c[4];
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) c[k] = u + k * kTriThreads < u1 ? (uint32_t)up[u + k * kTriThreads] & id_mask(a.w) : kReachNone;
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k)
        if (c[k] != kReachNone) atomicOr(&s_bits[c[k] >> 5], 1u << (c[k] & 31u));
    }
    __syncthreads();
    // (each wave takes every kWaves-th edge: neighbours' degrees differ most by wave otherwise)
    const uint32_t i = q.y + lane * kWaves + wid;
    uint32_t n = 0;
    if (i < end) {
      const uint4 e = a.edge[i];
      if (e.w) n = e.z;
      s_first[wid][lane] = e.y;
    }
    uint32_t h = 0;
    tri_flat<4>(s_flat[wid], n, [&](uint32_t from, uint32_t k) { return a.col[s_first[wid][from] + k]; },
                [&](uint32_t c) { h += (s_bits[c >> 5] >> (c & 31u)) & 1u; });
    hits += h;
    __syncthreads();
    // (few: word by word; else all of them)
    if (u1 - u0 <= kTriThreads) {
      if (u0 + tid < u1) s_bits[((uint32_t)up[u0 + tid] & id_mask(a.w)) >> 5] = 0;
    } else {
      for (uint32_t x = tid; x < WORDS; x += kTriThreads) s_bits[x] = 0;
    }
    __syncthreads();
  }
  tri_add(a, hits, &s_hits);
}

}  // namespace wg
