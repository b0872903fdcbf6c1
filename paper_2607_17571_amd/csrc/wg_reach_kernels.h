// Kernels of the row-at-a-time closure (see wg_reach.h).
#pragma once

#include "wg_reach_device.h"

namespace wg {

__device__ __forceinline__ bool reach_halted(const ReachCtl* rc) {
  return (__hip_atomic_load(&rc->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kReachHalt) != 0;
}

// ... or cancelled, from within a long row or slab (one thread)
__device__ __forceinline__ bool reach_look(const ReachArgs& a) { return reach_halted(a.rc) || cancelled(a.cancel, &a.rc->stop); }

// `n` pool entries (one thread); past the pool's end they are counted but not to be written.
__device__ __forceinline__ uint64_t reach_alloc(const ReachArgs& a, uint32_t n) {
  const unsigned long long at = atomicAdd(&a.rc->cursor, (unsigned long long)n);
  if (at + n > a.pool_cap)
    atomicOr(&a.rc->stop, (uint32_t)(at > kReachMaxTuples ? kReachPoolFull | kReachTooLarge : kReachPoolFull));
  return at;
}

// A row or slab with columns at a level past the last one allotted: the closure ends.
__device__ __forceinline__ void reach_deep(const ReachArgs& a) { atomicOr(&a.rc->stop, (uint32_t)kReachDeep); }

// Adds a level's counts to the block's LDS table (levels below kReachLdsLevels) or to memory.
__device__ __forceinline__ void reach_count(unsigned long long (*s_lev)[2], const ReachArgs& a, uint32_t lv,
                                            uint32_t n, unsigned long long d) {
  if (lv < kReachLdsLevels) {
    if (n) atomicAdd(&s_lev[lv][0], (unsigned long long)n);
    if (d) atomicAdd(&s_lev[lv][1], d);
  } else if (lv < a.lev_cap) {
    if (n) atomicAdd(&a.lev[lv].n[a.form], (unsigned long long)n);
    if (d) atomicAdd(&a.lev[lv].d[a.form], d);
  }
}

__device__ __forceinline__ void reach_levels_clear(unsigned long long (*s_lev)[2]) {
  for (uint32_t x = threadIdx.x; x < kReachLdsLevels; x += blockDim.x) s_lev[x][0] = s_lev[x][1] = 0;
}

// (after a barrier) the block's level counts into memory
__device__ __forceinline__ void reach_levels_flush(const unsigned long long (*s_lev)[2], const ReachArgs& a) {
  for (uint32_t x = threadIdx.x; x < kReachLdsLevels && x < a.lev_cap; x += blockDim.x) {
    if (s_lev[x][0]) atomicAdd(&a.lev[x].n[a.form], s_lev[x][0]);
    if (s_lev[x][1]) atomicAdd(&a.lev[x].d[a.form], s_lev[x][1]);
  }
}

// Next queued row of `tier` for this block (thread 0), kReachNone when all n are handed out.  The
// rows are dealt to the XCDs (blocks b, b + 8, ... run on one), whose counters stay in their own
// L2; a block whose share is used up takes from the others'.
__device__ __forceinline__ uint32_t reach_claim(ReachCtl* rc, int tier, uint32_t n, uint32_t& share) {
  for (; share < (uint32_t)kReachXcds; ++share) {
    const uint32_t x = (blockIdx.x + share) % kReachXcds;
    const uint32_t at = atomicAdd(&rc->claim[tier][x][0], 1u) * kReachXcds + x;
    if (at < n) return at;
  }
  return kReachNone;
}

// ---------------------------------------------------------------------------
// Ids by rank (wg_reach.h): the distinct ids of a sorted run, a static range of it per block, and each
// edge's two ids found among them by bisection.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_ids_gather(const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst,
                                                       uint64_t m, uint32_t* __restrict__ keys) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (uint64_t)gridDim.x * kBlock) {
    keys[i] = src[i];
    keys[m + i] = dst[i];
  }
}

constexpr uint32_t kIdsTile = kBlock;
__global__ __launch_bounds__(kBlock) void k_ids_count(const uint32_t* __restrict__ v, uint64_t n, uint64_t* __restrict__ part) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  uint64_t lo, hi, c = 0, total;
  block_range(n, kIdsTile, lo, hi);
  for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) c += i == 0 || v[i - 1] != v[i] ? 1 : 0;
  (void)block_excl_scan<uint64_t>(c, s_wave, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}
__global__ __launch_bounds__(kBlock) void k_ids_write(const uint32_t* __restrict__ v, uint64_t n, const uint64_t* __restrict__ part,
                                                      uint32_t* __restrict__ ids, uint32_t* __restrict__ n_ids) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  uint64_t before = 0, run;
  for (uint32_t x = threadIdx.x; x < blockIdx.x; x += kBlock) before += part[x];
  (void)block_excl_scan<uint64_t>(before, s_wave, run);
  uint64_t lo, hi;
  block_range(n, kIdsTile, lo, hi);
  for (uint64_t i0 = lo; i0 < hi; i0 += kBlock) {
    const uint64_t i = i0 + threadIdx.x;
    const bool head = i < hi && (i == 0 || v[i - 1] != v[i]);
    uint64_t total;
    const uint64_t at = run + block_excl_scan<uint64_t>(head ? 1 : 0, s_wave, total);
    if (head) ids[at] = v[i];
    run += total;
  }
  if (hi == n && lo < hi && threadIdx.x == 0) *n_ids = (uint32_t)run;
}

__device__ __forceinline__ uint32_t id_rank(const uint32_t* __restrict__ ids, uint32_t n, uint32_t id) {
  uint32_t lo = 0;
  for (uint32_t len = n; len > 1;) {
    const uint32_t half = len / 2;
    if (ids[lo + half] <= id) lo += half;
    len -= half;
  }
  return lo;
}
__global__ __launch_bounds__(kBlock) void k_ids_map(const uint32_t* __restrict__ ids, const uint32_t* __restrict__ n_ids,
                                                    const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst,
                                                    uint64_t m, uint32_t* __restrict__ src_out, uint32_t* __restrict__ dst_out) {
  const uint32_t n = *n_ids;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (uint64_t)gridDim.x * kBlock) {
    src_out[i] = id_rank(ids, n, src[i]);
    dst_out[i] = id_rank(ids, n, dst[i]);
  }
}
__global__ __launch_bounds__(kBlock) void k_ids_back(const uint32_t* __restrict__ ids, uint32_t* ranks, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock)
    ranks[i] = ids[ranks[i]];
}
template <typename K>
__global__ __launch_bounds__(kBlock) void k_ids_keys(const uint32_t* __restrict__ ids, const K* __restrict__ keys, uint64_t n,
                                                     int w, int out_w, uint64_t* __restrict__ out) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) {
    const K k = keys[i];
    out[i] = ((uint64_t)ids[(uint32_t)(k >> w)] << out_w) | ids[(uint32_t)k & id_mask(w)];
  }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void k_count_rows(Ctrl* ctrl, const K* __restrict__ E, int w) {
  __shared__ uint32_t s_rows;
  if (threadIdx.x == 0) s_rows = 0;
  __syncthreads();
  const uint64_t n = ctrl->m_unique;
  uint32_t rows = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock)
    rows += i == 0 || head_row<K>(E[i - 1], w) != head_row<K>(E[i], w) ? 1 : 0;
  rows = wave_sum<uint32_t>(rows);
  if (lane_id() == 0 && rows) atomicAdd(&s_rows, rows);
  __syncthreads();
  if (threadIdx.x == 0 && s_rows) atomicAdd(&ctrl->rows, s_rows);
}

// ---------------------------------------------------------------------------
// Renumbering.  Every edge flags its row's and its column's key (plain byte stores: no atomics);
// the flags become one 16-byte word per 32 keys with the bits and the ranks before them, so that
// a key's row or column number is one load; then the rows' starts, then the edge records.  A few
// launches of streaming work over the edges and the id range.
// ---------------------------------------------------------------------------
template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_mark(const Ctrl* ctrl, const K* __restrict__ E, ReachGraph g) {
  const uint64_t n = ctrl->m_unique;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) {
    const K e = E[i];
    const uint32_t row = head_row<K>(e, g.w);
    if (i == 0 || head_row<K>(E[i - 1], g.w) != row) g.flags[row] = 1;
    g.flags[g.span + col_key<K>(e, g.w)] = 1;
  }
}

// The bits of 32 flags (bytes 0 or 1).
__device__ __forceinline__ uint32_t flag_bits(const uint8_t* __restrict__ f) {
  const uint4* __restrict__ p = (const uint4*)f;
  uint32_t bits = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint4 v = p[q];
    const uint32_t x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      bits |= ((x[k] | (x[k] >> 7) | (x[k] >> 14) | (x[k] >> 21)) & 0xFu) << (16 * q + 4 * k);
  }
  return bits;
}

constexpr uint32_t kReachRankTile = kBlock;  // words

__global__ __launch_bounds__(kBlock) void k_reach_rank_sum(ReachGraph g, uint64_t* __restrict__ part) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  uint64_t lo, hi;
  block_range(g.span / 32, kReachRankTile, lo, hi);
  uint64_t sum = 0;  // rows << 32 | columns
  for (uint64_t x = lo + threadIdx.x; x < hi; x += kBlock) {
    const uint32_t rb = flag_bits(g.flags + 32 * x), cb = flag_bits(g.flags + g.span + 32 * x);
    sum += ((uint64_t)__popc(rb) << 32) | (uint32_t)__popc(cb);
  }
  uint64_t total;
  (void)block_excl_scan<uint64_t>(sum, s_wave, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// (one block needs no totals: part nullptr)
__global__ __launch_bounds__(kBlock) void k_reach_rank(const Ctrl* ctrl, ReachGraph g,
                                                       const uint64_t* __restrict__ part, ReachCtl* rc) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  const uint64_t words = g.span / 32;
  uint64_t run = 0;
  if (part) {
    // (block_prefix saturates at 40 bits: sum the halves apart)
    uint64_t rows = 0, cols = 0;
    for (uint32_t x = threadIdx.x; x < blockIdx.x; x += kBlock) {
      rows += part[x] >> 32;
      cols += part[x] & 0xFFFFFFFFull;
    }
    uint64_t tr, tc;
    (void)block_excl_scan<uint64_t>(rows, s_wave, tr);
    (void)block_excl_scan<uint64_t>(cols, s_wave, tc);
    run = (tr << 32) | tc;
  }
  uint64_t lo, hi;
  block_range(words, kReachRankTile, lo, hi);
  for (uint64_t x0 = lo; x0 < hi; x0 += kBlock) {
    const uint64_t x = x0 + threadIdx.x;
    uint32_t rb = 0, cb = 0;
    if (x < hi) {
      rb = flag_bits(g.flags + 32 * x);
      cb = flag_bits(g.flags + g.span + 32 * x);
    }
    uint64_t total;
    const uint64_t at = run + block_excl_scan<uint64_t>(((uint64_t)__popc(rb) << 32) | (uint32_t)__popc(cb), s_wave, total);
    if (x < hi) {
      RankWord r;
      r.rowbits = rb;
      r.colbits = cb;
      r.rowpre = (uint32_t)(at >> 32);
      r.colpre = (uint32_t)at;
      g.rank[x] = r;
      for (uint32_t k = r.colpre; cb; cb &= cb - 1, ++k) g.colkey[k] = (uint32_t)x * 32u + (uint32_t)__ffs(cb) - 1u;
    }
    run += total;
  }
  if (hi == words && lo < hi && threadIdx.x == 0) {  // the last block with words
    RankWord r;
    r.rowbits = r.colbits = 0;
    r.rowpre = rc->rows = (uint32_t)(run >> 32);
    r.colpre = rc->cols = (uint32_t)run;
    g.rank[words] = r;
    rc->edges = (uint32_t)ctrl->m_unique;
  }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_rows(const Ctrl* ctrl, const K* __restrict__ E, ReachGraph g,
                                                       const ReachCtl* rc) {
  const uint64_t n = ctrl->m_unique;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kBlock) {
    const uint32_t row = head_row<K>(E[i], g.w);
    if (i == 0 || head_row<K>(E[i - 1], g.w) != row) {
      const RankWord r = g.rank[row >> 5];
      const uint32_t at = r.rowpre + bits_below(r.rowbits, row);
      g.rowkey[at] = row;
      g.rstart[at] = (uint32_t)i;
    }
    if (i + 1 == n) g.rstart[rc->rows] = (uint32_t)n;
  }
}

template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_edges(const Ctrl* ctrl, const K* __restrict__ E, ReachGraph g,
                                                        ReachCtl* rc, int slabs) {
  __shared__ uint32_t s_inner;
  const uint64_t n = ctrl->m_unique;
  const uint32_t rows = rc->rows;
  if (threadIdx.x == 0) s_inner = 0;
  __syncthreads();
  uint32_t inner = 0;
  const bool slab = slabs && rows <= kSlabRows16;
  const uint32_t per = slab_per((uint32_t)n);
  const uint64_t end = slab ? (uint64_t)per * kSlabThreads : n;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < end; i += (uint64_t)gridDim.x * kBlock) {
    uint32_t from = rows, to = rows, c = kReachNone;  // (past the edges: an idle row)
    if (i < n) {
      const K e = E[i];
      const uint32_t row = head_row<K>(e, g.w), ck = col_key<K>(e, g.w);
      const bool last = i + 1 == n || head_row<K>(E[i + 1], g.w) != row;
      const RankWord r = g.rank[ck >> 5];
      c = r.colpre + bits_below(r.colbits, ck);
      uint32_t start = kReachNone;
      if ((r.rowbits >> (ck & 31u)) & 1u) {
        to = r.rowpre + bits_below(r.rowbits, ck);
        start = g.rstart[to];
        ++inner;
      }
      uint2 rec;
      rec.x = c | (last ? kReachLast : 0u);
      rec.y = start;
      g.edge[i] = rec;
      g.cstart[c] = start;  // (every edge into c writes the same)
      if (slab) {
        const RankWord q = g.rank[row >> 5];
        from = q.rowpre + bits_below(q.rowbits, row);
      }
    }
    if (slab) {
      const uint64_t at = (i % per) * kSlabThreads + i / per;
      g.slab_edge[at] = (from << 16) | to;
      g.slab_col[at] = c;
    }
  }
  if (slabs != 2) return;
  inner = wave_sum<uint32_t>(inner);
  if (lane_id() == 0 && inner) atomicAdd(&s_inner, inner);
  __syncthreads();
  if (threadIdx.x == 0 && s_inner) atomicAdd(&rc->inner[blockIdx.x % kReachXcds][0], s_inner);
}

// ---------------------------------------------------------------------------
// Thread tier: thread t takes row t, holds its columns in 16 registers (a membership test is 16
// compares, an insertion a shift) and the starts of the rows still to expand in LDS, and sorts the
// columns with a network over the registers at the end.  Every row steps through its edge lists and
// levels by itself, two edge records a step: level by level in lockstep, a wave took the widest of
// its 64 rows at every level.  A block's rows are consecutive, so their sorted columns are packed
// into one stretch of the pool.  Bound by instruction issue (about 40 per record).  1.65 million
// rows of 256 random graphs: in lockstep 364 us, so 144.
// ---------------------------------------------------------------------------
// (flip all ones: descending)
template <int N>
__device__ __forceinline__ void sort_regs(uint32_t (&v)[N], uint32_t flip = 0) {
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] ^= flip;
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int l = i ^ j;
        if (l > i) {
          const uint32_t lo = v[i] < v[l] ? v[i] : v[l], hi = v[i] < v[l] ? v[l] : v[i];
          v[i] = (i & k) == 0 ? lo : hi;
          v[l] = (i & k) == 0 ? hi : lo;
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < N; ++r) v[r] ^= flip;
}

constexpr uint32_t kReachFailBuf = 512;  // rows a block buffers before it appends them to a queue
constexpr int kReachLevCopies = 16;      // copies of a block's level counts (spread over the lanes)

__global__ __launch_bounds__(kBlock) void k_reach_thread(ReachArgs a) {
  constexpr int CAP = (int)kReachThreadCap;
  __shared__ uint32_t s_q[CAP * kBlock];  // starts to expand by (index, thread); then the sorted columns
  __shared__ uint16_t s_stat[CAP * kBlock];  // by (level, thread): tuples | degrees << 8
  __shared__ unsigned long long s_cnt[kReachLevCopies][kReachThreadCap];  // level: tuples | degrees << 32
  __shared__ uint32_t s_fail[kReachFailBuf];
  __shared__ uint32_t s_fn, s_flush;
  __shared__ uint32_t s_wave[kWavesPerBlock];
  __shared__ uint64_t s_pos;
  const uint32_t tid = threadIdx.x;
  for (uint32_t x = tid; x < (uint32_t)kReachLevCopies * CAP; x += kBlock) (&s_cnt[0][0])[x] = 0;
  if (tid == 0) s_fn = 0;
  const uint32_t n = a.rc->rows;
  if (n < a.min_rows) {  // (uniform over the launch)
    if (tid == 0 && blockIdx.x == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
    return;
  }
  const uint2* __restrict__ edge = a.g.edge;
  unsigned long long* const my = s_cnt[tid % kReachLevCopies];
  uint64_t chunk = 0;
  uint32_t left = 0;  // pool entries left of the block's chunk (uniform)
  const uint32_t ntiles = (n + kBlock - 1) / kBlock, stretch = xcd_stretch(ntiles, kReachTileStretch);
  __syncthreads();
  for (uint32_t iter = 0;; ++iter) {
    const uint32_t tile = xcd_tile(iter, stretch), next = xcd_tile(iter + 1, stretch);
    if (tile >= ntiles) break;
    const uint32_t row = tile * kBlock + tid;
    uint32_t q[CAP];
#pragma unroll
    for (int k = 0; k < CAP; ++k) q[k] = kReachNone;  // (no column: columns have 31 bits)
    uint32_t cnt = 0, pops = 0, lv = 0;
    bool fail = false;
    if (row < n) {
      uint32_t e = a.g.rstart[row], f = 0, hi = 0, prev = 0, found = 0, d = 0;
      bool on = true, first = true;
      for (;;) {
        if (!on) {
          if (f == hi) {
            // the level is expanded: its counts, then the level found
            if (!first) s_stat[lv++ * kBlock + tid] = (uint16_t)(found | (d << 8));
            first = false;
            found = cnt - prev;
            if (found == 0) break;
            prev = cnt;
            d = 0;
            hi = pops;
            if (f == hi) {
              s_stat[lv++ * kBlock + tid] = (uint16_t)found;
              break;
            }
          }
          e = s_q[f++ * kBlock + tid];
          on = true;
        }
        uint2 x[2];  // (readable past the last edge)
        x[0] = edge[e];
        x[1] = edge[e + 1];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (!on) continue;
          const uint32_t z = x[k].x & ~kReachLast;
          on = (x[k].x & kReachLast) == 0;
          ++d;
          bool dup = false;
#pragma unroll
          for (int r = 0; r < CAP; ++r) dup |= q[r] == z;
          if (dup) continue;
#pragma unroll
          for (int r = CAP - 1; r > 0; --r) q[r] = q[r - 1];
          q[0] = z;
          if (++cnt <= (uint32_t)CAP && x[k].y != kReachNone) s_q[pops++ * kBlock + tid] = x[k].y;
        }
        e += 2;
        fail = cnt > (uint32_t)CAP || d > 255u;
        if (fail) break;
      }
      if (fail) {
        cnt = 0;
      } else {
        for (uint32_t l = 0; l < lv; ++l) {
          const uint32_t x = s_stat[l * kBlock + tid];
          atomicAdd(&my[l], (unsigned long long)(x & 255u) | ((unsigned long long)(x >> 8) << 32));
        }
        sort_regs<CAP>(q);
      }
    }
    __syncthreads();  // s_q is free for the output
    uint32_t total;
    const uint32_t at = block_excl_scan<uint32_t>(cnt, s_wave, total);
    if (total > left) {  // (uniform)
      if (tid == 0) s_pos = reach_alloc(a, kReachChunk);
      __syncthreads();
      chunk = s_pos;
      left = kReachChunk;
    }
#pragma unroll
    for (int k = 0; k < CAP; ++k)
      if ((uint32_t)k < cnt) s_q[at + k] = q[k];
    if (fail) s_fail[atomicAdd(&s_fn, 1u)] = row;
    if (row < n) {
      a.cnt[row] = cnt;
      a.seg[row] = (uint32_t)(chunk + at);
    }
    __syncthreads();
    if (chunk + total <= a.pool_cap)
      for (uint32_t t = tid; t < total; t += kBlock) a.pool[chunk + t] = s_q[t];
    chunk += total;
    left -= total;
    // a buffer that a further tile could overfill goes out
    const uint32_t fn = s_fn;
    if (fn > 0 && (next >= ntiles || fn > kReachFailBuf - kBlock)) {
      if (tid == 0) s_flush = atomicAdd(&a.rc->queued[0], fn);
      __syncthreads();
      for (uint32_t t = tid; t < fn; t += kBlock) a.queue[0][s_flush + t] = s_fail[t];
      __syncthreads();
      if (tid == 0) s_fn = 0;
    }
    __syncthreads();
  }
  for (uint32_t lv = tid; lv < (uint32_t)CAP; lv += kBlock) {
    unsigned long long sn = 0, sd = 0;
    for (int c = 0; c < kReachLevCopies; ++c) {
      sn += s_cnt[c][lv] & 0xFFFFFFFFull;
      sd += s_cnt[c][lv] >> 32;
    }
    if (sn) atomicAdd(&a.lev[lv].n[0], sn);
    if (sd) atomicAdd(&a.lev[lv].d[0], sd);
  }
}

// ---------------------------------------------------------------------------
// Slabs.  A workgroup of 1,024 threads takes 32 (16) consecutive columns.  In LDS, for every row,
// D = the columns found at the last level and acc = those of the row's successors at that level;
// the columns found so far (S) are registers of the row's thread.  A level is two passes: each
// thread ORs D of the successors of its stretch of edges (kept in registers) and adds each row's
// part to acc with an LDS atomic; then every row takes acc & ~S as its new D.  The candidates are
// the new columns' degrees, summed through a table per byte of columns.  No memory traffic within
// a level; about 2 us per level at 30,000 edges, one workgroup per CU, every slab on its own.
// R-MAT scale 15 (7,546 rows, 7,535 columns): 236 slabs of 13 levels where the bits tier ran
// 180M candidates one by one.
// ---------------------------------------------------------------------------
// Whether the slabs take the rows (the same in every block of the launches before the tiers run).
__device__ __forceinline__ bool slab_chosen(const ReachArgs& a) {
  if (a.slab_mode == 0 || a.rc->rows > kSlabRows16) return false;
  if (a.slab_mode == 1) return true;
  if (2ull * a.rc->queued[0] < a.rc->rows) return false;
  const uint64_t rows = a.rc->rows, cols = a.rc->cols, level = (uint64_t)a.rc->edges * ((cols + 31) / 32);
  uint64_t inner = 0;
#pragma unroll
  for (int x = 0; x < kReachXcds; ++x) inner += a.rc->inner[x][0];
  return level <= kSlabLevel ? 2 * inner >= rows : cols <= 2 * rows && 2 * inner >= 3 * rows;
}

template <typename W, int RP>
__device__ __forceinline__ void slab_run(const ReachArgs& a, uint32_t* s_mem, unsigned long long (*s_lev)[2],
                                         uint32_t* s_tab, uint32_t* s_any, uint32_t* s_halt) {
  constexpr uint32_t B = 8 * sizeof(W);  // columns per slab
  constexpr uint32_t TH = kSlabThreads;
  constexpr int EREG = sizeof(W) == 4 ? (int)kSlabEdgeRegs : (int)kSlabEdgeRegs * 3 / 4;
  const uint32_t tid = threadIdx.x;
  const uint32_t rows = wave_uniform(a.rc->rows), cols = wave_uniform(a.rc->cols),
                 edges = wave_uniform(a.rc->edges);
  const uint32_t pitch = (rows / TH + 1) * TH;  // whole rounds of rows, an idle one among them
  W* const D = (W*)s_mem;
  W* const acc = D + pitch;
  const uint32_t per = slab_per(edges);
  const uint32_t* __restrict__ se = a.g.slab_edge;
  const uint32_t* __restrict__ sc = a.g.slab_col;
  W* const out = (W*)a.bits;
  const auto add = [&](uint32_t x, uint32_t v) {
    if constexpr (sizeof(W) == 4) atomicOr(&acc[x], v);
    else atomicOr((uint32_t*)acc + (x >> 1), v << (16u * (x & 1u)));
  };
  // the thread's first edges stay in registers for every level of every slab
  uint32_t er[EREG];
#pragma unroll
  for (int k = 0; k < EREG; ++k) {
    er[k] = (uint32_t)k < per ? se[(uint32_t)k * TH + tid] : (rows << 16) | rows;  // (an idle row)
    if (k % 4 == 3) WG_FENCE_LOADS;
  }
  const uint32_t slabs = (cols + B - 1) / B;
  for (uint32_t slab = blockIdx.x; slab < slabs; slab += gridDim.x) {
    // byte tables: s_tab[256 b + v] = degrees of the columns of byte b in v
    for (uint32_t x = tid; x < 256u * sizeof(W); x += TH) {
      uint32_t sum = 0;
      for (uint32_t v = x & 255u; v; v &= v - 1) {
        const uint32_t c = slab * B + (x >> 8) * 8u + (uint32_t)__ffs(v) - 1u;
        const uint32_t st = c < cols ? a.g.cstart[c] : kReachNone;
        if (st != kReachNone) {
          // degree: the row's start is among rstart (its index by the column's key)
          const uint32_t key = a.g.colkey[c];
          const RankWord r = a.g.rank[key >> 5];
          sum += a.g.rstart[r.rowpre + bits_below(r.rowbits, key) + 1] - st;
        }
      }
      s_tab[x] = sum;
    }
    for (uint32_t x = tid; x < pitch; x += TH) {
      D[x] = 0;
      acc[x] = 0;
    }
    W S[RP];
#pragma unroll
    for (int k = 0; k < RP; ++k) S[k] = 0;
    if (tid < 2) s_any[tid] = 0;
    if (tid == 0) *s_halt = reach_halted(a.rc);
    __syncthreads();
    if (*s_halt) break;
    for (uint32_t k = 0; k < per; ++k) {
      const uint32_t c = sc[k * TH + tid];
      if (c / B == slab) add(se[k * TH + tid] >> 16, 1u << (c % B));
    }
    __syncthreads();
    uint32_t look = min(kStopLevels, a.lev_cap);  // the next level to stop at, if need be
    for (uint32_t lv = 0;; ++lv) {
      uint32_t found = 0, deg = 0;  // (a thread's columns, 576 at most, have at most 2^20 edges each)
#pragma unroll
      for (int k = 0; k < RP; ++k) {
        if ((uint32_t)k * TH >= rows) continue;  // (uniform; rows past the last have no bits)
        const uint32_t x = (uint32_t)k * TH + tid;
        const W v = acc[x];
        const W nw = (W)(v & (W)~S[k]);
        if (v) acc[x] = 0;
        D[x] = nw;
        if (nw) {
          S[k] = (W)(S[k] | nw);
          found += (uint32_t)__popc((uint32_t)nw);
#pragma unroll
          for (int q = 0; q < (int)sizeof(W); ++q) deg += s_tab[256 * q + (((uint32_t)nw >> (8 * q)) & 255u)];
        }
        WG_FENCE_LOADS;  // (registers: one row's loads at a time)
      }
      found = wave_sum<uint32_t>(found);
      unsigned long long sum = wave_sum<uint32_t>(deg);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(deg >> 26 != 0) != 0, 0)) sum = wave_sum<uint64_t>(deg);  // (else below 2^32)
      if (lane_id() == 0 && found) {
        reach_count(s_lev, a, lv, found, sum);
        s_any[lv & 1u] = 1;
      }
      if (tid == 0) s_any[(lv + 1) & 1u] = 0;
      __syncthreads();
      if (!s_any[lv & 1u]) break;
      if (__builtin_expect(lv >= look, 0)) {
        if (lv >= a.lev_cap) {
          if (tid == 0) reach_deep(a);
          break;
        }
        if (tid == 0) *s_halt = reach_look(a);
        __syncthreads();
        if (*s_halt) break;
        look = min(lv + kStopLevels, a.lev_cap);
      }
      uint32_t cur = 0, v = 0;
      auto edge = [&](uint32_t x, uint32_t dx) {
        if (x != cur) {
          if (v) add(cur, v);
          v = 0;
          cur = x;
        }
        v |= dx;
      };
#pragma unroll
      for (int k = 0; k < EREG; k += 4) {  // four loads in flight
        if ((uint32_t)k >= per) continue;  // (uniform)
        uint32_t dv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          WG_OPAQUE(er[k + q]);
          dv[q] = (uint32_t)D[er[k + q] & 0xFFFFu];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) edge(er[k + q] >> 16, dv[q]);
        WG_FENCE_LOADS;
      }
      for (uint32_t k = EREG; k < per; k += 4) {
        uint32_t u[4], dv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = k + q < per ? se[(k + q) * TH + tid] : (rows << 16) | rows;
#pragma unroll
        for (int q = 0; q < 4; ++q) dv[q] = (uint32_t)D[u[q] & 0xFFFFu];
#pragma unroll
        for (int q = 0; q < 4; ++q) edge(u[q] >> 16, dv[q]);
      }
      if (v) add(cur, v);
      __syncthreads();
    }
    uint32_t left = rows > tid ? rows - tid : 0u;  // rows from the thread's first on
    WG_OPAQUE(left);
    W* const o = out + (uint64_t)slab * rows + tid;
#pragma unroll
    for (int k = 0; k < RP; ++k) {
      if ((uint32_t)k * TH < left) o[(uint32_t)k * TH] = S[k];
      WG_FENCE_LOADS;
    }
    __syncthreads();
  }
}

// One launch for both widths where there may be rows for the narrow one (a launch that finds nothing to do
// takes 5 us of a closure by tiers).
template <bool BOTH>
__global__ __launch_bounds__(kSlabThreads) void k_slab(ReachArgs a) {
  __shared__ uint32_t s_mem[kSlabLdsWords];
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  __shared__ uint32_t s_tab[1024];
  __shared__ uint32_t s_any[2], s_halt;
  const uint32_t rows = a.rc->rows;
  if (block_stop(!slab_chosen(a) || reach_halted(a.rc) || rows > (BOTH ? kSlabRows16 : kSlabRows32))) return;
  if (rows < a.min_rows) {
    if (threadIdx.x == 0 && blockIdx.x == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
    return;
  }
  const uint32_t B = BOTH && rows > kSlabRows32 ? 16 : 32;
  const uint64_t need = (uint64_t)((a.rc->cols + B - 1) / B) * rows * (B / 8);
  if (blockIdx.x == 0 && threadIdx.x == 0) a.rc->slab = B;  // read by later launches
  if (need > 4 * a.bits_words) {
    if (threadIdx.x == 0 && blockIdx.x == 0) atomicOr(&a.rc->stop, (uint32_t)kReachSlabFull);
    return;
  }
  a.form = 1;
  reach_levels_clear(s_lev);
  __syncthreads();
  if (BOTH && rows > kSlabRows32)
    slab_run<uint16_t, (int)((kSlabRows16 + kSlabThreads) / kSlabThreads)>(a, s_mem, s_lev, s_tab, s_any, &s_halt);
  else
    slab_run<uint32_t, (int)((kSlabRows32 + kSlabThreads) / kSlabThreads)>(a, s_mem, s_lev, s_tab, s_any, &s_halt);
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

__device__ __forceinline__ uint32_t result_rows(const ReachArgs& a) { return a.square ? a.rc->cols : a.rc->rows; }

// Tuples of each row over all slabs: 64 rows per block, its waves taking the slabs in turn.
__global__ __launch_bounds__(kBlock) void k_slab_count(ReachArgs a) {
  __shared__ uint32_t s_c[kWavesPerBlock][kWave];
  if (block_stop(a.rc->slab == 0 || (a.rc->stop & (kReachHalt | kReachSlabFull)) != 0)) return;
  const uint32_t rows = result_rows(a), B = a.rc->slab, slabs = (a.rc->cols + B - 1) / B;
  const uint32_t lane = (uint32_t)lane_id(), wid = threadIdx.x / kWave;
  for (uint32_t x0 = blockIdx.x * kWave; x0 < rows; x0 += gridDim.x * kWave) {
    const uint32_t x = x0 + lane;
    uint32_t c = 0;
    if (x < rows) {
      if (B == 32)
        for (uint32_t s = wid; s < slabs; s += kWavesPerBlock) c += (uint32_t)__popc(a.bits[(uint64_t)s * rows + x]);
      else
        for (uint32_t s = wid; s < slabs; s += kWavesPerBlock)
          c += (uint32_t)__popc((uint32_t)((const uint16_t*)a.bits)[(uint64_t)s * rows + x]);
    }
    s_c[wid][lane] = c;
    __syncthreads();
    if (wid == 0 && x < rows) {
      for (int q = 1; q < kWavesPerBlock; ++q) c += s_c[q][lane];
      a.cnt[x] = c;
    }
    __syncthreads();
  }
}

// Sorts the N x G values of G neighbouring lanes (lane gl holds values gl * N ...), a bitonic network: the
// steps within a lane are minima and maxima of registers, the few across lanes exchange them.
template <int N, int G>
__device__ __forceinline__ void sort_group(uint32_t (&v)[N], uint32_t gl) {
  sort_regs<N>(v, (gl & 1u) ? 0xFFFFFFFFu : 0u);
  auto across = [&](auto dist) {
    constexpr int D = decltype(dist)::value;
    // (down: this lane keeps the larger values; descending stretches are flipped)
    const bool up = (gl & D) != 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const uint32_t o = lane_xor<D>(v[r]);
      v[r] = (v[r] < o) != up ? v[r] : o;
    }
  };
#pragma unroll
  for (int k = 2; k <= G; k <<= 1) {
    const uint32_t flip = (gl & (uint32_t)k) && k < G ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] ^= flip;
    if (k > 4) across(std::integral_constant<int, 4>{});
    if (k > 2) across(std::integral_constant<int, 2>{});
    across(std::integral_constant<int, 1>{});
#pragma unroll
    for (int j = N / 2; j > 0; j >>= 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int l = i ^ j;
        if (l > i) {
          const uint32_t lo = v[i] < v[l] ? v[i] : v[l], hi = v[i] < v[l] ? v[l] : v[i];
          v[i] = lo;
          v[l] = hi;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] ^= flip;
  }
}

// ---------------------------------------------------------------------------
// Group tiers: G lanes take a row, 64 / G rows a wave.  The set is a hash table in LDS, beside it the
// starts of the rows still to expand (a ring) and the levels' counts.  Rows of these tiers are
// narrow (one to four vertices per level), so few lanes can work on one; every lane steps
// through an edge list of its own, takes the next from the ring when that ends, and a row moves to
// its next level by itself: a wave's rows wait for each other only at their end.  Bound by the
// steps' latency (a dependent load and an LDS compare-and-swap) over the rows in flight, which
// their LDS limits (192 of the small tier per CU, 48 of the large).  140,000 rows of 17 to some
// thousand tuples: one tier of 16 lanes and 128 tuples took 780 us and left 720 to the queue
// tier; 258, 249 and 219 so.
// ---------------------------------------------------------------------------
template <uint32_t H, uint32_t RING, uint32_t LMAX>
struct ReachRow {
  uint32_t hash[H];    // columns; then those alone
  uint32_t ring[RING];
  uint32_t lev[LMAX];  // tuples | degrees << 16
  uint32_t pad;        // (an odd stride: rows at the same place sit in different banks)
};

template <int TIER, int G, uint32_t CAP, uint32_t H, uint32_t RING, uint32_t LMAX, int NW>
__global__ __launch_bounds__(NW * kWave) void k_reach_group(ReachArgs a) {
  constexpr uint32_t PER = kWave / G;  // rows of a wave
  constexpr uint32_t kHashShift = 32 - __builtin_ctz(H);
  static_assert(H >= 2 * CAP && (H & (H - 1)) == 0 && (RING & (RING - 1)) == 0 && PER * CAP <= kReachChunk, "");
  __shared__ ReachRow<H, RING, LMAX> s_row[NW * PER];
  __shared__ uint32_t s_buf[NW][kWave];
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  const uint32_t n = a.rc->queued[TIER];
  const uint32_t tid = threadIdx.x;
  if (block_stop(n == 0 || a.rc->slab != 0 || reach_halted(a.rc))) return;
  reach_levels_clear(s_lev);
  __syncthreads();
  const int lane = lane_id();
  const uint32_t gl = (uint32_t)lane % G;
  const uint64_t gmask = ((1ull << G) - 1ull) << (lane & ~(G - 1));
  const uint64_t lt = lanemask_lt();
  ReachRow<H, RING, LMAX>& q = s_row[tid / G];
  const uint2* __restrict__ edge = a.g.edge;
  uint64_t chunk = 0;
  uint32_t left = 0;
  uint32_t* const buf = s_buf[tid / kWave];
  uint32_t* const next = TIER == 0 ? a.queue[1] : (a.after_groups == kThinTier ? a.queue[kThinTier] : a.queue[kQueueTier]);
  uint32_t* const queued = &a.rc->queued[TIER == 0 ? 1 : a.after_groups];
  uint32_t fn = 0;      // rows in the wave's buffer
  auto flush = [&]() {  // (the whole wave)
    if (fn == 0) return;
    wave_lds_sync();
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(queued, fn);
    at = __shfl(at, 0, kWave);
    if ((uint32_t)lane < fn) next[at + lane] = buf[lane];
    fn = 0;
    wave_lds_sync();
  };
  const uint32_t stretch = xcd_stretch((n + NW * PER - 1) / (NW * PER), kReachQueueStretch / (NW * PER));
  for (uint32_t iter = 0;; ++iter) {
    const uint64_t tile = (uint64_t)xcd_tile(iter, stretch) * (NW * PER);
    if (tile >= n) break;
    const uint64_t base = tile + (tid / kWave) * PER;
    if (iter % kStopRows == kStopRows - 1 && wave_uniform(reach_halted(a.rc))) break;
    const uint64_t k = base + (uint32_t)lane / G;
    const bool have = k < n;
    const uint32_t row = have ? a.queue[TIER][k] : 0u;
    for (uint32_t x = gl; x < H; x += G) q.hash[x] = kReachNone;
    // the row's own edges: one list, as if its vertex had been found before the first level
    uint32_t cnt = 0, prev = 0, pops = have ? 1u : 0u, lo = 0, hi = pops, f = gl + G, level = 0, found = 0, d = 0;
    bool fail = false, done = !have, first = true;
    bool on = have && gl == 0;
    uint32_t e = on ? a.g.rstart[row] : 0u;
    wave_lds_sync();
    for (;;) {
      const uint64_t busy = __builtin_amdgcn_ballot_w64(on) & gmask;
      const bool idle = busy == 0 && !done;
      if (__builtin_amdgcn_ballot_w64(idle)) {
        if (idle) {
          // the row's level is expanded: its counts, then the level found
          if (!first && gl == 0) q.lev[level] = found | (d << 16);
          if (!first) ++level;
          first = false;
          found = cnt - prev;
          fail = fail || (found != 0 && level >= LMAX);
          done = fail || found == 0;
          prev = cnt;
          d = 0;
          lo = hi;
          hi = pops;
          f = lo + gl;
          if (!done && f < hi) {
            e = q.ring[f % RING];
            on = true;
            f += G;
          }
        }
      }
      if (__builtin_amdgcn_ballot_w64(!done) == 0) break;
      uint2 rec[2];  // (readable past the last edge)
      rec[0].x = rec[0].y = rec[1].x = rec[1].y = kReachNone;
      if (on) {
        rec[0] = edge[e];
        rec[1] = edge[e + 1];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t z = rec[h].x & ~kReachLast;
        bool fresh = false;
        if (on) {
          uint32_t slot = (z * 0x9E3779B1u) >> kHashShift;
          for (;;) {
            const uint32_t old = atomicCAS(&q.hash[slot], kReachNone, z);
            fresh = old == kReachNone;
            if (fresh || old == z) break;
            slot = (slot + 1) % H;
          }
        }
        const uint64_t ob = __builtin_amdgcn_ballot_w64(on) & gmask;
        const uint64_t nb = __builtin_amdgcn_ballot_w64(fresh) & gmask;
        const uint64_t pb = __builtin_amdgcn_ballot_w64(fresh && rec[h].y != kReachNone) & gmask;
        if (fresh && rec[h].y != kReachNone) q.ring[(pops + (uint32_t)__popcll(pb & lt)) % RING] = rec[h].y;
        cnt += (uint32_t)__popcll(nb);
        pops += (uint32_t)__popcll(pb);
        d += (uint32_t)__popcll(ob);
        fail = fail || cnt > CAP || pops - lo > RING || d > 0xFFFFu;
        on = on && (rec[h].x & kReachLast) == 0 && !fail;
      }
      e += 2;
      wave_lds_sync();
      if (!on && !done && !fail && f < hi) {
        e = q.ring[f % RING];
        on = true;
        f += G;
      }
    }
    wave_lds_sync();
    const bool good = have && !fail;
    if (good && gl == 0 && level > a.lev_cap) reach_deep(a);
    if (good)
      for (uint32_t x = gl; x < level; x += G) reach_count(s_lev, a, x, q.lev[x] & 0xFFFFu, q.lev[x] >> 16);
    // pool entries of the wave's rows, side by side
    const uint32_t mine = good ? cnt : 0u;
    const uint32_t incl = wave_incl_scan<uint32_t>(gl == 0 ? mine : 0u);
    const uint32_t total = __shfl(incl, kWave - 1, kWave);
    const uint32_t before = __shfl(incl, lane & ~(G - 1), kWave) - mine;
    if (total > left) {
      uint64_t pos = 0;
      if (lane == 0) pos = reach_alloc(a, kReachChunk);
      chunk = __shfl(pos, 0, kWave);
      left = kReachChunk;
    }
    const bool fits = chunk + total <= a.pool_cap;
    // the columns alone
    {
      constexpr int SLOTS = (int)(H / G);
      uint32_t v[SLOTS], c = 0;
#pragma unroll
      for (int r = 0; r < SLOTS; ++r) {
        v[r] = q.hash[(uint32_t)r * G + gl];
        c += v[r] != kReachNone ? 1u : 0u;
      }
      const uint32_t ends = wave_incl_scan<uint32_t>(c);
      uint32_t at = ends - c;
      at -= __shfl(at, lane & ~(G - 1), kWave);
      wave_lds_sync();
#pragma unroll
      for (int r = 0; r < SLOTS; ++r)
        if (v[r] != kReachNone) q.hash[at++] = v[r];
      wave_lds_sync();
    }
    // sorted in registers
    {
      constexpr int N = (int)(CAP / G);
      uint32_t v[N];
#pragma unroll
      for (int r = 0; r < N; ++r) v[r] = gl * N + r < mine ? q.hash[gl * N + r] : kReachNone;
      sort_group<N, G>(v, gl);
      wave_lds_sync();
#pragma unroll
      for (int r = 0; r < N; ++r) q.hash[gl * N + r] = v[r];
      wave_lds_sync();
      if (fits)
        for (uint32_t x = gl; x < mine; x += G) a.pool[chunk + before + x] = q.hash[x];
    }
    if (good && gl == 0) {
      a.cnt[row] = cnt;
      a.seg[row] = (uint32_t)(chunk + before);
    }
    // rows sent on are buffered per wave (a same-address atomic costs 12 ns)
    const bool out = have && gl == 0 && fail;
    const uint64_t sent = __builtin_amdgcn_ballot_w64(out);
    if (out) buf[fn + (uint32_t)__popcll(sent & lt)] = row;
    fn += (uint32_t)__popcll(sent);
    if (fn > kWave - PER) flush();
    chunk += total;
    left -= total;
    wave_lds_sync();
  }
  flush();
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// The edges of the rows that start at `start` in each lane of a wave (kReachNone: none), each record
// through `visit(on, record)`: the first eight by their lane (four loads at a time), the rest of
// a longer row by the whole wave.  Returns edges; their sum over the lanes is what was visited.
template <typename Visit>
__device__ __forceinline__ uint32_t wave_expand(const uint2* __restrict__ edge, uint32_t edges, uint32_t start,
                                                Visit visit) {
  const uint32_t lane = (uint32_t)lane_id();
  bool on = start != kReachNone;
  uint32_t e = on ? start : 0u, d = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (__builtin_amdgcn_ballot_w64(on) == 0) return d;
    uint2 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k].x = x[k].y = kReachNone;
      if (on) x[k] = edge[e + k];  // (readable past the last edge)
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (__builtin_amdgcn_ballot_w64(on) == 0) break;
      visit(on, x[k]);
      d += on ? 1u : 0u;
      on = on && (x[k].x & kReachLast) == 0;
    }
    e += 4;
  }
  for (uint64_t big = __builtin_amdgcn_ballot_w64(on); big; big &= big - 1) {
    const int src = __ffsll((unsigned long long)big) - 1;
    uint32_t b = __shfl(e, src, kWave);
    for (;;) {
      uint2 x;
      x.x = kReachLast;
      x.y = kReachNone;
      if (b + lane < edges) x = edge[b + lane];
      const uint64_t ends = __builtin_amdgcn_ballot_w64((x.x & kReachLast) != 0);
      // the row's edges: up to and including the first end
      const bool in = ends == 0 || lane <= (uint32_t)(__ffsll((unsigned long long)ends) - 1);
      visit(in, x);
      d += in ? 1u : 0u;
      if (ends) break;
      b += kWave;
    }
  }
  return d;
}

// The columns of a row's instance: [base, base + width).
__device__ __forceinline__ void row_columns(const ReachArgs& a, uint32_t row, uint32_t& base, uint32_t& width) {
  if (a.g.instances <= 1) {
    base = 0;
    width = a.rc->cols;
    return;
  }
  const uint64_t first = a.g.rowkey[row] & ~id_mask(a.g.w);
  const uint64_t end = first + (1ull << a.g.w);
  base = rank_col(a.g.rank, first);
  width = rank_col(a.g.rank, end < a.g.span ? end : a.g.span) - base;
}

// ---------------------------------------------------------------------------
// Thin tier: one row per wave, the set a bitmap of the instance's columns in memory (the wave's own, in
// its XCD's L2), beside it in LDS a bit per 1,024 columns that has any and the levels' queues.  A level
// costs the latencies of an edge load and of an atomic in the L2, 1.2 us; what counts is how
// many rows are in flight, 24 per CU where a bitmap in LDS leaves one or two.  Only the stretches
// that have columns are read back and cleared.  A level that outgrows the queue sends the row on, and so
// does one that is not thin by the last level whose counts can still be taken back.
// ---------------------------------------------------------------------------
// Pool entries a wave reserves at a time, and rows between its looks at `stop`: both are on the one line that
// all waves' atomics queue for (a reservation and a look for every row: 2,000 cycles of 70 vertices
// 10.4 ms, 4.0 so).
constexpr uint32_t kThinChunk = 1024;
constexpr uint32_t kThinWaves = 4;  // (each for itself: a quarter of the blocks to start)
template <uint32_t QCAP, uint32_t GROUPS>  // stretches of 1,024 columns
__global__ __launch_bounds__(kThinWaves * kWave) void k_reach_thin(ReachArgs a) {
  constexpr uint32_t TH = kThinWaves * kWave;
  static_assert(4 * QCAP >= GROUPS && GROUPS % 32 == 0 && GROUPS / 32 <= kWave, "");
  struct Row {  // a wave's
    uint32_t front[2][QCAP];
    uint32_t any[GROUPS / 32];
    uint32_t ln[kReachLdsLevels], ld[kReachLdsLevels];
  };
  __shared__ Row s_row[kThinWaves];
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  const uint32_t lane = (uint32_t)lane_id(), wid = threadIdx.x / kWave;
  Row& r = s_row[wid];
  const uint32_t n = a.rc->queued[kThinTier];
  if (block_stop(n == 0 || a.rc->slab != 0 || reach_halted(a.rc))) return;
  if (n <= a.thin_rows) {  // (uniform over the launch)
    for (uint32_t i = blockIdx.x * TH + threadIdx.x; i < n; i += gridDim.x * TH) a.queue[kQueueTier][i] = a.queue[kThinTier][i];
    if (threadIdx.x == 0 && blockIdx.x == 0) a.rc->queued[kQueueTier] = n;
    return;
  }
  reach_levels_clear(s_lev);
  if (lane < GROUPS / 32) r.any[lane] = 0;
  __syncthreads();
  const uint64_t lt = lanemask_lt();
  const uint2* __restrict__ edge = a.g.edge;
  const uint32_t edges = a.rc->edges;
  uint32_t* const vis = a.vis + ((uint64_t)blockIdx.x * kThinWaves + wid) * a.vis_words;
  uint32_t share = 0, claims = 0, left = 0;
  uint64_t chunk = 0;  // pool entries left of the wave's
  for (;;) {
    uint32_t row = kReachNone;
    if (lane == 0 && !(claims++ % kStopRows == 0 && reach_look(a))) {
      const uint32_t at = reach_claim(a.rc, kThinTier, n, share);
      if (at != kReachNone) row = a.queue[kThinTier][at];
    }
    row = wave_uniform(row);
    if (row == kReachNone) break;
    uint32_t base, width;
    row_columns(a, row, base, width);
    if ((width + 31u) / 32u > min(a.vis_words, GROUPS * 32u)) {  // (the host sized it for the widest instance)
      if (lane == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
      break;
    }
    const uint32_t first = a.g.rstart[row], deg = a.g.rstart[row + 1] - first;
    int to = 0;
    uint32_t nq = 0, nf = 0;
    auto visit = [&](bool on, uint2 rec) {
      const uint32_t z = (rec.x & ~kReachLast) - base;
      bool fresh = false;
      if (on) {
        const uint32_t bit = 1u << (z & 31u);
        fresh = (__hip_atomic_fetch_or(&vis[z >> 5], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit) == 0;
        if (fresh) atomicOr(&r.any[z >> 15], 1u << ((z >> 10) & 31u));
      }
      const uint64_t nb = __builtin_amdgcn_ballot_w64(fresh);
      if (nb) {  // (uniform)
        const uint64_t pb = __builtin_amdgcn_ballot_w64(fresh && rec.y != kReachNone);
        const uint32_t at = nq + (uint32_t)__popcll(pb & lt);
        if (fresh && rec.y != kReachNone && at < QCAP) r.front[to][at] = rec.y;
        nq += (uint32_t)__popcll(pb);
        nf += (uint32_t)__popcll(nb);
      }
    };
    for (uint32_t j = 0; j < deg; j += kWave) {
      const bool on = j + lane < deg;
      uint2 rec;
      rec.x = rec.y = kReachNone;
      if (on) rec = edge[first + j + lane];
      visit(on, rec);
    }
    uint32_t lv = 0, cnt = 0, look = min(kStopLevels, a.lev_cap);
    bool fail = false;
    for (;;) {
      const int from = to;
      const uint32_t fn = nq, found = nf;
      cnt += found;
      if (found == 0) break;
      if (__builtin_expect(lv >= look, 0)) {
        if (lane == 0 && lv >= a.lev_cap) reach_deep(a);
        if (wave_uniform(lane == 0 && (lv >= a.lev_cap || reach_look(a)))) break;
        look = min(lv + kStopLevels, a.lev_cap);
      }
      if (fn > QCAP || (lv == kReachLdsLevels && fn > QCAP / 4)) {
        fail = true;
        break;
      }
      to ^= 1;
      nq = nf = 0;
      wave_lds_sync();
      uint32_t dsum = 0;
      for (uint32_t f = 0; f < fn; f += kWave)
        dsum += wave_expand(edge, edges, f + lane < fn ? r.front[from][f + lane] : kReachNone, visit);
      dsum = wave_sum<uint32_t>(dsum);
      wave_lds_sync();
      if (lane == 0) {
        if (lv < kReachLdsLevels) {
          r.ln[lv] = found;
          r.ld[lv] = dsum;
        } else {
          reach_count(s_lev, a, lv, found, dsum);
        }
      }
      ++lv;
    }
    wave_lds_sync();
    uint64_t pos = ~0ull;
    if (fail) {
      if (lane == 0) {
        if (lv > kReachLdsLevels) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);  // (counted already)
        else a.queue[kQueueTier][atomicAdd(&a.rc->queued[kQueueTier], 1u)] = row;
      }
    } else {
      for (uint32_t x = lane; x < lv && x < kReachLdsLevels; x += kWave) reach_count(s_lev, a, x, r.ln[x], r.ld[x]);
      if (cnt > left) {  // (uniform)
        left = max(cnt, kThinChunk);
        if (lane == 0) chunk = reach_alloc(a, left);
        chunk = __shfl(chunk, 0, kWave);
      }
      pos = chunk;
      chunk += cnt;
      left -= cnt;
      if (lane == 0) {
        a.cnt[row] = cnt;
        a.seg[row] = (uint32_t)pos;
      }
      if (chunk > a.pool_cap) pos = ~0ull;
    }
    // the stretches that have columns, in order (the queues are free)
    uint16_t* const list = (uint16_t*)&r.front[0][0];
    uint32_t v = lane < GROUPS / 32 ? r.any[lane] : 0u;
    const uint32_t c = (uint32_t)__popc(v), incl = wave_incl_scan<uint32_t>(c);
    const uint32_t groups = __shfl(incl, kWave - 1, kWave);
    for (uint32_t at = incl - c; v; v &= v - 1) list[at++] = (uint16_t)(lane * 32u + (uint32_t)__ffs(v) - 1u);
    if (lane < GROUPS / 32) r.any[lane] = 0;
    wave_lds_sync();
    // eight at a time, four words a lane
    for (uint32_t g0 = 0; g0 < groups; g0 += 8) {
      const uint32_t g = g0 + lane / 8;
      const uint32_t x0 = g < groups ? (uint32_t)list[g] * 32u + lane % 8 * 4u : 0u;
      uint32_t b[4], sum = 0;
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q)
        b[q] = g < groups ? __hip_atomic_load(&vis[x0 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        if (b[q]) __hip_atomic_store(&vis[x0 + q], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        sum += (uint32_t)__popc(b[q]);
      }
      if (pos != ~0ull) {
        const uint32_t ends = wave_incl_scan<uint32_t>(sum);
        uint64_t at = pos + ends - sum;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
          for (; b[q]; b[q] &= b[q] - 1) a.pool[at++] = base + (x0 + q) * 32u + (uint32_t)__ffs(b[q]) - 1u;
        pos += __shfl(ends, kWave - 1, kWave);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // (the words are zero before the next row's bits)
    wave_lds_sync();
  }
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// ---------------------------------------------------------------------------
// Queue tier: one row per block of NW waves (one wave where the columns' bitmap is at most 8 KB).
// The set is a bitmap of the instance's columns in LDS; a column whose bit a lane sets first is
// found, and its row, if it has one, goes to the next level's queue.  Thin, deep rows pay per level
// one edge load and a few LDS round trips (one wave keeps its counts in registers: a tenth less for
// the rows past 256 tuples of 256 random graphs), and 5 to 24 of them run per CU.  A level that outgrows the
// queue sends the row on.  The columns come out of the bitmap in order.
// ---------------------------------------------------------------------------
template <int NW, uint32_t WORDS, uint32_t QCAP>
__global__ __launch_bounds__(NW * kWave) void k_reach_queue(ReachArgs a) {
  constexpr uint32_t TH = NW * kWave;
  __shared__ uint32_t s_vis[WORDS];
  __shared__ uint32_t s_front[2][QCAP];
  __shared__ uint32_t s_n[2], s_f[2];  // queued, found
  __shared__ uint32_t s_row, s_d, s_halt;
  __shared__ uint32_t s_wave[NW];
  __shared__ uint64_t s_pos;
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  __shared__ uint32_t s_ln[kReachLdsLevels], s_ld[kReachLdsLevels];  // the row's levels so far
  const uint32_t tid = threadIdx.x;
  const uint32_t n = a.rc->queued[kQueueTier];
  if (block_stop(n == 0 || a.rc->slab != 0 || reach_halted(a.rc))) return;
  reach_levels_clear(s_lev);
  const int wid = (int)(tid / kWave);
  const int lane = lane_id();
  const uint64_t lt = lanemask_lt();
  const uint2* __restrict__ edge = a.g.edge;
  const uint32_t edges = a.rc->edges;
  uint32_t share = 0, claims = 0;
  for (uint32_t x = tid; x < WORDS; x += TH) s_vis[x] = 0;
  __syncthreads();
  for (;;) {
    if (tid == 0) {
      const bool over = claims++ % kStopRows == 0 && reach_look(a);
      const uint32_t at = over ? kReachNone : reach_claim(a.rc, kQueueTier, n, share);
      s_row = at == kReachNone ? kReachNone : a.queue[kQueueTier][at];
      s_n[0] = s_n[1] = s_f[0] = s_f[1] = 0;
    }
    __syncthreads();
    const uint32_t row = s_row;
    if (row == kReachNone) break;
    uint32_t base, width;
    row_columns(a, row, base, width);
    const uint32_t words = (width + 31u) / 32u;
    if (words > WORDS) {  // (the host sized WORDS for the widest instance)
      if (tid == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
      break;
    }
    const uint32_t first = a.g.rstart[row], deg = a.g.rstart[row + 1] - first;
    int to = 0;
    // (one wave: its counts are in registers)
    uint32_t nq = 0, nf = 0;
    auto visit = [&](bool on, uint2 rec) {
      const uint32_t z = (rec.x & ~kReachLast) - base;
      bool fresh = false;
      if (on) fresh = !((atomicOr(&s_vis[z >> 5], 1u << (z & 31u)) >> (z & 31u)) & 1u);
      const uint64_t nb = __builtin_amdgcn_ballot_w64(fresh);
      if (nb) {  // (uniform in the wave)
        const uint64_t pb = __builtin_amdgcn_ballot_w64(fresh && rec.y != kReachNone);
        uint32_t at = 0;
        if constexpr (NW == 1) {
          at = nq;
          nq += (uint32_t)__popcll(pb);
          nf += (uint32_t)__popcll(nb);
        } else {
          if (lane == 0) {
            at = atomicAdd(&s_n[to], (uint32_t)__popcll(pb));
            atomicAdd(&s_f[to], (uint32_t)__popcll(nb));
          }
          at = __shfl(at, 0, kWave);
        }
        at += (uint32_t)__popcll(pb & lt);
        if (fresh && rec.y != kReachNone && at < QCAP) s_front[to][at] = rec.y;
      }
    };
    for (uint32_t j = (uint32_t)wid * kWave; j < deg; j += TH) {
      const bool on = j + lane < deg;
      uint2 rec;
      rec.x = rec.y = kReachNone;
      if (on) rec = edge[first + j + lane];
      visit(on, rec);
    }
    __syncthreads();
    uint32_t lv = 0, cnt = 0, look = min(kStopLevels, a.lev_cap);  // the next level to stop at, if need be
    bool fail = false;
    for (;;) {
      const int from = to;
      const uint32_t fn = NW == 1 ? nq : s_n[from], found = NW == 1 ? nf : s_f[from];
      cnt += found;
      if (found == 0) break;
      if (__builtin_expect(fn > QCAP || lv >= look, 0)) {
        fail = fn > QCAP;
        if (fail) break;
        if (tid == 0) {
          s_halt = lv >= a.lev_cap || reach_look(a);
          if (lv >= a.lev_cap) reach_deep(a);
        }
        if constexpr (NW == 1) wave_lds_sync();
        else __syncthreads();
        if (s_halt) break;
        look = min(lv + kStopLevels, a.lev_cap);
      }
      to ^= 1;
      if constexpr (NW == 1) {
        nq = nf = 0;
        wave_lds_sync();
      } else {
        __syncthreads();
        if (tid == 0) s_n[to] = s_f[to] = s_d = 0;
        __syncthreads();
      }
      uint32_t dsum = 0;
      for (uint32_t f = (uint32_t)wid * kWave; f < fn; f += TH)
        dsum += wave_expand(edge, edges, f + lane < fn ? s_front[from][f + lane] : kReachNone, visit);
      dsum = wave_sum<uint32_t>(dsum);
      if constexpr (NW == 1) {
        wave_lds_sync();
      } else {
        if (lane == 0 && dsum) atomicAdd(&s_d, dsum);
        __syncthreads();
        dsum = s_d;
      }
      // (the row's counts: kept until it is done, or straight to memory once it is deeper than
      // the table, from where on it can no longer be sent back)
      if (tid == 0) {
        if (lv < kReachLdsLevels) {
          s_ln[lv] = found;
          s_ld[lv] = dsum;
        } else {
          reach_count(s_lev, a, lv, found, dsum);
        }
      }
      ++lv;
    }
    __syncthreads();
    if (fail) {
      if (tid == 0) {
        // (counted already, or no tier for it: the general path)
        if (lv > kReachLdsLevels || !a.bits_tier) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
        else a.queue[kBitsTier][atomicAdd(&a.rc->queued[kBitsTier], 1u)] = row;
      }
      for (uint32_t x = tid; x < words; x += TH) s_vis[x] = 0;
    } else {
      for (uint32_t x = tid; x < lv && x < kReachLdsLevels; x += TH) reach_count(s_lev, a, x, s_ln[x], s_ld[x]);
      if (tid == 0) {
        const uint64_t pos = reach_alloc(a, cnt);
        s_pos = pos + cnt > a.pool_cap ? ~0ull : pos;
        a.cnt[row] = cnt;
        a.seg[row] = (uint32_t)pos;
      }
      __syncthreads();
      const uint64_t pos = s_pos;
      uint32_t run = 0;
      for (uint32_t x0 = 0; x0 < words; x0 += TH) {
        const uint32_t x = x0 + tid;
        uint32_t bits = 0;
        if (x < words) {
          bits = s_vis[x];
          s_vis[x] = 0;
        }
        uint32_t total;
        uint32_t at = run + block_excl_scan<uint32_t, NW>((uint32_t)__popc(bits), s_wave, total);
        run += total;
        if (pos != ~0ull)
          for (; bits; bits &= bits - 1) a.pool[pos + at++] = base + x * 32u + (uint32_t)__ffs(bits) - 1u;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// ---------------------------------------------------------------------------
// Bits tier: one row per block of four waves, its set, its level and its next level three
// bitmaps in LDS.  The waves scan the level's halfwords interleaved (a power-law graph's hubs sit
// in few words), compact the columns they find into a list of their own and expand it with all
// lanes; a column not in the set has its bit ORed into the next level, which therefore needs no
// dedup at all (a repeat costs an LDS read and an atomic without return).  Between levels one
// pass joins the next level into the set.  Bound by LDS traffic and instruction issue per
// candidate.  The row goes out as its bitmap.
// ---------------------------------------------------------------------------
constexpr int kReachBitsWaves = 4;
template <uint32_t WORDS, typename ID>
__global__ __launch_bounds__(kReachBitsWaves * kWave) void k_reach_bits(ReachArgs a) {
  constexpr int NW = kReachBitsWaves;
  constexpr uint32_t TH = NW * kWave;
  constexpr uint32_t LCAP = kWave * 16;  // columns of 64 halfwords
  __shared__ uint32_t s_vis[WORDS], s_cur[WORDS], s_nxt[WORDS];
  __shared__ ID s_list[NW][LCAP];
  __shared__ uint32_t s_n[NW];
  __shared__ uint32_t s_row, s_at, s_any[2], s_halt;
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  const uint32_t tid = threadIdx.x;
  const uint32_t n = a.rc->queued[kBitsTier];
  if (block_stop(n == 0 || a.rc->slab != 0 || reach_halted(a.rc))) return;
  if (n > a.slots) {
    if (tid == 0 && blockIdx.x == 0) atomicOr(&a.rc->stop, (uint32_t)kReachSlotsFull);
    return;
  }
  reach_levels_clear(s_lev);
  const int wid = (int)(tid / kWave);
  const int lane = lane_id();
  const uint2* __restrict__ edge = a.g.edge;
  const uint32_t edges = a.rc->edges;
  const uint16_t* const cur16 = (const uint16_t*)s_cur;
  ID* const list = s_list[wid];
  uint32_t share = 0, claims = 0;
  for (uint32_t x = tid; x < WORDS; x += TH) s_vis[x] = s_cur[x] = s_nxt[x] = 0;
  __syncthreads();
  for (;;) {
    if (tid == 0) {
      const bool over = reach_halted(a.rc) || (++claims % kStopRows == 0 && cancelled(a.cancel, &a.rc->stop));
      const uint32_t at = over ? kReachNone : reach_claim(a.rc, kBitsTier, n, share);
      s_at = at;
      s_row = at == kReachNone ? kReachNone : a.queue[kBitsTier][at];
      s_any[0] = 0;
    }
    __syncthreads();
    const uint32_t row = s_row, slot = s_at;
    if (row == kReachNone) break;
    uint32_t base, width;
    row_columns(a, row, base, width);
    const uint32_t words = (width + 31u) / 32u, halves = words * 2;
    if (words > WORDS) {
      if (tid == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
      break;
    }
    const uint32_t first = a.g.rstart[row], deg = a.g.rstart[row + 1] - first;
    for (uint32_t j = tid; j < deg; j += TH) {
      const uint32_t z = (edge[first + j].x & ~kReachLast) - base;
      atomicOr(&s_nxt[z >> 5], 1u << (z & 31u));
    }
    __syncthreads();
    uint32_t cnt = 0;
    for (uint32_t lv = 0;; ++lv) {
      // the next level becomes the level and joins the set
      uint32_t mine = 0;
      for (uint32_t x = tid; x < words; x += TH) {
        const uint32_t b = s_nxt[x];
        s_cur[x] = b;
        if (b) {
          s_nxt[x] = 0;
          s_vis[x] |= b;
          mine += (uint32_t)__popc(b);
        }
      }
      if (mine) {
        reach_count(s_lev, a, lv, mine, 0);
        atomicAdd(&s_any[lv & 1u], mine);
      }
      if (tid == 0) {
        s_any[(lv + 1) & 1u] = 0;
        s_halt = lv % kStopLevels == kStopLevels - 1 && reach_look(a);
      }
      __syncthreads();
      const uint32_t found = s_any[lv & 1u];
      if (found != 0 && lv >= a.lev_cap && tid == 0) reach_deep(a);
      if (found == 0 || lv >= a.lev_cap || s_halt) break;
      cnt += found;
      uint32_t dsum = 0;
      for (uint32_t h0 = 0; h0 < halves; h0 += TH) {
        const uint32_t h = h0 + (uint32_t)lane * NW + (uint32_t)wid;
        uint32_t b = h < halves ? (uint32_t)cur16[h] : 0u;
        if (__builtin_amdgcn_ballot_w64(b != 0) == 0) continue;  // (uniform in the wave)
        if (lane == 0) s_n[wid] = 0;
        wave_lds_sync();
        if (b) {
          uint32_t at = atomicAdd(&s_n[wid], (uint32_t)__popc(b));
          for (; b; b &= b - 1) list[at++] = (ID)(h * 16u + (uint32_t)__ffs(b) - 1u);
        }
        wave_lds_sync();
        const uint32_t ln = s_n[wid];
        for (uint32_t f = 0; f < ln; f += kWave) {
          const uint32_t start = f + lane < ln ? a.g.cstart[base + (uint32_t)list[f + lane]] : kReachNone;
          dsum += wave_expand(edge, edges, start, [&](bool on, uint2 rec) {
            const uint32_t z = (rec.x & ~kReachLast) - base;
            if (on && !((s_vis[z >> 5] >> (z & 31u)) & 1u)) atomicOr(&s_nxt[z >> 5], 1u << (z & 31u));
          });
        }
        wave_lds_sync();
      }
      if (dsum) reach_count(s_lev, a, lv, 0, dsum);
      __syncthreads();
    }
    uint32_t* const out = a.bits + (uint64_t)slot * a.words;
    for (uint32_t x = tid; x < a.words; x += TH) {
      const bool in = x < words;
      out[x] = in ? s_vis[x] : 0u;
      if (in) s_vis[x] = 0;
    }
    if (tid == 0) {
      a.cnt[row] = cnt | kReachBitRow;
      a.seg[row] = slot;
    }
    __syncthreads();
  }
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// ---------------------------------------------------------------------------
// Row offsets: off[r] = tuples of the rows before r (off[rows] = all), from cnt in two launches as
// every scan here.
// ---------------------------------------------------------------------------
constexpr uint32_t kReachScanTile = kBlock * 8;

__global__ __launch_bounds__(kBlock) void k_reach_sum(ReachArgs a, uint64_t* __restrict__ part) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  if (block_stop(reach_halted(a.rc))) return;
  uint64_t lo, hi;
  block_range(result_rows(a), kReachScanTile, lo, hi);
  uint64_t sum = 0;
  for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) sum += a.cnt[i] & ~kReachBitRow;
  uint64_t total;
  (void)block_excl_scan<uint64_t>(sum, s_wave, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// (one block needs no totals: part nullptr)
template <int SCAN_MAX>
__global__ __launch_bounds__(kBlock) void k_reach_offsets(ReachArgs a, const uint64_t* __restrict__ part,
                                                          uint32_t* __restrict__ off) {
  __shared__ uint64_t s_pre[SCAN_MAX];
  __shared__ uint64_t s_wave[kWavesPerBlock];
  if (block_stop(reach_halted(a.rc))) return;
  const uint32_t n = result_rows(a);
  uint64_t run = 0;
  if (part) {
    (void)block_prefix<SCAN_MAX / kBlock>(part, (int)gridDim.x, s_pre, s_wave);
    run = s_pre[blockIdx.x];
  }
  uint64_t lo, hi;
  block_range(n, kReachScanTile, lo, hi);
  for (uint64_t base = lo; base < hi; base += kReachScanTile) {
    uint32_t c[8];
    uint64_t sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint64_t i = base + (uint64_t)threadIdx.x * 8 + k;
      c[k] = i < hi ? a.cnt[i] & ~kReachBitRow : 0u;
      sum += c[k];
    }
    uint64_t total;
    uint64_t at = run + block_excl_scan<uint64_t>(sum, s_wave, total);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint64_t i = base + (uint64_t)threadIdx.x * 8 + k;
      if (i < hi) off[i] = (uint32_t)at;
      at += c[k];
    }
    run += total;
  }
  if (hi == n && lo < hi && threadIdx.x == 0) off[n] = (uint32_t)run;
}

// ---------------------------------------------------------------------------
// Reading the result.  put(position, row key, id) stores a tuple.
// ---------------------------------------------------------------------------
// Rows with lists: tiles of outputs, so that rows of any length spread evenly; a tile's rows (at
// most one per output: every row has a tuple) are staged in LDS and each output finds its own by
// bisection.  Blocks take consecutive tiles, so only the first is searched over all rows.
constexpr uint32_t kReachOutTile = 2048;

template <typename Put>
__device__ __forceinline__ void reach_unpack_lists(const ReachResult& r, uint32_t bid, uint32_t nblocks, Put put) {
  constexpr uint32_t T = kReachOutTile;
  __shared__ uint32_t s_off[T], s_seg[T], s_row[T];
  __shared__ uint32_t s_r[2];
  const uint32_t tid = threadIdx.x;
  const uint32_t rows = r.rows;
  const uint64_t F = r.off[rows];
  const uint64_t ntiles = (F + T - 1) / T, per = (ntiles + nblocks - 1) / nblocks;
  const uint64_t t0 = (uint64_t)bid * per, t1 = min(t0 + per, ntiles);
  const int wid = (int)(tid / kWave);
  uint64_t from = 0;  // a row at or before the next tile's first output
  for (uint64_t tile = t0; tile < t1; ++tile) {
    const uint64_t p0 = tile * T, p1 = min(p0 + T, F);
    if (wid < 2) {
      const uint64_t p = wid == 0 ? p0 : p1 - 1;
      const uint64_t end = tile == t0 ? rows : min<uint64_t>(from + T + 1, rows);
      const uint64_t v = wave_partition(from, end, [&](uint64_t i) { return r.off[i] <= p; }) - 1;
      if (lane_id() == 0) s_r[wid] = (uint32_t)v;
    }
    __syncthreads();
    const uint32_t r0 = s_r[0], span = s_r[1] - r0 + 1;  // span <= T
    for (uint32_t x = tid; x < span; x += kBlock) {
      s_off[x] = r.off[r0 + x];
      s_seg[x] = r.seg[r0 + x];
      s_row[x] = (r.cnt[r0 + x] & kReachBitRow) ? kReachNone : r0 + x;  // (the bitmaps' blocks write those)
    }
    __syncthreads();
    for (uint32_t t = tid; t < (uint32_t)(p1 - p0); t += kBlock) {
      const uint32_t p = (uint32_t)(p0 + t);
      uint32_t lo = 0;
      for (uint32_t len = span; len > 1;) {
        const uint32_t half = len >> 1;
        lo = s_off[lo + half] <= p ? lo + half : lo;
        len -= half;
      }
      const uint32_t row = s_row[lo];
      if (row != kReachNone) put(p, r.rowkey[row], r.colkey[r.pool[(uint64_t)s_seg[lo] + (p - s_off[lo])]]);
    }
    from = s_r[1];
    __syncthreads();
  }
}

// Rows with bitmaps: a block per row expands 256 words at a time through LDS, so that the writes
// coalesce.
template <typename Put>
__device__ __forceinline__ void reach_unpack_bits(const ReachResult& r, uint32_t bid, uint32_t nblocks, Put put) {
  __shared__ uint16_t s_id[kBlock * 32];  // columns relative to the 256 words' first
  __shared__ uint32_t s_wave2[kWavesPerBlock];
  const uint32_t tid = threadIdx.x;
  for (uint64_t k = bid; k < r.n_bits; k += nblocks) {
    const uint32_t row = r.bit_rows[k], key = r.rowkey[row];
    const uint32_t base = rank_col(r.rank, key & ~id_mask(r.w));
    const uint32_t* __restrict__ b = r.bits + k * r.words;
    uint64_t out = r.off[row];
    for (uint32_t x0 = 0; x0 < r.words; x0 += kBlock) {
      uint32_t v = x0 + tid < r.words ? b[x0 + tid] : 0u;
      uint32_t total;
      uint32_t at = block_excl_scan<uint32_t>((uint32_t)__popc(v), s_wave2, total);
      for (; v; v &= v - 1) s_id[at++] = (uint16_t)(tid * 32u + (uint32_t)__ffs(v) - 1u);
      __syncthreads();
      for (uint32_t t = tid; t < total; t += kBlock) put(out + t, key, r.colkey[base + x0 * 32u + s_id[t]]);
      out += total;
      __syncthreads();
    }
  }
}

// Slabs: a wave per row takes 64 slabs at a time (a lane each), lists their columns in LDS and writes
// them out in order.  The eight waves of a block read neighbouring rows, that is the same lines of
// every slab.
constexpr int kSlabOutWaves = 8;
template <typename Put>
__device__ __forceinline__ void reach_unpack_slabs(const ReachResult& r, Put put) {
  __shared__ uint16_t s_col[kSlabOutWaves][kWave * 32];
  const int wid = (int)(threadIdx.x / kWave);
  const uint32_t lane = (uint32_t)lane_id();
  uint16_t* const mine = s_col[wid];
  const uint32_t B = r.slab, slabs = (r.cols + B - 1) / B;
  for (uint64_t row = (uint64_t)blockIdx.x * kSlabOutWaves + wid; row < r.rows;
       row += (uint64_t)gridDim.x * kSlabOutWaves) {
    const uint32_t key = r.rowkey[row];
    uint64_t out = r.off[row];
    for (uint32_t s0 = 0; s0 < slabs; s0 += kWave) {
      uint32_t v = 0;
      if (s0 + lane < slabs) {
        const uint64_t at = (uint64_t)(s0 + lane) * r.rows + row;
        v = B == 32 ? r.bits[at] : (uint32_t)((const uint16_t*)r.bits)[at];
      }
      const uint32_t c = (uint32_t)__popc(v);
      const uint32_t incl = wave_incl_scan<uint32_t>(c);
      const uint32_t total = __shfl(incl, kWave - 1, kWave);
      for (uint32_t at = incl - c; v; v &= v - 1) mine[at++] = (uint16_t)(lane * B + (uint32_t)__ffs(v) - 1u);
      wave_lds_sync();
      for (uint32_t t = lane; t < total; t += kWave) put(out + t, key, r.colkey[s0 * B + mine[t]]);
      out += total;
      wave_lds_sync();
    }
  }
}

struct PutPairs {
  uint32_t* src;
  uint32_t* dst;
  uint32_t mask;
  __device__ __forceinline__ void operator()(uint64_t p, uint32_t row, uint32_t col) const {
    src[p] = row & mask;
    dst[p] = col & mask;
  }
};
template <typename K>
struct PutKeys {
  K* keys;
  int w;
  uint32_t mask;
  __device__ __forceinline__ void operator()(uint64_t p, uint32_t row, uint32_t col) const {
    keys[p] = ((K)row << w) | (K)(col & mask);
  }
};

// Blocks [0, list_blocks) take the rows with lists, the others the bitmaps.
template <typename Put>
__global__ __launch_bounds__(kBlock) void k_reach_unpack(ReachResult r, uint32_t list_blocks, Put put) {
  if (blockIdx.x < list_blocks) reach_unpack_lists(r, blockIdx.x, list_blocks, put);
  else reach_unpack_bits(r, blockIdx.x - list_blocks, gridDim.x - list_blocks, put);
}
template <typename Put>
__global__ __launch_bounds__(kSlabOutWaves * kWave) void k_slab_unpack(ReachResult r, Put put) {
  reach_unpack_slabs(r, put);
}

// First tuple of every instance: that of its first row.
__global__ __launch_bounds__(kBlock) void k_reach_instances(ReachResult r, uint32_t num, uint64_t* __restrict__ out) {
  for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v <= num; v += (uint64_t)gridDim.x * kBlock) {
    uint64_t row = r.rows;
    if (v < num) {
      const RankWord q = r.rank[(v << r.w) >> 5];
      row = q.rowpre + bits_below(q.rowbits, (uint32_t)(v << r.w));
    }
    out[v] = r.off[row];
  }
}

}  // namespace wg
