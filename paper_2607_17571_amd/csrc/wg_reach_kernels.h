// Kernels of the row-at-a-time closure (see wg_reach.h).
#pragma once

#include "wg_device.h"
#include "wg_reach.h"

namespace wg {

// LDS written by one lane of a wave, read by another: the wave's LDS instructions execute in
// order, so only the compiler must keep them so.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ bool reach_halted(const ReachCtl* rc) {
  return (__hip_atomic_load(&rc->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kReachHalt) != 0;
}

// `n` pool entries (one thread); past the pool's end they are counted but not to be written.
__device__ __forceinline__ uint64_t reach_alloc(const ReachArgs& a, uint32_t n) {
  const unsigned long long at = atomicAdd(&a.rc->cursor, (unsigned long long)n);
  if (at + n > a.pool_cap)
    atomicOr(&a.rc->stop, (uint32_t)(at > kReachMaxTuples ? kReachPoolFull | kReachTooLarge : kReachPoolFull));
  return at;
}

// Adds a level's counts to the block's LDS table (levels below kReachLdsLevels) or to memory.
__device__ __forceinline__ void reach_count(unsigned long long (*s_lev)[2], const ReachArgs& a, uint32_t lv,
                                            uint32_t n, uint32_t d) {
  if (lv < kReachLdsLevels) {
    if (n) atomicAdd(&s_lev[lv][0], (unsigned long long)n);
    if (d) atomicAdd(&s_lev[lv][1], (unsigned long long)d);
  } else if (lv < a.lev_cap) {
    if (n) atomicAdd(&a.lev[lv].n, (unsigned long long)n);
    if (d) atomicAdd(&a.lev[lv].d, (unsigned long long)d);
  } else {
    atomicOr(&a.rc->stop, (uint32_t)kReachDeep);
  }
}

__device__ __forceinline__ void reach_levels_clear(unsigned long long (*s_lev)[2]) {
  for (uint32_t x = threadIdx.x; x < kReachLdsLevels; x += blockDim.x) s_lev[x][0] = s_lev[x][1] = 0;
}

// (after a barrier) the block's level counts into memory
__device__ __forceinline__ void reach_levels_flush(const unsigned long long (*s_lev)[2], const ReachArgs& a) {
  for (uint32_t x = threadIdx.x; x < kReachLdsLevels && x < a.lev_cap; x += blockDim.x) {
    if (s_lev[x][0]) atomicAdd(&a.lev[x].n, s_lev[x][0]);
    if (s_lev[x][1]) atomicAdd(&a.lev[x].d, s_lev[x][1]);
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
// Thread tier: thread t of a tile takes edge t if it is the first of its row, holds the row's
// ids in 16 registers (a membership test is 16 compares) with a copy in LDS to pop them by
// index, and sorts them with a network over the registers at the end.  A tile's rows are
// consecutive, so their sorted ids are packed into one stretch of the pool.  Bound by the
// dependent loads of a pop (index entry, then edges): 64 rows advance per wave, and blocks of
// 16 KB of LDS keep 8 in flight per CU.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void sort_regs(uint32_t (&v)[N]) {
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
}

constexpr uint32_t kReachFailBuf = 512;   // rows a block buffers before it appends them to a queue
constexpr int kReachLevCopies = 16;       // copies of a block's level counts (spread over the lanes)

template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_thread(const Ctrl* ctrl, const K* __restrict__ E, ReachArgs a) {
  constexpr int CAP = (int)kReachThreadCap;
  __shared__ uint32_t s_q[CAP * kBlock];  // ids by (index, thread); then the tile's sorted ids
  __shared__ unsigned long long s_cnt[kReachLevCopies][kReachThreadCap];  // level: tuples | degrees << 32
  __shared__ uint32_t s_fail[2][kReachFailBuf];
  __shared__ uint32_t s_fn[2];
  __shared__ uint32_t s_wave[kWavesPerBlock];
  __shared__ uint64_t s_pos;
  __shared__ uint32_t s_flush[2];
  const uint32_t tid = threadIdx.x;
  for (uint32_t x = tid; x < (uint32_t)kReachLevCopies * CAP; x += kBlock) (&s_cnt[0][0])[x] = 0;
  if (tid < 2) s_fn[tid] = 0;
  const uint64_t n = ctrl->m_unique;
  const uint32_t idm = a.w >= 32 ? 0xFFFFFFFFu : (1u << a.w) - 1u;
  const uint32_t* __restrict__ R = a.R;
  const uint32_t* __restrict__ Edst = a.Edst;
  unsigned long long* const my = s_cnt[tid % kReachLevCopies];
  uint64_t chunk = 0;
  uint32_t left = 0;  // pool entries left of the block's chunk (uniform)
  const uint64_t ntiles = (n + kBlock - 1) / kBlock;
  __syncthreads();
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t i = tile * kBlock + tid;
    uint32_t row = 0, fail = 0;  // fail: 1 to the next tier, 2 a hub
    bool head = false;
    if (i < n) {
      row = head_row<K>(E[i], a.w);
      head = i == 0 || head_row<K>(E[i - 1], a.w) != row;
    }
    uint32_t q[CAP];
#pragma unroll
    for (int k = 0; k < CAP; ++k) q[k] = kReachNone;  // (no id: ids have at most 20 bits here)
    uint32_t cnt = 0;
    unsigned long long degs = 0;  // 4 bits per popped id
    uint32_t starts = 1;          // bit f: id f opens a level
    if (head) {
      const uint32_t inst = row & ~idm;
      const uint32_t d = R[(uint64_t)row + 1] - (uint32_t)i;
      if (d > 15) {
        fail = d >= a.hub ? 2u : 1u;
      } else {
#pragma unroll
        for (int k = 0; k < 15; ++k)
          if ((uint32_t)k < d) {
            q[k] = Edst[i + k];
            s_q[k * kBlock + tid] = q[k];
          }
        cnt = d;
        uint32_t end = cnt;  // of the current level
        for (uint32_t f = 0; f < cnt && !fail; ++f) {
          if (f == end) {
            starts |= 1u << f;
            end = cnt;
          }
          const uint64_t v = inst | s_q[f * kBlock + tid];
          const uint32_t e0 = R[v], e1 = R[v + 1];
          const uint32_t dv = e1 - e0;
          if (dv > 15) {
            fail = dv >= a.hub ? 2u : 1u;
            break;
          }
          degs |= (unsigned long long)dv << (4 * f);
          for (uint32_t e = e0; e < e1; ++e) {
            const uint32_t z = Edst[e];
            bool dup = false;
#pragma unroll
            for (int k = 0; k < CAP; ++k) dup |= q[k] == z;
            if (dup) continue;
            if (cnt == (uint32_t)CAP) {
              fail = 1;
              break;
            }
#pragma unroll
            for (int k = 0; k < CAP; ++k) q[k] = (uint32_t)k == cnt ? z : q[k];
            s_q[cnt * kBlock + tid] = z;
            ++cnt;
          }
        }
      }
      if (fail) {
        cnt = 0;
      } else {
        uint32_t lv = 0, ln = 0, ld = 0;
        for (uint32_t f = 0; f < cnt; ++f) {
          if (f > 0 && ((starts >> f) & 1u)) {
            atomicAdd(&my[lv], (unsigned long long)ln | ((unsigned long long)ld << 32));
            ++lv;
            ln = ld = 0;
          }
          ++ln;
          ld += (uint32_t)(degs >> (4 * f)) & 15u;
        }
        atomicAdd(&my[lv], (unsigned long long)ln | ((unsigned long long)ld << 32));
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
    if (fail) {
      const int which = fail == 2 ? 1 : 0;
      s_fail[which][atomicAdd(&s_fn[which], 1u)] = row;
    }
    if (i < n) {
      a.cnt[i] = cnt;
      a.seg[i] = (uint32_t)(chunk + at);
    }
    __syncthreads();
    if (chunk + total <= a.pool_cap)
      for (uint32_t t = tid; t < total; t += kBlock) a.pool[chunk + t] = s_q[t];
    chunk += total;
    left -= total;
    // queue buffers that a further tile could overfill go out
    const bool last = tile + gridDim.x >= ntiles;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      const uint32_t fn = s_fn[which];
      const int tier = which ? a.hub_tier : a.tier_after[0];
      if (fn > 0 && (last || fn > kReachFailBuf - kBlock)) {
        if (tid == 0) {
          if (tier < 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
          else s_flush[which] = atomicAdd(&a.rc->queued[tier], fn);
        }
        __syncthreads();
        if (tier >= 0)
          for (uint32_t t = tid; t < fn; t += kBlock) a.queue[tier][s_flush[which] + t] = s_fail[which][t];
        __syncthreads();
        if (tid == 0) s_fn[which] = 0;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  for (uint32_t lv = tid; lv < (uint32_t)CAP; lv += kBlock) {
    unsigned long long sn = 0, sd = 0;
    for (int c = 0; c < kReachLevCopies; ++c) {
      sn += s_cnt[c][lv] & 0xFFFFFFFFull;
      sd += s_cnt[c][lv] >> 32;
    }
    if (sn) atomicAdd(&a.lev[lv].n, sn);
    if (sd) atomicAdd(&a.lev[lv].d, sd);
  }
}

// ---------------------------------------------------------------------------
// Group tier: 16 lanes per row, four rows per wave in lockstep.  The set is a hash table of 256
// slots (linear probing, at most half full), the ids in order of discovery are the queue whose
// stretches are the levels.  A lane pops a vertex and walks its edges.  Rows of this tier are
// narrow (a few vertices per level), so the lanes of 16 are about as many as a level can use, and
// the rows in flight (96 per CU) hide the loads.
// ---------------------------------------------------------------------------
constexpr int kReachGroup = 16;
constexpr int kReachGroupsPerBlock = kBlock / kReachGroup;

__global__ __launch_bounds__(kBlock) void k_reach_group(ReachArgs a) {
  constexpr uint32_t CAP = kReachGroupCap, H = kReachGroupSlots;
  constexpr int G = kReachGroup;
  __shared__ uint32_t s_hash[kReachGroupsPerBlock][H];
  __shared__ uint32_t s_ids[kReachGroupsPerBlock][CAP];
  __shared__ uint32_t s_buf[kWavesPerBlock][2][kWave];
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  const uint32_t n = a.rc->queued[0];
  const uint32_t tid = threadIdx.x;
  if (block_stop(n == 0 || reach_halted(a.rc))) return;
  reach_levels_clear(s_lev);
  __syncthreads();
  const int lane = lane_id();
  const uint32_t gl = (uint32_t)lane % G;
  const uint64_t gmask = 0xFFFFull << (lane & ~(G - 1));
  const uint64_t lt = lanemask_lt();
  const uint32_t grp = tid / G;
  uint32_t* const hash = s_hash[grp];
  uint32_t* const ids = s_ids[grp];
  const uint32_t* __restrict__ R = a.R;
  const uint32_t* __restrict__ Edst = a.Edst;
  const uint32_t idm = a.w >= 32 ? 0xFFFFFFFFu : (1u << a.w) - 1u;
  const uint32_t wave_id = blockIdx.x * kWavesPerBlock + tid / kWave;
  const uint32_t waves = gridDim.x * kWavesPerBlock;
  constexpr uint32_t PER = kWave / G;  // rows of a wave
  uint64_t chunk = 0;
  uint32_t left = 0;
  uint32_t(*const buf)[kWave] = s_buf[tid / kWave];
  uint32_t fn[2] = {0, 0};  // rows in the wave's buffers: outgrown, hub
  auto flush = [&](int which) {  // (the whole wave)
    if (fn[which] == 0) return;
    wave_lds_sync();
    const int tier = which ? a.hub_tier : a.tier_after[1];
    if (tier < 0) {
      if (lane == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
    } else {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&a.rc->queued[tier], fn[which]);
      at = __shfl(at, 0, kWave);
      if ((uint32_t)lane < fn[which]) a.queue[tier][at + lane] = buf[which][lane];
    }
    fn[which] = 0;
    wave_lds_sync();
  };
  for (uint64_t base = (uint64_t)wave_id * PER; base < n; base += (uint64_t)waves * PER) {
    if (__builtin_amdgcn_readfirstlane((int)reach_halted(a.rc))) break;
    const uint64_t k = base + (uint32_t)lane / G;
    const bool have = k < n;
    const uint32_t row = have ? a.queue[0][k] : 0u;
    const uint32_t inst = row & ~idm;
    uint32_t first = 0, cnt = 0, fail = 0;
    for (uint32_t x = gl; x < H; x += G) hash[x] = kReachNone;
    wave_lds_sync();
    // adds the ids of edges [e0, e1) of every lane (empty: none) to the lane's row
    auto expand = [&](uint32_t e0, uint32_t e1) {
      while (__builtin_amdgcn_ballot_w64(e0 < e1 && !fail)) {
        bool pending = e0 < e1 && !fail, fresh = false;
        const uint32_t z = pending ? Edst[e0] : 0u;
        ++e0;
        uint32_t slot = (z * 0x9E3779B1u) >> 24;
        while (__builtin_amdgcn_ballot_w64(pending)) {
          if (pending) {
            const uint32_t old = atomicCAS(&hash[slot], kReachNone, z);
            fresh = old == kReachNone;
            pending = !fresh && old != z;
            slot = (slot + 1) % H;
          }
        }
        const uint64_t nb = __builtin_amdgcn_ballot_w64(fresh) & gmask;
        const uint32_t at = cnt + (uint32_t)__popcll(nb & lt);
        if (fresh && at < CAP) ids[at] = z;
        cnt += (uint32_t)__popcll(nb);
        if (cnt > CAP) fail = 1;
      }
    };
    {
      uint32_t e1 = 0;
      if (have) {
        first = R[row];
        e1 = R[(uint64_t)row + 1];
        if (e1 - first > CAP) fail = e1 - first >= a.hub ? 2u : 1u;
      }
      // the row's own edges are distinct: lane l takes edges l, l + G, ...
      for (uint32_t e = first + gl; __builtin_amdgcn_ballot_w64(e < e1 && !fail); e += G)
        expand(e, e < e1 ? e + 1 : e);
    }
    wave_lds_sync();
    // level by level; the counts go out only once the row is done, so the levels' ends and
    // degrees stay in registers of the lanes (level l in lane l % G's slot l / G)
    uint32_t head = 0, end = cnt, levels = 0;
    constexpr int LREG = (int)(CAP / G);
    uint32_t lev_n[LREG], lev_d[LREG];
#pragma unroll
    for (int r = 0; r < LREG; ++r) lev_n[r] = lev_d[r] = 0;
    while (__builtin_amdgcn_ballot_w64(!fail && head < end)) {
      uint32_t dsum = 0;
      const bool act = !fail && head < end;
      const uint32_t lo = act ? head : 0u, hi = act ? end : 0u;
      for (uint32_t f = lo + gl; __builtin_amdgcn_ballot_w64(f < hi && !fail); f += G) {
        uint32_t e0 = 0, e1 = 0;
        if (f < hi && !fail) {
          const uint64_t v = inst | ids[f];
          e0 = R[v];
          e1 = R[v + 1];
          dsum += e1 - e0;
        }
        // a hub sends the whole row on (its edges alone outgrow the tier)
        const uint64_t big = __builtin_amdgcn_ballot_w64(e1 - e0 > CAP) & gmask;
        const uint64_t hub = __builtin_amdgcn_ballot_w64(e1 - e0 >= a.hub) & gmask;
        if (big) fail = hub ? 2u : 1u;
        expand(e0, e1);
        wave_lds_sync();
      }
#pragma unroll
      for (int d = G / 2; d >= 1; d >>= 1) dsum += __shfl_xor(dsum, d, kWave);
      if (act && levels % G == gl) {
#pragma unroll
        for (int r = 0; r < LREG; ++r)
          if ((uint32_t)r == levels / G) {
            lev_n[r] = hi - lo;
            lev_d[r] = dsum;
          }
      }
      if (act) {
        ++levels;
        head = end;
        end = cnt;
      }
    }
    const bool good = have && !fail;
    if (good) {
#pragma unroll
      for (int r = 0; r < LREG; ++r)
        if ((uint32_t)r * G + gl < levels) reach_count(s_lev, a, (uint32_t)r * G + gl, lev_n[r], lev_d[r]);
    }
    // pool entries of the wave's rows, side by side
    const uint32_t mine = good ? cnt : 0u;
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int q = 0; q < (int)PER; ++q) {
      const uint32_t c = __shfl(mine, q * G, kWave);
      before += q < lane / G ? c : 0u;
      total += c;
    }
    if (total > left) {
      uint64_t pos = 0;
      if (lane == 0) pos = reach_alloc(a, kReachChunk);
      chunk = __shfl(pos, 0, kWave);
      left = kReachChunk;
    }
    const bool fits = chunk + total <= a.pool_cap;
    // sorted by counting the smaller ids: every lane ranks its ids against each id of the row
    {
      uint32_t v[LREG], rank[LREG];
#pragma unroll
      for (int r = 0; r < LREG; ++r) {
        const uint32_t x = (uint32_t)r * G + gl;
        v[r] = x < mine ? ids[x] : kReachNone;
        rank[r] = 0;
      }
      for (uint32_t t = 0; t < mine; ++t) {
        const uint32_t y = ids[t];
#pragma unroll
        for (int r = 0; r < LREG; ++r) rank[r] += y < v[r] ? 1u : 0u;
      }
#pragma unroll
      for (int r = 0; r < LREG; ++r)
        if (fits && (uint32_t)r * G + gl < mine) a.pool[chunk + before + rank[r]] = v[r];
    }
    if (good && gl == 0) {
      a.cnt[first] = cnt;
      a.seg[first] = (uint32_t)(chunk + before);
    }
    // rows sent on are buffered per wave (a same-address atomic costs 12 ns)
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      const bool out = have && gl == 0 && fail == (uint32_t)which + 1;
      const uint64_t ob = __builtin_amdgcn_ballot_w64(out);
      if (out) buf[which][fn[which] + (uint32_t)__popcll(ob & lt)] = row;
      fn[which] += (uint32_t)__popcll(ob);
      if (fn[which] > kWave - PER) flush(which);
    }
    chunk += total;
    left -= total;
    wave_lds_sync();
  }
  flush(0);
  flush(1);
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// Edges of the vertices that the lanes of a wave hold, each id through `visit`: short lists by
// their lane, long ones by the whole wave, one after the other.
constexpr uint32_t kReachSerial = 8;
template <typename Visit>
__device__ __forceinline__ void wave_expand(const uint32_t* __restrict__ Edst, uint32_t e0, uint32_t deg, Visit visit) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t d = deg <= kReachSerial ? deg : 0u;
  for (uint32_t j = 0; __builtin_amdgcn_ballot_w64(j < d); ++j) {
    const uint32_t z = j < d ? Edst[e0 + j] : 0u;
    visit(j < d, z);
  }
  for (uint64_t big = __builtin_amdgcn_ballot_w64(deg > kReachSerial); big; big &= big - 1) {
    const int src = __ffsll((unsigned long long)big) - 1;
    const uint32_t b0 = __shfl(e0, src, kWave), bd = __shfl(deg, src, kWave);
    for (uint32_t j = 0; j < bd; j += kWave) {
      const bool on = j + lane < bd;
      const uint32_t z = on ? Edst[b0 + j + lane] : 0u;
      visit(on, z);
    }
  }
}

// ---------------------------------------------------------------------------
// Queue tier: one row per block of NW waves (one wave where the ids' bitmap is at most 8 KB).
// The set is a bitmap of the id space in LDS; an id whose bit a lane sets first goes to the
// next level's queue.  Thin, deep rows (a mesh: two hundred levels of a hundred vertices) pay
// per level one index load, one edge load and one LDS round trip, and up to 32 of them run per
// CU.  A level that outgrows the queue sends the row on.  The ids come out of the bitmap in
// order.
// ---------------------------------------------------------------------------
template <int NW, uint32_t WORDS, uint32_t QCAP, typename ID>
__global__ __launch_bounds__(NW * kWave) void k_reach_queue(ReachArgs a) {
  constexpr uint32_t TH = NW * kWave;
  __shared__ uint32_t s_vis[WORDS];
  __shared__ ID s_front[2][QCAP];
  __shared__ uint32_t s_n[2];
  __shared__ uint32_t s_row, s_d;
  __shared__ uint32_t s_wave[NW];
  __shared__ uint64_t s_pos;
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  __shared__ uint32_t s_ln[kReachLdsLevels], s_ld[kReachLdsLevels];  // the row's levels so far
  const uint32_t tid = threadIdx.x;
  const uint32_t n = a.rc->queued[1];
  if (block_stop(n == 0 || reach_halted(a.rc))) return;
  reach_levels_clear(s_lev);
  const uint32_t words = a.words;
  const int wid = (int)(tid / kWave);
  const int lane = lane_id();
  const uint64_t lt = lanemask_lt();
  const uint32_t* __restrict__ R = a.R;
  const uint32_t* __restrict__ Edst = a.Edst;
  const uint32_t idm = a.w >= 32 ? 0xFFFFFFFFu : (1u << a.w) - 1u;
  uint32_t share = 0;
  for (uint32_t x = tid; x < words; x += TH) s_vis[x] = 0;
  __syncthreads();
  for (;;) {
    if (tid == 0) {
      const uint32_t at = reach_halted(a.rc) ? kReachNone : reach_claim(a.rc, 1, n, share);
      s_row = at == kReachNone ? kReachNone : a.queue[1][at];
      s_n[0] = s_n[1] = 0;
    }
    __syncthreads();
    const uint32_t row = s_row;
    if (row == kReachNone) break;
    const uint32_t inst = row & ~idm;
    const uint32_t first = R[row], deg = R[(uint64_t)row + 1] - first;
    // sets the bit of z; a lane that set it first appends z to queue `to`
    int to = 0;
    auto visit = [&](bool on, uint32_t z) {
      bool fresh = false;
      if (on && !((s_vis[z >> 5] >> (z & 31u)) & 1u))
        fresh = !((atomicOr(&s_vis[z >> 5], 1u << (z & 31u)) >> (z & 31u)) & 1u);
      const uint64_t nb = __builtin_amdgcn_ballot_w64(fresh);
      if (nb) {  // (uniform in the wave)
        uint32_t at = 0;
        if constexpr (NW == 1) {
          at = s_n[to];
          wave_lds_sync();
          if (lane == 0) s_n[to] = at + (uint32_t)__popcll(nb);
          wave_lds_sync();
        } else {
          if (lane == 0) at = atomicAdd(&s_n[to], (uint32_t)__popcll(nb));
          at = __shfl(at, 0, kWave);
        }
        at += (uint32_t)__popcll(nb & lt);
        if (fresh && at < QCAP) s_front[to][at] = (ID)z;
      }
    };
    for (uint32_t j = (uint32_t)wid * kWave; j < deg; j += TH) {
      const bool on = j + lane < deg;
      visit(on, on ? Edst[first + j + lane] : 0u);
    }
    __syncthreads();
    uint32_t lv = 0, cnt = 0;
    bool fail = false;
    for (;;) {
      const int from = to;
      const uint32_t fn = s_n[from];
      cnt += fn;
      if (fn == 0) break;
      if (fn > QCAP) {
        fail = true;
        break;
      }
      to ^= 1;
      __syncthreads();
      if (tid == 0) {
        s_n[to] = 0;
        s_d = 0;
      }
      __syncthreads();
      uint32_t dsum = 0;
      for (uint32_t f = (uint32_t)wid * kWave; f < fn; f += TH) {
        uint32_t e0 = 0, d = 0;
        if (f + lane < fn) {
          const uint64_t v = inst | (uint32_t)s_front[from][f + lane];
          e0 = R[v];
          d = R[v + 1] - e0;
        }
        dsum += d;
        wave_expand(Edst, e0, d, visit);
      }
      if (dsum) atomicAdd(&s_d, dsum);
      __syncthreads();
      // (the row's counts: kept until it is done, or straight to memory once it is deeper than
      // the table, from where on it can no longer be sent back)
      if (tid == 0) {
        if (lv < kReachLdsLevels) {
          s_ln[lv] = fn;
          s_ld[lv] = s_d;
        } else {
          reach_count(s_lev, a, lv, fn, s_d);
        }
      }
      ++lv;
    }
    __syncthreads();
    if (fail && lv > kReachLdsLevels) {
      // counted already: a row this deep whose level outgrows the queue goes to the general path
      if (tid == 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
    } else if (fail) {
      if (tid == 0) {
        const int tier = a.tier_after[2];
        if (tier < 0) atomicOr(&a.rc->stop, (uint32_t)kReachUnsupported);
        else a.queue[tier][atomicAdd(&a.rc->queued[tier], 1u)] = row;
      }
      for (uint32_t x = tid; x < words; x += TH) s_vis[x] = 0;
    } else {
      for (uint32_t x = tid; x < lv && x < kReachLdsLevels; x += TH) reach_count(s_lev, a, x, s_ln[x], s_ld[x]);
      if (tid == 0) {
        const uint64_t pos = reach_alloc(a, cnt);
        s_pos = pos + cnt > a.pool_cap ? ~0ull : pos;
        a.cnt[first] = cnt;
        a.seg[first] = (uint32_t)pos;
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
          for (; bits; bits &= bits - 1) a.pool[pos + at++] = x * 32u + (uint32_t)__ffs(bits) - 1u;
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
// in few words), compact the ids they find into a list of their own and expand it with all
// lanes; an id not in the set has its bit ORed into the next level, which therefore needs no
// dedup at all (a repeated id costs an LDS read and an atomic without return).  Between levels
// one pass joins the next level into the set.  Bound by LDS traffic and instruction issue per
// candidate (a read of the set, an edge from L2); the bitmaps (12 KB at 15 bits) leave eight
// blocks per CU.  The row goes out as its bitmap: 2^w / 8 bytes instead of 4 per tuple.
// ---------------------------------------------------------------------------
constexpr int kReachBitsWaves = 4;
template <uint32_t WORDS, typename ID>
__global__ __launch_bounds__(kReachBitsWaves * kWave) void k_reach_bits(ReachArgs a) {
  constexpr int NW = kReachBitsWaves;
  constexpr uint32_t TH = NW * kWave;
  constexpr uint32_t LCAP = kWave * 16;  // ids of 64 halfwords
  __shared__ uint32_t s_vis[WORDS], s_cur[WORDS], s_nxt[WORDS];
  __shared__ ID s_list[NW][LCAP];
  __shared__ uint32_t s_n[NW];
  __shared__ uint32_t s_row, s_at, s_any[2];
  __shared__ unsigned long long s_lev[kReachLdsLevels][2];
  const uint32_t tid = threadIdx.x;
  const uint32_t n = a.rc->queued[2];
  if (block_stop(n == 0 || reach_halted(a.rc))) return;
  if (n > a.slots) {
    if (tid == 0 && blockIdx.x == 0) atomicOr(&a.rc->stop, (uint32_t)kReachSlotsFull);
    return;
  }
  reach_levels_clear(s_lev);
  const uint32_t words = a.words, halves = words * 2;
  const int wid = (int)(tid / kWave);
  const int lane = lane_id();
  const uint32_t* __restrict__ R = a.R;
  const uint32_t* __restrict__ Edst = a.Edst;
  const uint32_t idm = a.w >= 32 ? 0xFFFFFFFFu : (1u << a.w) - 1u;
  const uint16_t* const cur16 = (const uint16_t*)s_cur;
  ID* const list = s_list[wid];
  uint32_t share = 0;
  __syncthreads();
  for (;;) {
    if (tid == 0) {
      const uint32_t at = reach_halted(a.rc) ? kReachNone : reach_claim(a.rc, 2, n, share);
      s_at = at;
      s_row = at == kReachNone ? kReachNone : a.queue[2][at];
      s_any[0] = 0;
    }
    for (uint32_t x = tid; x < words; x += TH) s_vis[x] = s_cur[x] = s_nxt[x] = 0;
    __syncthreads();
    const uint32_t row = s_row, slot = s_at;
    if (row == kReachNone) break;
    const uint32_t inst = row & ~idm;
    const uint32_t first = R[row], deg = R[(uint64_t)row + 1] - first;
    for (uint32_t j = tid; j < deg; j += TH) {
      const uint32_t z = Edst[first + j];
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
      if (tid == 0) s_any[(lv + 1) & 1u] = 0;
      __syncthreads();
      const uint32_t found = s_any[lv & 1u];
      if (found == 0) break;
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
          uint32_t e0 = 0, d = 0;
          if (f + lane < ln) {
            const uint64_t v = inst | (uint32_t)list[f + lane];
            e0 = R[v];
            d = R[v + 1] - e0;
          }
          dsum += d;
          wave_expand(Edst, e0, d, [&](bool on, uint32_t z) {
            if (on && !((s_vis[z >> 5] >> (z & 31u)) & 1u)) atomicOr(&s_nxt[z >> 5], 1u << (z & 31u));
          });
        }
        wave_lds_sync();
      }
      if (dsum) reach_count(s_lev, a, lv, 0, dsum);
      __syncthreads();
    }
    uint32_t* const out = a.bits + (uint64_t)slot * words;
    for (uint32_t x = tid; x < words; x += TH) out[x] = s_vis[x];
    if (tid == 0) {
      a.cnt[first] = cnt | kReachBitRow;
      a.seg[first] = slot;
    }
    __syncthreads();
  }
  __syncthreads();
  reach_levels_flush(s_lev, a);
}

// ---------------------------------------------------------------------------
// Row offsets: off[i] = tuples of the rows before edge i (off[m] = all), from cnt in two
// launches as every scan here.
// ---------------------------------------------------------------------------
constexpr uint32_t kReachScanTile = kBlock * 8;

__global__ __launch_bounds__(kBlock) void k_reach_sum(const Ctrl* ctrl, ReachArgs a, uint64_t* __restrict__ part) {
  __shared__ uint64_t s_wave[kWavesPerBlock];
  if (block_stop(reach_halted(a.rc))) return;
  uint64_t lo, hi;
  block_range(ctrl->m_unique, kReachScanTile, lo, hi);
  uint64_t sum = 0;
  for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) sum += a.cnt[i] & ~kReachBitRow;
  uint64_t total;
  (void)block_excl_scan<uint64_t>(sum, s_wave, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

template <int SCAN_MAX>
__global__ __launch_bounds__(kBlock) void k_reach_offsets(const Ctrl* ctrl, ReachArgs a,
                                                          const uint64_t* __restrict__ part,
                                                          uint32_t* __restrict__ off) {
  __shared__ uint64_t s_pre[SCAN_MAX];
  __shared__ uint64_t s_wave[kWavesPerBlock];
  if (block_stop(reach_halted(a.rc))) return;
  const uint64_t n = ctrl->m_unique;
  const uint64_t all = block_prefix<SCAN_MAX / kBlock>(part, (int)gridDim.x, s_pre, s_wave);
  uint64_t lo, hi;
  block_range(n, kReachScanTile, lo, hi);
  uint64_t run = s_pre[blockIdx.x];
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
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    off[n] = (uint32_t)all;
    a.rc->edges = n;
  }
}

// ---------------------------------------------------------------------------
// Reading the result.  Rows with an id list: a tile of edges at a time, one output per thread and
// step (its row found by bisection over the tile's list rows in LDS); the tile's ids are
// mostly one stretch of the pool and its outputs one stretch of the result.  Rows with a bitmap:
// a block per row expands 256 words at a time through LDS, so that the writes coalesce.
// put(position, row, id) stores a tuple.
// ---------------------------------------------------------------------------

template <typename K, typename Put>
__device__ __forceinline__ void reach_unpack_lists(const ReachResult& r, const K* __restrict__ E, uint32_t bid,
                                                   uint32_t nblocks, Put put) {
  __shared__ uint32_t s_start[kBlock], s_seg[kBlock], s_off[kBlock], s_row[kBlock];
  __shared__ uint32_t s_wave[kWavesPerBlock];
  const uint32_t tid = threadIdx.x;
  const uint64_t ntiles = (r.m + kBlock - 1) / kBlock;
  for (uint64_t tile = bid; tile < ntiles; tile += nblocks) {
    const uint64_t i = tile * kBlock + tid;
    uint32_t c = 0;
    if (i < r.m) {
      c = r.cnt[i];
      if (c & kReachBitRow) c = 0;
      s_seg[tid] = r.seg[i];
      s_off[tid] = r.off[i];
      s_row[tid] = head_row<K>(E[i], r.w);
    }
    uint32_t total;
    s_start[tid] = block_excl_scan<uint32_t>(c, s_wave, total);
    __syncthreads();
    for (uint32_t t = tid; t < total; t += kBlock) {
      // the last entry starting at or before t (rows without a list share the next start)
      uint32_t lo = 0;
#pragma unroll
      for (uint32_t step = kBlock / 2; step >= 1; step >>= 1) lo = s_start[lo + step] <= t ? lo + step : lo;
      const uint32_t q = t - s_start[lo];
      put((uint64_t)s_off[lo] + q, s_row[lo], r.pool[(uint64_t)s_seg[lo] + q]);
    }
    __syncthreads();
  }
}

template <typename Put>
__device__ __forceinline__ void reach_unpack_bits(const ReachResult& r, uint32_t bid, uint32_t nblocks, Put put) {
  __shared__ uint16_t s_id[kBlock * 32];  // ids relative to the 256 words' first
  __shared__ uint32_t s_wave2[kWavesPerBlock];
  const uint32_t tid = threadIdx.x;
  for (uint64_t k = bid; k < r.n_bits; k += nblocks) {
    const uint32_t row = r.bit_rows[k];
    const uint32_t* __restrict__ b = r.bits + k * r.words;
    uint64_t out = r.off[r.R[row]];
    for (uint32_t x0 = 0; x0 < r.words; x0 += kBlock) {
      uint32_t v = x0 + tid < r.words ? b[x0 + tid] : 0u;
      uint32_t total;
      uint32_t at = block_excl_scan<uint32_t>((uint32_t)__popc(v), s_wave2, total);
      for (; v; v &= v - 1) s_id[at++] = (uint16_t)(tid * 32u + (uint32_t)__ffs(v) - 1u);
      __syncthreads();
      for (uint32_t t = tid; t < total; t += kBlock) put(out + t, row, x0 * 32u + s_id[t]);
      out += total;
      __syncthreads();
    }
  }
}

// Blocks [0, list_blocks) take the rows with lists, the others the bitmaps.
template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_unpack(ReachResult r, const K* __restrict__ E, uint32_t list_blocks,
                                                         uint32_t* __restrict__ src, uint32_t* __restrict__ dst) {
  const uint32_t idm = r.w >= 32 ? 0xFFFFFFFFu : (1u << r.w) - 1u;
  const auto put = [=](uint64_t p, uint32_t row, uint32_t id) {
    src[p] = row & idm;
    dst[p] = id;
  };
  if (blockIdx.x < list_blocks) reach_unpack_lists<K>(r, E, blockIdx.x, list_blocks, put);
  else reach_unpack_bits(r, blockIdx.x - list_blocks, gridDim.x - list_blocks, put);
}

// The same into packed keys (a result that leaves its engine).
template <typename K>
__global__ __launch_bounds__(kBlock) void k_reach_keys(ReachResult r, const K* __restrict__ E, uint32_t list_blocks,
                                                       K* __restrict__ keys) {
  const int w = r.w;
  const auto put = [=](uint64_t p, uint32_t row, uint32_t id) { keys[p] = ((K)row << w) | (K)id; };
  if (blockIdx.x < list_blocks) reach_unpack_lists<K>(r, E, blockIdx.x, list_blocks, put);
  else reach_unpack_bits(r, blockIdx.x - list_blocks, gridDim.x - list_blocks, put);
}

// First tuple of every instance: that of the first edge whose row is instance v's or later.
__global__ __launch_bounds__(kBlock) void k_reach_instances(ReachResult r, uint32_t num, uint64_t* __restrict__ out) {
  for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v <= num; v += (uint64_t)gridDim.x * kBlock)
    out[v] = v == num ? r.off[r.m] : r.off[r.R[v << r.w]];
}

}  // namespace wg
