// Transitive closure one source row at a time (gfx950, wave64).
//
// T(x,z) <- T(x,y), E(y,z) never changes x, so the semi-naive evaluation of Section II splits
// by source row: Delta^i restricted to row x is the set of vertices at distance i + 1 from
// x, its join with E is the expansion of those vertices' edges, and the dedup and the set
// difference against Full are one membership test in the set of vertices row x already
// holds.  A row's whole fixpoint therefore runs in one workgroup (or one wave, or one thread)
// with that set on chip -- no candidate is ever written to memory, sorted or merged, and no
// launch is needed per iteration.  The sizes the loop reports stay those of the iterations:
// |Delta^i| is the number of (row, vertex) pairs found at level i over all rows, and the
// candidates of iteration i + 1 the out-degrees of those vertices, both summed per level.
//
// Rows differ by orders of magnitude, so they go through tiers; a row that outgrows a tier is
// queued for the next one and starts over there (nothing of it has been counted yet):
//   thread  <= 16 tuples: the set in registers                         k_reach_thread
//   group   <= 128 tuples: 16 lanes, a hash set in LDS                 k_reach_group
//   wave    any size, thin levels: a bitmap of the id space and two    k_reach_queue
//           frontier queues in LDS (a block of 16 waves for wide ids)
//   block   any size, wide levels: three bitmaps in LDS                k_reach_bits
// The first three write a row's sorted dst ids to a pool of 32-bit entries, the last writes the
// row's bitmap.  The result stays in that form; reading it unpacks it (k_reach_unpack*).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wg_launch.h"

namespace wg {

constexpr int kReachTiers = 3;              // queues between the tiers: group, queue, bits
constexpr uint32_t kReachThreadCap = 16;    // tuples a thread's row holds
constexpr uint32_t kReachGroupCap = 128;    // ... a 16-lane group's
constexpr uint32_t kReachGroupSlots = 256;  // hash slots of a group (load at most 1/2)
constexpr uint32_t kReachChunk = 4096;      // pool entries a block or wave reserves at a time
constexpr uint32_t kReachLdsLevels = 128;   // levels counted in LDS (deeper ones in memory)
constexpr uint32_t kReachBitRow = 0x80000000u;  // flag in cnt[]: the row is a bitmap
constexpr uint32_t kReachNone = 0xFFFFFFFFu;
constexpr int kReachXcds = 8;

// ReachCtl::stop.  A pool or slots too small leave the counting on (the host then knows what is
// needed and runs the rows again); the others end every kernel at its next look.
enum : uint32_t {
  kReachPoolFull = 1,     // the pool is too small: ids were dropped
  kReachSlotsFull = 2,    // more bitmap rows than slots: the bits tier did not run
  kReachUnsupported = 4,  // a row beyond the tiers this id width has
  kReachDeep = 8,         // more levels than the host allotted
  kReachTooLarge = 16,    // more than 2^32 - 16 tuples
  kReachHalt = kReachUnsupported | kReachDeep | kReachTooLarge,
};
constexpr unsigned long long kReachMaxTuples = 0xFFFFFFF0ull;

struct ReachLevel {
  unsigned long long n;  // tuples found at this level, all rows
  unsigned long long d;  // their out-degrees: the candidates of the next iteration
};

struct ReachCtl {
  uint32_t queued[kReachTiers];  // rows queued for each tier
  uint32_t stop;                 // kReach* bits
  unsigned long long cursor;     // pool entries handed out
  unsigned long long edges;      // distinct edges (for the host, beside the above)
  unsigned long long pad[4];
  uint32_t claim[kReachTiers][kReachXcds][16];  // rows handed out, one counter per XCD (a 64 B line
                                                // each: same-address atomics of all XCDs serialise
                                                // at 12 ns)
};

struct ReachArgs {
  const uint32_t* R;     // dense edge index (row v: edges R[v] .. R[v + 1])
  const uint32_t* Edst;  // dst ids of the sorted, distinct edges
  int w;                 // id bits: row = instance << w | id
  int tier_after[kReachTiers];  // tier a row goes to when it outgrows: the thread, group, queue
                                // tier (0 group, 1 queue, 2 bits, -1 none)
  uint32_t hub;          // a row meeting a vertex of at least this degree skips to `hub_tier`
  int hub_tier;
  uint32_t* cnt;         // per edge: its row's tuples at the row's first edge, 0 elsewhere
  uint32_t* seg;         // per first edge: pool position of the row's ids, or its bitmap's slot
  uint32_t* queue[kReachTiers];
  uint32_t* pool;
  uint64_t pool_cap;
  uint32_t* bits;        // bitmap slots of `words` words
  uint32_t words;
  uint64_t slots;
  ReachCtl* rc;
  ReachLevel* lev;
  uint32_t lev_cap;
};

// A closure in this form, for reading it.
struct ReachResult {
  const uint32_t* cnt;
  const uint32_t* seg;
  const uint32_t* off;
  const uint32_t* R;
  const uint32_t* pool;
  const uint32_t* bits;
  const uint32_t* bit_rows;  // queued rows of the bits tier, slot by slot
  uint32_t n_bits;           // ... how many
  uint32_t words;
  uint64_t m;                // distinct edges
  int w;
};

// Every tier over the m (at most) edges of E, then the row offsets (off: m + 1 entries; part:
// g.scan entries of scratch).  `a` and its buffers are described above.
template <typename K>
void launch_reach(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const ReachArgs& a,
                  uint64_t* part, uint32_t* off);

// The result as src / dst arrays, as packed keys, and the instances' first tuples (num + 1).
template <typename K>
void launch_reach_unpack(hipStream_t s, const Grid& g, const ReachResult& r, const K* E, uint32_t* src,
                         uint32_t* dst);
template <typename K>
void launch_reach_keys(hipStream_t s, const Grid& g, const ReachResult& r, const K* E, K* keys);
void launch_reach_instances(hipStream_t s, const Grid& g, const ReachResult& r, uint32_t num, uint64_t* out);

}  // namespace wg
