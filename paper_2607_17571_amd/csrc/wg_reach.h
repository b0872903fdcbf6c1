// Transitive closure one source row at a time (gfx950, wave64).
//
// T(x,z) <- T(x,y), E(y,z) never changes x, so the semi-naive evaluation of Section II splits
// by source row: Delta^i restricted to row x is the set of vertices at distance i + 1 from
// x, its join with E is the expansion of those vertices' edges, and the dedup and the set
// difference against Full are one membership test in the set of vertices row x already
// holds.  A row's whole fixpoint therefore runs where that set is on chip -- no candidate is
// ever written to memory, sorted or merged, and no launch is needed per iteration.  The sizes
// the loop reports stay those of the iterations: |Delta^i| is the number of (row, vertex)
// pairs found at level i over all rows, and the candidates of iteration i + 1 the out-degrees of
// those vertices, both summed per level.
//
// The graph is renumbered first: rows are the vertices with out-edges, columns the vertices with
// in-edges, both in id order, so that ids of any width and spread, and the instances of a batch,
// become two dense ranges (a column's rank orders like its id, so sorted output stays sorted).
//
// Two ways to run the rows:
//
// Slabs (k_slab*), where most rows reach much of the graph: a workgroup takes 32 columns and
// holds, for every row, the bits of those columns found at the last level; a level ORs the bits
// of each row's successors.  The columns are independent, so a slab runs to its fixpoint alone.
//
// Tiers, where rows are short and differ by orders of magnitude: a row that outgrows a tier is
// queued for the next one and starts over there (nothing of it has been counted yet):
//   thread  <= 16 tuples: the set in registers                         k_reach_thread
//   groups  <= 64 tuples (4 lanes) and <= 256 (8): a hash set in LDS   k_reach_group
//   thin    (past 131,072 columns) any size, thin levels: two frontier
//           queues in LDS, a bitmap of the columns in memory          k_reach_thin
//   queue   any size, thin levels: a bitmap of the columns and two
//           frontier queues in LDS (one wave, or a block for wide ones) k_reach_queue
//   bits    any size, wide levels: three bitmaps in LDS                k_reach_bits
// All but the last write a row's sorted columns to a pool of 32-bit entries, the last writes the
// row's bitmap.  The result stays in its form; reading it unpacks it.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "wg_launch.h"

namespace wg {

constexpr int kReachTiers = 5;              // queues between the tiers: two groups, thin, queue, bits
constexpr int kThinTier = 2, kQueueTier = 3, kBitsTier = 4;
// The queue tier holds a row's bitmap of all columns in LDS: from this many words on one or two rows
// per CU.  The thin tier then takes the rows first, 24 per CU (ms a closure by the iterations' launches /
// with the queue tier alone / with the thin tier: 1,000 chains of 300 vertices 37.7 / 171 / 18.5, 800 of
// 300 36.2 / 69.5 / 14.9, 100 of 3,000 678 / 1,816 / 110; random graphs of 1,000,000 vertices with
// 950,000 edges 13.6 / 6.0 / 2.8, of 700,000 with 630,000 6.6 / 1.45 / 1.17).  Up to kThinRounds rows
// for each that the queue tier has in flight stay there: a binary tree of 2^18 vertices has 1,023, wide
// ones among them, 1.45 ms so and 1.54 through both.
constexpr uint32_t kThinWords = 4097;
constexpr uint32_t kThinQueue = 512;         // rows queued per level (256 and 1,024 alike)
constexpr uint32_t kThinRounds = 4;
constexpr uint32_t kThinGroups = 1024;       // of 1,024 columns each, 2^20 at most
constexpr uint64_t kThinBytes = 256u << 20;  // bitmaps of all rows in flight, at most
constexpr uint32_t kReachThreadCap = 16;    // tuples a thread's row holds
constexpr uint32_t kReachChunk = 4096;      // pool entries a block or wave reserves at a time
constexpr uint32_t kReachLdsLevels = 128;   // levels counted in LDS (deeper ones in memory)
constexpr uint32_t kReachBitRow = 0x80000000u;  // flag in cnt[]: the row is a bitmap
constexpr uint32_t kReachNone = 0xFFFFFFFFu;
constexpr uint32_t kReachLast = 0x80000000u;  // flag in an edge's column: the last of its row
constexpr int kReachXcds = 8;
// Tiles of 256 rows that go to one XCD together: the instances of a batch lie one after the other, so
// that an XCD's L2 then holds the edges its rows share (256 random graphs, 18 MB of edges: the
// small group tier a tenth less with it, the thread tier 351 -> 331 us).
constexpr uint32_t kReachTileStretch = 64;
constexpr uint32_t kReachQueueStretch = 512;  // queued rows likewise
constexpr uint32_t kReachEdgePad = 8;       // edge records readable past the last

// Fewer rows than this are left to the iterations' launches (TC): a fat row is a serial chain in one
// workgroup, where an iteration's launches spread its candidates over the chip (one vertex with 1,000,000
// leaves 2,118 us against 448, four instances with one row of 100,000 1,177 against 345; down to 180 rows
// the rows are ahead, 171 us against 256).
constexpr uint32_t kReachMinRows = 128;

// Slabs: LDS for two words per row (and one idle row).  32 columns per slab while the rows fit
// at 4 bytes, else 16.
constexpr uint32_t kSlabThreads = 1024;
constexpr uint32_t kSlabLdsWords = 36864;                    // 147,456 bytes
constexpr uint32_t kSlabRows32 = kSlabLdsWords / 2 - 1;      // rows at 32 columns per slab
constexpr uint32_t kSlabRows16 = kSlabLdsWords - 1;          // ... at 16
constexpr uint32_t kSlabEdgeRegs = 32;                       // edges a thread keeps in registers
// Where the host leaves the choice to the device (slab_mode 2), slabs take the rows if half of them
// outgrew the thread tier and the graph goes on: every second row at least has an edge to a vertex with
// edges, and a level over all slabs is at most kSlabLevel word operations (edges x columns / 32, 1.1e12
// a second), or rows reach further on average than to one other and the columns are not mostly leaves.
// (us a closure by the iterations' launches / by slabs / by tiers: 1,000 vertices with 800 leaves each
// 409 / 32,164 / 476, 20,000 with 20 349 / 21,174 / 277, 1,000 with 36 297 / 373 / 247, 30,000 with 17 of
// 60,000 leaves 326 / 4,919 / 303.)
constexpr uint64_t kSlabLevel = 128u << 20;

// ReachCtl::stop.  A pool or slots too small leave the counting on (the host then knows what is
// needed and runs the rows again); the others end every kernel at its next look.
enum : uint32_t {
  kReachPoolFull = 1,     // the pool is too small: ids were dropped
  kReachSlotsFull = 2,    // more bitmap rows than slots: the bits tier did not run
  kReachUnsupported = 4,  // a row beyond the tiers
  kReachDeep = 8,         // more levels than the host allotted
  kReachTooLarge = 16,    // more than 2^32 - 16 tuples
  kReachSlabFull = 32,    // the slabs' bits do not fit their buffer: the slabs did not run
  kReachCancelled = 64,   // the host's word said so (ReachArgs::cancel); so for SgCtl::stop
  kReachHalt = kReachUnsupported | kReachDeep | kReachTooLarge | kReachCancelled,
};
// Rows and slabs, and the tail of same-generation, look at `stop` and the host's word every so many levels
// (a load of 1 to 3 us every 64 levels of 1 us and more), tiers every so many rows or tiles of them: the
// look waits for the atomics on its line (the queue tier of 256 random graphs: every row 322 us, 228 so).
constexpr uint32_t kStopLevels = 64;
constexpr uint32_t kStopRows = 16;
constexpr unsigned long long kReachMaxTuples = 0xFFFFFFF0ull;

struct ReachLevel {          // [0]: by the tiers, [1]: by the slabs
  unsigned long long n[2];  // tuples found at this level, all rows
  unsigned long long d[2];  // their out-degrees: the candidates of the next iteration
};

struct alignas(64) ReachCtl {
  uint32_t queued[kReachTiers];  // rows queued for each tier
  uint32_t stop;                 // kReach* bits
  unsigned long long cursor;     // pool entries handed out
  uint32_t rows, cols, edges;    // of the renumbered graph
  uint32_t slab;                 // the slabs took the rows: columns per slab (32 or 16), else 0
  unsigned long long pad[2];
  uint32_t inner[kReachXcds][16];  // edges to a vertex that has edges, a counter on a line of its own per XCD
  uint32_t claim[kReachTiers][kReachXcds][16];  // rows handed out, one counter per XCD (a 64 B line
                                                // each: same-address atomics of all XCDs serialise
                                                // at 12 ns)
};

static_assert(offsetof(ReachCtl, claim) % 64 == 0 && sizeof(ReachCtl) % 64 == 0, "");

// Where the flags go that are read 16 at a time, behind `head` bytes of control blocks and levels.
constexpr size_t reach_flags_at(size_t head) { return (head + 15) & ~(size_t)15; }

// Ranks of 32 consecutive ids: which are rows and columns, and how many come before them.
struct RankWord {
  uint32_t rowbits, colbits, rowpre, colpre;
};

// The renumbered graph.  Keys are instance << w | id.
struct ReachGraph {
  uint32_t* rowkey;   // key of each row
  uint32_t* rstart;   // first edge of each row, rows + 1 entries
  uint32_t* colkey;   // key of each column
  uint32_t* cstart;   // first edge of the row of each column's vertex, kReachNone without one
  uint2* edge;        // {column | kReachLast, first edge of the column's row or kReachNone}
  uint32_t* slab_edge;  // slabs: row << 16 | successor row, 1,024 stretches interleaved
  uint32_t* slab_col;   // ... their columns
  RankWord* rank;     // by key / 32; one word past the last key
  uint8_t* flags;     // by key: row flags, then column flags (`span` each)
  uint64_t span;      // keys (a multiple of 32)
  uint32_t instances;
  int w;
};

struct ReachArgs {
  ReachGraph g;
  int bits_tier;         // rows that outgrow the queue tier go to the bits tier (else they stop)
  int slab_mode;         // 0: no slabs; 1: slabs; 2: slabs where slab_chosen says so (kSlabLevel)
  uint32_t* cnt;         // per row: its tuples (| kReachBitRow)
  uint32_t* seg;         // per row: pool position of its columns, or its bitmap's slot
  uint32_t* queue[kReachTiers];
  uint32_t* pool;
  uint64_t pool_cap;
  uint32_t* bits;        // bitmap slots of `words` words, or the slabs' bits
  int after_groups;      // the tier the groups send rows on to: kThinTier or kQueueTier
  uint32_t* vis;         // thin tier: a bitmap per wave, all zeros between launches
  uint32_t vis_words;    // ... its words (a multiple of 32)
  uint32_t thin_rows;    // rows up to which it leaves all of them to the queue tier
  uint32_t words;        // words of a row's bitmap: the columns of the widest instance (at most)
  uint64_t slots;
  uint64_t bits_words;   // words of `bits`
  ReachCtl* rc;
  ReachLevel* lev;
  uint32_t lev_cap;
  uint32_t min_rows;     // (kReachMinRows)
  uint32_t square;       // the result's rows are the columns (same-generation)
  const uint32_t* cancel;  // pinned: not 0 once the caller gives up (nullptr: never).  (A kernel on a
                           // stream of its own may be queued behind the very launches it is to end.)
  uint32_t form;         // which of a level's counts the kernel adds to
};

// A closure in this form, for reading it.
struct ReachResult {
  const uint32_t* cnt;
  const uint32_t* seg;
  const uint32_t* off;       // first tuple of every row, rows + 1 entries
  const uint32_t* rowkey;
  const uint32_t* colkey;
  const uint32_t* pool;
  const uint32_t* bits;
  const uint32_t* bit_rows;  // rows of the bits tier, slot by slot
  const RankWord* rank;
  uint32_t n_bits;           // ... how many
  uint32_t words;
  uint32_t rows, cols;
  uint32_t slab;             // columns per slab (bits: slab by slab, a word or halfword per row)
  int w;
};

// Counts the rows of the sorted distinct edges E (at most m) into ctrl->rows.
template <typename K>
void launch_count_rows(hipStream_t s, const Grid& g, Ctrl* ctrl, const K* E, uint64_t m, int w);
// Renumbers the sorted distinct edges E (ctrl->m_unique of them, at most m).
template <typename K>
void launch_reach_graph(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const ReachArgs& a,
                        uint64_t* part);
// Ids too far apart to rank by their value: replaced by their rank among the graph's ids, which keeps
// their order.  keys: the 2 m ids, gathered; sorted by the caller (count: where their number is);
// then the distinct ones into ids (n_ids: how many), and the edges by rank.
void launch_ids_gather(hipStream_t s, const Grid& g, const uint32_t* src, const uint32_t* dst, uint64_t m, uint32_t* keys);
void launch_ids(hipStream_t s, const Grid& g, const uint32_t* sorted, const uint32_t* src, const uint32_t* dst, uint64_t m,
                uint64_t* part, uint32_t* ids, uint32_t* n_ids, uint32_t* src_out, uint32_t* dst_out);
// Back: n ranks in place, and n packed keys of w-bit ranks as keys of ids.
void launch_ids_back(hipStream_t s, const Grid& g, const uint32_t* ids, uint32_t* ranks, uint64_t n);
template <typename K>
void launch_ids_keys(hipStream_t s, const Grid& g, const uint32_t* ids, const K* keys, uint64_t n, int w, int out_w,
                     uint64_t* out);

// Waves of the thin tier, for the bitmaps of `words` words, and the rows up to which it does nothing.
uint32_t thin_waves(const Grid& g, uint32_t words);
uint32_t thin_rows(const Grid& g, uint32_t words);

// The rows, then their offsets (off: rows + 1 entries; part: g.scan entries of scratch).
void launch_reach(hipStream_t s, const Grid& g, uint64_t m, const ReachArgs& a, uint64_t* part, uint32_t* off);

// The offsets of slabs alone (rows: at most m).
void launch_slab_offsets(hipStream_t s, const Grid& g, uint64_t m, const ReachArgs& a, uint64_t* part, uint32_t* off);

// The result (n tuples) as src / dst arrays, as packed keys, and the instances' first tuples (num + 1).
void launch_reach_unpack(hipStream_t s, const Grid& g, const ReachResult& r, uint64_t n, uint32_t* src,
                         uint32_t* dst);
template <typename K>
void launch_reach_keys(hipStream_t s, const Grid& g, const ReachResult& r, uint64_t n, K* keys);
void launch_reach_instances(hipStream_t s, const Grid& g, const ReachResult& r, uint32_t num, uint64_t* out);

}  // namespace wg
