// Same-generation on the renumbered graph (gfx950, wave64).
//
//   SG(x,y) <- E(p,x), E(p,y), x != y.      SG(x,y) <- E(a,x), SG(a,b), E(b,y).
//
// The relation is symmetric, and its semi-naive evaluation (Section VI) is a search over pairs from
// the base pairs: Delta^i are the pairs first found in round i.  Two forms, over the rows and
// columns of wg_reach.h:
//
// Matrices, where much of the pairs' square is reached: Delta and Full as bit matrices over the
// columns, 32 columns of every row to a word, slab by slab.  A round is Delta' = (A^T Delta A) \ Full:
// one launch ORs the rows of Delta into their children's rows (a slab per workgroup, in LDS) and
// writes the product transposed, the next does the same to that -- by symmetry the second factor --
// and takes the difference.  No candidate is formed: two ORs per edge and 32 columns.
//
// Pairs, where few are reached: each unordered pair once in a hash set in memory (both orders are
// counted and, at the end, written); a round expands the pairs found in the last one, a thread
// per candidate, and inserts their children's pairs with a compare-and-swap.  Rounds of a few hundred pairs run
// back to back in one workgroup.  One launch per round where the joins, sorts, differences and
// merges of sorted relations took about twenty.
#pragma once

#include "wg_reach.h"

namespace wg {

// Matrices from one base candidate per this many pairs of columns on (us with the line at 1/16, here,
// 1/4,096: random graph of 6,000 vertices 397 / 400 / 601; R-MAT scale 10 565 / 236 / 230, scale 14
// 337 / 347 / 323).
constexpr uint32_t kSgDense = 256;
// Largest out-degree the pair form takes: a wave expands up to 64 pairs, of at most 4,096 candidates
// each, by itself.
constexpr uint32_t kSgPairDegree = 64;
// Pairs to expand in a round that one workgroup takes alone (6 us for a thin one, 10 us as a launch of
// its own; us a pass on 500,000 vertices / a batch of 256 graphs: 128 pairs 894 / 598, 256 885 / 590,
// 512 876 / 574, 1,024 888 / 584, 2,048 930 / 613).
constexpr uint32_t kSgTail = 512;
// The pairs' cost is their number (0.35 ns each: a compare-and-swap in memory, the list, a sort), the
// iterations' and the matrices' mostly that of their rounds (100 us, 25 to 100).  So the pairs are left, to
// matrices where the columns allow and else to the iterations, once a round finds more than kSgGrowing
// and half as many again as the one before, or more than kSgHeavy (for matrices kSgGrowing) and not
// fewer by 5%; and rounds end early that find more than an eighth of kSgHeavy (kSgGrowing), or than
// twice the last one's, on average up to the next read.  (us, by pairs to the end / by the
// iterations / so: trees of 8 children, 3,000 vertices 3,324 / 791 / 755, 30,000 466,008 / 24,546 / 25,524;
// of 2, 30,000 52,464 / 13,067 / 13,333; random tree of 30,000 17,793 / 7,608 / 8,215; random graph of
// 100,000 vertices with 105,000 edges, 234 rounds, 20,124 / 48,167 / 20,576.)
constexpr uint64_t kSgGrowing = 1u << 17;
constexpr uint64_t kSgHeavy = 1u << 22;
constexpr uint32_t kSgProbes = 128;      // buckets of 4 slots probed before the table counts as full
constexpr uint32_t kSgThreads = 1024;
constexpr uint32_t kSgBuf = 2048;        // new pairs a block buffers
constexpr uint32_t kSgEdgeThreads = 1024;

enum : uint32_t { kSgTableFull = 1, kSgListFull = 2, kSgDeep = 4 };

struct SgLevel {
  unsigned long long n;      // matrices: pairs found in this round, both orders
  unsigned long long c;      // candidates of this round
  unsigned long long found;  // pairs: unordered pairs found (low half), of them to expand (high half)
  uint32_t diag;             // ... of them (x, x)
  uint32_t kstart, fstart;   // ... their stretches of the lists
  uint32_t pad;
};

struct SgCtl {
  unsigned long long base;   // base candidates: sum of deg (deg - 1)
  uint32_t wide;             // an out-degree past kSgPairDegree
  uint32_t pad;
  unsigned long long out;    // keys written by k_sg_emit
  uint32_t stop;             // kSg* bits
  uint32_t next;             // the tail's next round
  uint32_t diagonal;         // matrices: (x, x) tuples dropped
  uint32_t pad2;
};

struct SgArgs {
  ReachGraph g;
  ReachCtl* rc;
  SgCtl* sc;
  SgLevel* lev;
  uint32_t lev_cap;
  const uint32_t* cancel;    // (as for ReachArgs)
  uint4* edge;               // {column, first edge of its row, edges of its row, edges from this one
                             // to the end of its own row}
  // pairs: columns x <= y as x << 32 | y
  unsigned long long* tab;   // hash slots (a power of two), all ones when empty
  uint64_t mask;
  unsigned long long* keys;  // pairs in order of discovery
  uint64_t key_cap;          // ... that are kept: past it the rounds end
  uint4* front;              // ... {first edges of the two rows, edges of each} of those to expand
  uint64_t front_cap;
  // matrices: word [slab * cols + row]
  uint32_t* S;
  uint32_t* D;
  uint32_t* M;
  uint32_t* base_edge;       // row << 16 | column, 1,024 stretches interleaved
  uint32_t* step_edge;       // column of the source (cols: none) << 16 | column
  uint32_t* cdeg;            // out-degree of each column's vertex
};

// The edges' records, base candidates and whether a degree is large, after launch_reach_graph.
template <typename K>
void launch_sg_edges(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const SgArgs& a);

void launch_sg_pairs_base(hipStream_t s, const Grid& g, const Ctrl* ctrl, uint64_t m, const SgArgs& a);
void launch_sg_pairs_round(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t j);
void launch_sg_pairs_tail(hipStream_t s, const SgArgs& a, uint32_t j);
// Both orders of the n pairs found as packed keys (`diagonal` 0: without (x, x)), unsorted.
template <typename K>
void launch_sg_emit(hipStream_t s, const Grid& g, const SgArgs& a, uint64_t n, int diagonal, K* out);

template <typename K>
void launch_sg_matrix_base(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const SgArgs& a,
                           uint32_t slabs);
void launch_sg_matrix_round(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t j, uint32_t slabs);
// Drops (x, x) from S (counted in sc->diagonal).
void launch_sg_matrix_diagonal(hipStream_t s, const Grid& g, const SgArgs& a, uint32_t cols);

}  // namespace wg
