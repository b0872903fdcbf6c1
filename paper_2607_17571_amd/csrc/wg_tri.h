// Triangle counting on the renumbered graph (gfx950, wave64).
//
// The directed triangles E(a,b), E(b,c), E(c,a) come in rotations: one of three distinct edges is
// counted three times.  They are counted at the rotation whose a comes last in the order of
// out-degrees (ties by number): only edges a -> b with b before a ("down") and c -> a with c before a
// ("up") take part, so that hubs are joined with their hub neighbours once and not through every
// leaf.  On a power-law graph of 65,536 vertices that leaves an eighth of the two-paths.  (a, a, a) is no
// rotation of another and is counted by itself.
//
// For each a the vertices c of its up edges are either looked up in the sorted out-edges of each b
// (few pairs (b, c)), or set as bits in LDS against which the out-edges of every b are tested.
#pragma once

#include "wg_reach.h"

namespace wg {

// Pairs (b, c) of a vertex that are looked up; more: bits.  A lookup is a chain of about ten loads
// in one lane, a piece of a row about 5 us of one workgroup.  R-MAT (us a count; 65,536 vertices
// with 524,288 edges / with 100,000 / 8,192 with 60,000): 16 pairs 302 / 220 / 235, 32 302 / 222 /
// 234, 64 302 / 223 / 234, 256 314 / 241 / 254, 1,024 324 / 275 / 266.
constexpr uint32_t kTriPairs = 32;
// Out-edges of a vertex per workgroup with bits: the hubs' 180,000 tests each spread over the chip,
// and few workgroups read the same up edges (64 and 128 alike, 256 2% slower).
constexpr uint32_t kTriPiece = 128;
// Fewer edges are left to the join's launches, which are fewer than the renumbering's (us a count,
// there / here: 9,000 edges 196 / 216, 16,400 204 / 213, 33,000 216 / 217, 60,000 345 / 234,
// 524,288 3,972 / 302).
constexpr uint64_t kTriMinEdges = 32768;
constexpr uint32_t kTriThreads = 512;
constexpr uint32_t kTriWords = 2048;      // words of bits: up to 65,536 columns (8 KB)
constexpr uint32_t kTriWordsWide = 32768;  // ... up to 1,048,576 (128 KB)

struct TriCtl {
  unsigned long long two_paths;  // sum over the edges (a, b) of b's out-degree
  unsigned long long hits;       // rotations found
  unsigned long long up;         // up edges
  uint32_t loops, pieces;
};

struct TriArgs {
  ReachGraph g;
  ReachCtl* rc;
  TriCtl* tc;
  uint4* edge;       // a -> b: {b's column, first edge of b's row, edges of b's row, 1: down}
  uint32_t* col;     // ... b's column alone
  uint32_t* ustart;  // per row: its up edges [ustart, uend) in up order
  uint32_t* uend;
  uint2* piece;      // {row, first edge}, at most rows + edges / kTriPiece
  int w;             // up keys: a's row << w | c's column
};

// The edges' records, counts, and the up edges as keys (unsorted).
template <typename K>
void launch_tri_edges(hipStream_t s, const Grid& g, const Ctrl* ctrl, const K* E, uint64_t m, const TriArgs& a, K* up);
// From the up edges sorted by row: the count.
template <typename K>
void launch_tri_count(hipStream_t s, const Grid& g, uint64_t m, const TriArgs& a, const K* up, bool wide);

}  // namespace wg
