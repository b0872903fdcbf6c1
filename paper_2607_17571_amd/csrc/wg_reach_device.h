// Device-side pieces shared by the kernels on the renumbered graph (wg_reach.h, wg_sg.h).
#pragma once

#include <type_traits>

#include "wg_device.h"
#include "wg_reach.h"

// Makes a register's value unknown to the compiler from here on (it would otherwise keep what it
// derives from a loop's invariants in registers of their own).
#ifndef WG_OPAQUE
#define WG_OPAQUE(x) asm volatile("" : "+v"(x))
#endif
// Keeps loads on their side of this point (fewer of them, and of their registers, in flight).
#define WG_FENCE_LOADS asm volatile("" ::: "memory")

namespace wg {

// LDS written by one lane of a wave, read by another: the wave's LDS instructions execute in
// order, so only the compiler must keep them so.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A barrier for what the block's waves hand each other in LDS: loads and stores in flight to memory
// are not waited for.
__device__ __forceinline__ void block_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// v of lane ^ D, D a power of two below 8.
template <int D>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
#ifdef __HIP_DEVICE_COMPILE__
  if constexpr (D == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);  // quads 1 0 3 2
  if constexpr (D == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);  // quads 2 3 0 1
#endif
  return __shfl_xor(v, D, kWave);
}

// The stretch in which n tiles go to the XCDs in turn: `most` tiles at most, as many stretches for each
// (36,000 vertices, 18,256 edges: 63 tiles in stretches of 64, all of them one XCD's, took 326 us a closure,
// 255 so).
__device__ __forceinline__ uint32_t xcd_stretch(uint32_t n, uint32_t most) {
  const uint32_t rounds = (n + kReachXcds * most - 1) / (kReachXcds * most);
  return rounds ? (n + kReachXcds * rounds - 1) / (kReachXcds * rounds) : 1u;
}

// Tile `v` of this block's XCD (blocks go to the XCDs in turn, each with an L2 of its own): stretches of
// C tiles go to the XCDs in turn, so that what neighbouring tiles share is read into one L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t iter, uint32_t C) {
  if (gridDim.x % kReachXcds) return blockIdx.x + iter * gridDim.x;
  const uint32_t x = blockIdx.x % kReachXcds, v = blockIdx.x / kReachXcds + iter * (gridDim.x / kReachXcds);
  return (v / C) * (C * kReachXcds) + x * C + v % C;
}

// A value that every lane holds, in a scalar register.
__device__ __forceinline__ uint32_t wave_uniform(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

__host__ __device__ __forceinline__ uint32_t id_mask(int w) { return w >= 32 ? 0xFFFFFFFFu : (1u << w) - 1u; }

template <typename K>
__device__ __forceinline__ uint32_t col_key(K k, int w) {  // instance << w | dst
  const uint32_t m = id_mask(w);
  return (head_row<K>(k, w) & ~m) | ((uint32_t)k & m);
}

__device__ __forceinline__ uint32_t bits_below(uint32_t v, uint32_t key) {
  return (uint32_t)__popc(v & ((1u << (key & 31u)) - 1u));
}
__device__ __forceinline__ uint32_t rank_col(const RankWord* __restrict__ rank, uint64_t key) {
  const RankWord r = rank[key >> 5];
  return r.colpre + bits_below(r.colbits, (uint32_t)key);
}

// Whether the caller has given up (one thread; then `stop` says so to the others).
__device__ __forceinline__ bool cancelled(const uint32_t* cancel, uint32_t* stop) {
  if (!cancel || __hip_atomic_load(cancel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == 0) return false;
  atomicOr(stop, (uint32_t)kReachCancelled);
  return true;
}

// Edge i's place among the slabs' 1,024 stretches of `per` edges: thread i / per reads its k-th edge
// at k * 1,024 + thread.
__device__ __forceinline__ uint32_t slab_per(uint32_t edges) { return (edges + kSlabThreads - 1) / kSlabThreads; }

}  // namespace wg
