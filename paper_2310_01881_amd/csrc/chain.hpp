// chain.hpp -- single-pass prefix sums across the blocks of one launch (chained scan with
// look-back; Merrill and Garland, "Single-pass parallel prefix scan with decoupled look-back",
// 2016): every block publishes the sum of its own part, adds up what the blocks before it have
// published, and publishes the total up to and including itself.
//
// Blocks take their number from a ticket when they start, so every block that a block waits
// for is already running and publishes its own sum without waiting for anyone: the wait
// always ends.  A state word holds the value and its status together and is read and written
// with device-scope atomics, so nothing else has to be ordered between blocks (which sit
// behind different L2 caches).  The words and the ticket must be zero before the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace amn {

constexpr uint64_t kChainSum = 1ull << 62;      // the block's own sum
constexpr uint64_t kChainPrefix = 2ull << 62;   // the sum of all blocks up to this one
constexpr uint64_t kChainValue = kChainSum - 1; // values stay below 2^62

// The next block number of this launch (one thread of the block calls it).
__device__ __forceinline__ uint32_t chain_ticket(uint64_t* ticket) {
  return (uint32_t)__hip_atomic_fetch_add(ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Called by one whole wave of block `blk`, `sum` being the block's own sum in every lane:
// the sum of all blocks before it.  64 predecessors are looked at per step.
__device__ __forceinline__ uint64_t chain_prefix(uint64_t* state, uint32_t blk, uint64_t sum, int lane) {
  if (lane == 0)
    __hip_atomic_store(&state[blk], (blk == 0 ? kChainPrefix : kChainSum) | sum, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (blk == 0) return 0;
  uint64_t before = 0;
  int64_t at = (int64_t)blk - 1;
  while (true) {
    const int64_t i = at - lane;
    uint64_t s = i >= 0 ? 0ull : kChainPrefix;
    uint64_t full, need;
    while (true) {
      if ((s >> 62) == 0u) s = __hip_atomic_load(&state[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      full = __ballot((s >> 62) == 2u);
      // lanes up to the nearest block whose prefix is known (all 64 if there is none)
      need = full ? (((full & (~full + 1ull)) << 1) - 1ull) : ~0ull;
      if ((__ballot((s >> 62) == 0u) & need) == 0) break;
      __builtin_amdgcn_s_sleep(2);
    }
    before += wave_sum_u64((need >> lane) & 1ull ? s & kChainValue : 0ull);
    if (full) break;
    at -= 64;
  }
  if (lane == 0)
    __hip_atomic_store(&state[blk], kChainPrefix | (before + sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return before;
}

}  // namespace amn
