// Small device helpers shared by the contraction kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace sht {

// Work item of this workgroup.  The hardware deals workgroups to the 8 XCDs
// round-robin (workgroup b runs on XCD b % 8); work lists hold 8 slices of
// `per` items, one per XCD, so slice x is processed in order on XCD x.
__device__ __forceinline__ int2 take_work(const int2* __restrict__ work, int per) {
  const int slot = (blockIdx.x % 8) * per + blockIdx.x / 8;
  return work[slot];
}

}  // namespace sht

namespace sht {

// Global-memory (address space 1) views of generic pointers: accesses
// through them compile to global_* instead of flat_* instructions, which also
// count against the LDS counter, so that the next wait for LDS waits for them.
typedef __attribute__((address_space(1))) float gfloat;
__device__ __forceinline__ gfloat* as_global(float* p) { return (gfloat*)p; }

// Race-check build (SHT_DEBUG_BARRIERS defined, libsht_debug.so): every
// barrier below first drains all of the wave's memory counters and meets the
// workgroup once more, so no load or store of one stage overlaps another
// stage's work.  Its results must equal the release build's bit for bit; a
// difference points at a missing wait or barrier.
#ifdef SHT_DEBUG_BARRIERS
constexpr bool kDebugBarriers = true;
#else
constexpr bool kDebugBarriers = false;
#endif

__device__ __forceinline__ void debug_drain() {
  if constexpr (kDebugBarriers) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);  // vmcnt, expcnt and lgkmcnt all zero
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// Workgroup barrier for data exchanged through LDS only: the wave waits for
// its own LDS operations (lgkmcnt(0)), then s_barrier.  Unlike
// __syncthreads(), whose release fence also waits for every outstanding
// global load and store (vmcnt(0)), it leaves prefetches in flight.
__device__ __forceinline__ void lds_barrier() {
  debug_drain();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt unconstrained
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

}  // namespace sht
