// What the row kernels share: workgroup shape, row cache sizes, the work counter.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/saki.h"
#include "row_engine.hpp"

namespace saki {

constexpr int NT = 256;
constexpr int WG_PER_CU = 2;
// bf16 rows of up to CACHED_MAXC chunks (262,144 entries) use the variant with
// a row cache of CACHE_KC chunks per wave: 4 KiB of chunk masses and 64 KiB of
// cached chunks per workgroup, two workgroups in the 160 KiB of LDS of a CU.
// The cached chunks are read once per row instead of three times.
constexpr int CACHED_MAXC = 256;
constexpr int CACHE_KC = 4;
template <int KC>
using RowSharedK = RowShared<NT, (KC > 0 ? CACHED_MAXC : MAX_CHUNKS), KC>;

__device__ __forceinline__ float nanf_() { return __builtin_nanf(""); }

// The next index from a work counter in device memory (a global atomic: the
// pointer's address space spares the check that a flat one needs).
template <typename C>
__device__ __forceinline__ C take_index(C* counter) {
  return __hip_atomic_fetch_add((__attribute__((address_space(1))) C*)counter, C{1}, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

// Takes the next work item (row or block) for the whole workgroup: thread 0
// takes it from the counter with a device atomic and posts it in LDS, and
// readfirstlane makes the index, and so the caller's loop exit, uniform in
// every wave, so all threads reach the same barriers.
__device__ __forceinline__ unsigned int take_next(unsigned int* counter, unsigned int* slot) {
  if (threadIdx.x == 0) *slot = take_index(counter);
  __syncthreads();
  const unsigned int v = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(*slot)));
  __syncthreads();
  return v;
}

// The kernel's only argument, read where it is used: the pointer is opaque to
// the compiler at each call, so fields are loaded again (from the scalar cache)
// instead of being held in scalar registers across the sweeps, where 30 pointers
// spill into lanes of vector registers and every row pays for reading them back.
template <typename S>
__device__ __forceinline__ const __attribute__((address_space(4))) S* kernel_args() {
  auto p = (const __attribute__((address_space(4))) S*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// A condition that every lane of a wave computes alike (from LDS or uniform
// data), as one the compiler knows to be uniform: a branch on it that leaves or
// restarts a loop with barriers is then a scalar branch, never a masked one.
__device__ __forceinline__ bool uniform(bool c) { return __builtin_amdgcn_readfirstlane(c ? 1 : 0) != 0; }

}  // namespace saki
