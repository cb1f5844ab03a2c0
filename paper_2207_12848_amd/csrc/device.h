// Device functions that the kernels of several files use.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sweep {

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2 cache: this
// renumbering gives each XCD one contiguous range of the grid, so that the workgroups an
// XCD runs together belong to few units and share those units' arrays in its L2.
__device__ __forceinline__ int xcd_block(int b, int nb) {
  constexpr int kXcd = 8;
  const int per = nb / kXcd, rem = nb % kXcd;
  const int x = b % kXcd;
  return x * per + min(x, rem) + b / kXcd;
}

// Lanes of `m` below this one.
__device__ __forceinline__ int rank_in(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

}  // namespace sweep
