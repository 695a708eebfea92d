// Block order over the 8 XCDs.  Included by the HIP kernels only.
#pragma once

#include <hip/hip_runtime.h>

namespace mssa {

// Blocks are dispatched round-robin over the 8 XCDs: block b of n takes work
// item xcd_remap(b, n), so that each XCD has a contiguous eighth of the items
// and its L2 serves few heads.
__device__ inline int xcd_remap(int b, int n) {
  const int q = n / 8, r = n % 8, x = b % 8, j = b / 8;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}

}  // namespace mssa
