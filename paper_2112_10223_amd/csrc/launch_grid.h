// Grids of launches whose blocks may be too many for one grid dimension: HIP takes fewer
// than 2^32 work-items (blocks times threads) along each.
#pragma once
#include <hip/hip_runtime.h>

namespace spk {

// Blocks of this many threads that one dimension takes.
constexpr long long grid_row(int threads) { return ((1LL << 32) - 1) / threads; }

// At least `blocks` blocks of `threads` threads, in one row as long as they fit.  The kernel
// numbers them with block_number() and leaves those past the end.
inline dim3 grid_rows(long long blocks, int threads) {
  const long long rows = (blocks + grid_row(threads) - 1) / grid_row(threads);
  return rows <= 1 ? dim3((unsigned)blocks) : dim3((unsigned)((blocks + rows - 1) / rows), (unsigned)rows);
}

__device__ __forceinline__ long long block_number() {
  return (long long)blockIdx.y * gridDim.x + blockIdx.x;
}

}  // namespace spk
