// Large windows on a grid of two levels (nsgc_large_grid.hip).
#ifndef NSGC_LARGE_GRID_HPP_
#define NSGC_LARGE_GRID_HPP_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstddef>

namespace nsgc {

// Persistent grids and table size of the kernels it shares with the grid windows.
struct LargeGridLaunch {
  uint32_t cus, links, wide, rounds, rowcol, sweeps;
  size_t lds_rowcol, lds_sweeps;
  uint32_t rc_slots_log2;
};

// Workspace bytes for a window of n packets, or 0 if the window is outside the
// range this path takes.
size_t large_grid_bytes(unsigned long long n);

// Enqueues the nine statistics of src[0..n), dst[0..n) into out[0..9), whose
// first word carries the invalid mark if a cell or bucket was too crowded.
hipError_t large_grid_stats(const uint32_t* src, const uint32_t* dst, unsigned long long n, void* ws,
                            unsigned long long* out, const LargeGridLaunch& L, hipStream_t s);

// Lets its kernels use up to `bytes` of dynamic LDS.
hipError_t large_grid_allow_lds(size_t bytes);

}  // namespace nsgc

#endif  // NSGC_LARGE_GRID_HPP_
