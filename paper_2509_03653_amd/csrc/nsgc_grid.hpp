// Grid windows (nsgc_grid.hip): launchers and shapes of their kernels.
#ifndef NSGC_GRID_HPP_
#define NSGC_GRID_HPP_

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "nsgc_plan.h"

namespace nsgc {

size_t lds_grid_part_bytes(uint32_t tile_log2, uint32_t max_cells);
size_t lds_grid_rc_bytes(uint32_t slots_log2);
size_t lds_grid_sweep_bytes(uint32_t slots_log2);

// Workgroups per compute unit that can be resident.  which: 0 partition (by
// tile_log2), 1 / 2 link aggregation of small / big cells, 3 row/column
// aggregation, 4 that of the entity counts.
hipError_t grid_resident_blocks(int which, uint32_t tile_log2, size_t lds, int* blocks);
hipError_t grid_allow_large_lds(size_t bytes);

hipError_t launch_grid_heavy(const nsgc_dev_plan* P, uint32_t tile_log2, uint32_t grid, hipStream_t s);
hipError_t launch_grid_partition(const nsgc_dev_plan* P, uint32_t tile_log2, uint32_t max_cells,
                                 uint32_t grid, hipStream_t s, bool keys = false);
// keys: the windows' packets are link keys (tiles of 2^14).
// which: 0 windows of small cells, 1 of big cells, 2 what the latter left over
hipError_t launch_grid_links(const nsgc_dev_plan* P, int which, uint32_t grid, hipStream_t s);
hipError_t launch_grid_rounds(const nsgc_dev_plan* P, bool after_wide, uint32_t grid, hipStream_t s);
hipError_t launch_grid_rowcol(const nsgc_dev_plan* P, uint32_t grid, size_t lds, hipStream_t s);
// k_finish (nsgc_kernels.hip) of a plan of one grid window.
hipError_t launch_grid_finish(const nsgc_dev_plan* P, hipStream_t s);
// Instead of the row/column aggregation and its sweeps, for entity counts.
hipError_t launch_grid_ent(const nsgc_dev_plan* P, uint32_t grid, hipStream_t s);
hipError_t launch_grid_sweeps(const nsgc_dev_plan* P, uint32_t grid, size_t lds, hipStream_t s);

}  // namespace nsgc

#endif  // NSGC_GRID_HPP_
