// Windows that one workgroup takes whole (nsgc_whole.hip).
#ifndef NSGC_WHOLE_HPP_
#define NSGC_WHOLE_HPP_

#include <hip/hip_runtime.h>

#include <cstdint>

#include "nsgc_plan.h"

namespace nsgc {

// which: the size, 0 .. NSGC_WHOLE - 1.
hipError_t launch_whole(const nsgc_dev_plan* P, int which, uint32_t grid, hipStream_t s);
// Whether that many windows can come with the launch instead of a plan, and
// their launch (all of one size).
bool whole_few(size_t windows);
hipError_t launch_whole_few(int which, const nsgc_small_desc* list, size_t windows, const uint32_t* src,
                            const uint32_t* dst, void* out, hipStream_t s);
hipError_t whole_resident_blocks(int which, int* blocks);

}  // namespace nsgc

#endif  // NSGC_WHOLE_HPP_
