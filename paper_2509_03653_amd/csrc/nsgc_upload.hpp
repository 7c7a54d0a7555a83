// Plans to the device (nsgc_upload.hip).
#ifndef NSGC_UPLOAD_HPP_
#define NSGC_UPLOAD_HPP_

#include <hip/hip_runtime.h>

#include <cstddef>

#include "nsgc_plan.h"

namespace nsgc {

// Plans of up to this many bytes travel in kernel arguments.
constexpr size_t kArgPlan = 3840;

// Copies `bytes` (a multiple of 16, at most kArgPlan) from `plan` to the device
// address `dev` and clears the `clear` bytes (a multiple of 16) at `to_clear`.
// `plan` may be reused on return.
hipError_t upload_by_args(const void* plan, size_t bytes, char* dev, char* to_clear, size_t clear, hipStream_t s);
// The same from pinned host memory, which must stay as it is until the stream
// has passed.
hipError_t upload_pinned(const char* stage, size_t bytes, char* dev, char* to_clear, size_t clear, hipStream_t s);
// The same with the sizes the plan's header holds when the kernel runs (at most
// `cap` bytes in all): for a captured graph.
hipError_t upload_captured(const char* stage, char* dev, size_t cap, hipStream_t s);

}  // namespace nsgc

#endif  // NSGC_UPLOAD_HPP_
