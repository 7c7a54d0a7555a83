// Plans to the device by kernel: in the arguments of a launch up to 3840 bytes,
// read from pinned host memory above (one trip over the link, every unit by a
// thread of its own).  A copy by the runtime in front of a call's kernels held
// them up by 5 to 10 us: one window of 8000 packets 33 us with it and 23
// without, 2000 windows of up to 1500 packets 44 and 30, nine windows of up to
// 2^22 packets 183 and 171, a graph of one window 36 and 29.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "nsgc_device.hpp"
#include "nsgc_upload.hpp"

namespace nsgc {

namespace {

constexpr uint32_t UT = 256;

struct ArgPlan {
  v4u32* dev;
  v4u32* to_clear;
  uint32_t n, clear;
  uint32_t pad[2];
  v4u32 words[kArgPlan / 16];
};
static_assert(sizeof(ArgPlan) <= 3968, "kernel arguments");

__global__ __launch_bounds__(UT) void k_upload_args(ArgPlan) {
  // (the arguments where they lie: indexed, they would be copied first)
  const ArgPlan* A = (const ArgPlan*)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t i = threadIdx.x;
  if (i < A->n) gptr(A->dev)[i] = A->words[i];
  const v4u32 z = {0u, 0u, 0u, 0u};
  for (uint32_t k = i; k < A->clear; k += UT) gptr(A->to_clear)[k] = z;
}
static_assert(kArgPlan / 16 <= UT, "one pass");

__global__ __launch_bounds__(UT) void k_upload(const v4u32* stage, v4u32* dev, uint32_t n, v4u32* to_clear,
                                               uint32_t clear) {
  const v4u32 z = {0u, 0u, 0u, 0u};
  for (uint32_t i = blockIdx.x * UT + threadIdx.x; i < n; i += gridDim.x * UT) gptr(dev)[i] = gptr(stage)[i];
  for (uint32_t i = blockIdx.x * UT + threadIdx.x; i < clear; i += gridDim.x * UT) gptr(to_clear)[i] = z;
}

// The sizes are read with the first units: one trip to host memory.
__global__ __launch_bounds__(UT) void k_upload_captured(const v4u32* stage, v4u32* dev, uint32_t cap) {
  const uint32_t i0 = blockIdx.x * UT + threadIdx.x;
  const nsgc_dev_plan* H = reinterpret_cast<const nsgc_dev_plan*>(stage);
  const v4u32 first = gptr(stage)[min(i0, cap - 1u)];
  const uint32_t n = gptr(&H->upload16)[0], clear = gptr(&H->clear16)[0];
  if (i0 < n) gptr(dev)[i0] = first;
  for (uint32_t i = i0 + gridDim.x * UT; i < n; i += gridDim.x * UT) gptr(dev)[i] = gptr(stage)[i];
  const v4u32 z = {0u, 0u, 0u, 0u};
  for (uint32_t i = i0; i < clear; i += gridDim.x * UT) gptr(dev)[n + i] = z;
}

}  // namespace

hipError_t upload_by_args(const void* plan, size_t bytes, char* dev, char* to_clear, size_t clear,
                          hipStream_t s) {
  ArgPlan a;
  a.dev = reinterpret_cast<v4u32*>(dev);
  a.to_clear = reinterpret_cast<v4u32*>(to_clear);
  a.n = uint32_t(bytes / 16);
  a.clear = uint32_t(clear / 16);
  std::memcpy(a.words, plan, bytes);
  hipLaunchKernelGGL(k_upload_args, dim3(1), dim3(UT), 0, s, a);
  return hipGetLastError();
}

hipError_t upload_pinned(const char* stage, size_t bytes, char* dev, char* to_clear, size_t clear,
                         hipStream_t s) {
  const uint32_t n = uint32_t(bytes / 16), c = uint32_t(clear / 16);
  const uint32_t grid = std::min<uint32_t>((std::max(n, c) + UT - 1) / UT, 256);
  hipLaunchKernelGGL(k_upload, dim3(std::max(grid, 1u)), dim3(UT), 0, s,
                     reinterpret_cast<const v4u32*>(stage), reinterpret_cast<v4u32*>(dev), n,
                     reinterpret_cast<v4u32*>(to_clear), c);
  return hipGetLastError();
}

hipError_t upload_captured(const char* stage, char* dev, size_t cap, hipStream_t s) {
  const uint32_t units = uint32_t(cap / 16);
  hipLaunchKernelGGL(k_upload_captured, dim3(std::min<uint32_t>((units + UT - 1) / UT, 64)), dim3(UT), 0, s,
                     reinterpret_cast<const v4u32*>(stage), reinterpret_cast<v4u32*>(dev), units);
  return hipGetLastError();
}

}  // namespace nsgc
