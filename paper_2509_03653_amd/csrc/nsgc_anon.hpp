// Address anonymization (nsgc_anon.hip), host-side launcher.
#ifndef NSGC_ANON_HPP_
#define NSGC_ANON_HPP_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstddef>

namespace nsgc {

// Workspace bytes anonymize needs for n packets (about 36 bytes per packet).
size_t anonymize_bytes(unsigned long long n);

// Lets its kernels use the LDS they need.
hipError_t anonymize_allow_lds();

// Anonymized columns of n packets (n < 2^31) into asrc / adst (device; may be
// src / dst themselves) and the number of unique addresses into *num
// (device).  ws holds anonymize_bytes(n) bytes.  Asynchronous on s.
hipError_t anonymize(const uint32_t* src, const uint32_t* dst, unsigned long long n,
                     unsigned long long seed, uint32_t* asrc, uint32_t* adst,
                     unsigned long long* num, void* ws, hipStream_t s);

}  // namespace nsgc

#endif  // NSGC_ANON_HPP_
