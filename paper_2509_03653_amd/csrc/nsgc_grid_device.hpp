// Device code shared by the grid windows (nsgc_grid.hip) and the large windows'
// outer cells (nsgc_large_grid.hip).
#ifndef NSGC_GRID_DEVICE_HPP_
#define NSGC_GRID_DEVICE_HPP_

#include "nsgc_device.hpp"
#include "nsgc_plan.h"

namespace nsgc {

// The partition looks dominant ids up in a direct-mapped table of 512 entries
// per view, indexed by nine bits of the hashed id from bit `shift` on; no two
// dominant ids of a view share an entry.  k_grid_heavy picks the shift among
// eight, so that the least frequent addresses are left out.
constexpr uint32_t HT = 512;
constexpr uint32_t HEAVY_SHIFTS = 8;
__device__ __forceinline__ uint32_t heavy_index(uint32_t id, uint32_t shift) { return (id >> shift) & (HT - 1); }

// The distance 1 .. 2^k - 1 (k >= 1) by which a link of a dominant address is
// moved off its home strip, from the other address' hashed id.  It takes bits
// 3 .. 18, which decide neither that address' strip and bucket (top bits) nor,
// with one address fixed, the link's table slot.
__device__ __forceinline__ uint32_t strip_shift(uint32_t other, uint32_t k) {
  return 1u + ((((other >> 3) & 0xFFFFu) * ((1u << k) - 1u)) >> 16);
}

// What entry i of a table holds while it is free: an id that belongs to
// another entry.
__device__ __forceinline__ uint32_t free_entry(uint32_t i, uint32_t shift) { return ((i & (HT - 1)) ^ 1u) << shift; }

// Four consecutive packets at any 4-byte aligned address.
typedef uint32_t v4u32_any __attribute__((ext_vector_type(4), aligned(4)));

}  // namespace nsgc

#endif  // NSGC_GRID_DEVICE_HPP_
