// How a list is dealt to the workgroups of a launch: contiguous ranges.
#ifndef NSGC_RANGES_HPP_
#define NSGC_RANGES_HPP_

#include <stdint.h>

namespace nsgc {

struct ListRange {
  uint64_t beg, end;
};

// Part `part` of `parts` of a list of n elements, in whole steps of `step`
// elements (the last one excepted).  In 64 bits: lists reach 2^32 - 1 elements,
// and rounding such a length up to steps does not fit 32.
constexpr ListRange list_range(uint64_t n, uint32_t step, uint32_t parts, uint32_t part) {
  const uint64_t steps = (n + step - 1) / step, per = (steps + parts - 1) / parts * step;
  const uint64_t beg = part * per < n ? part * per : n;
  return {beg, n - beg < per ? n : beg + per};
}

}  // namespace nsgc

#endif  // NSGC_RANGES_HPP_
