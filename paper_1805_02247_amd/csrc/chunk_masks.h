// Lane masks of one 64-particle chunk of the CIC paints (bit l: lane l), for the device and the
// host compiler.
#pragma once
#include <cstdint>

namespace pmr {

// Lanes that continue the run of the lane below: the keys agree (`same`) and both lanes hold a
// particle (`ok`). A lane without one may carry any key: no key is free to mark it, as the cells
// of a mesh can take all 2^32.
constexpr uint64_t run_joins(uint64_t same, uint64_t ok) {
  return same & (ok & (ok << 1));
}

// The last lane of every run.
constexpr uint64_t run_ends(uint64_t joins, uint64_t ok) { return ok & ~(joins >> 1); }

}  // namespace pmr
