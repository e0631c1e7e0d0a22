// Lane masks of one 64-particle chunk of the CIC paints (bit l: lane l), for the device and the
// host compiler.
#pragma once
#include <cstdint>

namespace pmr {

// Key of a lane without a particle. It differs from lane to lane, but on meshes of 2^32 cells in
// all it is also the key of one of the last 64 cells, which the lane below may hold.
constexpr uint32_t empty_lane_key(uint32_t lane) { return 0xffffffffu - lane; }

// Lanes that continue the run of the lane below: the keys agree (`same`) and both lanes hold a
// particle (`ok`).
constexpr uint64_t run_joins(uint64_t same, uint64_t ok) { return same & ok & (ok << 1); }

// The last lane of every run.
constexpr uint64_t run_ends(uint64_t joins, uint64_t ok) { return ok & ~(joins >> 1); }

}  // namespace pmr
