// Which launches a grid or a batch of grids takes: rules on sizes, in plain
// C++ (no HIP), so that they can be checked on the CPU alone.
#pragma once

#include <vector>

namespace sbp {

// Cuts a batch's tile-kernel grids (the bytes of their fields, in the order in
// which they run) into groups; returns the end of each.  A group's grids run
// all their steps before the next group's, in launches they share, so its
// fields should stay in the 256 MB memory-side cache from stage to stage: at
// most kGroupBytes, and as few groups as that takes, of like size (one grid
// left over fills the chip worst).
constexpr double kGroupBytes = 240e6;
std::vector<int> tile_groups(const std::vector<double>& bytes);

}  // namespace sbp
