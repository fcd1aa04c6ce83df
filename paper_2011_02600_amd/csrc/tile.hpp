// The tile stage kernel: launchers.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace sbp {

// mode 0: Runge-Kutta stage; mode 1: the right-hand side into dq alone
template <typename T>
hipError_t launch_tile(int order, int mode, const TileArgs<T>& a, hipStream_t st);
// a stage of several grids of one order: b.first holds the prefix sums of
// their tile counts
template <typename T>
hipError_t launch_tile_batch(int order, const BatchArgs<T, TileArgs<T>>& b, hipStream_t st);
// largest scratch (private segment) size of its kernels, bytes per lane;
// (size_t)-1 if it cannot be queried
template <typename T>
std::size_t tile_scratch(int order);

}  // namespace sbp
