// Which launches a grid or a batch of grids takes: rules on sizes, in plain
// C++ (no HIP), so that they can be checked on the CPU alone.
#pragma once

#include <cstddef>
#include <vector>

#include "tile_shape.hpp"

namespace sbp {

// A grid as the rules see it: points, interior order (= closure rows), reach of
// the stencil, bytes per value, bytes of its fields.
struct RouteGrid {
  int nq, nr, ns;
  int order, r, q;
  int es;
  double bytes;
};

// Tile bounds of the stage kernel's march: a balanced split of [0, N) into
// tiles of width <= W whose first and last tile hold at least m points (so that
// SBP closure rows never straddle a tile edge), and one along q into tiles of
// width <= 64 whose starts are multiples of `align` points (128-byte lines).
std::vector<int> tile_bounds(int N, int W, int m);
std::vector<int> tile_bounds_aligned(int N, int align, int m);
// 1 if the edge kernel also takes the last r row (no tile of ty rows is then
// shorter than that)
int edge_row(int nr, int ty);

// Chunks along s of a march over `cols` tiles: the s queues of a chunk start
// with `warm` planes, and the blocks run in waves of one per compute unit; the
// number of chunks that minimises the planes of a unit, waves x (planes + warm).
struct MarchSplit {
  int chunks;
  long long planes;
};
MarchSplit march_split(long long cols, int ns, int warm, int cus);

// Whether a stage of a single grid is faster as one launch of the tile kernel
// than as the march with its edge and penalty launches.
constexpr std::size_t kTileNodes = 1750000;
bool tile_stage(const RouteGrid& g);
// The same for a right-hand side alone, without penalties.
constexpr std::size_t kTileRhsNodes = 4500000;
bool tile_rhs(const RouteGrid& g);

// Estimated us per stage of the tile kernel on one grid of a batch.  Fields above
// kOwnBytes do not stay in the memory-side cache from stage to stage.
constexpr double kOwnBytes = 240e6;
double tile_us(const RouteGrid& g);

// Planes per s-chunk of a batch's work list over `cus` compute units: the length
// that minimises waves of one block per unit times the planes of a block (its
// chunk plus the warm-up planes).
int list_chunk(const std::vector<RouteGrid>& grids, int cus);
// Estimated us per stage of a batch over the work list (no grids: 0; 1e30 if the
// list could be longer than kMaxItems, with chunks of 8 planes, or does not serve
// the orders).
constexpr int kMaxItems = 65536;
double list_us(const std::vector<RouteGrid>& grids);

// Cuts a batch's tile-kernel grids (the bytes of their fields and faces, in the
// order in which they run) into groups; returns the end of each.  A group's grids
// run all their steps before the next group's, in launches they share per order,
// so what they read should stay in the 256 MB memory-side cache from stage to
// stage: at most kGroupBytes, and as few groups as that takes, of like size (one
// grid left over fills the chip worst).
constexpr double kGroupBytes = 250e6;
std::vector<int> tile_groups(const std::vector<double>& bytes);

}  // namespace sbp
