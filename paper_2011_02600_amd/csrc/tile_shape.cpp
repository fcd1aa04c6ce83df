// Launch shape of the tile kernel.
#include <algorithm>

#include "tile_shape.hpp"

namespace sbp {

namespace {

// tiles along r: at most W rows, balanced, or with full first and last tiles
TileAxis split_r(int n, int W, int m) {
  TileAxis a{};
  a.n = n;
  a.T = (n + W - 1) / W;
  if (a.T <= 1) {
    a.T = 1;
    a.e0 = n;
    return a;
  }
  const int p = n / a.T, r = n % a.T;
  if (p >= m) {  // balanced, the larger tiles last
    a.e0 = a.p = p;
    a.thr = a.T - r - 1;
    return a;
  }
  const int mid = n - 2 * W, tm = a.T - 2;
  a.e0 = W;
  a.p = mid / tm;
  a.thr = tm - mid % tm;
  return a;
}

// tiles along q: 32 columns, so that they start on 128-byte lines; a single
// column past the last joins it (the 2^k + 1 points of refined grids), a few
// columns take 16 from the tile before
TileAxis split_q(int n, int m, bool wide) {
  TileAxis a{};
  a.n = n;
  a.e0 = a.p = 32;
  a.thr = 1 << 30;
  const int r = n % 32;
  a.T = n / 32 + (r ? 1 : 0);
  a.last = n - 32 * (a.T - 1);
  if (a.T > 1 && r == 1 && wide) {
    --a.T;
    a.last = 33;
  } else if (a.T > 1 && r && r < m) {
    a.last = r + 16;
  }
  return a;
}

}  // namespace

// Tiles of 32 columns (or a last one of 33, see tile_kernel) x 8 rows, 7 where
// a tile has 33 columns.  The first and last tile of an axis hold all m
// closure rows of its ends (so order 8, m = 8, takes no tiles of 33).
TileShape tile_shape(int nq, int nr, int ns, int m) {
  TileShape s{};
  s.q = split_q(nq, m, m < kTileH);
  s.r = split_r(nr, s.q.last == kTileW ? kTileH - 1 : kTileH, m);
  s.ntiles = s.q.T * s.r.T * ns;
  return s;
}

}  // namespace sbp
