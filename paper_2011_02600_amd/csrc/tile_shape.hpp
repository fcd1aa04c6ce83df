// The tile stage kernel's launch shape (no HIP: the host side is also built for
// the CPU alone).
#pragma once

namespace sbp {

// Split of n points into T tiles: the first e0 points, then tiles of p
// points, those after tile thr of p + 1; with last > 0 the last tile holds
// `last` points.
struct TileAxis {
  int n, T, e0, p, thr, last;
#if defined(__HIPCC__)
  __host__ __device__
#endif
  int start(int t) const {
    if (t <= 0) return 0;
    if (t >= T) return n;
    if (t == T - 1 && last > 0) return n - last;
    const int u = t - 1;
    return e0 + u * p + (u > thr ? u - thr : 0);
  }
};

// launch shape of the tile kernel: tiles along q and r, one plane each
struct TileShape {
  TileAxis q, r;
  int ntiles;
  int part;  // nodes computed: 0 all, 1 i < nq-1 and j < nr-ey, 2 the others
};

// largest tile width (q) and height (r); threads per block
constexpr int kTileW = 33, kTileH = 8, kTileNT = 256;

// launch shape for nq x nr x ns points and m closure rows
TileShape tile_shape(int nq, int nr, int ns, int m);

}  // namespace sbp
