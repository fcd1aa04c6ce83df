// CPU-only check of the rules that choose a grid's and a batch's launches
// (csrc/route.cpp), built by tests/test_route_rules.py.  Prints what fails
// and returns non-zero.
#include <cstdio>
#include <vector>

#include "../../paper_2011_02600_amd/csrc/route.hpp"

using namespace sbp;

static int bad = 0;
static void check(bool ok, const char* what) {
  if (!ok) {
    std::printf("failed: %s\n", what);
    ++bad;
  }
}

// bytes of the fields of an nq x nr x ns grid: rows of nq - 1 nodes in whole
// 128-byte lines, and the last column
static double bytes(int nq, int nr, int ns, int es) {
  const int line = 128 / es;
  return 39.0 * es * ((double)((nq - 1 + line - 1) / line * line) + 1) * nr * ns;
}

// and of its face coefficients, 10 per face node
static double cube(int n, int es) { return bytes(n, n, n, es) + 60.0 * es * n * n; }

static void groups() {
  check(tile_groups({}).empty(), "no grids");
  check(tile_groups({1e9}) == std::vector<int>{1}, "one grid over the limit");
  check(tile_groups({1e9, 1e9, 1e9}) == std::vector<int>({1, 2, 3}), "grids over the limit");
  // 16 and 9 shots of 64^3 (41.5 MB of fields): groups of like size
  check(tile_groups(std::vector<double>(16, cube(64, 4))) == std::vector<int>({4, 8, 12, 16}), "16 of 64^3");
  check(tile_groups(std::vector<double>(9, cube(64, 4))).size() == 2, "9 of 64^3");
  check(tile_groups(std::vector<double>(9, cube(64, 8))).back() == 9, "9 of 64^3 in double precision");
  // padded rows: 40^3 fills 64 of its rows' places
  const std::vector<double> b(47, cube(40, 4));
  for (std::size_t n = 1, i = 0; n <= 64; ++n) {
    // rising sizes
    std::vector<double> v;
    for (i = 0; i < n; ++i) v.push_back(5e6 * (1 + i));
    std::size_t at = 0;
    for (int end : tile_groups(v)) {
      double sum = 0.0;
      check((int)at < end && end <= (int)n, "groups in order, none empty");
      const std::size_t first = at;
      for (; (int)at < end; ++at) sum += v[at];
      check(sum <= kGroupBytes || at == first + 1, "a group of several grids within the limit");
    }
    check(at == n, "every grid in a group");
  }
  std::size_t at = 0;
  for (int end : tile_groups(b)) {
    check((end - at) * b[0] <= kGroupBytes, "47 of 40^3 within the limit");
    at = end;
  }
}

// measured us per stage, tile kernel and march (one GPU, steps with a source)
static void stages() {
  struct Row {
    int es, order, nq, nr, ns;
    double tile, march;
  };
  static const Row rows[] = {
      {4, 2, 97, 97, 97, 33.6, 79.5},      {4, 2, 40, 40, 1000, 155.3, 136.3},  {4, 2, 20, 260, 330, 173.4, 216.7},
      {4, 4, 65, 65, 400, 71.9, 105.6},    {4, 4, 40, 40, 1000, 177.0, 148.8},  {4, 4, 20, 20, 4000, 197.5, 264.5},
      {4, 6, 65, 65, 49, 18.0, 82.0},      {4, 6, 257, 257, 26, 102.8, 119.4},  {4, 6, 40, 40, 1000, 190.0, 161.3},
      {4, 6, 1001, 40, 40, 94.8, 124.9},   {4, 7, 40, 40, 1000, 201.6, 167.7},  {4, 7, 513, 200, 16, 103.0, 143.2},
      {4, 3, 34, 167, 171, 138.8, 112.9},  {4, 5, 34, 180, 180, 173.9, 132.6},  {4, 3, 33, 180, 180, 44.0, 99.8},
      {4, 5, 100, 120, 130, 169.9, 133.3}, {4, 5, 66, 120, 130, 67.2, 127.0},   {4, 6, 130, 130, 100, 138.6, 153.1},
      {4, 3, 40, 160, 160, 74.0, 105.9},   {4, 7, 68, 140, 160, 155.5, 172.2},  {4, 3, 45, 150, 150, 61.5, 95.6},
      {4, 8, 65, 65, 65, 38.2, 93.8},      {4, 8, 97, 97, 97, 95.9, 105.7},     {4, 8, 65, 65, 400, 181.0, 126.9},
      {4, 8, 120, 120, 120, 158.5, 146.0}, {4, 8, 20, 260, 260, 187.5, 249.3},  {4, 8, 40, 40, 1000, 230.9, 184.0},
      {8, 3, 117, 117, 117, 186.2, 231.9}, {8, 6, 120, 120, 120, 247.5, 277.2}, {8, 8, 65, 65, 400, 350.4, 479.0},
  };
  static const int r[9] = {0, 0, 0, 1, 1, 2, 2, 3, 3}, q[9] = {0, 0, 2, 2, 3, 3, 4, 4, 5};
  for (const Row& x : rows) {
    const bool tile = tile_stage({x.nq, x.nr, x.ns, x.order, r[x.order], q[x.order], x.es, bytes(x.nq, x.nr, x.ns, x.es)});
    if (tile != (x.tile < x.march)) {
      std::printf("order %d %d x %d x %d (%d bytes): %s\n", x.order, x.nq, x.nr, x.ns, x.es, tile ? "tile" : "march");
      ++bad;
    }
  }
  check(!tile_stage({130, 130, 104, 6, 2, 4, 8, bytes(130, 130, 104, 8)}), "above the limit");
  // the whole transposed operator, in single precision
  static const Row rhs[] = {
      {4, 8, 65, 65, 1000, 1065.8, 947.6}, {4, 8, 65, 65, 400, 468.7, 442.4},  {4, 8, 40, 40, 2500, 1351.6, 1280.9},
      {4, 8, 257, 257, 60, 833.3, 794.0},  {4, 8, 72, 72, 330, 478.9, 524.4},  {4, 8, 65, 65, 200, 260.9, 272.6},
      {4, 4, 72, 72, 330, 436.4, 480.2},   {4, 2, 40, 40, 1000, 484.4, 505.6}, {4, 6, 33, 33, 1500, 424.4, 483.8},
      {4, 6, 100, 190, 139, 702.7, 674.1}, {4, 8, 103, 153, 209, 930.5, 850.5}, {4, 6, 34, 285, 239, 916.0, 880.8},
      {4, 4, 20, 20, 4000, 646.3, 737.9},  {4, 2, 257, 257, 60, 709.6, 736.6}, {4, 6, 117, 117, 117, 416.3, 426.8},
  };
  for (const Row& x : rhs) {
    const RouteGrid g{x.nq, x.nr, x.ns, x.order, r[x.order], q[x.order], x.es, bytes(x.nq, x.nr, x.ns, x.es)};
    if (tile_rhs(g) != (x.tile < x.march)) {
      std::printf("right-hand side, order %d %d x %d x %d: %s\n", x.order, x.nq, x.nr, x.ns, tile_rhs(g) ? "tile" : "march");
      ++bad;
    }
  }
  check(tile_rhs({129, 129, 129, 6, 2, 4, 4, bytes(129, 129, 129, 4)}), "129^3");
  check(!tile_rhs({129, 129, 129, 6, 2, 4, 8, bytes(129, 129, 129, 8)}), "129^3 in double precision");
  check(!tile_rhs({166, 166, 166, 6, 2, 4, 4, bytes(166, 166, 166, 4)}), "above the right-hand sides' limit");
}

// measured us per stage of k grids in groups of the tile kernel and on the work
// list, where no group keeps their fields in the cache
static void lists() {
  struct Row {
    int es, order, nq, nr, ns, k;
    double tile, list;
  };
  static const Row rows[] = {
      {8, 6, 103, 91, 109, 3, 526, 464},
      {4, 4, 96, 109, 149, 2, 126, 240},
      {8, 6, 109, 98, 89, 4, 620, 537},
      {8, 6, 101, 108, 100, 4, 755, 649},
      {8, 6, 108, 112, 98, 4, 747, 658},
      {8, 4, 133, 173, 32, 4, 312, 569},
      {8, 6, 105, 91, 103, 5, 832, 680},
      {4, 6, 117, 117, 117, 3, 388, 347},
      {8, 6, 117, 117, 117, 3, 715, 607},
      {8, 6, 113, 113, 113, 4, 886, 713},
      {4, 8, 65, 65, 200, 8, 807, 603},
  };
  static const int r[9] = {0, 0, 0, 1, 1, 2, 2, 3, 3}, q[9] = {0, 0, 2, 2, 3, 3, 4, 4, 5};
  for (const Row& x : rows) {
    const RouteGrid g{x.nq, x.nr, x.ns, x.order, r[x.order], q[x.order], x.es, bytes(x.nq, x.nr, x.ns, x.es)};
    if ((x.k * tile_us(g) <= list_us(std::vector<RouteGrid>(x.k, g))) != (x.tile < x.list)) {
      std::printf("%d of %d x %d x %d, order %d (%d bytes): tile %.0f list %.0f\n", x.k, x.nq, x.nr, x.ns, x.order, x.es,
                  x.k * tile_us(g), list_us(std::vector<RouteGrid>(x.k, g)));
      ++bad;
    }
  }
  check(list_us({}) == 0.0, "empty list");
  const RouteGrid thin{4, 106000, 4, 2, 0, 2, 4, bytes(4, 106000, 4, 4)};
  check(list_us({thin, thin, thin, thin}) < 1e30, "a list that fits");
  check(list_us(std::vector<RouteGrid>(5, thin)) == 1e30, "a list that could be too long");
}

int main() {
  groups();
  stages();
  lists();
  std::printf(bad ? "%d failed\n" : "OK\n", bad);
  return bad ? 1 : 0;
}
