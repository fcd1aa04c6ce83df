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

static void groups() {
  check(tile_groups({}).empty(), "no grids");
  check(tile_groups({1e9}) == std::vector<int>{1}, "one grid over the limit");
  check(tile_groups({1e9, 1e9, 1e9}) == std::vector<int>({1, 2, 3}), "grids over the limit");
  // 16 and 9 shots of 64^3: groups of like size
  check(tile_groups(std::vector<double>(16, bytes(64, 64, 64, 4))) == std::vector<int>({4, 8, 12, 16}), "16 of 64^3");
  check(tile_groups(std::vector<double>(9, bytes(64, 64, 64, 4))).size() == 2, "9 of 64^3");
  check(tile_groups(std::vector<double>(9, bytes(64, 64, 64, 8))).back() == 9, "9 of 64^3 in double precision");
  // padded rows: 40^3 fills 64 of its rows' places
  const std::vector<double> b(47, bytes(40, 40, 40, 4));
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

int main() {
  groups();
  std::printf(bad ? "%d failed\n" : "OK\n", bad);
  return bad ? 1 : 0;
}
