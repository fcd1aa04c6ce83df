#include "route.hpp"

#include <algorithm>
#include <functional>

namespace sbp {

std::vector<int> tile_bounds(int N, int W, int m) {
  std::vector<int> b;
  if (N <= W) return {0, N};
  int T = (N + W - 1) / W;
  for (int t = 0; t <= T; ++t) b.push_back((int)((long long)t * N / T));
  if (b[1] - b[0] >= m && b[T] - b[T - 1] >= m) return b;
  // fall back: full first and last tiles, balanced middle
  b.assign(1, 0);
  b.push_back(W);
  const int mid = N - 2 * W;
  if (mid > 0) {
    const int Tm = (mid + W - 1) / W;
    for (int t = 1; t <= Tm; ++t) b.push_back(W + (int)((long long)t * mid / Tm));
  }
  if (b.back() != N - W) b.push_back(N - W);
  b.push_back(N);
  return b;
}

std::vector<int> tile_bounds_aligned(int N, int align, int m) {
  std::vector<int> b{0};
  while (N - b.back() > 64) b.push_back(b.back() + 64);
  b.push_back(N);
  // a last tile narrower than m: move its start back by one line at a time
  while (b.size() > 2 && b[b.size() - 1] - b[b.size() - 2] < m) {
    const int s = b[b.size() - 2] - align;
    if (s <= b[b.size() - 3]) break;
    b[b.size() - 2] = s;
  }
  bool ok = b.size() >= 2;
  for (std::size_t t = 0; t + 1 < b.size(); ++t) ok = ok && b[t + 1] - b[t] <= 64 && b[t + 1] > b[t];
  ok = ok && (b.size() == 2 || (b[1] - b[0] >= m && b[b.size() - 1] - b[b.size() - 2] >= m));
  return ok ? b : tile_bounds(N, 64, m);
}

int edge_row(int nr, int ty) { return (nr - 1) % ty == 0 && nr - 1 >= 2 * ty ? 1 : 0; }

MarchSplit march_split(long long cols, int ns, int warm, int cus) {
  MarchSplit best{1, -1};
  for (int nz = 1; nz <= std::max(1, ns / 8); ++nz) {
    const long long waves = (cols * nz + cus - 1) / cus;
    const long long planes = waves * ((ns + nz - 1) / nz + warm);
    if (best.planes < 0 || planes < best.planes) best = {nz, planes};
  }
  return best;
}

// tiles of the stage kernel's march, 8 rows high, per plane
static long long march_cols(const RouteGrid& g) {
  return (long long)(tile_bounds_aligned(g.nq - 1, 128 / g.es, g.order).size() - 1) *
         (long long)(tile_bounds(g.nr - edge_row(g.nr, 8), 8, g.order).size() - 1);
}

// What the estimates below depend on: millions of lanes of the tile kernel's
// tiles, used or not; millions of elements of a field with its padded rows;
// whether rows of 64, 128 or 256 elements keep whole fields on few memory
// channels, and whether the tiles then also start inside a line (a last tile of
// 16 + r columns for r < m left over; not where one column more joins it).
struct RouteSize {
  double lanes, padded;
  bool even, split;
  long long planes;  // of the march, per compute unit
};
static RouteSize route_size(const RouteGrid& g) {
  RouteSize z;
  const TileShape t = tile_shape(g.nq, g.nr, g.ns, g.order);
  const int line = 128 / g.es, pitch = (g.nq - 1 + line - 1) / line * line;
  z.lanes = 1e-6 * kTileNT * t.ntiles;
  z.padded = 1e-6 * (pitch + 1.0) * g.nr * g.ns;
  z.even = (pitch == 64 || pitch == 128 || pitch == 256) && t.q.last != kTileW;
  z.split = z.even && t.q.T > 1 && g.nq % 32 && g.nq % 32 < g.order;
  z.planes = march_split(march_cols(g), g.ns, g.r + g.q + 1, 256).planes;
  return z;
}

// The tile kernel reads the planes around a node again for every node, which
// costs little while the caches hold them; the march reads them once, in a chain
// of planes whose latency small grids cannot hide.  Near-cubic grids meet
// between 1.6 and 2.1 million nodes (us per stage, tile and march: order 6
// single 1.44e6 nodes 96 and 120, 2.15e6 141 and 136; double 1.44e6 214 and 231,
// 2.15e6 311 and 298).  Below that the shape decides in single precision.  The
// tile kernel's time goes with its lanes while the fields fit the memory-side
// cache, else with their padded bytes, more of them on rows of 64 and 128
// elements; the march's with the planes of a compute unit, the bytes and the
// faces.  The constants (us) are fitted to 306 grids of 2e4 to 1.75e6 nodes, orders
// 2 to 8, where the rule is more than 1 % slower than the march on one (6 %, order
// 8 at 1001 x 40 x 40) and gives away at most 7 % of the tile kernel's gains; by
// nodes alone the tile kernel was slower on 60, by up to 43 % (order 8 at 65 x 65 x
// 400 181 and 127 us, order 5 at 100 x 120 x 130 170 and 133, order 3 at 34 x 167 x
// 171 139 and 113).  In double precision, where the march has two more launches
// and is bound by its registers, the tile kernel is ahead on 200 of 203 grids and
// at most 3 % behind (order 6 at 65 x 65 x 400: 262 and 253 us).
bool tile_stage(const RouteGrid& g) {
  if ((std::size_t)g.nq * g.nr * g.ns > kTileNodes) return false;
  if (g.es == 8) return true;
  const RouteSize z = route_size(g);
  const int o = g.order, o8 = o == 8;
  const double out = std::min(1.0, std::max(0.0, (g.bytes - 255e6) / 30e6));  // share beyond the cache
  const double tile = 11.0 + (1.0 - out) * (15.9 + 4.2 * o + 17.6 * o8) * z.lanes +
                      out * (42.0 + 3.3 * o + 10.7 * o8 + 6.6 * z.even + 13.9 * z.split) * z.padded;
  const double march = 18.6 + (3.3 + 0.07 * o) * z.planes + 13.8 * z.padded + 7.8e-5 * g.nq * (g.nr + g.ns);
  return tile <= march;
}

// A right-hand side stores 9 words per node fewer than a stage, which the march,
// bound by its chain, gains nothing from: in single precision the tile kernel is
// ahead up to some 4.5 million nodes (order 6: 2.15e6 nodes 119 and 136 us, 4.17e6
// 43 us less than the march with its edge launch, 7.19e6 13 us more), except on
// many shapes at order 8, whose tiles leave lanes idle, and on rows of 64 and 128
// elements (whole transposed operator, us: order 8 at 65 x 65 x 1000 1066 and 948,
// at 257 x 257 x 60 833 and 794, at 72 x 72 x 330 479 and 524; order 6 at 100 x 190 x
// 139 703 and 674).  The constants are fitted to 198 grids of up to 4.5e6 nodes,
// orders 2 to 8; the rule costs at most 3 % against the better of both.  In double
// precision both take turns above kTileNodes.
bool tile_rhs(const RouteGrid& g) {
  if (g.es == 8) return tile_stage(g);
  if ((std::size_t)g.nq * g.nr * g.ns > kTileRhsNodes) return false;
  const RouteSize z = route_size(g);
  const int o8 = g.order == 8;
  return (1.5 + 1.6 * g.order - 12.0 * o8 + 4.1 * z.even + 8.4 * z.split) * z.padded + (14.7 + 14.0 * o8) * z.lanes <=
         13.3 + 3.0 * z.planes - 1.1e-4 * g.nr * g.ns;
}

double tile_us(const RouteGrid& g) {
  static const double rate[2][2][7] = {{{36, 36, 42, 45, 48, 55, 80}, {58, 60, 64, 67, 70, 74, 85}},
                                       {{82, 82, 90, 103, 112, 120, 130}, {99, 105, 109, 114, 130, 130, 142}}};
  return rate[g.es == 8][g.bytes > kOwnBytes][g.order - 2] * 1e-6 * kTileNT *
         tile_shape(g.nq, g.nr, g.ns, g.order).ntiles;
}

int list_chunk(const std::vector<RouteGrid>& grids, int cus) {
  int nsmax = 0;
  std::vector<long long> cols;
  for (const RouteGrid& g : grids) {
    nsmax = std::max(nsmax, g.ns);
    cols.push_back(march_cols(g));
  }
  long long best = -1;
  int bestL = nsmax;
  for (int L = nsmax; L >= 8; L = L * 3 / 4) {
    long long tiles = 0, planes = 0;
    for (std::size_t i = 0; i < grids.size(); ++i) {
      const RouteGrid& g = grids[i];
      const int Lg = std::min(L, g.ns), nz = (g.ns + Lg - 1) / Lg;
      tiles += cols[i] * nz;
      planes = std::max<long long>(planes, (g.ns + nz - 1) / nz + g.r + g.q + 1);
    }
    const long long cost = (tiles + cus - 1) / cus * planes;
    if (best < 0 || cost < best) {
      best = cost;
      bestL = L;
    }
  }
  return bestL;
}

// The list's blocks in the order in which the launch takes them: 8 segments of
// equal cost (grids largest first), one per XCD, whose 32 compute units take
// each the next longest block; an edge block counts as 4 planes.  The time is
// that of the last unit, at rates fitted to 80 batches, most of two to five
// grids whose fields do not fit the cache: there the list was from 1.34 times
// as fast as the tile kernel to 1.9 times as slow.  Choosing by the estimates
// costs 0.5 % on average against the better of both (always the tile kernel
// 2.4 %; us per stage, tile kernel and list: 3 of 117^3, order 6, single 388 and
// 347, double 715 and 607; 8 of 65 x 65 x 200, order 8, single 807 and 603).  With
// orders that take launches per order instead of the list (7 and 8 in double
// precision) the tile kernel was ahead throughout, by 1.1 to 3 times.
double list_us(const std::vector<RouteGrid>& grids) {
  if (grids.empty()) return 0.0;
  int order = 0;
  std::vector<RouteGrid> by = grids;
  std::stable_sort(by.begin(), by.end(), [](const RouteGrid& a, const RouteGrid& b) {
    return (long long)a.nq * a.nr * a.ns > (long long)b.nq * b.nr * b.ns;
  });
  const int L = list_chunk(grids, 256);
  struct Run {  // `n` blocks of `planes` planes
    long long n;
    int planes;
  };
  std::vector<Run> runs;
  long long total = 0, items = 0;
  for (const RouteGrid& g : by) {
    order = std::max(order, g.order);
    const int Lg = std::min(L, g.ns), nz = (g.ns + Lg - 1) / Lg;
    const int edge = (g.nr + 63) / 64 + (edge_row(g.nr, 8) ? (g.nq - 1 + 63) / 64 : 0);
    runs.push_back({march_cols(g) * nz, (g.ns + nz - 1) / nz + g.r + g.q + 1});
    runs.push_back({(long long)edge * ((g.ns + 7) / 8), 4});
    items += (march_cols(g) + edge) * ((g.ns + 7) / 8);
    for (std::size_t i = runs.size() - 2; i < runs.size(); ++i) total += runs[i].n * runs[i].planes;
  }
  if (items > kMaxItems || (grids[0].es == 8 && order >= 7)) return 1e30;
  long long last = 0, acc = 0;
  std::size_t at = 0;
  for (int x = 0; x < 8; ++x) {
    std::vector<Run> part;
    for (const long long goal = total * (x + 1) / 8; at < runs.size() && acc < goal;) {
      const long long n = std::min(runs[at].n, (goal - acc + runs[at].planes - 1) / runs[at].planes);
      part.push_back({n, runs[at].planes});
      acc += n * runs[at].planes;
      if ((runs[at].n -= n) == 0) ++at;
    }
    std::stable_sort(part.begin(), part.end(), [](const Run& a, const Run& b) { return a.planes > b.planes; });
    std::vector<long long> unit(32, 0);  // a heap, the earliest first
    for (const Run& r : part)
      for (long long i = 0; i < r.n; ++i) {
        std::pop_heap(unit.begin(), unit.end(), std::greater<long long>());
        unit.back() += r.planes;
        std::push_heap(unit.begin(), unit.end(), std::greater<long long>());
      }
    last = std::max(last, *std::max_element(unit.begin(), unit.end()));
  }
  return grids[0].es == 8 ? 150.0 + 8.0 * last : (order == 8 ? 150.0 + 6.6 * last : 60.0 + 5.1 * last);
}

// us per stage of 16 shots of 64^3, order 4 (43 MB each in single precision),
// with the work list and in groups of 1, 2, 3, 4, 6, 8 and 16: single
// precision 289, and 355, 286, 258, 233, 258, 294, 288; double 562, and 570,
// 476, 469, 538, 532, 520, 507.  The bytes are those of the padded rows and the
// face coefficients: counted by nodes, groups of grids whose rows fill their lines
// badly leave the cache (47 of 40^3, order 4: 337 us, 278 in groups of the right
// size, 327 with the work list; 31 of 34 x 101 x 29, order 6: 516, 415 and 431).
// 250 MB in groups of like size, by order: over 112 batches of one shape 2.6 % and
// over 53 uneven ones 3.7 % less time than 1.28 million nodes a group by size,
// none slower by more than 2 %; 240 MB of fields by size were 13 % slower on a
// batch that just exceeds them.
std::vector<int> tile_groups(const std::vector<double>& bytes) {
  double left = 0.0, sum = 0.0;
  int groups = bytes.empty() ? 0 : 1;
  for (double b : bytes) {
    left += b;
    if (sum > 0.0 && sum + b > kGroupBytes) {
      ++groups;
      sum = 0.0;
    }
    sum += b;
  }
  std::vector<int> end;
  sum = 0.0;
  for (int i = 0; i < (int)bytes.size(); ++i) {
    // (left: the bytes from this group's first grid on)
    if (sum > 0.0 && (sum + bytes[i] > kGroupBytes || (groups > 1 && sum + 0.5 * bytes[i] > left / groups))) {
      end.push_back(i);
      left -= sum;
      sum = 0.0;
      if (groups > 1) --groups;
    }
    sum += bytes[i];
  }
  if (!bytes.empty()) end.push_back((int)bytes.size());
  return end;
}

}  // namespace sbp
