#include "route.hpp"

namespace sbp {

// us per stage of 16 shots of 64^3, order 4 (41.5 MB each in single precision),
// with the work list and in groups of 1, 2, 3, 4, 6, 8 and 16: single
// precision 289, and 355, 286, 258, 233, 258, 294, 288; double 562, and 570,
// 476, 469, 538, 532, 520, 507.  The bytes are those of the padded rows: counted
// by nodes, groups of grids whose rows fill their lines badly leave the cache
// (47 of 40^3, order 4: 337 us, 278 in groups of the right size, 327 with the
// work list; 31 of 34 x 101 x 29, order 6: 516, 415 and 431).  Over 112 batches
// of random shapes 240 MB is best: 200 and 225 MB halve groups of two grids of
// 104 and 120 MB (480 to 576 us, 233 to 256), 250 MB costs up to 14 % on small
// grids.
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
