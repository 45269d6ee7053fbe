// Column width of the Legendre contraction's tiles: host-compilable, so that
// the rule can be checked without a GPU.
#pragma once

namespace sht {
namespace legw {

// Field groups per column chunk for a segment of `groups` groups with `tiles`
// (order, parity, row tile) items and `steps` K steps, at most `limit`; `others`:
// items times (columns + 1.5) of the plan's other segments.
//
// Where the chip is full, a chunk of cb groups costs about cb + 1.5 (the 1.5 for
// the table's loads and splits), so the widest chunks are best, unless the last
// one is ragged.  Up to two steps a tile wider than four, which needs a second
// data piece a wave and leaves three workgroups instead of four on a CU, costs a
// fifth more; at one step a workgroup's start and end weigh more, 2.4 and a
// third.  Where it is not full, a tile's own time decides, about cb + 3, and
// chunks are made narrower until some 420 (columns + 1.5) are at work.  Measured,
// kernel us, float32, analysis / synthesis, at the width of the full chip -> as
// chosen: 33 x 64 x 64 fields 10.6 / 8.6 -> 7.0 / 6.8, 73 x 144 x 64 13.1 / 12.3 ->
// 9.3 / 8.6, 121 x 240 x 128 21.7 / 18.3 -> 18.1 / 17.5, 181 x 360 x 64 22.1 / 21.6 ->
// 19.0 / 18.0; 181 x 360 x 128 and wider plans keep theirs.
inline int width(int groups, int limit, long long tiles, int steps, double others) {
  const int most = groups < limit ? groups : limit;
  int best = 1;
  double best_cost = -1.0;
  for (int cb = groups > 1 ? 2 : 1; cb <= most; ++cb) {
    const double chunks = (groups + cb - 1) / cb;
    double work = chunks * static_cast<double>(tiles) * (steps == 1 ? 1.4 * (cb + 2.4) : cb + 1.5);
    if (cb > 4 && steps <= 2) work *= steps == 1 ? 1.3 : 1.19;
    const double full = (others + work) / 420.0, own = cb + 3.0;
    const double cost = full > own ? full : own;
    if (best_cost < 0.0 || cost <= best_cost) {
      best = cb;
      best_cost = cost;
    }
  }
  return best;
}

}  // namespace legw
}  // namespace sht
