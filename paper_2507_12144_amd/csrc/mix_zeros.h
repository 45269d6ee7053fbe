// Who writes the zeros (m > l) of a channel mix: host-compilable, so that the
// split can be checked without a GPU.
//
// For degree l the column tiles cover all batch x mmax columns (b, m), of which
// only batch x mcount hold products.  The tiles past those have nothing else to
// do and share the zeros, unless the waves of the tiles with products have a row
// (b, c') each at most: 16 x 1 channels, lmax 360, 77 us a mix by those, 88 by
// the tiles past them, which then no longer end at once; 4 x 32 channels 59 and
// 54, 4 x 256 807 and 798.  A wave takes several rows at a time when a row has
// fewer zeros than lanes.  (By the tiles with products alone, a wave per row, the
// zeros of few degrees and many members were the whole time: 64 x 64 channels,
// lmax 8, 174 us a mix, now 11.)
#pragma once

namespace sht {
namespace mixz {

constexpr int kWaves = 4;  // waves of a workgroup

struct Share {
  int first, tiles;  // column tiles first .. first + tiles - 1 write zeros
  int shift;         // 2^shift lanes per row
};

// tiles: column tiles of the grid, live: those with products, rows of the
// workgroup's row tile, zeros of a row
constexpr bool by_live_tiles(int tiles, int live, int rows) { return live == tiles || rows <= kWaves * live; }
constexpr Share share(int tiles, int live, int rows, int zeros) {
  Share s{by_live_tiles(tiles, live, rows) ? 0 : live, 0, 0};
  s.tiles = s.first == 0 ? live : tiles - live;
  while (s.shift < 6 && (1 << s.shift) < zeros) ++s.shift;
  return s;
}

// rows first_row(), first_row() + row_step(), ... and orders (counted from the
// first zero) first_order(), first_order() + order_step(), ... of a lane of
// column tile `tile`
constexpr int first_row(const Share& s, int tile, int wave, int lane) {
  return ((tile - s.first) * kWaves + wave) * (64 >> s.shift) + (lane >> s.shift);
}
constexpr int row_step(const Share& s) { return s.tiles * kWaves * (64 >> s.shift); }
constexpr int first_order(const Share& s, int lane) { return lane & ((1 << s.shift) - 1); }
constexpr int order_step(const Share& s) { return 1 << s.shift; }

}  // namespace mixz
}  // namespace sht
