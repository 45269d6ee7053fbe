// Items of the ring DFT kernels on the 8 XCDs: host-compilable, so that the
// deal can be checked without a GPU.
//
// A field group has 2 nk items (ring pair kk, half hh), in the order (kk, hh).
// Every XCD has a list of `chunk` entries per group, and takes the items of one
// eighth of the group; chunk is a multiple of four: the four items of two
// neighbouring ring pairs, which complete one 128-byte line of W, run together
// on one XCD.  With few rings the first chunks hold all items (17 northern rings:
// 34 items in five chunks of 8), so from group to group (and segment to segment)
// the chunks go on with the XCD after the last one that had any, and every
// eight groups one further, so that the ragged chunk moves too.  Measured,
// forward / inverse, us, fixed -> moved: 33 x 64 x 1000 fields 14.4 / 14.2 -> 11.1
// / 11.1, 97 x 192 x 1000 55 / 43 -> 47 / 37, 193 x 384 x 1000 169 / 177 -> 148 /
// 165.  Where all eight chunks have items they stay (Gauss 360 x 720 x 1024, the
// eighth half empty: 470 / 518 fixed, 487 / 498 moved).
#pragma once

namespace sht {
namespace dfti {

constexpr int kXcds = 8;

constexpr int chunk(int nk) { return ((2 * nk + kXcds - 1) / kXcds + 3) / 4 * 4; }
// XCDs from one group to the next
constexpr int step(int nk) { return (2 * nk + chunk(nk) - 1) / chunk(nk) % kXcds; }
// item (2 kk + hh) of a group's entry on an XCD; may be past the last item
constexpr int item(int xcd, int segment, int group, int entry, int chunk, int step) {
  const unsigned n = static_cast<unsigned>(segment) + static_cast<unsigned>(group);
  const unsigned first = step == 0 ? 0u : (n * step + n / kXcds) % kXcds;  // XCD of the first chunk
  return static_cast<int>((static_cast<unsigned>(xcd) + kXcds - first) % kXcds) * chunk + entry;
}

}  // namespace dfti
}  // namespace sht
