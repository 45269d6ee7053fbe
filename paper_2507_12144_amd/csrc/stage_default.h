// Default staging of the spectrum through order-major tiles: host-compilable, so
// that the rule can be checked without a GPU.
#pragma once

namespace sht {
namespace staging {

// Staged, the contraction reads and writes whole lines, but each transform takes
// one more launch and moves the spectrum twice.  Direct, the 8-byte entries of
// 16 orders share a line of the spectrum, and a line is moved once only if it
// stays in its XCD's L2 (4 MiB) until the orders of a work chunk are done: the
// lines that a chunk has open (one for every field and degree), and the table
// that streams past them meanwhile, taken at 0.6 of eight orders' (16 bytes a
// degree and northern ring).
inline double open_bytes(long long fields, int lmax, int rings) {
  return 128.0 * fields * lmax + 0.6 * 16.0 * lmax * rings;
}
// The line lies at 3.2 MB.  SHT, ISHT, us, direct / staged: 33 x 64 x 1280 fields (5.3
// MB) 37 / 37, 39 / 37, x 1792 (7.4) 49 / 44, 53 / 44; 61 x 120 x 364 (2.8) 25 / 27,
// 22 / 27, x 509 (3.9) 31 / 29, 28 / 29; 121 x 240 x 182 (2.9) 35 / 35, 31 / 34, x 364
// (5.7) 64 / 55, 59 / 54; 181 x 360 x 113 (2.8) 43 / 42, 41 / 41, x 364 (8.5) 148 /
// 120, 110 / 112; 361 x 720 x 28 (1.9) 47 / 48, 51 / 49, x 91 (4.8) 136 / 130, 140 /
// 126; 721 x 1440 x 5 (3.0) 121 / 124, 111 / 119, x 15 (3.9) 174 / 170, 165 / 158.
// (By the size of the whole spectrum, 20 MiB and more staged, the same shapes
// lay up to 50% off the better choice, in the mean 1.7%; by this rule 22% and
// 0.6%.)
constexpr double kOpenBytes = 3.2e6;

inline bool segment(long long fields, int lmax, int rings) { return open_bytes(fields, lmax, rings) >= kOpenBytes; }

}  // namespace staging
}  // namespace sht
