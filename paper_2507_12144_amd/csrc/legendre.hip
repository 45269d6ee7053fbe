// Entry points of the Legendre contraction (kernels in legendre.h, instantiated
// per form and direction in legendre_{f32,bf16,bf16x2,bf16x3}_{ana,syn}.hip).
#include <algorithm>

#include "legendre.h"
#include "legendre_width.h"

namespace sht {

using legk::launch;

int legendre_ring_pad(int nk) { return nk <= kMaxRings ? (nk + 31) / 32 * 32 : -1; }

bool legendre_ncb_supported(int ncb) { return ncb >= 2 && ncb <= 4; }

int legendre_column_blocks(Storage form, bool synthesis, int groups, int ncb, long long tiles, int steps,
                           double others) {
  int limit = ncb == 2 ? legk::kMaxCb : ncb == 3 ? 6 : 4;
  if (form == Storage::BF16X3 && !synthesis) limit = std::min(limit, legk::max_cb<Storage::BF16X3, false>);
  return legw::width(groups, limit, tiles, steps, others);
}

int legendre_row_tiles(int row_blocks) { return (row_blocks + legk::kTileBlocks - 1) / legk::kTileBlocks; }

hipError_t launch_legendre_analysis(const BatchArgs& b, Storage form, float2* y, float c_rest, hipStream_t st) {
  switch (form) {
    case Storage::F32: return launch<Storage::F32, false>(b, nullptr, y, c_rest, st);
    case Storage::BF16: return launch<Storage::BF16, false>(b, nullptr, y, c_rest, st);
    case Storage::BF16X2: return launch<Storage::BF16X2, false>(b, nullptr, y, c_rest, st);
    case Storage::BF16X3: return launch<Storage::BF16X3, false>(b, nullptr, y, c_rest, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_legendre_synthesis(const BatchArgs& b, Storage form, const float2* y, hipStream_t st) {
  switch (form) {
    case Storage::F32: return launch<Storage::F32, true>(b, y, nullptr, 1.f, st);
    case Storage::BF16: return launch<Storage::BF16, true>(b, y, nullptr, 1.f, st);
    case Storage::BF16X2: return launch<Storage::BF16X2, true>(b, y, nullptr, 1.f, st);
    case Storage::BF16X3: return launch<Storage::BF16X3, true>(b, y, nullptr, 1.f, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace sht
