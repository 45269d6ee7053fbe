// Analysis kernels of the bf16 form (see legendre.h); one translation unit per
// form and direction so that they compile in parallel.
#include "legendre.h"

namespace sht {
namespace legk {
template hipError_t launch<Storage::BF16, false>(const BatchArgs&, const float2*, float2*, float, hipStream_t);
}  // namespace legk
}  // namespace sht
