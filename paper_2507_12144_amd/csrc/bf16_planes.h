// Float32 values as sums of bf16 planes, for the bf16 matrix cores
// (v_mfma_f32_16x16x32_bf16) to take in the place of the float32 ones.
#pragma once

#include <hip/hip_runtime.h>

namespace sht {
namespace planes {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Global address-space views: the pointers come from the segment table in
// memory, and accesses through them as generic pointers would be flat ones,
// which count as LDS operations too, so that the LDS barrier of every step
// would wait for the loads in flight.
typedef __attribute__((address_space(1))) const v4f gcv4f;
typedef __attribute__((address_space(1))) const float gcfloat;
typedef __attribute__((address_space(1))) floatx4 gfloatx4;

// Float32 operands are split after an exact scaling by 2^16: every float32 is
// a multiple of 2^-149, so each plane of the scaled value is a multiple of
// 2^-133, the smallest bf16 (the conversions and the matrix cores keep
// subnormals).  Unscaled, the third plane, 2^-16 to 2^-24 of the value, fell
// off below 1e-33.
constexpr float kSplitScale = 65536.f;

// Two float32 values rounded to nearest-even bf16, packed (v_cvt_pk_bf16_f32).
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  const f32x2 v = {x, y};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// 8 float32 values as ND bf16 planes (residuals in float32, exact).  A value
// that rounds to an infinite bf16 leaves a NaN in the last plane.
template <int ND>
__device__ __forceinline__ void split8(const float* v, bf16x8* out) {
  u32x4 bits[ND];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = v[2 * e], y = v[2 * e + 1];
#pragma unroll
    for (int pl = 0; pl < ND; ++pl) {
      const unsigned b = pack_bf16(x, y);
      bits[pl][e] = b;
      if (pl + 1 < ND) {
        x -= __builtin_bit_cast(float, b << 16);
        y -= __builtin_bit_cast(float, b & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int pl = 0; pl < ND; ++pl) out[pl] = __builtin_bit_cast(bf16x8, bits[pl]);
}

}  // namespace planes
}  // namespace sht
