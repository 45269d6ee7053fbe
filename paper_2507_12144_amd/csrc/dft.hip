// Ring DFT kernels: the longitude step of the SHT (the "2 pi * FFT_1D_R2C
// along W, then keep m < mmax" of Alg. 1) and its inverse.
//
// Design (gfx950):
//  * A workgroup owns one ring pair (k, nlat-1-k) for 4 fields.  The two
//    real rings of a field are packed as one complex sequence z = u_k + i u_k'
//    (the mirrored ring), so one complex FFT of length nlon yields both real
//    spectra, and the pair is exactly what the equatorial fold of the
//    Legendre step needs: S = X_k + X_k' and A = X_k - X_k'.
//  * The complex FFT is a Stockham autosort in LDS, in place, in at most four
//    (for the widths in use three) passes of radix 2 .. 16 butterflies, each
//    a composite DFT held in registers.  The widths of the 0.25 / 0.5 / 1
//    degree and small test grids (1440, 720, 360, 64) have their radices and
//    indices fixed at compile time; every other width 2^a 3^b 5^c runs the
//    same passes with run-time ones (72
//    fields, us, forward / inverse, against the ping-pong path with radices
//    up to 5 that they had: 649 x 1296: 393 / 420 -> 143 / 155, 271 x 540: 46 /
//    48 -> 29 / 27, 513 x 1024: 207 / 212 -> 86 / 107).
//  * Twiddles: a pass of radix R after P points needs w^(q k), q < R, k < P.
//    LDS holds them for the q of a two-digit basis (q < B and the multiples
//    of B, B = 4, for radix 9 B = 3), ordered by k: a thread reads those few
//    at consecutive addresses and forms the others by one product.
//  * Workspace layout W[m][p][g][k][16]: g = group of 8 fields, 16 floats =
//    (re, im) of those fields.  A workgroup writes / reads 32-byte runs; the
//    workgroups completing one 128-byte line run together on the same XCD
//    (which merges them in its L2).
// Bound: the memory phases.  721 x 1440 x 72 fields: 156 / 155 us, forward /
// inverse, for 661 / 601 MB (4.2 / 3.9 TB/s; at the start of the in-place form
// with two-level twiddles 165 / 166); 361 x 720 x 72: 40 / 35 (49 / 41), Gauss
// 360 x 720 x 1024: 472 / 517 (552 / 623).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "dft_items.h"
#include "internal.h"
#include "kernel_common.h"

namespace sht {
namespace {

constexpr int FGW = 4;     // fields per workgroup

// Threads of a workgroup and the widest ring that they serve.  A narrow ring
// keeps few threads of a large workgroup busy (a 72-point pass of radix 9 has
// 32 butterflies), and every loop is unrolled for the widest ring, so a plan
// takes the smallest block that covers its widest one; without the wide
// rings' registers the run-time radices need 58 VGPRs (eight waves per SIMD)
// instead of 80.  Measured, 1000 fields, us, forward / inverse, one block of
// 512 threads for every width against these: 36 x 19 27 / 29 -> 9.6 / 9.3, 72
// x 37 49 / 48 -> 16 / 16, 144 x 73 83 / 79 -> 31 / 29, 256 x 129 153 / 167 ->
// 87 / 92, 384 x 193 267 / 310 -> 169 / 178, 480 x 241 305 / 386 -> 241 / 251,
// 640 x 321 500 / 640 -> 431 / 425; 288 fields: 1000 x 501 271 / 346 -> 259 /
// 315, 1080 x 541 291 / 373 -> 295 / 339.
template <int NT_, int WIDEST_>
struct Block {
  static constexpr int NT = NT_, WIDEST = WIDEST_;
};
using Narrow = Block<128, 192>;
using Middle = Block<256, 384>;
using Middle2 = Block<256, 768>;
using Wide = Block<512, 1152>;
using Widest = Block<512, kMaxNlon>;
// The forward step leaves two blocks earlier than the inverse one: more
// workgroups in flight keep more partly written lines of W in flight (see
// dft_paired).  Forward, 1000 fields, us, 256 / 512 threads: 576 x 289 367 /
// 410, 600 x 301 402 / 380, 640 x 321 526 / 431 (inverse 425 / 546); Wide /
// Widest at 288 fields: 1000 x 501 259 / 271, 1080 x 541 394 / 322 (inverse
// 358 / 405).
constexpr int kForwardMiddle2 = 576, kForwardWide = 1024;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// global address space: the pointers come from the segment table
typedef __attribute__((address_space(1))) const f32x2 gcf32x2;
typedef __attribute__((address_space(1))) const f32x4 gcf32x4;

// Complex values from one field's sequence to the next in LDS: two fields
// apart the same index falls half a bank period away, so that a pair of lanes
// on one order of two fields (see the W accesses) does not conflict.
__host__ __device__ constexpr int field_stride(int n) { return n + ((8 - n) & 15); }

struct DftArgs {
  int nlat, nlon, lmax, mmax, nk, F, kpad, G;
  long long wslab;         // floats per (m, parity) slab of W
  int ntw;                 // twiddles in LDS
  int npass;
  const int* radix;        // the segment's radix plan (device memory)
  float c_rest;
};

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// multiply by +i (sg = +1) or -i (sg = -1)
__device__ __forceinline__ float2 mul_i(float2 a, float sg) { return make_float2(-sg * a.y, sg * a.x); }

// cos / sin of 2 pi e / R for the composite radices (e < R).
template <int R>
__device__ __forceinline__ float root_cos(int e);
template <int R>
__device__ __forceinline__ float root_sin(int e);

#define SHT_ROOTS(R, ...)                                                    \
  template <>                                                                \
  __device__ __forceinline__ float root_cos<R>(int e) {                      \
    constexpr float c[R] = {__VA_ARGS__};                                    \
    return c[e];                                                             \
  }
SHT_ROOTS(8, 1.f, 0.70710678118654752f, 0.f, -0.70710678118654752f, -1.f, -0.70710678118654752f, 0.f,
          0.70710678118654752f)
SHT_ROOTS(9, 1.f, 0.76604444311897804f, 0.17364817766693035f, -0.5f, -0.93969262078590838f,
          -0.93969262078590838f, -0.5f, 0.17364817766693035f, 0.76604444311897804f)
SHT_ROOTS(10, 1.f, 0.80901699437494742f, 0.30901699437494742f, -0.30901699437494742f, -0.80901699437494742f,
          -1.f, -0.80901699437494742f, -0.30901699437494742f, 0.30901699437494742f, 0.80901699437494742f)
SHT_ROOTS(16, 1.f, 0.92387953251128676f, 0.70710678118654752f, 0.38268343236508977f, 0.f,
          -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128676f, -1.f, -0.92387953251128676f,
          -0.70710678118654752f, -0.38268343236508977f, 0.f, 0.38268343236508977f, 0.70710678118654752f,
          0.92387953251128676f)
SHT_ROOTS(6, 1.f, 0.5f, -0.5f, -1.f, -0.5f, 0.5f)
SHT_ROOTS(12, 1.f, 0.86602540378443871f, 0.5f, 0.f, -0.5f, -0.86602540378443871f, -1.f, -0.86602540378443882f, -0.5f, 0.f, 0.5f, 0.86602540378443837f)
SHT_ROOTS(15, 1.f, 0.91354545764260087f, 0.66913060635885824f, 0.30901699437494745f, -0.10452846326765333f, -0.5f, -0.80901699437494734f, -0.97814760073380569f, -0.97814760073380569f, -0.80901699437494756f, -0.5f, -0.10452846326765423f, 0.30901699437494723f, 0.66913060635885846f, 0.91354545764260098f)
#undef SHT_ROOTS
// sin(2 pi e / R) = cos(2 pi (e - R/4) / R) for R divisible by 4; listed
// explicitly for the odd-quarter radices.
template <>
__device__ __forceinline__ float root_sin<8>(int e) {
  constexpr float s[8] = {0.f, 0.70710678118654752f, 1.f, 0.70710678118654752f, 0.f, -0.70710678118654752f, -1.f,
                          -0.70710678118654752f};
  return s[e];
}
template <>
__device__ __forceinline__ float root_sin<9>(int e) {
  constexpr float s[9] = {0.f, 0.64278760968653933f, 0.98480775301220806f, 0.86602540378443865f,
                          0.34202014332566873f, -0.34202014332566873f, -0.86602540378443865f,
                          -0.98480775301220806f, -0.64278760968653933f};
  return s[e];
}
template <>
__device__ __forceinline__ float root_sin<10>(int e) {
  constexpr float s[10] = {0.f, 0.58778525229247313f, 0.95105651629515357f, 0.95105651629515357f,
                           0.58778525229247313f, 0.f, -0.58778525229247313f, -0.95105651629515357f,
                           -0.95105651629515357f, -0.58778525229247313f};
  return s[e];
}
template <>
__device__ __forceinline__ float root_sin<16>(int e) {
  constexpr float s[16] = {0.f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128676f, 1.f,
                           0.92387953251128676f, 0.70710678118654752f, 0.38268343236508977f, 0.f,
                           -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128676f, -1.f,
                           -0.92387953251128676f, -0.70710678118654752f, -0.38268343236508977f};
  return s[e];
}

template <>
__device__ __forceinline__ float root_sin<6>(int e) {
  constexpr float s[6] = {0.f, 0.8660254037844386f, 0.86602540378443871f, 0.f, -0.86602540378443837f, -0.8660254037844386f};
  return s[e];
}
template <>
__device__ __forceinline__ float root_sin<12>(int e) {
  constexpr float s[12] = {0.f, 0.5f, 0.8660254037844386f, 1.f, 0.86602540378443871f, 0.5f, 0.f, -0.5f, -0.86602540378443837f, -1.f, -0.8660254037844386f, -0.5f};
  return s[e];
}
template <>
__device__ __forceinline__ float root_sin<15>(int e) {
  constexpr float s[15] = {0.f, 0.40673664307580015f, 0.74314482547739413f, 0.95105651629515353f, 0.9945218953682734f, 0.86602540378443871f, 0.58778525229247325f, 0.20791169081775931f, -0.20791169081775907f, -0.58778525229247303f, -0.86602540378443837f, -0.99452189536827329f, -0.95105651629515364f, -0.74314482547739402f, -0.40673664307580015f};
  return s[e];
}

// In-register DFT of length R: A_s = sum_q a_q e^{sg 2 pi i q s / R}.
template <int R>
struct Codelet;

template <>
struct Codelet<2> {
  __device__ static __forceinline__ void run(float2* a, float) {
    const float2 t = a[1];
    a[1] = csub(a[0], t);
    a[0] = cadd(a[0], t);
  }
};

template <>
struct Codelet<4> {
  __device__ static __forceinline__ void run(float2* a, float sg) {
    const float2 s02 = cadd(a[0], a[2]), d02 = csub(a[0], a[2]);
    const float2 s13 = cadd(a[1], a[3]), d13 = mul_i(csub(a[1], a[3]), sg);
    a[0] = cadd(s02, s13);
    a[2] = csub(s02, s13);
    a[1] = cadd(d02, d13);
    a[3] = csub(d02, d13);
  }
};

template <>
struct Codelet<3> {
  __device__ static __forceinline__ void run(float2* a, float sg) {
    const float h = 0.86602540378443864676f;  // sin(2 pi / 3)
    const float2 t = cadd(a[1], a[2]);
    const float2 d = mul_i(cscale(csub(a[1], a[2]), h), sg);
    const float2 b = make_float2(a[0].x - 0.5f * t.x, a[0].y - 0.5f * t.y);
    a[0] = cadd(a[0], t);
    a[1] = cadd(b, d);
    a[2] = csub(b, d);
  }
};

template <>
struct Codelet<5> {
  __device__ static __forceinline__ void run(float2* a, float sg) {
    const float c1 = 0.30901699437494742410f;   // cos(2 pi / 5)
    const float c2 = -0.80901699437494742410f;  // cos(4 pi / 5)
    const float s1 = 0.95105651629515357212f;   // sin(2 pi / 5)
    const float s2 = 0.58778525229247312917f;   // sin(4 pi / 5)
    const float2 t1 = cadd(a[1], a[4]), d1 = csub(a[1], a[4]);
    const float2 t2 = cadd(a[2], a[3]), d2 = csub(a[2], a[3]);
    const float2 r1 = make_float2(a[0].x + c1 * t1.x + c2 * t2.x, a[0].y + c1 * t1.y + c2 * t2.y);
    const float2 r2 = make_float2(a[0].x + c2 * t1.x + c1 * t2.x, a[0].y + c2 * t1.y + c1 * t2.y);
    const float2 i1 = mul_i(make_float2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y), sg);
    const float2 i2 = mul_i(make_float2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y), sg);
    a[0] = make_float2(a[0].x + t1.x + t2.x, a[0].y + t1.y + t2.y);
    a[1] = cadd(r1, i1);
    a[4] = csub(r1, i1);
    a[2] = cadd(r2, i2);
    a[3] = csub(r2, i2);
  }
};

// Composite R = R1 * R2 (Cooley-Tukey in registers): inputs n = R2 n1 + n2,
// outputs k = k1 + R1 k2, inner twiddles e^{sg 2 pi i n2 k1 / R}.
template <int R1, int R2>
struct Composite {
  __device__ static __forceinline__ void run(float2* a, float sg) {
    constexpr int R = R1 * R2;
    float2 t[R];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
      float2 u[R1];
#pragma unroll
      for (int n1 = 0; n1 < R1; ++n1) u[n1] = a[R2 * n1 + n2];
      Codelet<R1>::run(u, sg);
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) {
        const int e = (n2 * k1) % R;
        if (e == 0) {
          t[n2 * R1 + k1] = u[k1];
        } else {
          t[n2 * R1 + k1] = cmul(u[k1], make_float2(root_cos<R>(e), sg * root_sin<R>(e)));
        }
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      float2 u[R2];
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) u[n2] = t[n2 * R1 + k1];
      Codelet<R2>::run(u, sg);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) a[k1 + R1 * k2] = u[k2];
    }
  }
};

template <>
struct Codelet<6> : Composite<2, 3> {};
template <>
struct Codelet<12> : Composite<3, 4> {};
template <>
struct Codelet<15> : Composite<3, 5> {};
template <>
struct Codelet<8> : Composite<2, 4> {};
template <>
struct Codelet<9> : Composite<3, 3> {};
template <>
struct Codelet<10> : Composite<2, 5> {};
template <>
struct Codelet<16> : Composite<4, 4> {};

// Digits of the twiddle basis of radix R: q = lo + BASE hi.
__host__ __device__ constexpr int twiddle_base(int R) { return R == 9 ? 3 : 4; }
__host__ __device__ constexpr int twiddle_los(int R) { return R - 1 < twiddle_base(R) - 1 ? R - 1 : twiddle_base(R) - 1; }
__host__ __device__ constexpr int twiddle_his(int R) { return (R - 1) / twiddle_base(R); }

// a * w, or a * conj(w) (the tables hold e^{-i ...})
template <bool INV>
__device__ __forceinline__ float2 twmul(float2 a, float2 w) {
  return INV ? make_float2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y) : cmul(a, w);
}

// v[q] *= w^(q k) for 1 <= q < R; tab points at k of the pass's table.
template <int R, bool INV>
__device__ __forceinline__ void apply_twiddles(float2* v, const float2* tab, int P) {
  constexpr int B = twiddle_base(R), NL = twiddle_los(R), NH = twiddle_his(R);
  float2 lo[NL > 0 ? NL : 1], hi[NH > 0 ? NH : 1];
#pragma unroll
  for (int i = 0; i < NL; ++i) lo[i] = tab[i * P];
#pragma unroll
  for (int i = 0; i < NH; ++i) hi[i] = tab[(NL + i) * P];
#pragma unroll
  for (int q = 1; q < R; ++q) {
    const int l = q % B, h = q / B;
    const float2 w = h == 0 ? lo[l - 1] : l == 0 ? hi[h - 1] : cmul(lo[l - 1], hi[h - 1]);
    v[q] = twmul<INV>(v[q], w);
  }
}

// a / b and the remainder for 0 <= a < 2^20, 0 < b < 2^12 (exact: the
// quotient is off a whole number by at least 1 / (2 b))
__device__ __forceinline__ int small_div(int a, float rb) { return static_cast<int>((a + 0.5f) * rb); }

// One in-place Stockham pass of radix R over FGW sequences of N points held
// in LDS; P is the product of the radices of the earlier passes (NC, PC: N
// and P where they are known at compile time).  Every thread first gathers
// the inputs of all its butterflies (at most PER) into registers, then,
// after a barrier, overwrites the buffer with their outputs.
template <int NT, int R, int PER, int NC, int PC, bool INV>
__device__ __forceinline__ void pass_inplace(float2* buf, const float2* tw, int n, int p) {
  const int N = NC > 0 ? NC : n, P = PC > 0 ? PC : p;
  const int FS = field_stride(N);
  const int NB = N / R, TOT = FGW * NB;
  const float rnb = 1.f / NB, rp = 1.f / P;
  float2 v[PER][R];
  int base[PER], kk[PER];
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int bi = threadIdx.x + b * NT;
    if (bi < TOT) {
      const int f = NC > 0 ? bi / NB : small_div(bi, rnb);
      const int t = bi - f * NB;
      kk[b] = PC == 1 ? 0 : PC > 0 ? t % P : t - P * small_div(t, rp);
      base[b] = f * FS + (t - kk[b]) * R + kk[b];
#pragma unroll
      for (int q = 0; q < R; ++q) v[b][q] = buf[f * FS + t + q * NB];
    }
  }
  lds_barrier();
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int bi = threadIdx.x + b * NT;
    if (bi < TOT) {
      if (PC != 1 && P > 1) apply_twiddles<R, INV>(v[b], tw + kk[b], P);
      Codelet<R>::run(v[b], INV ? 1.f : -1.f);
#pragma unroll
      for (int q = 0; q < R; ++q) buf[base[b] + q * P] = v[b][q];
    }
  }
  lds_barrier();
}

constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ constexpr int pass_twiddles(int R, int P) { return P > 1 ? P * (twiddle_los(R) + twiddle_his(R)) : 0; }

// Widths with compile-time radices.
template <class BLK, int N_, int R1, int R2, int R3>
struct FixedFFT {
  static constexpr int NT = BLK::NT, WIDEST = N_;
  static constexpr int N = N_;
  static constexpr int PASSES = R3 > 1 ? 3 : 2;
  static constexpr int RADIX[3] = {R1, R2, R3};
  static constexpr int TWIDDLES = pass_twiddles(R2, R1) + (R3 > 1 ? pass_twiddles(R3, R1 * R2) : 0);
  template <bool INV>
  __device__ static __forceinline__ void run(float2* buf, const float2* tw, const DftArgs&) {
    static_assert(R1 * R2 * R3 == N, "radix plan");
    pass_inplace<NT, R1, ceil_div(FGW * N / R1, NT), N, 1, INV>(buf, tw, N, 1);
    pass_inplace<NT, R2, ceil_div(FGW * N / R2, NT), N, R1, INV>(buf, tw, N, R1);
    if constexpr (R3 > 1)
      pass_inplace<NT, R3, ceil_div(FGW * N / R3, NT), N, R1 * R2, INV>(buf, tw + pass_twiddles(R2, R1), N, R1 * R2);
  }
};

// Run-time radices (make_dft_plan): any N = 2^a 3^b 5^c <= kMaxNlon.  The
// butterflies per thread cover the largest width a radix is chosen for.
template <class BLK>
struct GenericFFT {
  static constexpr int NT = BLK::NT, WIDEST = BLK::WIDEST;
  static constexpr int N = 0, TWIDDLES = 0;
  template <bool INV>
  __device__ static __forceinline__ void run(float2* buf, const float2* tw, const DftArgs& a) {
    int p = 1;
    for (int s = 0; s < a.npass; ++s) {
      const int R = a.radix[s];
      // keeps the index arithmetic of every radix inside its case: hoisted
      // out of the loop it takes 240 VGPRs
      int n = __builtin_amdgcn_readfirstlane(a.nlon);
      asm volatile("" : "+s"(n));
      switch (R) {
#define SHT_PASS(RR)                                                                                              \
  case RR:                                                                                                        \
    pass_inplace<NT, RR, ceil_div(FGW * max_width(RR) / RR, NT), 0, 0, INV>(buf, tw, n, p);                       \
    tw += pass_twiddles(RR, p);                                                                                   \
    break;
        SHT_PASS(2)
        SHT_PASS(3)
        SHT_PASS(4)
        SHT_PASS(5)
        SHT_PASS(6)
        SHT_PASS(8)
        SHT_PASS(9)
        SHT_PASS(10)
        SHT_PASS(12)
        SHT_PASS(15)
        default:
        SHT_PASS(16)
#undef SHT_PASS
      }
      p *= R;
    }
  }
  // widest ring a radix is chosen for: radices above 10 take one butterfly a
  // thread, so that no pass holds more than 20 complex values
  __host__ __device__ static constexpr int max_width(int R) {
    return R > 10 && NT * R / FGW < WIDEST ? NT * R / FGW : WIDEST;
  }
};

// The twiddle tables into LDS: all loads first, issued right behind the
// thread's data loads, so that the workgroup still waits for one round trip
// (ahead of them they cost the 720-point forward kernel 518 -> 547 us at
// 1024 fields, in a loop of load and store the 1440-point one 163 -> 174).  A width has fewer twiddles than points
// (make_dft_plan).
template <class FFT>
struct TwiddleCopy {
  static constexpr int NT = FFT::NT;
  static constexpr int PER = ceil_div(FFT::N > 0 ? FFT::TWIDDLES : FFT::WIDEST, NT);
  f32x2 v[PER];
  __device__ __forceinline__ void load(const DftArgs& a, const float2* tw) {
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int i = threadIdx.x + b * NT;
      if (i < a.ntw) v[b] = ((gcf32x2*)tw)[i];
    }
  }
  __device__ __forceinline__ void store(const DftArgs& a, float2* ltw) const {
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int i = threadIdx.x + b * NT;
      if (i < a.ntw) ltw[i] = make_float2(v[b][0], v[b][1]);
    }
  }
};

// Item (field group g, ring pair kk, half hh).
struct Item {
  int g, kk, hh;
  bool valid;
};

__device__ __forceinline__ size_t wrow(const DftArgs& a, int m, int p, int g, int kk) {
  return static_cast<size_t>(2 * m + p) * a.wslab + (static_cast<size_t>(g) * a.kpad + kk) * 16;
}

template <class FFT, bool PAIRED>
__device__ __forceinline__ void dft_forward_body(const DftArgs& a, const Item& it, const float* __restrict__ x,
                                                 float* __restrict__ W, const float2* __restrict__ tw,
                                                 const float* __restrict__ ring_scale, float2* lds,
                                                 float* __restrict__ zonal) {
  constexpr int NF = FFT::N, NT = FFT::NT;
  const int N = NF > 0 ? NF : a.nlon;
  const int kk = it.kk;
  const int ks = a.nlat - 1 - kk;
  const bool eq = (ks == kk);
  const int f0 = 8 * it.g + 4 * it.hh;
  const int FS = field_stride(N);
  float2* ltw = lds + FGW * FS;
  TwiddleCopy<FFT> twc;
  // Load 4 fields x 2 rings, packed as complex (north, mirrored ring).  Every
  // load of the thread is issued before the first LDS store, so that the
  // workgroup waits for one memory round trip, not one per iteration.
  auto load_rings = [&](auto vec_c) {
    constexpr int V = decltype(vec_c)::value;  // longitudes per load
    typedef float vec __attribute__((ext_vector_type(V)));
    typedef __attribute__((address_space(1))) const vec gvec;
    constexpr int PER = ceil_div(FGW * FFT::WIDEST / V, NT);
    const int nq = N / V;
    const float rnq = 1.f / nq;
    vec vn[PER], vs[PER];
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int idx = threadIdx.x + b * NT;
      const int fl = NF > 0 ? idx / nq : small_div(idx, rnq);
      const int j = V * (idx - fl * nq);
      const int fi = f0 + fl;
      vn[b] = 0.f;
      vs[b] = 0.f;
      if (fl < FGW && fi < a.F) {
        vn[b] = *(gvec*)(x + (static_cast<size_t>(fi) * a.nlat + kk) * N + j);
        if (!eq) vs[b] = *(gvec*)(x + (static_cast<size_t>(fi) * a.nlat + ks) * N + j);
      }
    }
    twc.load(a, tw);
    twc.store(a, ltw);
#pragma unroll
    for (int b = 0; b < PER; ++b) {
      const int idx = threadIdx.x + b * NT;
      const int fl = NF > 0 ? idx / nq : small_div(idx, rnq);
      if (fl < FGW) {
        float2* d = lds + fl * FS + V * (idx - fl * nq);
#pragma unroll
        for (int i = 0; i < V; ++i) d[i] = make_float2(vn[b][i], vs[b][i]);
      }
    }
  };
  if (NF > 0 ? NF % 4 == 0 : (N & 3) == 0) {
    load_rings(std::integral_constant<int, 4>{});
  } else if ((N & 1) == 0) {
    load_rings(std::integral_constant<int, 2>{});
  } else {
    twc.load(a, tw);
    twc.store(a, ltw);
    for (int idx = threadIdx.x; idx < FGW * N; idx += NT) {
      const int fl = idx / N;
      const int j = idx - fl * N;
      const int fi = f0 + fl;
      float re = 0.f, im = 0.f;
      if (fi < a.F) {
        re = x[(static_cast<size_t>(fi) * a.nlat + kk) * N + j];
        if (!eq) im = x[(static_cast<size_t>(fi) * a.nlat + ks) * N + j];
      }
      lds[fl * FS + j] = make_float2(re, im);
    }
  }
  lds_barrier();
  FFT::template run<false>(lds, ltw, a);
  const float2* Z = lds;
  const float sc = ring_scale[kk];
  if (zonal) {
    // zonal power spectra of the two rings: sc |X|^2 with the zonal scale
    for (int m = threadIdx.x; m < a.mmax; m += NT) {
#pragma unroll
      for (int fl = 0; fl < FGW; ++fl) {
        const int fi = f0 + fl;
        if (fi >= a.F) continue;
        const float2 zm = Z[fl * FS + m];
        const float2 zr = Z[fl * FS + (m == 0 ? 0 : N - m)];
        const float2 xn = make_float2(0.5f * (zm.x + zr.x), 0.5f * (zm.y - zr.y));
        const float2 xs = make_float2(0.5f * (zm.y + zr.y), -0.5f * (zm.x - zr.x));
        zonal[(static_cast<size_t>(fi) * a.nlat + kk) * a.mmax + m] = sc * (xn.x * xn.x + xn.y * xn.y);
        if (!eq) zonal[(static_cast<size_t>(fi) * a.nlat + ks) * a.mmax + m] = sc * (xs.x * xs.x + xs.y * xs.y);
      }
    }
    return;
  }
  // S and A of field fl at order m
  auto fold = [&](int fl, int m, float* Sv, float* Av) {
    const float2 zm = Z[fl * FS + m];
    const float2 zr = Z[fl * FS + (m == 0 ? 0 : N - m)];
    // spectra of the two packed real rings
    const float2 xn = make_float2(0.5f * (zm.x + zr.x), 0.5f * (zm.y - zr.y));
    const float2 xs = make_float2(0.5f * (zm.y + zr.y), -0.5f * (zm.x - zr.x));
    float2 S, A;
    if (eq) {
      S = cscale(xn, sc);
      A = make_float2(0.f, 0.f);
    } else {
      S = cscale(cadd(xn, xs), sc);
      A = cscale(csub(xn, xs), sc);
    }
    if (m == 0) {
      S.y = 0.f;
      A.y = 0.f;
    }
    Sv[0] = S.x;
    Sv[1] = S.y;
    Av[0] = A.x;
    Av[1] = A.y;
  };
  if constexpr (PAIRED) {
    // a pair of lanes writes the 32 bytes of one order and parity
    for (int idx = threadIdx.x; idx < 2 * a.mmax; idx += NT) {
      const int m = idx >> 1, h = idx & 1;
      float S[4], A[4];
      fold(2 * h, m, S, A);
      fold(2 * h + 1, m, S + 2, A + 2);
      float* w = W + wrow(a, m, 0, it.g, kk) + 8 * it.hh + 4 * h;
      *reinterpret_cast<float4*>(w) = make_float4(S[0], S[1], S[2], S[3]);
      *reinterpret_cast<float4*>(w + a.wslab) = make_float4(A[0], A[1], A[2], A[3]);
    }
  } else {
    // one lane writes them
    for (int m = threadIdx.x; m < a.mmax; m += NT) {
      float S[8], A[8];
#pragma unroll
      for (int fl = 0; fl < FGW; ++fl) fold(fl, m, S + 2 * fl, A + 2 * fl);
      float* w = W + wrow(a, m, 0, it.g, kk) + 8 * it.hh;
      float4* ps = reinterpret_cast<float4*>(w);
      float4* pa = reinterpret_cast<float4*>(w + a.wslab);
      ps[0] = make_float4(S[0], S[1], S[2], S[3]);
      ps[1] = make_float4(S[4], S[5], S[6], S[7]);
      pa[0] = make_float4(A[0], A[1], A[2], A[3]);
      pa[1] = make_float4(A[4], A[5], A[6], A[7]);
    }
  }
}

template <class FFT>
__device__ __forceinline__ void dft_inverse_body(const DftArgs& a, const Item& it, const float* __restrict__ W,
                                                 float* __restrict__ x, const float2* __restrict__ tw,
                                                 const float* __restrict__ ring_scale, float2* lds) {
  constexpr int NF = FFT::N, NT = FFT::NT;
  const int N = NF > 0 ? NF : a.nlon;
  const int kk = it.kk;
  const int ks = a.nlat - 1 - kk;
  const bool eq = (ks == kk);
  const int f0 = 8 * it.g + 4 * it.hh;
  const int FS = field_stride(N);
  float2* ltw = lds + FGW * FS;
  TwiddleCopy<FFT> twc;
  const float hc = 0.5f * a.c_rest;
  // E = W[m][0], O = W[m][1] of this item's 4 fields -> spectra of the two
  // rings, placed at bins m and N - m of the packed sequence
  // (a pair of lanes reads the 32 bytes of one order and parity: fields 2 h
  // and 2 h + 1)
  auto place = [&](int m, int h, f32x4 e, f32x4 o) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float2* d = lds + (2 * h + i) * FS;
      const float2 E = make_float2(e[2 * i], e[2 * i + 1]);
      const float2 O = make_float2(o[2 * i], o[2 * i + 1]);
      const float2 yn = cadd(E, O);
      const float2 ys = eq ? make_float2(0.f, 0.f) : csub(E, O);
      if (m == 0) {
        d[0] = make_float2(yn.x, ys.x);
      } else {
        const float2 hn = cscale(yn, hc), hs = cscale(ys, hc);
        d[m] = make_float2(hn.x - hs.y, hn.y + hs.x);
        d[N - m] = make_float2(hn.x + hs.y, -hn.y + hs.x);
      }
    }
  };
  // all loads of the thread first (m < mmax <= N / 2), then the zeros of the
  // bins above the truncation and the loaded bins; order m has odd-parity
  // degrees only when m + 1 < lmax
  constexpr int PER = ceil_div(FFT::WIDEST, NT);
  f32x4 e[PER], o[PER];
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int idx = threadIdx.x + b * NT, m = idx >> 1;
    if (m < a.mmax) {
      const float* w = W + wrow(a, m, 0, it.g, kk) + 8 * it.hh + 4 * (idx & 1);
      e[b] = *(gcf32x4*)w;
      o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (m + 1 < a.lmax) o[b] = *(gcf32x4*)(w + a.wslab);
    }
  }
  twc.load(a, tw);
  twc.store(a, ltw);
  const int gap = N - 2 * a.mmax + 1;  // bins mmax .. N - mmax
  for (int i = threadIdx.x; i < gap; i += NT)
#pragma unroll
    for (int fl = 0; fl < FGW; ++fl) lds[fl * FS + a.mmax + i] = make_float2(0.f, 0.f);
#pragma unroll
  for (int b = 0; b < PER; ++b) {
    const int idx = threadIdx.x + b * NT, m = idx >> 1;
    if (m < a.mmax) place(m, idx & 1, e[b], o[b]);
  }
  lds_barrier();
  FFT::template run<true>(lds, ltw, a);
  const float2* Z = lds;
  const float sc = ring_scale[kk];
  const int nq = N / 4;
  const float rnq = 1.f / nq;
  if ((N & 3) == 0) {
    for (int idx = threadIdx.x; idx < FGW * nq; idx += NT) {
      const int fl = NF > 0 ? idx / nq : small_div(idx, rnq);
      const int j = 4 * (idx - fl * nq);
      const int fi = f0 + fl;
      if (fi >= a.F) continue;
      const float2* z = Z + fl * FS + j;
      const float2 z0 = z[0], z1 = z[1], z2 = z[2], z3 = z[3];
      *reinterpret_cast<float4*>(x + (static_cast<size_t>(fi) * a.nlat + kk) * N + j) =
          make_float4(z0.x * sc, z1.x * sc, z2.x * sc, z3.x * sc);
      if (!eq)
        *reinterpret_cast<float4*>(x + (static_cast<size_t>(fi) * a.nlat + ks) * N + j) =
            make_float4(z0.y * sc, z1.y * sc, z2.y * sc, z3.y * sc);
    }
  } else {
    for (int idx = threadIdx.x; idx < FGW * N; idx += NT) {
      const int fl = idx / N;
      const int j = idx - fl * N;
      const int fi = f0 + fl;
      if (fi >= a.F) continue;
      const float2 z = Z[fl * FS + j];
      x[(static_cast<size_t>(fi) * a.nlat + kk) * N + j] = z.x * sc;
      if (!eq) x[(static_cast<size_t>(fi) * a.nlat + ks) * N + j] = z.y * sc;
    }
  }
}

__device__ __forceinline__ DftArgs seg_args(const SegDev& sd, float c_rest) {
  DftArgs a;
  a.nlat = sd.g.nlat;
  a.nlon = sd.g.nlon;
  a.lmax = sd.g.lmax;
  a.mmax = sd.g.mmax;
  a.nk = sd.g.nk;
  a.F = sd.g.F;
  a.kpad = sd.g.kpad;
  a.G = sd.g.groups;
  a.wslab = sd.g.wslab;
  a.ntw = sd.ntw;
  a.npass = sd.npass;
  a.radix = sd.radix;
  a.c_rest = c_rest;
  return a;
}

template <class BLK>
using F1440 = FixedFFT<BLK, 1440, 9, 10, 16>;
template <class BLK>
using F720 = FixedFFT<BLK, 720, 9, 5, 16>;
template <class BLK>
using F360 = FixedFFT<BLK, 360, 9, 5, 8>;
template <class BLK>
using F64 = FixedFFT<BLK, 64, 4, 16, 1>;

// Batched kernels: workgroup b runs on XCD b % 8 and takes entry b / 8 of that
// XCD's list, segment after segment, field group after field group (segment s
// owns entries [dft_begin, dft_begin + groups * dft_chunk) of every list).
// Of a group's 2 nk items (ring pair kk, half hh) an XCD has one eighth
// (dft_items.h): all XCDs are on the same field group at a time, so that the
// part of W in flight, whose 128-byte lines are a stride of one order apart,
// stays within the last-level cache until a slab's neighbouring rings have
// joined (1024 fields at 360 x 720, forward: 528 -> 485 us against one
// contiguous slice of the whole numbering per XCD; 72 fields at 721 x 1440: 160
// -> 158).
__device__ __forceinline__ int segment_of(const SegDev* __restrict__ segs, int nseg, int slot) {
  int s = 0;
  while (s + 1 < nseg && slot >= segs[s + 1].dft_begin) ++s;
  return s;
}
__device__ __forceinline__ Item item_of(const SegDev& sd, int seg, int local) {
  Item it;
  it.g = local / sd.dft_chunk;
  const int i = dfti::item(blockIdx.x % 8, seg, it.g, local - it.g * sd.dft_chunk, sd.dft_chunk, sd.dft_step);
  it.kk = i >> 1;
  it.hh = i & 1;
  it.valid = it.kk < sd.g.nk && 8 * it.g + 4 * it.hh < sd.g.F;
  return it;
}

// GENERIC: some segment's width takes run-time radices.  Plans without one
// get kernels without that path: in the blocks of 512 threads it needs 77 to
// 80 VGPRs (six waves per SIMD), the compile-time widths 57 (eight), which is
// four workgroups on a CU instead of three up to width 720 (361 x 720 x 72
// fields, inverse: 41 -> 50 us with the shared kernel, 38 without).
// PAIRED: the form of the stores to W (dft_paired), a plan's choice and not
// a branch in the kernel: with both forms in one kernel the pairs' gain was
// lost (181 x 360 x 360 fields: 65 us instead of 54).
// mode 0: unit ring scale, 1: (2 pi / nlon) w_k, 2: zonal PSD into `zonal`
template <class BLK, bool GENERIC, bool PAIRED>
__global__ __launch_bounds__(BLK::NT) __attribute__((amdgpu_waves_per_eu(GENERIC ? 6 : 8))) void dft_forward_batched(
    const SegDev* __restrict__ segs, int nseg, const float* __restrict__ x, int mode,
    float* __restrict__ zonal) {
  extern __shared__ float2 lds[];
  const int slot = blockIdx.x / 8;
  const int seg = segment_of(segs, nseg, slot);
  const SegDev& sd = segs[seg];
  const DftArgs a = seg_args(sd, 1.f);
  const Item it = item_of(sd, seg, slot - sd.dft_begin);
  if (!it.valid) return;
  const float* xs = x + sd.grid_off;
  const float* scale = mode == 1 ? sd.scale_sht : mode == 2 ? sd.scale_zonal : sd.scale_one;
  float* zs = mode == 2 ? zonal : nullptr;
  auto run = [&](auto fft) { dft_forward_body<decltype(fft), PAIRED>(a, it, xs, sd.work, sd.tw, scale, lds, zs); };
  const int n = sd.g.nlon;
  if constexpr (BLK::WIDEST >= 1440)
    if (n == 1440) return run(F1440<BLK>());
  if constexpr (BLK::WIDEST >= 720)
    if (n == 720) return run(F720<BLK>());
  if constexpr (BLK::WIDEST >= 360)
    if (n == 360) return run(F360<BLK>());
  if (n == 64) return run(F64<BLK>());
  if constexpr (GENERIC) run(GenericFFT<BLK>());
}

template <class BLK, bool GENERIC>
__global__ __launch_bounds__(BLK::NT) __attribute__((amdgpu_waves_per_eu(GENERIC ? 6 : 8))) void dft_inverse_batched(
    const SegDev* __restrict__ segs, int nseg, float* __restrict__ x, int sht_scale, float c_rest) {
  extern __shared__ float2 lds[];
  const int slot = blockIdx.x / 8;
  const int seg = segment_of(segs, nseg, slot);
  const SegDev& sd = segs[seg];
  const DftArgs a = seg_args(sd, c_rest);
  const Item it = item_of(sd, seg, slot - sd.dft_begin);
  if (!it.valid) return;
  float* xs = x + sd.grid_off;
  const float* scale = sht_scale ? sd.scale_sht : sd.scale_one;
  auto run = [&](auto fft) { dft_inverse_body<decltype(fft)>(a, it, sd.work, xs, sd.tw, scale, lds); };
  const int n = sd.g.nlon;
  if constexpr (BLK::WIDEST >= 1440)
    if (n == 1440) return run(F1440<BLK>());
  if constexpr (BLK::WIDEST >= 720)
    if (n == 720) return run(F720<BLK>());
  if constexpr (BLK::WIDEST >= 360)
    if (n == 360) return run(F360<BLK>());
  if (n == 64) return run(F64<BLK>());
  if constexpr (GENERIC) run(GenericFFT<BLK>());
}

hipError_t prepare_lds(const void* k, size_t lds_bytes) {
  if (lds_bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
}

}  // namespace

namespace {

// Fewest passes; then an odd first radix (the first pass writes at a stride
// of its radix: an even one conflicts in the LDS banks), then the smallest
// largest radix.
struct RadixSearch {
  int n;
  int cur[kMaxRadices], best[kMaxRadices];
  int nbest = kMaxRadices + 1, best_odd = 0, best_max = 0;
  void go(int rest, int depth) {
    if (rest == 1) {
      const int odd = depth > 0 && cur[0] % 2 == 1;
      int mx = 0;
      for (int i = 0; i < depth; ++i) mx = std::max(mx, cur[i]);
      if (depth < nbest || (depth == nbest && (odd > best_odd || (odd == best_odd && mx < best_max)))) {
        nbest = depth;
        best_odd = odd;
        best_max = mx;
        std::copy(cur, cur + depth, best);
      }
      return;
    }
    if (depth >= kMaxRadices || depth >= nbest) return;
    for (int r : {16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2}) {
      if (rest % r || n > GenericFFT<Widest>::max_width(r)) continue;
      cur[depth] = r;
      go(rest / r, depth + 1);
    }
  }
};

template <class F>
bool fixed_plan(int n, DftPlan* p) {
  if (n != F::N) return false;
  p->npass = F::PASSES;
  for (int i = 0; i < F::PASSES; ++i) p->radix[i] = F::RADIX[i];
  return true;
}

}  // namespace

bool make_dft_plan(int n, DftPlan* p) {
  p->n = n;
  p->npass = 0;
  for (int i = 0; i < kMaxRadices; ++i) p->radix[i] = 1;
  if (!(fixed_plan<F1440<Widest>>(n, p) || fixed_plan<F720<Widest>>(n, p) || fixed_plan<F360<Widest>>(n, p) || fixed_plan<F64<Widest>>(n, p))) {
    RadixSearch s;
    s.n = n;
    s.go(n, 0);
    if (s.nbest > kMaxRadices) return false;
    p->npass = s.nbest;
    std::copy(s.best, s.best + s.nbest, p->radix);
  }
  int pr = 1;
  p->ntw = 0;
  for (int i = 0; i < p->npass; ++i) {
    p->ntw += pass_twiddles(p->radix[i], pr);
    pr *= p->radix[i];
  }
  return p->ntw <= n;
}

void dft_twiddles(const DftPlan& p, std::vector<float2>* out) {
  out->clear();
  int pr = 1;
  for (int i = 0; i < p.npass; ++i) {
    const int R = p.radix[i], B = twiddle_base(R);
    if (pr > 1) {
      for (int j = 0; j < twiddle_los(R) + twiddle_his(R); ++j) {
        const int q = j < twiddle_los(R) ? j + 1 : B * (j - twiddle_los(R) + 1);
        for (int k = 0; k < pr; ++k) {
          const double t = -2.0 * M_PI * static_cast<double>(q * k) / (static_cast<double>(pr) * R);
          out->push_back(make_float2(static_cast<float>(std::cos(t)), static_cast<float>(std::sin(t))));
        }
      }
    }
    pr *= R;
  }
}

// Forward stores of W.  A pair of lanes per 32-byte run makes half the L2
// requests of one lane with two 16-byte stores.  It loses where the lines in
// flight on an XCD (24 quads of workgroups x 2 mmax lines of 128 bytes) pass
// its 4 MiB of L2 and the workspace passes what the last-level cache can
// hold: lines are then written back before their four writers are done.
// Measured, forward, us, pair / single: 721 x 1440 (720 orders) at 72 fields
// (318 MB) 158 / 164, 80 (354 MB) 175 / 180, 96 (424 MB) 240 / 223, 144 (637
// MB) 360 / 308, 432 1060 / 885; 649 x 1296 (648 orders) at 144 fields 250 /
// 259; 541 x 1080 at 288 fields 322 / 331.  The Wide block has four workgroups
// on a CU, 32 quads: 451 x 900 (450 orders, 288 fields) 223 / 240, 481 x 960
// 261 / 247 to 291 / 247, 501 x 1000 321 / 259 (72 fields, 76 / 84).  Below it
// pairs never lost more than 2%: 289 x 576 (288 orders, 1000 fields) 357 /
// 350, 241 x 480 241 / 239, 201 x 400 171 / 185, 181 x 360 132 / 141.  A plan
// takes pairs when every segment does.
bool dft_paired(const SegGeom& g, int widest) {
  const int orders = widest > kForwardMiddle2 && widest <= kForwardWide ? 456 : 656;
  return g.mmax <= orders || 8LL * g.mmax * g.wslab <= (384LL << 20);
}

int dft_chunk(int nk) { return dfti::chunk(nk); }
int dft_step(int nk) { return dfti::step(nk); }

size_t dft_lds_bytes(const DftPlan& p) {
  return (static_cast<size_t>(FGW) * field_stride(p.n) + p.ntw) * sizeof(float2);
}

bool dft_is_fixed(const DftPlan& p) {
  return p.n == F1440<Widest>::N || p.n == F720<Widest>::N || p.n == F360<Widest>::N || p.n == F64<Widest>::N;
}

namespace {

// f(kernel, threads) for the kernel of a plan
template <class BLK, class F>
auto of_block_forward(const BatchArgs& b, F f) {
  if constexpr (BLK::WIDEST > Middle2::WIDEST)
    if (!b.dft_paired)
      return f(b.dft_generic ? dft_forward_batched<BLK, true, false> : dft_forward_batched<BLK, false, false>,
               BLK::NT);
  return f(b.dft_generic ? dft_forward_batched<BLK, true, true> : dft_forward_batched<BLK, false, true>, BLK::NT);
}
template <class F>
auto with_forward(const BatchArgs& b, F f) {
  const int w = b.dft_widest;
  if (w <= Narrow::WIDEST) return of_block_forward<Narrow>(b, f);
  if (w <= Middle::WIDEST) return of_block_forward<Middle>(b, f);
  if (w <= kForwardMiddle2) return of_block_forward<Middle2>(b, f);
  if (w <= kForwardWide) return of_block_forward<Wide>(b, f);
  return of_block_forward<Widest>(b, f);
}
template <class BLK, class F>
auto of_block_inverse(const BatchArgs& b, F f) {
  return f(b.dft_generic ? dft_inverse_batched<BLK, true> : dft_inverse_batched<BLK, false>, BLK::NT);
}
template <class F>
auto with_inverse(const BatchArgs& b, F f) {
  const int w = b.dft_widest;
  if (w <= Narrow::WIDEST) return of_block_inverse<Narrow>(b, f);
  if (w <= Middle::WIDEST) return of_block_inverse<Middle>(b, f);
  if (w <= Middle2::WIDEST) return of_block_inverse<Middle2>(b, f);
  if (w <= Wide::WIDEST) return of_block_inverse<Wide>(b, f);
  return of_block_inverse<Widest>(b, f);
}

hipError_t launch_forward(const BatchArgs& b, const float* x, int mode, float* zonal, hipStream_t st) {
  return with_forward(b, [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(8 * b.dft_per)), dim3(threads), b.dft_lds, st, b.segs,
                       b.nseg, x, mode, zonal);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t prepare_dft_kernels(const BatchArgs& b) {
  auto prepare = [&](auto kernel, int) { return prepare_lds(reinterpret_cast<const void*>(kernel), b.dft_lds); };
  const hipError_t e = with_forward(b, prepare);
  return e != hipSuccess ? e : with_inverse(b, prepare);
}

hipError_t launch_dft_forward_batched(const BatchArgs& b, const float* x, bool sht_scale, hipStream_t st) {
  return launch_forward(b, x, sht_scale ? 1 : 0, nullptr, st);
}

hipError_t launch_zonal_psd(const BatchArgs& b, const float* x, float* out, hipStream_t st) {
  return launch_forward(b, x, 2, out, st);
}

hipError_t launch_dft_inverse_batched(const BatchArgs& b, float* x, bool sht_scale, float c_rest, hipStream_t st) {
  return with_inverse(b, [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(8 * b.dft_per)), dim3(threads), b.dft_lds, st, b.segs,
                       b.nseg, x, sht_scale ? 1 : 0, c_rest);
    return hipGetLastError();
  });
}

}  // namespace sht
