// Per-degree complex channel mix: out[b,c',l,m] = sum_c W[l,c',c] in[b,c,l,m]
// (adjoint: conj(W[l,c,c'])), the multi-channel per-degree filter of the
// spectral convolution (App. B.4, eq. s2_spectral_conv: the filter depends on
// l only, never on m), and its weight gradient
// dW[l,c',c] = sum_{b,m<=l} g[b,c',l,m] conj(in[b,c,l,m]).
//
// For each degree l all three are a complex matrix product C = A B:
//   mix     : A = W_l   (C x C),  B = X_l (C x columns (b, m), m <= min(l, mmax-1))
//   adjoint : A = W_l^H,          B = X_l
//   dW      : A = G_l   (C x columns), B = X_l^H
// computed on the bf16 matrix cores with every float32 value split into three
// bf16 planes (six products, float32 accumulation; see bf16_planes.h), which
// carry the whole float32 value at 2.7 times the float32 matrix cores' rate.
// Both operands enter the split times 2^16 and the sums leave times 2^-32;
// outputs that are not finite (sums beyond 2^96, or of an infinity) are taken
// again on the float32 matrix cores.
//
// The contraction index runs over (re, im) pairs: a packed pair of bf16 is
// one complex value's plane, so the operand planes come straight from memory
// order.  With A's pairs (a_re, a_im) as they are, the real part of the
// product takes B's pairs as (b_re, -b_im) and the imaginary part as
// (b_im, b_re) (mix; the other two differ in signs): B's planes are stored
// to LDS in both arrangements, once per workgroup.
//
// Tile: 128 rows x 64 columns per workgroup; wave w has rows 32 w .. 32 w +
// 31 (two row blocks) and all four column blocks.  Its rows of A are its own
// (memory -> registers, one step of 16 complex values ahead); of B each wave
// loads and splits one column block per step.  Column blocks past the last
// column are left out (the columns of degree l are B (l + 1), so a tile is
// often ragged).  64 accumulator VGPRs and two 24 KiB LDS slots let three
// workgroups share a CU.
//
// Bound: instruction issue and the matrix cores.  Measured, us per launch,
// before (float32 matrix cores, 64 x 64 tiles, a separate kernel for the zeros
// of m > l, included) and now, mix / adjoint / weight gradient: 4 x 256
// channels, lmax 360: 1483 / 1610 / 1330 -> 799 / 860 / 661 (0.95 to
// 1.24 PFLOP/s of bf16 products); 1 x 677: 3074 / 3338 / 2510 -> 1575 / 1594 /
// 1333; 4 x 57, lmax 180: 52 / 57 / 90 -> 35 / 36 / 48.
#include "bf16_planes.h"
#include "internal.h"
#include "kernel_common.h"
#include "mix_members.h"
#include "mix_zeros.h"

namespace sht {
namespace {

using namespace planes;

enum class Product { Mix, MixAdjoint, WeightGrad };

constexpr int kRows = 128, kCols = 64;  // workgroup tile
constexpr int kStep = mixm::kStep;      // complex contraction indices per step
constexpr int kSlot = 4 * 2 * 3 * 64;   // v4f of one LDS slot: column blocks x arrangements x planes

constexpr float kSumScale = 1.f / (kSplitScale * kSplitScale);

// 16 bytes at 8-byte alignment (complex rows of odd length).
typedef float f32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef __attribute__((address_space(1))) const f32x4_a8 gc4_a8;
typedef __attribute__((address_space(1))) const f32x2 gc2;

// Workgroup -> (degree l, tile) with every tile of a degree on one XCD (the
// hardware deals workgroup b to XCD b % 8), so that the operands of degree l
// are fetched into one L2; the degrees with the most columns first.  The
// grid has 8 * ceil(lmax / 8) * T workgroups.
struct DegreeTile {
  int l, tile;
  __device__ __forceinline__ DegreeTile(int lmax, int T) {
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    l = lmax - 1 - (xcd + 8 * (slot / T));
    tile = slot % T;
  }
};

__device__ __forceinline__ bf16x8 flip(bf16x8 v, unsigned mask, bool swap) {
  u32x4 u = __builtin_bit_cast(u32x4, v);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (swap) u[i] = __builtin_amdgcn_alignbit(u[i], u[i], 16);
    u[i] ^= mask;
  }
  return __builtin_bit_cast(bf16x8, u);
}

__device__ __forceinline__ void split(const float* v, bf16x8* pl) {
  float up[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) up[e] = v[e] * kSplitScale;
  split8<3>(up, pl);
}

// B's second arrangement: (b_im, b_re), the signs as above; the first is
// (b_re, -b_im) for the mix and (b_re, b_im) for the other two.
template <Product P>
__device__ __forceinline__ bf16x8 first_arrangement(bf16x8 v) {
  return flip(v, P == Product::Mix ? 0x80000000u : 0u, false);
}
template <Product P>
__device__ __forceinline__ bf16x8 second_arrangement(bf16x8 v) {
  return flip(v, P == Product::Mix ? 0u : P == Product::MixAdjoint ? 0x80000000u : 0x00008000u, true);
}

// The operands of one degree.  A lane (li, lk) of a step holds row (or column)
// li and the four complex contraction indices 4 lk .. 4 lk + 3.
template <Product P>
struct Degree {
  static constexpr bool DW = P == Product::WeightGrad;
  int B, C, lmax, mmax, l;
  const float2 *Ap, *Bp;
  float2* out;
  int mcount;  // orders m <= l
  int ncols;
  int steps;
  bool one_row;       // mix_members.h
  float rmc;
  size_t plane;  // complex values of one field
  size_t wl;

  __device__ __forceinline__ Degree(int B, int C, int lmax, int mmax, int l, const float2* Ap, const float2* Bp,
                                    float2* out)
      : B(B), C(C), lmax(lmax), mmax(mmax), l(l), Ap(Ap), Bp(Bp), out(out) {
    mcount = (l + 1 < mmax) ? l + 1 : mmax;
    ncols = DW ? C : B * mcount;
    plane = static_cast<size_t>(lmax) * mmax;
    one_row = DW && mixm::one_row(B, mcount, C * plane);
    steps = DW ? mixm::steps(B, mcount, C * plane) : (C + kStep - 1) / kStep;
    rmc = 1.f / mcount;
    wl = static_cast<size_t>(l) * C * C;
  }
  // a column of B and a row of A, clamped
  __device__ __forceinline__ const float2* column(int col) const {
    col = min(col, ncols - 1);
    if constexpr (DW)
      return Bp + (static_cast<size_t>(col) * lmax + l) * mmax;
    else
      return Bp + (static_cast<size_t>(col / mcount) * C * lmax + l) * mmax + col % mcount;
  }
  __device__ __forceinline__ const float2* row(int row) const {
    row = min(row, C - 1);
    if constexpr (P == Product::Mix)
      return Ap + wl + static_cast<size_t>(row) * C;
    else if constexpr (P == Product::MixAdjoint)
      return Ap + wl + row;
    else
      return Ap + (static_cast<size_t>(row) * lmax + l) * mmax;
  }
  // output (0, col), and the distance from one row to the next
  __device__ __forceinline__ float2* output(int col) const {
    if constexpr (DW)
      return out + wl + col;
    else
      return out + (static_cast<size_t>(col / mcount) * C * lmax + l) * mmax + col % mcount;
  }
  __device__ __forceinline__ size_t ostride() const { return DW ? static_cast<size_t>(C) : plane; }

  // four complex values of this lane, contraction indices i0 .. i0 + 3 below
  // `end` (zero from there on), consecutive or `stride` complex values apart
  __device__ __forceinline__ static void load_run(const float2* p, int i0, int end, float* v) {
    if (i0 + 4 <= end) {
      gc4_a8* q = (gc4_a8*)(p + i0);
      const f32x4_a8 a = q[0], b = q[1];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = a[i];
        v[4 + i] = b[i];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f32x2 a = *(gc2*)(p + min(i0 + e, end - 1));
        v[2 * e] = i0 + e < end ? a[0] : 0.f;
        v[2 * e + 1] = i0 + e < end ? a[1] : 0.f;
      }
    }
  }
  __device__ __forceinline__ static void load_strided(const float2* p, size_t stride, int i0, int end, float* v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x2 a = *(gc2*)(p + static_cast<size_t>(min(i0 + e, end - 1)) * stride);
      v[2 * e] = i0 + e < end ? a[0] : 0.f;
      v[2 * e + 1] = i0 + e < end ? a[1] : 0.f;
    }
  }
  // A step of the contraction: its number, and of the weight gradient member by
  // member the member and its first order.
  struct Step {
    int s, b, i;
  };
  __device__ __forceinline__ Step first() const { return Step{0, 0, 0}; }
  __device__ __forceinline__ void next(Step& t) const {
    ++t.s;
    if constexpr (DW) {
      t.i += kStep;
      if (t.i >= mcount) {
        t.i = 0;
        ++t.b;
      }
    }
  }
  // Offsets of a lane's four columns (b, m) of a step, in one row; the same for
  // every row of A and column of B.
  struct Four {
    size_t at[4];
    int i0;
  };
  __device__ __forceinline__ Four four(int lk, int s) const {
    Four f;
    f.i0 = s * kStep + 4 * lk;
    const unsigned past = static_cast<unsigned>(C * plane - mcount);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = min(f.i0 + e, B * mcount - 1);
      f.at[e] = static_cast<unsigned long long>(static_cast<unsigned>(mixm::member_of(i, rmc))) * past + i;
    }
    return f;
  }
  __device__ __forceinline__ void load_four(const float2* p, const Four& f, int s, float* v) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x2 a = *(gc2*)(p + f.at[e]);
      v[2 * e] = a[0];
      v[2 * e + 1] = a[1];
    }
    if (s + 1 == steps) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (f.i0 + e >= B * mcount) v[2 * e] = v[2 * e + 1] = 0.f;
    }
  }
  // the same member by member
  __device__ __forceinline__ void load_member(const float2* p, int lk, const Step& t, float* v) const {
    load_run(p + t.b * (C * plane), t.i + 4 * lk, mcount, v);
  }
  // step t of N rows of A, and of a column of B
  template <int N>
  __device__ __forceinline__ void load_rows(const float2* const* base, int lk, const Step& t, float (*v)[8]) const {
    if constexpr (DW) {
      if (one_row) {
        const Four f = four(lk, t.s);
#pragma unroll
        for (int n = 0; n < N; ++n) load_four(base[n], f, t.s, v[n]);
        return;
      }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
      if constexpr (DW)
        load_member(base[n], lk, t, v[n]);
      else if constexpr (P == Product::Mix)
        load_run(base[n], t.s * kStep + 4 * lk, C, v[n]);
      else
        load_strided(base[n], static_cast<size_t>(C), t.s * kStep + 4 * lk, C, v[n]);
    }
  }
  __device__ __forceinline__ void load_column(const float2* base, int lk, const Step& t, float* v) const {
    if constexpr (DW)
      load_rows<1>(&base, lk, t, reinterpret_cast<float(*)[8]>(v));
    else
      load_strided(base, plane, t.s * kStep + 4 * lk, C, v);
  }

  // The 16 x 16 block at (row0, col0) on the float32 matrix cores, for the
  // outputs 4 lk + i, i in the bits of `want`, of this lane's column: float32's
  // own range, infinities included.  Straight from memory (4 x 256 channels,
  // lmax 360, every output beyond the range, us: mix 3587, adjoint 3412, weight
  // gradient 4690; a tiled kernel on these matrix cores 1425 / 1608 / 1332).
  __device__ __forceinline__ void exact_block(int row0, int col0, unsigned want, int li, int lk) const {
    const int col = col0 + li;
    const float2 *ab = row(row0 + li), *bb = column(col);
    floatx4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
    // an output whose row or column holds a NaN has its result
    float na = 0.f, nb = 0.f;
    for (Step t = first(); t.s < steps; next(t)) {
      float a[1][8], b[8];
      load_rows<1>(&ab, lk, t, a);
      load_column(bb, lk, t, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        na += a[0][e] != a[0][e] ? 1.f : 0.f;
        nb += b[e] != b[e] ? 1.f : 0.f;
      }
    }
    auto fold = [](unsigned long long v) { return static_cast<unsigned>(v | v >> 16 | v >> 32 | v >> 48) & 0xffffu; };
    const unsigned arows = fold(__ballot(na > 0.f)), bcols = fold(__ballot(nb > 0.f));
    want &= ~(arows >> (4 * lk));
    if ((bcols >> li) & 1) want = 0;
    if (!__any(want)) return;
    for (Step t = first(); t.s < steps; next(t)) {
      float a[1][8], b[8];
      load_rows<1>(&ab, lk, t, a);
      load_column(bb, lk, t, b);
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float br = b[e], bi = b[e + 1];
        re = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][e], br, re, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][e + 1], P == Product::Mix ? -bi : bi, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][e], DW ? -bi : bi, im, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][e + 1], P == Product::MixAdjoint ? -br : br, im, 0, 0, 0);
      }
    }
    if (col >= ncols) return;
    float2* o = output(col);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = row0 + 4 * lk + i;
      if (((want >> i) & 1) && r < C) o[static_cast<size_t>(r) * ostride()] = make_float2(re[i], im[i]);
    }
  }
};

template <Product P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void degree_product_kernel(
    int B, int C, int lmax, int mmax, const float2* __restrict__ Ap, const float2* __restrict__ Bp,
    float2* __restrict__ out) {
  constexpr bool DW = P == Product::WeightGrad;
  __shared__ v4f lds[2 * kSlot];
  const int tc = ((DW ? C : B * mmax) + kCols - 1) / kCols, tr = (C + kRows - 1) / kRows;
  const DegreeTile dt(lmax, tc * tr);
  if (dt.l < 0) return;
  const Degree<P> d(B, C, lmax, mmax, dt.l, Ap, Bp, out);
  const int mcount = d.mcount, ncols = d.ncols, steps = d.steps;
  const int r0 = (dt.tile / tc) * kRows, j0 = (dt.tile % tc) * kCols;
  const int tile = j0 / kCols, live = (ncols + kCols - 1) / kCols, nrow = min(kRows, C - r0) * B;
  if (tile >= live && (DW || mixz::by_live_tiles(tc, live, nrow))) return;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  // zeros of out (m > l), by the column tiles that mix_zeros.h names
  if constexpr (!DW) {
    const int nz = mmax - mcount;
    const mixz::Share z = mixz::share(tc, live, nrow, nz);
    if (nz > 0 && tile >= z.first && mixz::first_row(z, tile, 0, 0) < nrow) {
      for (int r = mixz::first_row(z, tile, threadIdx.x >> 6, lane); r < nrow; r += mixz::row_step(z)) {
        const int b = r % B, c = r0 + r / B;
        float2* o = out + ((static_cast<size_t>(b) * C + c) * lmax + dt.l) * mmax + mcount;
        for (int m = mixz::first_order(z, lane); m < nz; m += mixz::order_step(z)) o[m] = make_float2(0.f, 0.f);
      }
    }
    if (tile >= live) return;
  }
  // wave roles rotate, so that ragged row tiles do not load one SIMD more
  const int wave = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + (blockIdx.x >> 3)) & 3;
  const int row0 = r0 + 32 * wave;
  // this lane's column (of column block `wave`) and rows in the loads
  const float2* bbase = d.column(j0 + 16 * wave + li);
  const float2* abase[2] = {d.row(row0 + li), d.row(row0 + 16 + li)};
  // both arrangements of this wave's column block
  auto store_b = [&](int slot, const float* v) {
    bf16x8 pl[3];
    split(v, pl);
    v4f* t = lds + slot * kSlot + wave * 6 * 64 + lane;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      t[i * 64] = __builtin_bit_cast(v4f, first_arrangement<P>(pl[i]));
      t[(3 + i) * 64] = __builtin_bit_cast(v4f, second_arrangement<P>(pl[i]));
    }
  };

  // R row blocks of this wave, Q column blocks of the workgroup; returns the
  // outputs that are not finite, bit 4 (4 t + q) + i
  auto run = [&](auto r_c, auto q_c) {
    constexpr int R = decltype(r_c)::value, Q = decltype(q_c)::value, RR = R > 0 ? R : 1;
    floatx4 acc[RR][Q][2];
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[t][q][0] = acc[t][q][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    float araw[RR][8], braw[8];
    const bool bw = wave < Q;  // this wave has a column block to load
    auto ta = d.first(), tb = ta;  // the steps loaded last
    if (bw) d.load_column(bbase, lk, tb, braw);
    d.template load_rows<R>(abase, lk, ta, araw);
    if (bw) {
      store_b(0, braw);
      d.next(tb);
      if (steps > 1) d.load_column(bbase, lk, tb, braw);
    }
    lds_barrier();
    for (int s = 0; s < steps; ++s) {
      bf16x8 a[RR][3];
#pragma unroll
      for (int t = 0; t < R; ++t) split(araw[t], a[t]);
      d.next(ta);
      if (s + 1 < steps) d.template load_rows<R>(abase, lk, ta, araw);
      if constexpr (R > 0) {
        const v4f* slot = lds + (s & 1) * kSlot + lane;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          bf16x8 b[2][3];
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 3; ++i) b[h][i] = __builtin_bit_cast(bf16x8, slot[(q * 6 + h * 3 + i) * 64]);
          // products of the smaller planes first
#pragma unroll
          for (int k = 2; k >= 0; --k)
#pragma unroll
            for (int ia = 0; ia <= k; ++ia)
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < R; ++t)
                  acc[t][q][h] =
                      __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][ia], b[h][k - ia], acc[t][q][h], 0, 0, 0);
        }
      }
      if (s + 1 < steps && bw) {
        store_b((s + 1) & 1, braw);
        d.next(tb);
        if (s + 2 < steps) d.load_column(bbase, lk, tb, braw);
      }
      lds_barrier();
    }
    float zero = 0.f;  // NaN once a sum is not finite
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) zero = fmaf(acc[t][q][1][i], 0.f, fmaf(acc[t][q][0][i], 0.f, zero));
    unsigned bad = 0;
    if (__any(zero != zero)) {
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (!(fabsf(acc[t][q][0][i]) < __builtin_inff() && fabsf(acc[t][q][1][i]) < __builtin_inff()))
              bad |= 1u << (4 * (4 * t + q) + i);
    }
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[t][q][h] = acc[t][q][h] * kSumScale;
    // lane (li, lk) holds rows 4 lk + i of column li
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int col = j0 + 16 * q + li;
      if (col >= ncols) continue;
      float2* o = d.output(col);
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = row0 + 16 * t + 4 * lk + i;
          if (row < C)
            o[static_cast<size_t>(row) * d.ostride()] = make_float2(acc[t][q][0][i], acc[t][q][1][i]);
        }
    }
    return bad;
  };
  const int nq = min(4, (ncols - j0 + 15) >> 4);
  auto rows = [&](auto q_c) {
    if (row0 + 16 < C) return run(std::integral_constant<int, 2>{}, q_c);
    if (row0 < C) return run(std::integral_constant<int, 1>{}, q_c);
    return run(std::integral_constant<int, 0>{}, q_c);
  };
  unsigned bad;
  switch (nq) {
    case 1: bad = rows(std::integral_constant<int, 1>{}); break;
    case 2: bad = rows(std::integral_constant<int, 2>{}); break;
    case 3: bad = rows(std::integral_constant<int, 3>{}); break;
    default: bad = rows(std::integral_constant<int, 4>{}); break;
  }
  if (__any(bad)) {
    int lane1 = lane;  // the addresses are formed anew, not held through the main loop
    asm volatile("" : "+v"(lane1));
    for (int tq = 0; tq < 8; ++tq) {
      const unsigned want = (bad >> (4 * tq)) & 15u;
      if (__any(want)) d.exact_block(row0 + 16 * (tq >> 2), j0 + 16 * (tq & 3), want, lane1 & 15, lane1 >> 4);
    }
  }
}

// The weight gradient by waves of one 16 x 16 block each, for products whose
// 128 x 64 tiles leave most of the chip idle (64 channels are one tile a degree):
// no LDS and no barrier, both operands straight to registers kAhead steps ahead,
// the same steps and products in the same order (the same bits).  Bound: a
// wave's instructions, about 0.9 us a step (a tile's step 1.9 to 2.3 us), and
// with many waves their sum, about 1 ns a wave and step.
constexpr int kAhead = 3;
__global__ __launch_bounds__(256) void gradient_block_kernel(int B, int C, int lmax, int mmax,
                                                             const float2* __restrict__ g,
                                                             const float2* __restrict__ x, float2* __restrict__ dW) {
  constexpr Product P = Product::WeightGrad;
  const int nb = (C + 15) / 16;
  const DegreeTile dt(lmax, (nb * nb + 3) / 4);
  const int block = 4 * dt.tile + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (dt.l < 0 || block >= nb * nb) return;
  const Degree<P> d(B, C, lmax, mmax, dt.l, g, x, dW);
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4, steps = d.steps;
  const int row0 = 16 * (block / nb), col = 16 * (block % nb) + li;
  const float2 *abase = d.row(row0 + li), *bbase = d.column(col);
  floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
  auto run = [&](auto one_row_c) {
    float a[kAhead][8], b[kAhead][8];
    auto t = d.first();  // the step to load next
    auto load = [&](float* va, float* vb) {
      if (t.s >= steps) return;
      if constexpr (decltype(one_row_c)::value) {
        const auto f = d.four(lk, t.s);
        d.load_four(abase, f, t.s, va);
        d.load_four(bbase, f, t.s, vb);
      } else {
        d.load_member(abase, lk, t, va);
        d.load_member(bbase, lk, t, vb);
      }
      d.next(t);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(a[u], b[u]);
    for (int s0 = 0; s0 < steps; s0 += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (s0 + u >= steps) break;
        bf16x8 pa[3], pb[2][3];
        split(a[u], pa);
        split(b[u], pb[0]);
        load(a[u], b[u]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          pb[1][i] = second_arrangement<P>(pb[0][i]);
          pb[0][i] = first_arrangement<P>(pb[0][i]);
        }
#pragma unroll
        for (int k = 2; k >= 0; --k)
#pragma unroll
          for (int ia = 0; ia <= k; ++ia)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[ia], pb[h][k - ia], acc[h], 0, 0, 0);
      }
    }
  };
  if (d.one_row)
    run(std::true_type{});
  else
    run(std::false_type{});
  unsigned bad = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!(fabsf(acc[0][i]) < __builtin_inff() && fabsf(acc[1][i]) < __builtin_inff())) bad |= 1u << i;
    const int row = row0 + 4 * lk + i;
    if (row < C && col < C)
      d.output(col)[static_cast<size_t>(row) * d.ostride()] = make_float2(acc[0][i] * kSumScale, acc[1][i] * kSumScale);
  }
  if (__any(bad)) d.exact_block(row0, 16 * (block % nb), bad, li, lk);
}

// Isotropic per-channel filter, the single-channel form of eq.
// s2_spectral_conv: out[b,c,l,m] = k[c,l] in[b,c,l,m] (adjoint: conj(k)),
// 0 for m > l.  Elementwise and HBM-bound: one thread per coefficient,
// consecutive threads on consecutive m.
// Grid: x = spectral row (b, c, l), y = 256-order slice; 32-bit indices.
__global__ __launch_bounds__(256) void isotropic_filter_kernel(int C, int lmax, int mmax,
                                                               const float2* __restrict__ k,
                                                               const float2* __restrict__ in,
                                                               float2* __restrict__ out, int adjoint) {
  const int row = static_cast<int>(blockIdx.x);
  const int m = static_cast<int>(blockIdx.y) * 256 + static_cast<int>(threadIdx.x);
  if (m >= mmax) return;
  const int f = row / lmax;
  const int l = row - f * lmax;
  const int c = f % C;
  const long long i = static_cast<long long>(row) * mmax + m;
  if (m > l) {
    out[i] = make_float2(0.f, 0.f);
    return;
  }
  const float2 kv = k[static_cast<long long>(c) * lmax + l];
  const float ki = adjoint ? -kv.y : kv.y;
  const float2 x = in[i];
  out[i] = make_float2(kv.x * x.x - ki * x.y, kv.x * x.y + ki * x.x);
}

// Filter gradient dk[c,l] = sum_b sum_{m <= min(l, mmax-1)} g conj(x): one
// wave per (c, l); lanes over m, members in order, a fixed-order wave sum.
__global__ __launch_bounds__(256) void isotropic_filter_grad_kernel(int B, int C, int lmax, int mmax,
                                                                    const float2* __restrict__ g,
                                                                    const float2* __restrict__ x,
                                                                    float2* __restrict__ dk) {
  const int lane = threadIdx.x & 63;
  const long long row = static_cast<long long>(blockIdx.x) * 4 + (threadIdx.x >> 6);  // c * lmax + l
  if (row >= static_cast<long long>(C) * lmax) return;
  const int l = static_cast<int>(row % lmax);
  const int mend = min(l + 1, mmax);
  float re = 0.f, im = 0.f;
  for (int b = 0; b < B; ++b) {
    const long long base = (static_cast<long long>(b) * C * lmax + row) * mmax;
    for (int m = lane; m < mend; m += 64) {
      const float2 gv = g[base + m], xv = x[base + m];
      re += gv.x * xv.x + gv.y * xv.y;
      im += gv.y * xv.x - gv.x * xv.y;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    re += __shfl_xor(re, off, 64);
    im += __shfl_xor(im, off, 64);
  }
  if (lane == 0) dk[row] = make_float2(re, im);
}

}  // namespace

hipError_t launch_channel_mix_weight_grad(int batch, int channels, int lmax, int mmax, const float2* g,
                                          const float2* x, float2* dW, hipStream_t stream) {
  const long long tiles =
      static_cast<long long>((channels + kCols - 1) / kCols) * ((channels + kRows - 1) / kRows);
  const long long blocks = 8LL * ((lmax + 7) / 8) * tiles;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // Blocks where their waves, weighted with the share of the longest
  // contraction that their degree has, are few enough for a wave's own time to
  // decide.  Measured, us, tiles / blocks, at the weighted number of waves: 64 x
  // 64 channels, lmax 32 (264) 278 / 112, 4 x 57, 180 (1448) 89 / 48, 4 x 96, 120
  // (2178) 59 / 49, 64 x 256, 16 (2176) 172 / 143, 16 x 96, 64 x 10 orders (2142)
  // 24 / 29, 2 x 200, 30 (2620) 13.5 / 13.3, 1 x 57, 360 (2888) 46 / 43, 64 x 96,
  // 200 x 4 (7146) 55 / 122, 4 x 256, 90 (11648) 61 / 132.
  const long long nb = (channels + 15) / 16;
  const double orders = mmax * (mmax + 1) / 2.0 + static_cast<double>(lmax - mmax) * mmax;  // of all degrees
  if (orders / mmax * nb * nb <= 2200.0) {
    const long long block_groups = 8LL * ((lmax + 7) / 8) * ((nb * nb + 3) / 4);
    hipLaunchKernelGGL(gradient_block_kernel, dim3(static_cast<unsigned>(block_groups)), dim3(256), 0, stream, batch,
                       channels, lmax, mmax, g, x, dW);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(degree_product_kernel<Product::WeightGrad>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                     stream, batch, channels, lmax, mmax, g, x, dW);
  return hipGetLastError();
}

hipError_t launch_channel_mix(int batch, int channels, int lmax, int mmax, const float2* W,
                              const float2* in, float2* out, int adjoint, hipStream_t stream) {
  const long long tiles = (static_cast<long long>(batch) * mmax + kCols - 1) / kCols * ((channels + kRows - 1) / kRows);
  const long long blocks = 8LL * ((lmax + 7) / 8) * tiles;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const long long rows = static_cast<long long>(batch) * channels * lmax;
  if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks));
  if (adjoint)
    hipLaunchKernelGGL(degree_product_kernel<Product::MixAdjoint>, grid, dim3(256), 0, stream, batch, channels, lmax,
                       mmax, W, in, out);
  else
    hipLaunchKernelGGL(degree_product_kernel<Product::Mix>, grid, dim3(256), 0, stream, batch, channels, lmax, mmax, W,
                       in, out);
  return hipGetLastError();
}

}  // namespace sht

namespace sht {

hipError_t launch_isotropic_filter(int batch, int channels, int lmax, int mmax, const float2* k, const float2* in,
                                   float2* out, int adjoint, hipStream_t stream) {
  const long long rows = static_cast<long long>(batch) * channels * lmax;
  if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
  if (rows == 0 || mmax <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(rows), static_cast<unsigned>((mmax + 255) / 256));
  hipLaunchKernelGGL(isotropic_filter_kernel, grid, dim3(256), 0, stream, channels, lmax, mmax, k, in, out,
                     adjoint);
  return hipGetLastError();
}

hipError_t launch_isotropic_filter_grad(int batch, int channels, int lmax, int mmax, const float2* g,
                                        const float2* x, float2* dk, hipStream_t stream) {
  const long long rows = static_cast<long long>(channels) * lmax;
  hipLaunchKernelGGL(isotropic_filter_grad_kernel, dim3(static_cast<unsigned>((rows + 3) / 4)), dim3(256), 0, stream,
                     batch, channels, lmax, mmax, g, x, dk);
  return hipGetLastError();
}

}  // namespace sht
