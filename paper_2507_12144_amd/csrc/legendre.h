// Legendre contraction kernels: the per-order-m dense contraction of Alg. 1
// (xc_{bclm} = sum_k L_{mlk} x_{bckm}) and its synthesis counterpart
// (eq. isht), on CDNA4's bf16 matrix cores (v_mfma_f32_16x16x32_bf16,
// float32 accumulation) in every precision form.
//
// Folded form.  With nodes symmetric about the equator,
// P^_l^m(-x) = (-1)^(l+m) P^_l^m(x), so for each m the degrees split by
// parity p = (l - m) & 1 and only the northern rings k < nk are needed:
//   analysis : u^[l] = sum_{k<nk} P^_l^m(x_k) (p == 0 ? S_k : A_k)
//   synthesis: E_k = sum_{p=0 rows} P^ u^,  O_k = sum_{p=1 rows} P^ u^,
//              north ring = E + O, mirrored ring = E - O
// which halves the multiply-adds.  S, A, E, O live in the workspace
// W[m][p][g][k][16] (g = group of 8 fields, 16 = their re/im).
//
// Precision forms.  The table a and the data b enter the matrix cores as
// bf16 planes, a = sum_i a_i, b = sum_j b_j, each plane the rounding to
// nearest of what the earlier ones left:
//   float32 : the table is held in float32 and split into three planes in
//             registers; all a_i b_j with i + j < 3 (six products).  Three
//             planes of 8 significant bits carry the whole float32 value;
//             the largest products left out, a_1 b_2 and a_2 b_1, are at most
//             2^-24 of a term each.  Against the
//             float64 oracle the results are nearer than those of the
//             float32 matrix cores (fewer roundings per sum: 6 per 32 terms
//             instead of one per term), which have a tenth of the rate.
//             Range: table and data enter the planes times 2^16, so that the
//             third plane of the smallest subnormal is a bf16 value, and the
//             sums leave times 2^-32.  Sums that pass 2^96 (or whose data
//             hold an infinity or NaN) come out non-finite; the columns they
//             are in are taken again on the float32 matrix cores.
//   bf16    : one plane of each, a_0 b_0
//   bf16x2  : two table planes (split from float64), three data planes,
//             a_0 b_0 + a_0 b_1 + a_1 b_0 + a_0 b_2 + a_1 b_1
//   bf16x3  : three table planes, three data planes, six products
//
// Tiling.  Per (segment, m, parity) both directions are one matrix product
// C[rows][columns] = A[rows][K] B[K][columns] with A the table (analysis:
// rows = degrees of the parity, K = rings; synthesis: rows = rings, K =
// degrees) and B the data (columns = re/im of the fields).  A workgroup of
// four waves computes a tile of at most 8 row blocks of 16 rows by CB column
// blocks of 16 columns (CB <= 9 field groups) through K steps of 32.
//  * A is private to a wave (row blocks w and w + 4 of the tile): its
//    fragments go straight from memory to registers, 16 bytes a lane, one
//    step ahead.  Every table entry is read by one wave per column chunk,
//    and 72 fields (9 groups) are a single chunk: the table streams from HBM
//    once per transform.
//  * B is shared: each wave loads whole 32 x 16 pieces (2 KiB) one step
//    ahead, splits them once per workgroup and stores the planes to LDS in
//    fragment order.  LDS barriers only, which leave the loads of the
//    following step in flight.
// C stays in registers (at most 18 blocks, 72 VGPRs a lane).
//
// Bound: memory at few column chunks (721 x 1440, 72 fields, float32: about
// 0.9 GB of table, workspace and tiles in 0.21 ms), instruction issue (splits
// and matrix instructions) at many.  What decides is that three waves share a
// SIMD, so that one's matrix instructions run while the others load, split or
// wait at a barrier; see single_slot.  Measured, us per launch, analysis /
// synthesis with staged spectra: 721 x 1440 x 72 fields 223 / 199 (float32
// matrix cores with an LDS ring for the table: 320 / 359), x 128 fields
// 339 / 321 (503 / 532), Gauss 360 x 720 x 1024 fields 455 / 487 (615 / 663);
// split bf16, 721 x 1440 x 72: 223 / 193 (252 / 255).  Of the float32 figures the
// scaling and the test of the sums are 0 to 3% (without: 225 / 196, 331 / 313,
// 449 / 474), up to 6% of a synthesis of few degrees (361 x 720 x 72: 41.8, 44.3).
#pragma once

#include <type_traits>

#include "bf16_planes.h"
#include "internal.h"
#include "kernel_common.h"

namespace sht {
namespace legk {

using namespace planes;

// Planes of a form: table pieces of 1 KiB per (16-row block, K step), table
// planes and data planes in the products.
template <Storage S>
struct Form;
template <>
struct Form<Storage::F32> {
  static constexpr int PIECES = 2, NP = 3, ND = 3;
};
template <>
struct Form<Storage::BF16> {
  static constexpr int PIECES = 1, NP = 1, ND = 1;
};
template <>
struct Form<Storage::BF16X2> {
  static constexpr int PIECES = 2, NP = 2, ND = 3;
};
template <>
struct Form<Storage::BF16X3> {
  static constexpr int PIECES = 3, NP = 3, ND = 3;
};

// The table fragment of a row block in planes, from its raw pieces.
template <Storage S>
__device__ __forceinline__ void table_planes(const v4f* raw, bf16x8* out) {
  if constexpr (S == Storage::F32) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = raw[e >> 2][e & 3];
    split8<3>(v, out);
  } else {
#pragma unroll
    for (int pl = 0; pl < Form<S>::NP; ++pl) out[pl] = __builtin_bit_cast(bf16x8, raw[pl]);
  }
}

// Powers of two by which float32 operands are scaled up before a split.
template <Storage S>
constexpr float kSplitUp = S == Storage::F32 ? planes::kSplitScale : 1.f;
template <Storage S>
constexpr float kSumDown = 1.f / (kSplitUp<S> * kSplitUp<S>);

constexpr int kTileBlocks = 8;  // row blocks of 16 per workgroup tile (two per wave)
constexpr int kMaxCb = 9;       // column blocks (field groups) per workgroup tile
// The three-plane form keeps its analysis's correction products in a sum of
// their own (rel-L2 against float64 at 360 x 720: 1.2e-7; in one sum 1.7e-7,
// which is the float32 form's), for twice the accumulators: narrower tiles.
template <Storage S, bool SYN>
constexpr bool own_corrections = S == Storage::BF16X3 && !SYN;
template <Storage S, bool SYN>
constexpr int max_cb = own_corrections<S, SYN> ? 4 : kMaxCb;

// Data slots in LDS, CB blocks x ND planes x 1 KiB each.  Two slots take one
// barrier per step.  At nine column blocks two slots of three planes are
// 54 KiB, which leaves room for only two workgroups on a CU (160 KiB), and a
// wave needs 181 VGPRs (two waves per SIMD); one slot with a second barrier
// and one column block's fragments at a time (164 VGPRs) lets three in:
// 721 x 1440 x 72 fields, float32, analysis / synthesis 254 / 230 -> 226 /
// 201 us, 181 x 360 x 360 fields 54 / 52 -> 47 / 44.  With eight blocks three
// fit either way and the single slot measured the same (325 / 309 against
// 330 / 308 us at 128 fields).
constexpr bool single_slot(int cb) { return cb == kMaxCb; }
template <Storage S>
constexpr int lds_v4(int cb) {
  return (single_slot(cb) ? 1 : 2) * cb * Form<S>::ND * 64;
}

// One tile.  Work item: order m, parity p, row tile rt, column chunk c of
// `cbs` field groups (the last one may be ragged).  Column block q of the
// tile is field group c * cbs + q; blocks past the last group repeat it and
// are not stored.
//
// Fragments: lane (li, lk) of a K step holds row (or column) li and the
// eight contraction indices 32 s + 4 e + lk, e < 8, of table and data alike.
// The data is the matrix cores' first operand, so that a lane receives
// columns 4 lk .. 4 lk + 3 of row li: 16 bytes, a block is 1 KiB contiguous.
template <Storage S, int CB, bool SYN, bool STG>
__device__ __forceinline__ void tile_body(const SegDev& sd, int m, int p, int rt, int c, int cbs, int rot,
                                          const float2* __restrict__ yin, float2* __restrict__ yout, float c_rest,
                                          v4f* lds, unsigned* bad) {
  using FM = Form<S>;
  constexpr int ND = FM::ND, NP = FM::NP, PIECES = FM::PIECES;
  constexpr int UN = (CB + 3) / 4;  // data pieces per wave and step
  constexpr bool SINGLE = single_slot(CB);
  constexpr int Q2 = SINGLE ? 1 : 2;  // column blocks worked on at a time
  const SegGeom& g = sd.g;
  const int lane = threadIdx.x & 63;
  // wave roles rotate with the workgroup, so that tiles with fewer row blocks
  // than waves do not load one SIMD of every CU more than the others
  const int wave = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + rot) & 3;
  const int li = lane & 15, lk = lane >> 4;
  const int n0 = (g.lmax - m + 1) >> 1;             // degrees of parity 0
  const int np = p ? (g.lmax - m) >> 1 : n0;        // of this parity
  const int nb16 = (n0 + 15) >> 4;                  // 16-row blocks of a parity region
  const int kst = g.kpad >> 5;                      // K steps over the rings
  const int steps = SYN ? (np + 31) >> 5 : kst;
  const int steps_mem = SYN ? (n0 + 31) >> 5 : kst; // as laid out
  const int rows_mem = SYN ? (g.nk + 15) >> 4 : nb16;
  const int nblk = SYN ? rows_mem : (np + 15) >> 4; // row blocks with content
  const int ntile = (nblk + kTileBlocks - 1) / kTileBlocks;
  // even split of the row blocks over the tiles
  const int rb0 = nblk * rt / ntile, rb1 = nblk * (rt + 1) / ntile;
  const int ra = rb0 + wave, rb = rb0 + wave + 4;
  const bool va = ra < rb1, vb = rb < rb1;

  auto table = [&](int lane) {
    return (gcv4f*)(SYN ? sd.tab_syn : sd.tab_ana) +
           static_cast<size_t>(SYN ? sd.syn_off[m] : sd.ana_off[m]) * PIECES * 64 +
           static_cast<size_t>(p) * rows_mem * steps_mem * PIECES * 64 + lane;
  };
  gcv4f* tab = table(lane);
  gcv4f* ta = tab + static_cast<size_t>(va ? ra : rb0) * steps_mem * PIECES * 64;
  gcv4f* tb = tab + static_cast<size_t>(vb ? rb : rb0) * steps_mem * PIECES * 64;

  // data pieces of this wave: column blocks wave, wave + 4, ...
  struct Source {
    int lk;
    gcfloat* at[UN];
    int step[UN];  // floats from one degree of the parity to the next (direct synthesis)
  };
  auto source = [&](int wave, int lane) {
    Source b;
    const int li = lane & 15;
    b.lk = lane >> 4;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int q = wave + 4 * u < CB ? wave + 4 * u : CB - 1;
      const int gi = c * cbs + q < g.groups ? c * cbs + q : g.groups - 1;
      b.step[u] = 0;
      if constexpr (!SYN) {
        b.at[u] = (gcfloat*)sd.work + static_cast<size_t>(2 * m + p) * g.wslab + static_cast<size_t>(gi) * g.kpad * 16 + lane;
      } else if constexpr (STG) {
        b.at[u] = (gcfloat*)sd.ystage + sd.ystage_off[m] + (static_cast<size_t>(p) * g.groups + gi) * nb16 * 256 + li;
      } else {
        // re (li even) or im of field 8 gi + li / 2 (field 0 past the last one)
        const int f = 8 * gi + (li >> 1) < g.F ? 8 * gi + (li >> 1) : 0;
        b.at[u] = (gcfloat*)yin + ((static_cast<size_t>(f) * g.lmax + m + p) * g.mmax + m) * 2 + (li & 1);
        b.step[u] = 4 * g.mmax;
      }
    }
    return b;
  };
  auto load_b = [&](const Source& b, int s, float (*raw)[8]) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (wave + 4 * u < CB) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if constexpr (!SYN) {
            raw[u][e] = b.at[u][s * 512 + e * 64];
          } else {
            // rows past the parity's last degree are zero whatever memory holds
            const int i = 32 * s + 4 * e + b.lk;
            const int ic = i < np ? i : 0;
            const float v = STG ? b.at[u][ic * 16] : b.at[u][static_cast<size_t>(ic) * b.step[u]];
            raw[u][e] = i < np ? v : 0.f;
          }
        }
      }
    }
  };
  auto store_b = [&](int slot, float (*raw)[8]) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      if (wave + 4 * u < CB) {
        bf16x8 pl[ND];
        float up[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) up[e] = raw[u][e] * kSplitUp<S>;
        split8<ND>(up, pl);
        v4f* d = lds + slot * (CB * ND * 64) + (wave + 4 * u) * ND * 64 + lane;
#pragma unroll
        for (int i = 0; i < ND; ++i) d[i * 64] = __builtin_bit_cast(v4f, pl[i]);
      }
    }
  };

  // The tile on the float32 matrix cores, for the columns flagged in `bad`:
  // float32's own range, infinities included.  One LDS slot of raw values, no
  // loads ahead: what takes this path is out of the range of data in earnest
  // (721 x 1440 x 72 fields, us, analysis / synthesis: 224 / 193, of size
  // 1e36 600 / 597; a pipelined kernel on these matrix cores 309 / 375).
  auto exact_range = [&](auto r_c, auto& put, float ms) {
    constexpr int R = decltype(r_c)::value, RR = R > 0 ? R : 1;
    // its addresses are formed anew: held through the main loop they would
    // spill (the synthesis, from six column blocks on)
    int lane1 = threadIdx.x & 63, w1 = wave;
    asm volatile("" : "+v"(lane1), "+s"(w1));
    const Source src = source(w1, lane1);
    gcv4f* tab1 = table(lane1);
    // a column with a NaN in it has its result: NaN in every row
    float sum[UN] = {};
    for (int s = 0; s < steps; ++s) {
      float braw[UN][8];
      load_b(src, s, braw);
#pragma unroll
      for (int u = 0; u < UN; ++u)
        if (wave + 4 * u < CB)
#pragma unroll
          for (int e = 0; e < 8; ++e) sum[u] += braw[u][e] != braw[u][e] ? 1.f : 0.f;
    }
    lds_barrier();  // every wave has seen that the workgroup takes this path
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (wave + 4 * u < CB && sum[u] > 0.f) atomicAnd(&bad[wave + 4 * u], ~(1u << li));
    lds_barrier();
    unsigned any = 0;
#pragma unroll
    for (int q = 0; q < CB; ++q) any |= bad[q];
    if (!__builtin_amdgcn_readfirstlane(any)) return;
    floatx4 acc[RR][CB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < CB; ++q) acc[r][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < steps; ++s) {
      float braw[UN][8];
      load_b(src, s, braw);
      if (s > 0) lds_barrier();  // every wave has read the slot
#pragma unroll
      for (int u = 0; u < UN; ++u)
        if (wave + 4 * u < CB) {
          v4f* d = lds + (wave + 4 * u) * 2 * 64 + lane;
          d[0] = v4f{braw[u][0], braw[u][1], braw[u][2], braw[u][3]};
          d[64] = v4f{braw[u][4], braw[u][5], braw[u][6], braw[u][7]};
        }
      v4f a[RR][2];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i) a[r][i] = tab1[((r ? rb : ra) * steps_mem + s) * PIECES * 64 + i * 64] * (1.f / kSplitUp<S>);
      lds_barrier();
#pragma unroll
      for (int q = 0; q < CB; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const v4f b = lds[(q * 2 + h) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < R; ++r)
              acc[r][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[r][h][e], acc[r][q], 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < CB; ++q) put(r, q, acc[r][q] * ms, (bad[q] >> (4 * lk)) & 15u);
  };

  // R row blocks of this wave (2, 1 or none)
  auto run = [&](auto r_c) {
    constexpr int R = decltype(r_c)::value;
    constexpr bool CORR = own_corrections<S, SYN>;
    const Source src = source(wave, lane);
    floatx4 acc[R > 0 ? R : 1][CB], corr[R > 0 ? R : 1][CORR ? CB : 1];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        acc[r][q] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (CORR) corr[r][q] = acc[r][q];
      }
    v4f araw[R > 0 ? R : 1][PIECES];
    float braw[UN][8];
    auto load_a = [&](int s) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < PIECES; ++i) araw[r][i] = (r ? tb : ta)[(s * PIECES + i) * 64];
    };
    if constexpr (S == Storage::F32)
      if (threadIdx.x < CB) bad[threadIdx.x] = 0;
    load_b(src, 0, braw);
    load_a(0);
    store_b(0, braw);
    if (steps > 1) load_b(src, 1, braw);
    lds_barrier();
    for (int s = 0; s < steps; ++s) {
      bf16x8 a[R > 0 ? R : 1][NP];
#pragma unroll
      for (int r = 0; r < R; ++r) table_planes<S>(araw[r], a[r]);
      if (s + 1 < steps) load_a(s + 1);
      const v4f* slot = lds + (SINGLE ? 0 : s & 1) * (CB * ND * 64) + lane;
      if constexpr (R > 0) {
        // R * Q2 independent accumulator chains
#pragma unroll
        for (int q = 0; q < CB; q += Q2) {
          bf16x8 b[Q2][ND];
#pragma unroll
          for (int h = 0; h < Q2; ++h)
            if (q + h < CB) {
#pragma unroll
              for (int i = 0; i < ND; ++i) b[h][i] = __builtin_bit_cast(bf16x8, slot[((q + h) * ND + i) * 64]);
            }
          // products of the smaller planes first: what a step adds to a sum
          // that is still small is rounded at the small sum's size
#pragma unroll
          for (int d = ND - 1; d >= 0; --d)
#pragma unroll
            for (int ia = 0; ia <= d && ia < NP; ++ia) {
#pragma unroll
              for (int h = 0; h < Q2; ++h)
                if (q + h < CB) {
#pragma unroll
                  for (int r = 0; r < R; ++r) {
                    floatx4& t = CORR && d > 0 ? corr[r][CORR ? q + h : 0] : acc[r][q + h];
                    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h][d - ia], a[r][ia], t, 0, 0, 0);
                  }
                }
            }
        }
      }
      if (s + 1 < steps) {
        if constexpr (SINGLE) lds_barrier();  // every wave has read the slot
        store_b(SINGLE ? 0 : (s + 1) & 1, braw);
        if (s + 2 < steps) load_b(src, s + 2, braw);
      }
      lds_barrier();
    }
    const float ms = (SYN || m == 0) ? 1.f : c_rest;
    // components of v: columns 4 lk .. 4 lk + 3 of column block q at row li
    // of the wave's row block r; those in `cols` are stored
    auto put = [&](int r, int q, floatx4 v, unsigned cols) {
      const int blk = r ? rb : ra, gi = c * cbs + q;
      if (gi >= g.groups || q >= cbs) return;
      auto store4 = [&](gfloat* d) {
        if (cols == 15u) {
          *(gfloatx4*)d = v;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((cols >> i) & 1) d[i] = v[i];
        }
      };
      if constexpr (SYN) {
        // the padding rings stay zero, whatever the data held
        if (16 * blk + li >= g.nk) return;
        store4(as_global(sd.work) + static_cast<size_t>(2 * m + p) * g.wslab +
               (static_cast<size_t>(gi) * g.kpad + 16 * blk + li) * 16 + 4 * lk);
      } else if constexpr (STG) {
        store4(as_global(sd.ystage) + sd.ystage_off[m] +
               ((static_cast<size_t>(p) * g.groups + gi) * nb16 + blk) * 256 + li * 16 + 4 * lk);
      } else {
        // re / im of fields 8 gi + 2 lk and the next at degree l
        const int i = 16 * blk + li, l = m + p + 2 * i, f = 8 * gi + 2 * lk;
        if (i >= np) return;
        float2* d = yout + (static_cast<size_t>(f) * g.lmax + l) * g.mmax + m;
        float2* d1 = d + static_cast<size_t>(g.lmax) * g.mmax;
        if (cols == 15u) {
          if (f < g.F) d[0] = make_float2(v[0], v[1]);
          if (f + 1 < g.F) d1[0] = make_float2(v[2], v[3]);
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if ((cols >> h) & 1 && f < g.F) (&d->x)[h] = v[h];
            if ((cols >> (2 + h)) & 1 && f + 1 < g.F) (&d1->x)[h] = v[2 + h];
          }
        }
      }
    };
    if constexpr (S == Storage::F32) {
      // NaN once a sum is not finite.  Four chains, and the rare paths marked as
      // such, so that their code lies behind the tile's: 0.2 of 45.5 us of the
      // four transforms at 121 x 240 x 15 fields.
      float zero[4] = {};
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < CB; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) zero[i] = fmaf(acc[r][q][i], 0.f, zero[i]);
      // columns (of fields that exist) with such a sum, a bit mask per column
      // block
      if (__builtin_expect(__any(!((zero[0] + zero[1]) + (zero[2] + zero[3]) == 0.f)), 0)) {
#pragma unroll
        for (int q = 0; q < CB; ++q) {
          unsigned cols = 0;
          const int f = 8 * (c * cbs + q) + 2 * lk;
#pragma unroll
          for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (!(fabsf(acc[r][q][i]) < __builtin_inff()) && f + (i >> 1) < g.F && q < cbs) cols |= 1u << (4 * lk + i);
          if (cols) atomicOr(&bad[q], cols);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < CB; ++q) {
        floatx4 v = acc[r][q];
        if constexpr (CORR) v = v + corr[r][q];
        if constexpr (!SYN || S == Storage::F32) v = v * (ms * kSumDown<S>);
        put(r, q, v, 15u);
      }
    if constexpr (S == Storage::F32) {
      lds_barrier();
      unsigned any = 0;
#pragma unroll
      for (int q = 0; q < CB; ++q) any |= bad[q];
      if (__builtin_expect(__builtin_amdgcn_readfirstlane(any) != 0, 0)) exact_range(r_c, put, ms);
    }
  };
  if (steps > 0 && ntile > 0) {
    if (vb)
      run(std::integral_constant<int, 2>{});
    else if (va)
      run(std::integral_constant<int, 1>{});
    else
      run(std::integral_constant<int, 0>{});
  }
  // Zeros of the spectrum (entries l < m'), direct form: the first tile of
  // order m writes those of degree l = m for its fields, y[f][m][m+1 ..
  // mmax-1], one contiguous run per field (staged: the transpose does).
  if constexpr (!SYN && !STG) {
    if (p == 0 && rt == 0) {
      const int fbeg = 8 * cbs * c;
      const int fend = min(g.F, fbeg + 8 * cbs);
      const int len = g.mmax - 1 - m;
      for (int ff = fbeg; ff < fend; ++ff) {
        float2* row = yout + (static_cast<size_t>(ff) * g.lmax + m) * g.mmax + m + 1;
        for (int e = threadIdx.x; e < len; e += 256) row[e] = make_float2(0.f, 0.f);
      }
    }
  }
}

// Batched kernels: a workgroup takes its item {m | p << 16 | row tile << 17,
// (segment << 16) | chunk} from the plan-wide work list.  The launch's CB
// covers the widest segment.
//
// MIXED: a segment of fewer groups than the launch's CB takes a tile of half or a
// quarter of its width (rounded up) where its chunks fit: at the full width it
// would load, split and multiply the repeated columns too (181 x 360 x 72 fields
// and 721 x 1440 x 8 in one plan, float32, analysis / synthesis: 160 / 156 ->
// 115 / 113 us).  Plans without such a segment keep a kernel of one width: with
// the others' code in it 721 x 1440 x 128 fields took 331 / 311 us, without 326 /
// 305, Gauss 360 x 720 x 1024 457 / 482 and 452 / 475.
constexpr int half_cb(int cb) { return (cb + 1) / 2; }
constexpr int quarter_cb(int cb) { return (cb + 3) / 4; }
template <Storage S, int CB, bool MIXED>
constexpr int lds_widest =
    MIXED && lds_v4<S>(half_cb(CB)) > lds_v4<S>(CB) ? lds_v4<S>(half_cb(CB)) : lds_v4<S>(CB);
template <Storage S, int CB, bool SYN, bool MIXED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void legendre_batched(
    const SegDev* __restrict__ segs, const int2* __restrict__ work, int per, const float2* __restrict__ yin,
    float2* __restrict__ yout, float c_rest, int staged) {
  __shared__ v4f lds[lds_widest<S, CB, MIXED>];
  __shared__ unsigned bad[CB];  // float32: columns with a sum that is not finite
  const int2 wk = take_work(work, per);
  if (wk.x < 0) return;
  const SegDev& sd = segs[wk.y >> 16];
  const int m = wk.x & 0xffff, p = (wk.x >> 16) & 1, rt = wk.x >> 17, c = wk.y & 0xffff;
  const int rot = blockIdx.x >> 3, cbs = SYN ? sd.syn_cb : sd.ana_cb;
  yin += sd.spec_off;
  yout += sd.spec_off;
  auto run = [&](auto cb_c) {
    constexpr int W = decltype(cb_c)::value;
    if (staged)
      tile_body<S, W, SYN, true>(sd, m, p, rt, c, cbs, rot, yin, yout, c_rest, lds, bad);
    else
      tile_body<S, W, SYN, false>(sd, m, p, rt, c, cbs, rot, yin, yout, c_rest, lds, bad);
  };
  if constexpr (MIXED && quarter_cb(CB) < half_cb(CB))
    if (cbs <= quarter_cb(CB)) return run(std::integral_constant<int, quarter_cb(CB)>{});
  if constexpr (MIXED && half_cb(CB) < CB)
    if (cbs <= half_cb(CB)) return run(std::integral_constant<int, half_cb(CB)>{});
  run(std::integral_constant<int, CB>{});
}

template <Storage S, bool SYN, int CB>
hipError_t launch_cb(int cb, dim3 grid, const BatchArgs& b, const int2* work, int per, const float2* in, float2* out,
                     float c_rest, int staged, hipStream_t st) {
  if (cb == CB) {
    auto start = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, b.segs, work, per, in, out, c_rest, staged);
      return hipGetLastError();
    };
    if constexpr (half_cb(CB) < CB)
      if ((SYN ? b.syn_least : b.ana_least) <= half_cb(CB)) return start(legendre_batched<S, CB, SYN, true>);
    return start(legendre_batched<S, CB, SYN, false>);
  }
  if constexpr (CB > 1) return launch_cb<S, SYN, CB - 1>(cb, grid, b, work, per, in, out, c_rest, staged, st);
  return hipErrorInvalidValue;
}

// Launch of one form and direction (explicitly instantiated in a translation
// unit of its own, legendre_{f32,bf16,bf16x2,bf16x3}_{ana,syn}.hip).
template <Storage S, bool SYN>
hipError_t launch(const BatchArgs& b, const float2* in, float2* out, float c_rest, hipStream_t st) {
  const int per = SYN ? b.syn_per : b.ana_per;
  const int2* work = SYN ? b.syn_work : b.ana_work;
  const int staged = SYN ? (b.staged >> 1) & 1 : b.staged & 1;
  const dim3 grid(static_cast<unsigned>(8 * per));
  return launch_cb<S, SYN, max_cb<S, SYN>>(SYN ? b.syn_cb : b.ana_cb, grid, b, work, per, in, out, c_rest, staged, st);
}

#define SHT_LEG_EXTERN(S)                                                                                     \
  extern template hipError_t launch<S, false>(const BatchArgs&, const float2*, float2*, float, hipStream_t); \
  extern template hipError_t launch<S, true>(const BatchArgs&, const float2*, float2*, float, hipStream_t);
SHT_LEG_EXTERN(Storage::F32)
SHT_LEG_EXTERN(Storage::BF16)
SHT_LEG_EXTERN(Storage::BF16X2)
SHT_LEG_EXTERN(Storage::BF16X3)
#undef SHT_LEG_EXTERN

}  // namespace legk
}  // namespace sht
