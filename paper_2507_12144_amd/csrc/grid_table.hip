// Plan-time float64 kernels: latitude nodes and quadrature weights (App. B.1)
// and the table of orthonormal associated Legendre functions by their
// three-term recurrence (App. B.3, eq. spherical_harmonics).  These are the
// only float64 kernels; every operation of the transforms themselves is
// float32 (or bf16 on the matrix cores).
#include "internal.h"
#include "bf16.h"
#include "bf16_planes.h"

namespace sht {
namespace {

constexpr double kPi = 3.14159265358979323846;

// Legendre polynomial P_n and P_{n-1} at x by the Bonnet recurrence.
__device__ void legendre_pn(int n, double x, double* pn, double* pn1) {
  double p0 = 1.0, p1 = x;
  if (n == 0) { *pn = 1.0; *pn1 = 0.0; return; }
  for (int k = 2; k <= n; ++k) {
    double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
    p0 = p1;
    p1 = p2;
  }
  *pn = p1;
  *pn1 = p0;
}

// One thread per ring.  Nodes are generated for the northern half and
// mirrored, so x_{nlat-1-k} = -x_k exactly and the equator (odd nlat) has
// x = 0 exactly; the equatorial fold of the contraction relies on this.
__global__ void grid_kernel(int nlat, int kind, double* __restrict__ xo, double* __restrict__ so,
                            double* __restrict__ wo) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nlat) return;
  const int kn = (k < nlat - 1 - k) ? k : nlat - 1 - k;  // northern mirror index
  const bool south = kn != k;
  const bool equator = (2 * kn == nlat - 1);
  double x, s, w;
  if (kind == 1) {
    // Gauss-Legendre: Newton on P_nlat from the asymptotic guess.
    x = cos(kPi * (kn + 0.75) / (nlat + 0.5));
    for (int it = 0; it < 100; ++it) {
      double pn, pn1;
      legendre_pn(nlat, x, &pn, &pn1);
      const double dp = nlat * (pn1 - x * pn) / ((1.0 - x) * (1.0 + x));
      const double dx = pn / dp;
      x -= dx;
      if (fabs(dx) < 1e-16) break;
    }
    if (equator) x = 0.0;
    double pn, pn1;
    legendre_pn(nlat, x, &pn, &pn1);
    const double dp = nlat * (pn1 - x * pn) / ((1.0 - x) * (1.0 + x));
    w = 2.0 / ((1.0 - x) * (1.0 + x) * dp * dp);
    s = sqrt((1.0 - x) * (1.0 + x));
  } else {
    // Pole-inclusive equiangular grid: t_k = pi k / (nlat - 1).
    const int N = nlat - 1;
    const double t = static_cast<double>(kn) / N;
    x = equator ? 0.0 : cospi(t);
    s = sinpi(t);
    if (kind == 2) {
      w = (kPi / N) * s;  // sin(t) dt
    } else {
      // Clenshaw-Curtis: w_k = (c_k/N)(1 - sum_j b_j cos(2 j t_k)/(4 j^2 - 1)),
      // the exact integral of the degree-N Chebyshev interpolant.
      double acc = 1.0;
      for (int j = 1; 2 * j <= N; ++j) {
        const double b = (2 * j == N) ? 1.0 : 2.0;
        // cos(2 j t_k) = cospi(2 j kn / N), argument reduced exactly mod 2N
        const long long r = (2LL * j * kn) % (2LL * N);
        acc -= b * cospi(static_cast<double>(r) / N) / (4.0 * j * j - 1.0);
      }
      const double c = (kn == 0) ? 1.0 : 2.0;
      w = c * acc / N;
    }
  }
  xo[k] = south ? -x : x;
  so[k] = s;
  wo[k] = w;
}

// Position of ring k, row d = l - m of order m in the two fragment tables:
// fragment, lane and element.
struct FragPos {
  int kst, nb, nr, ns;
  int a_step, a_lk, a_e, s_blk, s_li;
  size_t a0, s0;
  __device__ __forceinline__ FragPos(const SegGeom& g, int m, int k, const int64_t* ana_off, const int64_t* syn_off) {
    const int n0 = (g.lmax - m + 1) >> 1;
    kst = g.kpad / 32;
    nb = (n0 + 15) / 16;
    nr = (g.nk + 15) / 16;
    ns = (n0 + 31) / 32;
    a_step = k >> 5;
    a_lk = k & 3;
    a_e = (k & 31) >> 2;
    s_blk = k >> 4;
    s_li = k & 15;
    a0 = static_cast<size_t>(ana_off[m]);
    s0 = static_cast<size_t>(syn_off[m]);
  }
  __device__ __forceinline__ void at(int d, size_t* ba, int* la, int* ea, size_t* bs, int* ls, int* es) const {
    const int p = d & 1, i = d >> 1;
    *ba = a0 + static_cast<size_t>(p * nb + (i >> 4)) * kst + a_step;
    *la = 16 * a_lk + (i & 15);
    *ea = a_e;
    *bs = s0 + static_cast<size_t>(p * nr + s_blk) * ns + (i >> 5);
    *ls = 16 * (i & 3) + s_li;
    *es = (i & 31) >> 2;
  }
};

// Legendre table in MFMA fragment order.  One thread per (ring k < nk,
// order m) runs the float64 recurrence of eq. spherical_harmonics
//   P^_0^0 = 1/sqrt(4 pi),  P^_m^m = -sqrt((2m+1)/(2m)) sin t P^_{m-1}^{m-1}
//   P^_{m+1}^m = sqrt(2m+3) x P^_m^m
//   P^_l^m = a_lm (x P^_{l-1}^m - b_lm P^_{l-2}^m)
//   a_lm = sqrt((4l^2-1)/(l^2-m^2)),  b_lm = sqrt(((l-1)^2-m^2)/(4(l-1)^2-1))
// and rounds every value, times 2^16 (bf16_planes.h), once to float32.  Degree
// l of order m has parity p = (l-m) & 1 and row i = (l-m) >> 1 of its parity
// block; rows come in blocks of 16 (ib = i / 16).  Each value is written to two tables of
// fragments (16 rows x 32 contraction indices), laid out so that a wave of
// the contraction kernels reads its operand of one K step as two contiguous
// 1 KiB pieces, 16 bytes a lane.  Lane 16 lk + li of a fragment holds row li
// and the contraction indices 4 e + lk, e < 8 (e = 4 h + q: piece h,
// component q), of its K step:
//  * analysis  (rows = degrees i, contraction = rings k, K step k / 32):
//      ((ana_off[m] + (p*nb + i/16)*(kpad/32) + k/32)*2 + h)*256 + lane*4 + q
//  * synthesis (rows = rings k, contraction = degrees i, K step i / 32):
//      ((syn_off[m] + (p*nr + k/16)*ns + i/32)*2 + h)*256 + lane*4 + q
// with nb = ceil(ceil((lmax-m)/2) / 16), ns = ceil(ceil((lmax-m)/2) / 32) and
// nr = ceil(nk / 16).
// Values too small for float64 flush to zero; none of them can grow back to
// a significant size before l = 768 on the supported grids.
__global__ void frag_table_kernel(SegGeom g, const double* __restrict__ xs, const double* __restrict__ ss,
                                  const int64_t* __restrict__ ana_off, const int64_t* __restrict__ syn_off,
                                  float* __restrict__ ta, float* __restrict__ tsyn) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  if (k >= g.nk || m >= g.mmax) return;
  const FragPos f(g, m, k, ana_off, syn_off);
  auto put = [&](int l, double v) {
    size_t ba, bs;
    int ea, es, la, ls;
    f.at(l - m, &ba, &la, &ea, &bs, &ls, &es);
    const float r = __double2float_rn(v * planes::kSplitScale);
    ta[(ba * 2 + (ea >> 2)) * 256 + la * 4 + (ea & 3)] = r;
    tsyn[(bs * 2 + (es >> 2)) * 256 + ls * 4 + (es & 3)] = r;
  };
  const double x = xs[k];
  const double sn = ss[k];
  double pmm = 1.0 / sqrt(4.0 * kPi);
  for (int i = 1; i <= m; ++i) pmm = -sqrt((2.0 * i + 1.0) / (2.0 * i)) * sn * pmm;
  if (m >= g.lmax) return;
  put(m, pmm);
  if (m + 1 >= g.lmax) return;
  double p2 = pmm;
  double p1 = sqrt(2.0 * m + 3.0) * x * pmm;
  put(m + 1, p1);
  const double mm = static_cast<double>(m) * m;
  for (int l = m + 2; l < g.lmax; ++l) {
    const double dl = l;
    const double a = sqrt((4.0 * dl * dl - 1.0) / (dl * dl - mm));
    const double b = sqrt(((dl - 1.0) * (dl - 1.0) - mm) / (4.0 * (dl - 1.0) * (dl - 1.0) - 1.0));
    const double p = a * (x * p1 - b * p2);
    p2 = p1;
    p1 = p;
    put(l, p);
  }
}

// bf16 planes of the same table.  Each float64 value v is split into NP bf16
// planes, each rounded to nearest-even from the float64 residual: hi =
// bf16(v), next = bf16(v - hi), ...  The fragments are those of the float32
// table; each holds NP planes of 1 KiB, a lane's eight values contiguous:
//      (fragment*NP + plane)*512 + lane*8 + e
template <int NP>
__global__ void frag_table_bf16_kernel(SegGeom g, const double* __restrict__ xs, const double* __restrict__ ss,
                                       const int64_t* __restrict__ ana_off, const int64_t* __restrict__ syn_off,
                                       uint16_t* __restrict__ ta, uint16_t* __restrict__ tsyn) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  if (k >= g.nk || m >= g.mmax) return;
  const FragPos f(g, m, k, ana_off, syn_off);
  auto put = [&](int l, double v) {
    size_t ba, bs;
    int ea, es, la, ls;
    f.at(l - m, &ba, &la, &ea, &bs, &ls, &es);
    double r = v;
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
      const uint16_t b = bf16_rn_from_double(r);
      r -= bf16_bits_to_double(b);
      ta[(ba * NP + pl) * 512 + la * 8 + ea] = b;
      tsyn[(bs * NP + pl) * 512 + ls * 8 + es] = b;
    }
  };
  const double x = xs[k];
  const double sn = ss[k];
  double pmm = 1.0 / sqrt(4.0 * kPi);
  for (int i = 1; i <= m; ++i) pmm = -sqrt((2.0 * i + 1.0) / (2.0 * i)) * sn * pmm;
  if (m >= g.lmax) return;
  put(m, pmm);
  if (m + 1 >= g.lmax) return;
  double p2 = pmm;
  double p1 = sqrt(2.0 * m + 3.0) * x * pmm;
  put(m + 1, p1);
  const double mm = static_cast<double>(m) * m;
  for (int l = m + 2; l < g.lmax; ++l) {
    const double dl = l;
    const double a = sqrt((4.0 * dl * dl - 1.0) / (dl * dl - mm));
    const double b = sqrt(((dl - 1.0) * (dl - 1.0) - mm) / (4.0 * (dl - 1.0) * (dl - 1.0) - 1.0));
    const double p = a * (x * p1 - b * p2);
    p2 = p1;
    p1 = p;
    put(l, p);
  }
}

}  // namespace

hipError_t launch_grid(int nlat, int kind, double* x, double* s, double* w, hipStream_t st) {
  const int threads = 64;
  hipLaunchKernelGGL(grid_kernel, dim3((nlat + threads - 1) / threads), dim3(threads), 0, st, nlat,
                     kind, x, s, w);
  return hipGetLastError();
}

hipError_t launch_frag_table(const SegGeom& g, const double* x, const double* s, const int64_t* ana_off,
                             const int64_t* syn_off, float* ta, float* tsyn, hipStream_t stream) {
  hipLaunchKernelGGL(frag_table_kernel, dim3((g.nk + 63) / 64, g.mmax), dim3(64), 0, stream, g, x, s, ana_off, syn_off,
                     ta, tsyn);
  return hipGetLastError();
}

hipError_t launch_frag_table_bf16(const SegGeom& g, int planes, const double* x, const double* s,
                                  const int64_t* ana_off, const int64_t* syn_off, uint16_t* ta, uint16_t* tsyn,
                                  hipStream_t stream) {
  const dim3 grid((g.nk + 63) / 64, g.mmax);
#define SHT_FRAG_CASE(N)                                                                                        \
  case N:                                                                                                       \
    hipLaunchKernelGGL(frag_table_bf16_kernel<N>, grid, dim3(64), 0, stream, g, x, s, ana_off, syn_off, ta, tsyn); \
    break;
  switch (planes) {
    SHT_FRAG_CASE(1)
    SHT_FRAG_CASE(2)
    SHT_FRAG_CASE(3)
    default: return hipErrorInvalidValue;
  }
#undef SHT_FRAG_CASE
  return hipGetLastError();
}

}  // namespace sht
