"""Ring DFT at widths that take every radix and pass count of its plan: the
forward and inverse longitude step of all four transforms against the FP64
oracle, with every order the width has (mmax = nlon // 2, so that all bins
take part) and with a truncation (zeros above it).

Tolerance: a DFT of at most four passes of radix <= 16 rounds at most
2 log2(16) + 4 times per pass (butterfly levels, twiddle, its factors), a
Legendre sum of `steps` times six products once each; relative to the size of
the terms: 2^-24 (12 passes + 6 steps + 4), doubled for cancelling terms.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

WIDTHS = [2, 3, 5, 6, 8, 9, 10, 12, 15, 16, 18, 25, 32, 45, 50, 75, 81, 128, 150, 240, 243, 256, 288, 375, 512, 540, 625,
          648, 720, 729, 768, 1000, 1024, 1080, 1250, 1296, 1440, 1458, 1536, 1600, 1875, 1920, 2000, 2025, 2048]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("nlon", WIDTHS)
def test_ring_dft_width(pkg, nlon):
    print("ring width", nlon, flush=True)
    nlat, fields, grid = 3, 5, 0
    rng = np.random.default_rng(nlon)
    u = rng.standard_normal((1, fields, nlat, nlon)).astype(np.float32)
    for mmax in sorted({max(1, nlon // 2), max(1, nlon // 5)}):
        lmax = mmax
        a = rng.standard_normal((1, fields, lmax, mmax, 2)).astype(np.float32)
        a = (a[..., 0] + 1j * a[..., 1]).astype(np.complex64)
        a[..., np.arange(lmax)[:, None] < np.arange(mmax)[None, :]] = 0
        a[..., 0] = a[..., 0].real
        u64, a64 = u.astype(np.float64), a.astype(np.complex128)
        refs = (oracle.sht(u64, lmax, mmax, grid), oracle.isht(a64, nlat, nlon, grid),
                oracle.sht_T(a64, nlat, nlon, grid), oracle.isht_T(u64, lmax, mmax, grid))
        plan = pkg.Plan(dict(nlat=nlat, nlon=nlon, lmax=lmax, mmax=mmax, grid="equiangular", channels=fields))
        du, da = torch.from_numpy(u).cuda(), torch.from_numpy(a).cuda()
        outs = [t.cpu().numpy() for t in (plan.sht(du), plan.isht(da), plan.sht_T(da), plan.isht_T(du))]
        tol = 2 * 2.0 ** -24 * (12 * 4 + 6 * math.ceil(lmax / 2 / 32) + 4)
        errs = [rel_l2(o, r) for o, r in zip(outs, refs)]
        print(f"  mmax {mmax}: rel-L2", ["%.2e" % e for e in errs], "tolerance %.2e" % tol, flush=True)
        assert max(errs) <= tol, (nlon, mmax, errs)
        plan.close()
