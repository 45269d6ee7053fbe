"""Ring DFT by the widest ring of a plan: the workgroup sizes change at 192,
384, 576 (forward), 768 (inverse), 1024 (forward) and 1152 (inverse) points,
and a plan's narrower segments run in the widest one's kernel; a large
workspace of many orders takes the single-lane stores.  FP64 oracle.

Tolerance: as for a single ring width (butterfly levels, twiddles, six
products per 32-term step): 2^-24 (12 passes + 6 steps + 4), doubled.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


def tolerance(lmax):
    return 2 * 2.0 ** -24 * (12 * 4 + 6 * math.ceil(lmax / 2 / 32) + 4)


@pytest.mark.parametrize("widest", [48, 192, 200, 384, 400, 576, 600, 768, 800, 1024, 1080, 1152, 1200])
def test_segments_of_unequal_width(pkg, widest):
    print("widest ring", widest, flush=True)
    rng = np.random.default_rng(widest)
    shapes = [(5, 36, 9), (7, widest, 24), (6, 64, 32) if widest >= 64 else (6, 24, 12), (3, 20, 4)]
    fields = 6
    descs = [dict(nlat=h, nlon=w, lmax=l, mmax=l, grid="equiangular", channels=fields) for h, w, l in shapes]
    plan = pkg.Plan(descs)
    us, cs = [], []
    flat, spec = np.zeros(plan.grid_elems, np.float32), np.zeros(plan.spec_elems, np.complex64)
    for i, (h, w, l) in enumerate(shapes):
        u = rng.standard_normal((fields, h, w)).astype(np.float32)
        a = (rng.standard_normal((fields, l, l)) + 1j * rng.standard_normal((fields, l, l))).astype(np.complex64)
        a = np.tril(a)
        a[..., 0] = a[..., 0].real
        go, so = plan.segment(i)
        flat[go:go + u.size], spec[so:so + a.size] = u.reshape(-1), a.reshape(-1)
        us.append(u)
        cs.append(a)
    y = plan.sht(torch.from_numpy(flat).cuda()).cpu().numpy()
    x = plan.isht(torch.from_numpy(spec).cuda()).cpu().numpy()
    for i, ((h, w, l), u, c) in enumerate(zip(shapes, us, cs)):
        go, so = plan.segment(i)
        ref_y = oracle.sht(u.astype(np.float64)[None], l, l, 0)[0]
        ref_x = oracle.isht(c.astype(np.complex128)[None], h, w, 0)[0]
        got_y = y[so:so + c.size].reshape(c.shape)
        got_x = x[go:go + u.size].reshape(u.shape)
        errs = (rel_l2(got_y, ref_y), rel_l2(got_x, ref_x))
        print("  %d x %d: rel-L2 %.2e %.2e, tolerance %.2e" % ((h, w) + errs + (tolerance(l),)), flush=True)
        assert max(errs) <= tolerance(l), (widest, h, w, errs)
    plan.close()


@pytest.mark.parametrize("nlon,fields", [(960, 1700), (1440, 1100)])
def test_single_lane_stores(pkg, nlon, fields):
    print("ring width", nlon, "fields", fields, flush=True)
    nlat, m = 3, nlon // 2
    g = torch.Generator(device="cuda").manual_seed(nlon)
    u = torch.randn((1, fields, nlat, nlon), generator=g, device="cuda")
    plan = pkg.Plan(dict(nlat=nlat, nlon=nlon, lmax=m, mmax=m, grid="equiangular", channels=fields))
    y = plan.sht(u)
    pick = [0, 3, 4, 7, fields // 2, fields - 1]
    ref = oracle.sht(u[:, pick].cpu().numpy().astype(np.float64), m, m, 0)
    err = rel_l2(y[:, pick].cpu().numpy(), ref)
    print("  rel-L2 %.2e, tolerance %.2e" % (err, tolerance(m)), flush=True)
    assert err <= tolerance(m)
    plan.close()
