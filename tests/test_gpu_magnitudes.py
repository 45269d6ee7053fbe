"""Float32 transforms over the magnitudes that float32 holds, against the FP64
oracle: data near the smallest and the largest normal numbers, tables that are
small where the data are not, and fields of very unequal size, infinities and
NaN side by side.

Float32 operands are split into three bf16 planes after a scaling by 2^16;
sums beyond 2^96 are taken again on the float32 matrix cores.

Tolerance: as for the tiles' edges, per output element 2^-24 times the
roundings of the sums (`steps` matrix instructions of six products; of 32
float32 terms where the sums are taken again), the DFT (2 log2(nlon)) and the
table and scale factors (4), doubled for cancelling terms.  The scales leave
every intermediate result at least 2^26 above the subnormals' spacing.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# nlat, nlon, lmax, mmax, grid, channels
SHAPES = [(33, 64, 33, 17, 0, 9), (64, 128, 258, 20, 1, 88)]
# exponents of the scale of each transform's input: the ring scale (2^-7 to
# 2^-9 here) meets the data before (sht) or after (sht_T) the sums
SMALL = {"sht": -118, "isht": -124, "sht_T": -120, "isht_T": -124}


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


def inputs(shape, seed):
    nlat, nlon, lmax, mmax, grid, C = shape
    rng = np.random.default_rng(seed)
    u = rng.standard_normal((1, C, nlat, nlon)).astype(np.float32)
    a = (rng.standard_normal((1, C, lmax, mmax)) + 1j * rng.standard_normal((1, C, lmax, mmax))).astype(np.complex64)
    a[..., np.arange(lmax)[:, None] < np.arange(mmax)[None, :]] = 0
    a[..., 0] = a[..., 0].real
    return u, a


def reference(op, v, shape):
    nlat, nlon, lmax, mmax, grid, _ = shape
    if op in ("sht", "isht_T"):
        return getattr(oracle, op)(v.astype(np.float64), lmax, mmax, grid)
    return getattr(oracle, op)(v.astype(np.complex128), nlat, nlon, grid)


def make_plan(pkg, shape):
    nlat, nlon, lmax, mmax, grid, C = shape
    return pkg.Plan(dict(nlat=nlat, nlon=nlon, lmax=lmax, mmax=mmax, grid=grid, channels=C))


@pytest.mark.parametrize("size", ["small", "border", "large"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_L{s[2]}M{s[3]}_F{s[5]}")
def test_scaled_inputs(pkg, shape, size):
    print("magnitudes", shape, size, flush=True)
    u, a = inputs(shape, 3)
    plan = make_plan(pkg, shape)
    steps = math.ceil(max((shape[0] + 1) // 2, (shape[2] + 1) // 2) / 32)
    tol = 2 * 2.0 ** -24 * ((6 if size == "small" else 32) * steps + 2 * math.log2(shape[1]) + 4)
    for op in ("sht", "isht", "sht_T", "isht_T"):
        e = {"small": SMALL[op], "border": 78, "large": 114}[size]
        v = (u if op in ("sht", "isht_T") else a) * np.float32(2.0 ** e)
        ref = reference(op, v, shape)
        for staged in (0, 3):
            plan.set_schedule(8, 0, 2, staged)
            got = getattr(plan, op)(torch.from_numpy(v).cuda()).cpu().numpy()
            # the norms of such numbers squared are beyond float32's range, not beyond float64's
            err = rel_l2(got.astype(ref.dtype), ref)
            print(f"  {op} 2^{e} staged {staged}: rel-L2 {err:.2e} (tolerance {tol:.2e})", flush=True)
            assert err <= tol, (op, e, staged, err)
    plan.close()


def test_small_table(pkg):
    """One order of high m: next to the poles every table value is small and
    the field is nothing else, so each ring is held to the tolerance."""
    shape = (129, 128, 48, 29, 0, 8)
    nlat, nlon, lmax, mmax, grid, C = shape
    _, a = inputs(shape, 4)
    a[..., :28] = 0
    plan = make_plan(pkg, shape)
    ref = reference("isht", a, shape)[0]
    got = plan.isht(torch.from_numpy(a).cuda()).cpu().numpy()[0].astype(np.float64)
    tol = 8 * 2.0 ** -24 * (6 + 2 * math.log2(nlon) + 4)
    size = np.abs(ref).max(axis=(0, 2))
    rings = np.nonzero((size > 1e-36) & (size < 1e-30))[0]
    print("rings", rings, "of size", size[rings], flush=True)
    assert len(rings) >= 2
    for k in rings:
        err = rel_l2(got[:, k], ref[:, k])
        print(f"  ring {k}: rel-L2 {err:.2e} (tolerance {tol:.2e})", flush=True)
        assert err <= tol, (k, err)
    plan.close()


def test_largest_coefficient(pkg):
    shape = (33, 64, 33, 17, 0, 3)
    _, a = inputs(shape, 5)
    a[0, 1] = 0
    a[0, 1, 0, 0] = np.finfo(np.float32).max
    plan = make_plan(pkg, shape)
    ref = reference("isht", a, shape)
    got = plan.isht(torch.from_numpy(a).cuda()).cpu().numpy().astype(np.float64)
    tol = 2 * 2.0 ** -24 * (32 * 2 + 12 + 4)
    for f in range(3):
        assert rel_l2(got[0, f], ref[0, f]) <= tol, f
    plan.close()


@pytest.mark.parametrize("staged", [0, 3])
def test_fields_apart(pkg, staged):
    """What a field holds changes no bit of another one."""
    shape = (33, 64, 33, 17, 0, 20)
    u, a = inputs(shape, 6)
    size = np.array([1, 2.0 ** 100, 2.0 ** -118, 2.0 ** 80, 1, 0, 2.0 ** 60, 1, 2.0 ** 110, 3] * 2, np.float32)
    u, a = u * size[:, None, None], a * size[:, None, None]
    u[0, 4, 5, 6], a[0, 4, 5, 2] = np.inf, np.inf
    u[0, 7, 8, 9], a[0, 7, 6, 1] = np.nan, np.nan
    plan = make_plan(pkg, shape)
    plan.set_schedule(8, 0, 2, staged)

    def same(x, y):
        x, y = (torch.view_as_real(t) if t.is_complex() else t for t in (x, y))
        return bool(((x == y) | (torch.isnan(x) & torch.isnan(y))).all())

    for op in ("sht", "isht", "sht_T", "isht_T"):
        v = torch.from_numpy(u if op in ("sht", "isht_T") else a).cuda()
        every = getattr(plan, op)(v)
        for f in range(shape[5]):
            alone = torch.zeros_like(v)
            alone[0, f] = v[0, f]
            assert same(every[0, f], getattr(plan, op)(alone)[0, f]), (op, f)
        assert all(bool(torch.isfinite(torch.view_as_real(every[0, f]) if every.is_complex() else every[0, f]).all())
                   for f in range(shape[5]) if f not in (4, 7))
    plan.close()
