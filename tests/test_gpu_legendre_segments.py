"""Segments of unequal field counts in one plan: a narrow segment's tiles run at
a part of the launch's width, with the results of a plan of its own, bit for bit."""
import pytest

from _util import ensure_built

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# field groups of the segments: every width up to the widest tile's, and its
# half and quarter
GROUPS = [[9, 1, 2, 3, 4, 5, 6, 7, 8], [8, 1, 2, 3, 4, 5], [7, 2, 3, 4], [6, 2, 3, 4], [5, 2, 3], [4, 1, 2, 3], [3, 1, 2], [2, 1],
          [19, 1, 4]]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("precision", ["fp32", "bf16", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("groups", GROUPS, ids=lambda g: "-".join(map(str, g)))
def test_unequal_segments(pkg, groups, precision):
    print("unequal segments", groups, precision, flush=True)
    shapes = [(17, 32, 16), (35, 64, 31), (70, 150, 66)]
    descs = []
    for i, n in enumerate(groups):
        nlat, nlon, L = shapes[i % 3]
        descs.append(dict(nlat=nlat, nlon=nlon, lmax=L, mmax=L, grid="equiangular", channels=8 * n - (3 if i % 2 else 0)))
    plan = pkg.Plan(descs, precision=precision)
    g = torch.Generator(device="cuda").manual_seed(len(groups))
    u = torch.randn(plan.grid_elems, generator=g, device="cuda")
    a = torch.view_as_complex(torch.randn((plan.spec_elems, 2), generator=g, device="cuda"))
    alone = [pkg.Plan(d, precision=precision) for d in descs]
    for staged in (0, 3):
        plan.set_schedule(8, 0, 2, staged)
        outs = {op: getattr(plan, op)(u if op in ("sht", "isht_T") else a) for op in ("sht", "isht", "sht_T", "isht_T")}
        for i, one in enumerate(alone):
            one.set_schedule(8, 0, 2, staged)
            go, so = plan.segment(i)
            x = u[go:go + one.grid_elems][:torch.Size(one.grid_shape()).numel()].reshape(one.grid_shape()).clone()
            y = a[so:so + one.spec_elems][:torch.Size(one.spec_shape()).numel()].reshape(one.spec_shape()).clone()
            for op, out in outs.items():
                ref = getattr(one, op)(x if op in ("sht", "isht_T") else y).reshape(-1)
                at = so if op in ("sht", "isht_T") else go
                assert torch.equal(torch.view_as_real(out[at:at + ref.numel()]) if out.is_complex() else out[at:at + ref.numel()],
                                   torch.view_as_real(ref) if ref.is_complex() else ref), (staged, i, op)
    for p in alone + [plan]:
        p.close()
