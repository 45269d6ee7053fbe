"""Lazily conjugated and negated tensors (torch keeps a bit beside memory that
holds the values before the conjugation): every call gives what it gives for
the same values written out, bit for bit, and refuses such a tensor where the
memory itself is what counts (outputs, buffers of a captured sequence).
"""
import pytest

from _util import ensure_built

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

B, C, L, NLAT, NLON = 2, 3, 12, 13, 24


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.fixture(scope="module")
def plan(pkg):
    return pkg.Plan(dict(nlat=NLAT, nlon=NLON, lmax=L, mmax=L, grid="equiangular", batch=B, channels=C))


def draw(seed, *shape):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


def cdraw(seed, *shape):
    return torch.view_as_complex(draw(seed, *shape, 2))


CALLS = {
    "isht": lambda p, s, x: p.isht(s(0)),
    "sht_T": lambda p, s, x: p.sht_T(s(0)),
    "sht": lambda p, s, x: p.sht(x(0)),
    "isht_T": lambda p, s, x: p.isht_T(x(0)),
    "mix": lambda p, s, x: p.mix(s(1, L, C, C), s(0)),
    "mix adjoint": lambda p, s, x: p.mix(s(1, L, C, C), s(0), adjoint=True),
    "mix_weight_grad": lambda p, s, x: p.mix_weight_grad(s(0), s(2)),
    "filter": lambda p, s, x: p.filter(s(1, C, L), s(0)),
    "filter_grad": lambda p, s, x: p.filter_grad(s(0), s(2)),
    "psd": lambda p, s, x: p.psd(s(0)),
    "zonal_psd": lambda p, s, x: p.zonal_psd(x(0)),
    "spectral_crps": lambda p, s, x: p.spectral_crps(s(0), s(1, C, L, L), grad=True),
    "spatial_crps": lambda p, s, x: p.spatial_crps(x(0), x(1, C, NLAT, NLON), grad=True),
}


@pytest.mark.parametrize("name", list(CALLS))
def test_lazy_inputs(plan, name):
    print("lazy view into", name, flush=True)
    results = []
    for lazy in (True, False):
        def spec(seed, *shape):
            t = cdraw(seed, *(shape or plan.spec_shape())).conj()
            assert t.is_conj() and t.is_contiguous()
            return t if lazy else t.resolve_conj()

        def grid(seed, *shape):
            t = torch._neg_view(draw(seed, *(shape or plan.grid_shape())))
            assert t.is_neg() and t.is_contiguous()
            return t if lazy else t.resolve_neg()

        r = CALLS[name](plan, spec, grid)
        results.append(r if isinstance(r, tuple) else (r,))
    assert all(torch.equal(a, b) for a, b in zip(*results)), name


def test_lazy_gradients(pkg, plan):
    """Autograd hands the conjugate's gradient on as a lazy view."""
    w, W, k = cdraw(5, *plan.spec_shape()), cdraw(6, L, C, C), cdraw(7, C, L)
    seen = []
    for op, back in ((lambda x: pkg.SHT.apply(x, plan), lambda g: plan.sht_T(g)),
                     (lambda x: pkg.ChannelMix.apply(x, W, plan), lambda g: plan.mix(W, g, adjoint=True)),
                     (lambda x: pkg.IsotropicFilter.apply(x, k, plan), lambda g: plan.filter(k, g, adjoint=True))):
        x = (draw(8, *plan.grid_shape()) if not seen else cdraw(9, *plan.spec_shape())).requires_grad_(True)
        y = op(x)
        y.register_hook(lambda g: seen.append(g))
        (y.conj() * w).real.sum().backward()
        g = seen[-1]
        assert g.is_conj()
        assert torch.equal(x.grad, back(g.resolve_conj()))


def test_lazy_outputs_and_graphs_are_refused(plan):
    y, x = cdraw(1, *plan.spec_shape()), draw(2, *plan.grid_shape())
    with pytest.raises(ValueError):
        plan.sht(x, out=y.conj())
    with pytest.raises(ValueError):
        plan.isht(y, out=torch._neg_view(x))
    with pytest.raises(ValueError):
        plan.mix(cdraw(3, L, C, C), y, out=torch.empty_like(y).conj())
    with pytest.raises(ValueError):
        plan.graph([("isht", y.conj(), x)])
    with pytest.raises(ValueError):
        plan.graph([("sht", x, y.conj())])
