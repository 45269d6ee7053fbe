"""Ensemble CRPS losses of infinite values, for every kind of member count: an
infinite member gives NaN (its skill term less its spread term, its own
difference among them: inf - inf), an infinite observation an infinite loss, as
the spread-skill sums give in float64; other channels are finite.  And losses and gradients of finite values at the edges
of the ranges of member counts that share a kernel, against the oracle: a loss
within 2 N + 8 roundings of its skill terms, a gradient within five of its terms
(its signs and their sums are exact)."""
import numpy as np
import pytest

import oracle
from _util import ensure_built

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

NLAT, NLON, L, C = 9, 16, 8, 3


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("N", [1, 2, 16, 17, 24, 25, 33, 64])
def test_infinite_values(pkg, N):
    print("crps values", N, flush=True)
    rng = np.random.default_rng(N)
    plan = pkg.Plan(dict(nlat=NLAT, nlon=NLON, lmax=L, mmax=L, grid="equiangular", batch=N, channels=C))
    for spectral in (False, True):
        shape = (L, L) if spectral else (NLAT, NLON)
        draw = lambda *s: rng.standard_normal(s + shape).astype(np.float32)  # noqa: E731
        ens, obs = draw(N, C), draw(C)
        if spectral:
            ens, obs = ens + 1j * draw(N, C), obs + 1j * draw(C)
        ens[N - 1, 0, 3, 1] = np.inf
        obs[1, 4, 2] = -np.inf
        crps = plan.spectral_crps if spectral else plan.spatial_crps
        de, do = (torch.from_numpy(v.astype(np.complex64 if spectral else np.float32)).cuda() for v in (ens, obs))
        losses = [crps(de, do), crps(de, do, grad=True)[0]]
        if N > 1:
            losses.append(crps(de, do, fair=True))
        with np.errstate(invalid="ignore"):
            one = oracle.crps_spread_skill(ens.real[:, 0, 3, 1], obs.real[0, 3, 1])
        assert np.isnan(one)
        for loss in losses:
            a, b, c = (float(v) for v in loss)
            assert np.isnan(a) and b == np.inf and np.isfinite(c), (spectral, N, a, b, c)
    plan.close()


@pytest.mark.parametrize("N", [17, 18, 23, 24, 25, 26, 31, 32, 33, 34, 63, 64])
def test_member_counts(pkg, N):
    print("crps member counts", N, flush=True)
    rng = np.random.default_rng(100 + N)
    plan = pkg.Plan(dict(nlat=NLAT, nlon=NLON, lmax=L, mmax=L, grid="equiangular", batch=N, channels=C))
    ens = rng.standard_normal((N, C, NLAT, NLON)).astype(np.float32)
    obs = rng.standard_normal((C, NLAT, NLON)).astype(np.float32)
    w = 2 * np.pi / NLON * plan.grid()[1].numpy()[:, None] / (4 * np.pi)
    e, o = ens.astype(np.float64), obs.astype(np.float64)
    for fair in (False, True):
        de, do = torch.from_numpy(ens).cuda(), torch.from_numpy(obs).cuda()
        loss, g = plan.spatial_crps(de, do, fair=fair, grad=True)
        alone = plan.spatial_crps(de, do, fair=fair)
        D = N * (N - 1) if fair else N * N
        rank = sum(np.sign(e - e[i]) for i in range(N))
        ref = w * oracle.crps_spread_skill_grad(e, o, fair)
        assert np.all(np.abs(g.cpu().numpy() - ref) <= 5 * 2.0 ** -24 * w * (1.0 / N + np.abs(rank) / D))
        ref = (w * oracle.crps_spread_skill(e, o, fair)).sum((1, 2))
        size = (w * np.abs(e - o).mean(0)).sum((1, 2))
        for got in (loss, alone):
            assert np.all(np.abs(got.cpu().numpy() - ref) <= 2.0 ** -24 * (2 * N + 8) * size), (N, fair)
    plan.close()
