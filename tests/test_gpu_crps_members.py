"""Ensemble CRPS gradients at every kind of member count (a kernel of its own
up to 16 members, shared ones of 32 and 64 above) and at the values where a
pair's sign can go wrong: ties, differences of one denormal, infinities and
NaN.

The gradient of a member is w (sign(v_e - obs) / N - sum_i sign(v_e - v_i) / D),
D = N^2 or N (N - 1), with the sign of a tie and of a NaN difference 0.  The
signs and their sum are whole numbers that both sides take exactly; what is
left are the roundings of 1/N, 1/D and w, two products, a difference and the
product with w: the difference from float64 is at most 5 * 2^-24 of
w (1/N + |sum| / D).  Losses of finite ensembles: at most 2 N + log2(points)
roundings, relative to the sum of the skill terms.
"""
import math

import numpy as np
import pytest

from _util import ensure_built

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

NLAT, NLON, C = 9, 16, 2


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


def _sign(d):
    return np.where(np.isnan(d), 0.0, np.sign(d))


@pytest.mark.parametrize("fair", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 15, 16, 17, 33, 64])
def test_gradient_signs(pkg, N, fair):
    if fair and N < 2:
        pytest.skip("the fair form needs two members")
    print("crps members", N, fair, flush=True)
    rng = np.random.default_rng(N)
    ens = rng.standard_normal((N, C, NLAT, NLON)).astype(np.float32)
    obs = rng.standard_normal((C, NLAT, NLON)).astype(np.float32)
    ens[0, 0, 2, 3] = obs[0, 2, 3]
    if N > 1:
        ens[1, 0, 3] = ens[0, 0, 3]                                  # a ring of ties
        ens[1, 0, 4] = np.nextafter(ens[0, 0, 4], np.float32(9))     # neighbours
        ens[0, 0, 5, 0], ens[1, 0, 5, 0] = 0.0, np.float32(1e-45)    # one denormal apart
        ens[0, 0, 5, 1], ens[1, 0, 5, 1] = 0.0, -0.0
        ens[0, 1, 2, 0], ens[N - 1, 1, 2, 1] = np.inf, -np.inf
        ens[0, 1, 3, 0] = np.nan
        ens[:, 1, 4, 0] = np.inf
    plan = pkg.Plan(dict(nlat=NLAT, nlon=NLON, lmax=4, mmax=4, grid="equiangular", batch=N, channels=C))
    loss, g = plan.spatial_crps(torch.from_numpy(ens).cuda(), torch.from_numpy(obs).cuda(), fair=fair, grad=True)
    loss0 = plan.spatial_crps(torch.from_numpy(ens).cuda(), torch.from_numpy(obs).cuda(), fair=fair)
    w = (2 * math.pi / NLON * plan.grid()[1].numpy() / (4 * math.pi))[:, None]
    e, o = ens.astype(np.float64), obs.astype(np.float64)
    with np.errstate(invalid="ignore"):
        rank = sum(_sign(e - e[i]) for i in range(N))
        skill = _sign(e - o)
        D = N * (N - 1) if fair else N * N
        ref = w * (skill / N - rank / D)
        size = w * (np.abs(skill) / N + np.abs(rank) / D)
        assert np.all(np.abs(g.cpu().numpy() - ref) <= 5 * 2.0 ** -24 * size)
        # the channel without special values (and every one of a lone member)
        for c in range(C) if N == 1 else [0]:
            terms = np.abs(e[:, c] - o[c]).sum(0) / N
            val = float((w * (terms - sum(np.abs(e[:, c] - e[i, c]).sum(0) for i in range(N)) / (2 * D))).sum())
            for got in (loss, loss0):
                assert abs(float(got[c]) - val) <= 2.0 ** -24 * (2 * N + 8) * float((w * terms).sum())
    plan.close()
