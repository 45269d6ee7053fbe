"""Weight gradient over many members of few orders, where the contraction takes
the (member, order) columns in one row and a lane's four columns can lie in up
to four members, against the FP64 oracle.

Tolerance: a sum of `steps` matrix instructions of six products each, every one
rounding once relative to the terms' size, twice for cancelling terms.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# batch, channels, lmax, mmax
SHAPES = [(33, 17, 9, 9), (64, 20, 3, 1), (5, 65, 40, 17), (16, 129, 24, 24), (2, 16, 34, 33), (7, 5, 5, 5),
          (1, 1, 1, 1), (40, 33, 16, 16), (2, 49, 70, 64), (3, 240, 40, 12), (1, 300, 20, 20), (2, 257, 33, 33), (1, 384, 17, 16)]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}C{}L{}M{}".format(*s))
def test_weight_gradient_members(pkg, shape):
    B, C, L, M = shape
    print("weight gradient members", shape, flush=True)
    rng = np.random.default_rng(31)
    draw = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)  # noqa: E731
    g, x = draw(B, C, L, M), draw(B, C, L, M)
    live = np.arange(L)[:, None] >= np.arange(M)[None, :]
    ref = oracle.channel_mix_dW(np.where(live, g, 0).astype(np.complex128), np.where(live, x, 0).astype(np.complex128))
    plan = pkg.Plan(dict(nlat=L + 1, nlon=max(2, 2 ** math.ceil(math.log2(2 * M))), lmax=L, mmax=M, grid="gauss",
                         batch=B, channels=C))
    # entries m > l are no part of the spectra
    nan = np.complex64(complex(float("nan"), float("nan")))
    dg, dx = (torch.from_numpy(np.where(live, v, nan)).cuda() for v in (g, x))
    got = plan.mix_weight_grad(dg, dx).cpu().numpy()
    for l in range(L):
        tol = 2.0 ** -24 * max(4, 12 * math.ceil(B * min(l + 1, M) / 16))
        e = rel_l2(got[l], ref[l])
        assert e <= tol, (l, e, tol)
    plan.close()
