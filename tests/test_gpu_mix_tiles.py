"""Per-degree channel mix, its adjoint and its weight gradient at the edges of
their tiles, against the FP64 oracle.

A workgroup's tile is 128 rows (output channels) x 64 columns ((member,
order) pairs, or channels for the weight gradient), four column blocks of 16;
the contraction (channels, or the orders of one member) runs in steps of 16
complex values.  The shapes put the channels at and around 16, 32, 64 and 128
and the columns of the highest degrees at and around multiples of 16 and 64.

Tolerance: an output is a sum of `steps` matrix instructions of six products
each, every one rounding once relative to the terms' size, twice for
cancelling terms: 2 * 2^-24 * 6 * steps, and at least four roundings.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# batch, channels, lmax, mmax
SHAPES = [(1, 1, 1, 1), (1, 15, 17, 17), (2, 16, 16, 9), (1, 17, 33, 32), (3, 33, 22, 22), (1, 64, 65, 64),
          (2, 65, 40, 33), (1, 128, 20, 20), (1, 129, 18, 18), (4, 160, 17, 16)]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}C{}L{}M{}".format(*s))
def test_mix_tile_edges(pkg, shape):
    B, C, L, M = shape
    print("mix tile edges", shape, flush=True)
    rng = np.random.default_rng(21)
    draw = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)  # noqa: E731
    W, x, g = draw(L, C, C), draw(B, C, L, M), draw(B, C, L, M)
    live = np.arange(L)[:, None] >= np.arange(M)[None, :]
    x0, g0 = np.where(live, x, 0).astype(np.complex128), np.where(live, g, 0).astype(np.complex128)
    refs = (oracle.channel_mix(x0, W), oracle.channel_mix_T(x0, W), oracle.channel_mix_dW(g0, x0))
    plan = pkg.Plan(dict(nlat=L + 1, nlon=max(2, 2 ** math.ceil(math.log2(2 * M))), lmax=L, mmax=M, grid="gauss",
                         batch=B, channels=C))
    # entries m > l are no part of the spectra
    nan = np.complex64(complex(float("nan"), float("nan")))
    dW, dx, dg = (torch.from_numpy(v).cuda() for v in (W, np.where(live, x, nan), np.where(live, g, nan)))
    outs = [t.cpu().numpy() for t in (plan.mix(dW, dx), plan.mix(dW, dx, adjoint=True), plan.mix_weight_grad(dg, dx))]
    steps = (math.ceil(C / 16), math.ceil(C / 16), B * math.ceil(M / 16))
    for name, o, r, n in zip(("mix", "adjoint", "weight gradient"), outs, refs, steps):
        tol = 2.0 ** -24 * max(4, 12 * n)
        e = rel_l2(o, r)
        print(f"  {name}: rel-L2 {e:.2e} (tolerance {tol:.2e})", flush=True)
        assert e <= tol, (name, e, tol)
    for o in outs[:2]:
        assert np.all(o[..., ~live] == 0)
    plan.close()
