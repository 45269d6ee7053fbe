"""Channel mix, adjoint and weight gradient over the magnitudes that float32
holds, against the FP64 oracle: operands near the smallest and the largest
normal numbers, and an infinity or NaN among ordinary values.

Float32 operands are split into three bf16 planes after a scaling by 2^16;
outputs of sums beyond 2^96 are taken again on the float32 matrix cores.

Tolerance: as for the tiles' edges, 2 * 2^-24 times the roundings of a sum:
six a step of 16 complex terms, or one a product (4 * 16 a step) where the sums
are taken again.
"""
import math

import numpy as np
import pytest

import oracle
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# batch, channels, lmax, mmax: several row and column tiles, ragged ones
B, C, L, M = 3, 145, 24, 22
SCALES = [(0, -120), (-120, 0), (-60, -60), (110, -110), (-126, 30), (60, 60), (126, -40), (90, -20)]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


def operands():
    rng = np.random.default_rng(8)
    draw = lambda *s: (rng.uniform(-1, 1, s) + 1j * rng.uniform(-1, 1, s)).astype(np.complex64)  # noqa: E731
    W, x, g = draw(L, C, C), draw(B, C, L, M), draw(B, C, L, M)
    live = np.arange(L)[:, None] >= np.arange(M)[None, :]
    return W, np.where(live, x, 0), np.where(live, g, 0)


def make_plan(pkg):
    return pkg.Plan(dict(nlat=L + 1, nlon=48, lmax=L, mmax=M, grid="gauss", batch=B, channels=C))


def run(plan, W, x, g):
    dW, dx, dg = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (W, x, g))
    return plan.mix(dW, dx), plan.mix(dW, dx, adjoint=True), plan.mix_weight_grad(dg, dx)


@pytest.mark.parametrize("ew,ex", SCALES)
def test_scaled_operands(pkg, ew, ex):
    print("mix magnitudes", ew, ex, flush=True)
    W, x, g = operands()
    sw, sx = np.float32(2.0 ** ew), np.float32(2.0 ** ex)
    W, x, g = W * sw, x * sx, g * sw
    plan = make_plan(pkg)
    outs = [t.cpu().numpy().astype(np.complex128) for t in run(plan, W, x, g)]
    W, x, g = (v.astype(np.complex128) for v in (W, x, g))
    refs = (oracle.channel_mix(x, W), oracle.channel_mix_T(x, W), oracle.channel_mix_dW(g, x))
    again = max(ew, ex) + 16 > 127 or ew + ex + 32 > 110
    steps = (math.ceil(C / 16), math.ceil(C / 16), B * math.ceil(M / 16))
    for name, o, r, n in zip(("mix", "adjoint", "weight gradient"), outs, refs, steps):
        tol = 2 * 2.0 ** -24 * (64 if again else 6) * n
        e = rel_l2(o, r)
        print(f"  {name}: rel-L2 {e:.2e} (tolerance {tol:.2e})", flush=True)
        assert e <= tol, (name, e, tol)
    plan.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_one_special_value(pkg, value):
    """An infinite or NaN part of one operand value: the outputs it enters are
    what float32 products and sums of the same terms give, the others the same
    bits as without it."""
    print("mix special value", value, flush=True)
    W, x, g = operands()
    plan = make_plan(pkg)
    clean = run(plan, W, x, g)
    b, c, c2, l, m = 1, 130, 37, 20, 5
    for which in ("W", "x", "g"):
        W1, x1, g1 = W.copy(), x.copy(), g.copy()
        if which == "W":
            W1[l, c, c2] = complex(value, 0.5)
        else:
            (x1 if which == "x" else g1)[b, c2, l, m] = complex(value, 0.5)
        outs = run(plan, W1, x1, g1)
        hit = [torch.zeros_like(t, dtype=torch.bool) for t in outs]
        if which == "W":
            hit[0][:, c, l, : min(l + 1, M)] = True
            hit[1][:, c2, l, : min(l + 1, M)] = True
        elif which == "x":
            hit[0][b, :, l, m] = hit[1][b, :, l, m] = True
            hit[2][l, :, c2] = True
        else:
            hit[2][l, c2, :] = True
        # float64 products of the real and imaginary parts, as the kernels form them
        with np.errstate(invalid="ignore"):
            Wd, xd, gd = (v.astype(np.complex128) for v in (W1[l], x1[:, :, l], g1[:, :, l]))

            def product(ar, ai, br, bi):
                return ar @ br - ai @ bi, ar @ bi + ai @ br

            cols = xd.transpose(1, 0, 2).reshape(C, -1)
            grad = gd.transpose(1, 0, 2).reshape(C, -1)
            mix = product(Wd.real, Wd.imag, cols.real, cols.imag)
            adj = product(Wd.real.T, -Wd.imag.T, cols.real, cols.imag)
            dw = product(grad.real, grad.imag, cols.real.T, -cols.imag.T)
        for name, o, cl, h, r in zip(("mix", "adjoint", "weight gradient"), outs, clean, hit, (mix, adj, dw)):
            assert torch.equal(torch.view_as_real(o)[~h], torch.view_as_real(cl)[~h]), (which, name)
            got = o[l] if name == "weight gradient" else o[:, :, l].transpose(0, 1).reshape(C, -1)
            at = (h[l] if name == "weight gradient" else h[:, :, l].transpose(0, 1).reshape(C, -1)).cpu().numpy()
            for part, ref in zip((got.real, got.imag), r):
                part = part.cpu().numpy()[at].astype(np.float64)
                assert np.array_equal(part, ref[at], equal_nan=True), (which, name)
    plan.close()
