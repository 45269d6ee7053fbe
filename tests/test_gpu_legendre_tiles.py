"""Legendre contraction at the edges of its tiles, against the FP64 oracle.

A workgroup's tile is at most 8 blocks of 16 rows by at most 9 column blocks
(groups of 8 fields), the contraction runs in steps of 32.  Rows are degrees
of one parity (analysis) or northern rings (synthesis), and the other of the
two is contracted, so the edges are: northern rings and degrees of a parity
at and around multiples of 16, 32 and 128, and field groups at and around the
chunk widths.

Tolerance: per output element a sum of `steps` matrix instructions of at most
six products each, every one rounding once, after a DFT of log2(nlon) levels
of two roundings and table and scale factors of four more, all relative to
the terms' size: 2^-24 (6 steps + 2 log2(nlon) + 4), doubled for cancelling
terms.  bf16x2 adds its table's representation error, at most 2^-16.
"""
import math

import numpy as np
import pytest

import oracle
import synth
from _util import ensure_built, rel_l2

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# nlat, nlon, lmax, mmax, grid, batch, channels
SHAPES = [
    (31, 64, 31, 32 - 1, 1, 1, 8),     # 16 northern rings: half a step, one group
    (33, 64, 33, 17, 0, 1, 9),         # 17 rings: two ring blocks; two groups, one ragged
    (63, 128, 64, 40, 1, 1, 72),       # 32 rings: one step; nine groups in one chunk
    (65, 128, 66, 33, 0, 1, 73),       # 33 rings; ten groups in two chunks
    (64, 128, 256, 20, 1, 1, 88),      # 128 degrees of a parity: one full tile; eleven groups, ragged last chunk
    (64, 128, 258, 5, 1, 1, 3),        # 129: two tiles, the smaller with four row blocks
    (257, 90, 290, 3, 0, 1, 5),        # 129 rings: two ring tiles, degrees beyond a step's end
    (511, 64, 20, 4, 1, 2, 65),        # 256 rings: two full ring tiles, one short step of degrees
]


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


@pytest.mark.parametrize("prec", ["fp32", "bf16x2", "bf16x3"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_L{s[2]}M{s[3]}_F{s[5] * s[6]}")
def test_tile_edges(pkg, shape, prec):
    nlat, nlon, lmax, mmax, grid, B, C = shape
    print("tile edges", shape, prec, flush=True)
    rng = np.random.default_rng(11)
    u = rng.standard_normal((B, C, nlat, nlon)).astype(np.float32)
    a = synth.coefficients(12, B, C, lmax, mmax).astype(np.complex64)
    u64, a64 = u.astype(np.float64), a.astype(np.complex128)
    refs = (oracle.sht(u64, lmax, mmax, grid), oracle.isht(a64, nlat, nlon, grid),
            oracle.sht_T(a64, nlat, nlon, grid), oracle.isht_T(u64, lmax, mmax, grid))
    steps = math.ceil(max((nlat + 1) // 2, (lmax + 1) // 2) / 32)
    tol = 2 * 2.0 ** -24 * (6 * steps + 2 * math.log2(nlon) + 4) + (2.0 ** -16 if prec == "bf16x2" else 0.0)
    plan = pkg.Plan(dict(nlat=nlat, nlon=nlon, lmax=lmax, mmax=mmax, grid=grid, batch=B, channels=C), precision=prec)
    du, da = torch.from_numpy(u).cuda(), torch.from_numpy(a).cuda()
    # entries l < m of the input are not part of the spectrum
    l, m = torch.arange(lmax, device="cuda")[:, None], torch.arange(mmax, device="cuda")[None, :]
    da = torch.where(l >= m, da, torch.full_like(da, float("nan")))
    first = None
    for staged in (0, 3):
        plan.set_schedule(8, 0, 2, staged)
        outs = (plan.sht(du), plan.isht(da), plan.sht_T(da), plan.isht_T(du))
        errs = [rel_l2(o.cpu().numpy(), r) for o, r in zip(outs, refs)]
        print(f"  staged {staged}: rel-L2", ["%.2e" % e for e in errs], "tolerance %.2e" % tol, flush=True)
        assert max(errs) <= tol, (staged, errs, tol)
        if first is None:
            first = outs
        else:
            assert all(torch.equal(o, f) for o, f in zip(outs, first))
    plan.close()
