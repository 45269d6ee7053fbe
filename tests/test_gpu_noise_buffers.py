"""Noise.step checks the buffer it is given before the kernels write to it."""
import pytest

from _util import ensure_built

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    ensure_built()
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_12144_amd as P
    return P


def test_output_buffer(pkg):
    plan = pkg.Plan(dict(nlat=9, nlon=16, lmax=8, mmax=8, grid="equiangular", batch=2, channels=2))
    noise = pkg.Noise(plan, 0.1, 1.0, 1.0, seed=3)
    shape, n = plan.grid_shape(), 2 * 2 * 9 * 16
    bad = [torch.empty(n - 1, device="cuda"), torch.empty(shape, dtype=torch.float16, device="cuda"), torch.empty(shape),
           torch.empty(shape + (2,), device="cuda")[..., 0], torch._neg_view(torch.empty(shape, device="cuda")), "field"]
    before = noise.state.clone()
    for out in bad:
        with pytest.raises(ValueError):
            noise.step(out=out)
    assert torch.equal(noise.state, before)
    # a buffer with room for the field, of any shape, is filled from its start
    flat = torch.zeros(n + 5, device="cuda")
    _, out = noise.step(out=flat)
    assert out is flat
    other = pkg.Noise(plan, 0.1, 1.0, 1.0, seed=3)
    _, field = other.step()
    assert torch.equal(flat[:n], field.reshape(-1)) and not flat[n:].any()
    other.close()
    noise.close()
    plan.close()
