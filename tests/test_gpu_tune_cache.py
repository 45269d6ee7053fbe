"""The tuner's cache file gives the schedule that was measured, whatever
schedule a plan has when it is tuned again."""
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


@pytest.mark.parametrize("precision", ["fp32", "bf16x2"])
def test_cached_schedule(pkg, tmp_path, precision):
    print("tuner cache", precision, flush=True)
    cache = tmp_path / "tuned"
    desc = dict(nlat=33, nlon=64, lmax=32, mmax=32, grid="equiangular", channels=24)
    plan = pkg.Plan(desc, precision=precision)
    _, ms = plan.tune(cache)
    assert ms > 0
    best = plan.schedule()
    for staged in range(4):
        other = pkg.Plan(desc, precision=precision)
        other.set_schedule(16, 1, 2, staged)
        index, ms = other.tune(cache)
        assert ms == -1.0 and other.schedule() == best, (staged, other.schedule(), best)
        other.close()
    again, ms = plan.tune(cache)
    assert ms == -1.0 and plan.schedule() == best
    # a line that holds no schedule of the tuner is measured again
    key = cache.read_text().splitlines()[-1].rsplit("\t", 1)[0]
    for broken in ("", "3", "7 7 7 7", "8 0 2"):
        cache.write_text(key + "\t" + broken + "\n")
        assert plan.tune(cache)[1] > 0, broken
    plan.close()
