"""How far smoothing carries a value that is not finite."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_14671_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("sigma", [2.2, 3.0, 4.1])
def test_smoothing_of_a_nan_stays_within_reach(ctx, sigma):
    """Outputs are summed eight at a time from the samples that the eight reach: a NaN changes
    none farther away than the filter's radius and seven."""
    n = 96
    mid = (40, 51, 45)
    for axis in range(3):
        x = torch.zeros((3, n, n, n), device="cuda")
        x[(1,) + mid] = 1.0
        hit = (ctx.smooth(x, sigma)[1] != 0).nonzero()[:, axis] - mid[axis]
        radius = int(hit.abs().max())
        assert 0 < radius < n // 2 - 16
        x[(1,) + mid] = float("nan")
        y = ctx.smooth(x, sigma)
        at = (~torch.isfinite(y[1])).nonzero()[:, axis] - mid[axis]
        print(f"sigma {sigma} axis {axis}: radius {radius}, NaN to {int(at.abs().max())}", flush=True)
        assert radius <= int(at.abs().max()) <= radius + 7
        assert torch.isfinite(y[0]).all() and torch.isfinite(y[2]).all()
