"""The periodic Gaussian against the oracle where its staging can go wrong: lines shorter than a
chunk of outputs and than the taps, taps over the whole line, the longest rows and taps, and
tiles with a few lines left over."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import muster_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_14671_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dims,sigma", [
    ((1, 1, 1), 1.0), ((2, 3, 5), 3.0), ((7, 8, 9), 0.4), ((5, 257, 3), 0.4), ((65, 33, 17), 3.0),
    ((3, 4, 4096), 2.0), ((2, 300, 130), 22.0), ((300, 2, 31), 20.0), ((128, 9, 127), 1.5)])
def test_smooth_at_the_ends_of_its_tiles(ctx, dims, sigma):
    rng = np.random.Generator(np.random.PCG64(sum(dims)))
    v = rng.standard_normal((3,) + dims).astype(np.float32)
    got = ctx.smooth(torch.from_numpy(v).cuda(), sigma).cpu().numpy()
    want = O.smooth(v.astype(np.float64), sigma)
    # three passes of at most 257 taps that sum to 1 in magnitude (ringing ones to 2): rounding
    # 2^-24 of the largest value per term, growing with the root of the terms
    tol = 3 * 16 * 2.0 ** -24 * 2 * np.abs(v).max()
    err = np.abs(got - want).max()
    print(f"smooth {dims} sigma {sigma}: {err:.1e} of {tol:.1e}", flush=True)
    assert err < tol
