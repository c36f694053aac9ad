"""The regulariser's value where it is asked for by itself or with a loss: squares of fp32
differences, exact in 64 bits, summed in 64 bits."""
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


def whole(shape, seed):
    """A field of whole numbers: its differences are exact in fp32, their squares are not."""
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng.integers(-(2 ** 13) - 1, 2 ** 13 + 2, (3,) + shape).astype(np.float32)


@pytest.mark.parametrize("shape", [(2, 3, 2), (5, 9, 33), (17, 16, 64)])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** 70, 2.0 ** -70])
def test_value_is_formed_in_64_bits(ctx, shape, scale):
    """Also of fields whose squares are beyond fp32's range, either way."""
    f = whole(shape, sum(shape)) * np.float32(scale)
    want = O.reg_ss(f.astype(np.float64))
    # a sum of n squares in 64 bits, and one over the slots: n 2^-53 at most
    tol = f.size * 2.0 ** -53
    for grad in (False, True):
        val = ctx.reg(torch.from_numpy(f).cuda(), grad=grad)
        val = val[0] if grad else val
        print(f"{shape} scale {scale:.0e} grad {grad}: {abs(val / want - 1):.1e}", flush=True)
        assert abs(val - want) <= tol * want


def test_loss_value_holds_the_same_sum(ctx):
    """The loss of fields whose squares are beyond fp32's range is finite, and is the similarity
    plus alpha times the mean of the regularisers."""
    from paper_2412_14671_amd import MusterParams
    from paper_2412_14671_amd.api import loss_value
    shape, alpha = (12, 14, 16), 0.25
    rng = np.random.Generator(np.random.PCG64(3))
    imgs = torch.from_numpy(rng.random((3,) + shape, dtype=np.float32)).cuda()
    svf = np.stack([whole(shape, 5), whole(shape, 6)]) * np.float32(2.0 ** 70)
    p = MusterParams(K=4, window=3, metric="silncc", alpha_ss=alpha)
    got = loss_value(torch.from_numpy(svf).cuda(), imgs, p, ctx)
    want = alpha / 2 * sum(O.reg_ss(f.astype(np.float64)) for f in svf)
    # the similarity of unit images is nothing beside 2^140
    assert np.isfinite(got) and abs(got - want) <= svf.size * 2.0 ** -53 * want
