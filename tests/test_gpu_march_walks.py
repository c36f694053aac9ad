"""The marching kernels where a block walks a long chunk of z with near and far voxels mixed, and
at grids around the 8 x 32 columns of a block."""
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


def fields(shape, vmax, K, seed):
    """A rough field whose last squaring samples up to vmax voxels away, a quarter of it on
    multiples of a quarter voxel, and a gradient of unit scale."""
    rng = np.random.Generator(np.random.PCG64(seed))
    u = vmax * (2.0 * rng.random((3,) + shape) - 1.0)
    snap = rng.random(shape) < 0.25
    u = np.where(snap, np.round(4.0 * u) / 4.0, u)
    return (2.0 * u).astype(np.float32), rng.standard_normal((3,) + shape).astype(np.float32)


def check(ctx, shape, vmax, K, modes):
    phi, G = fields(shape, vmax, K, seed=sum(shape) + K)
    us = O.exp_fwd(phi.astype(np.float64), K)
    # a squaring's Jacobian amplifies the rounding (2^-22 of the largest displacement) that the
    # steps before it left
    amp = sum((1.0 + 6.0 * vmax) ** s for s in range(K))
    got = ctx.exp(torch.from_numpy(phi).cuda(), K).cpu().numpy()
    err, tol = np.abs(got - us[-1]).max(), 2.0 ** -22 * np.abs(us[-1]).max() * amp
    print(f"exp {shape} vmax {vmax} K {K}: {err:.2e} of {tol:.2e}", flush=True)
    assert err < tol
    want = 2.0 ** -K * O.exp_bwd(us, G.astype(np.float64))
    # far voxels are summed in fixed point, 2^-21 max|G| per contribution at most, some tens of
    # them on a voxel
    tol = 2.0 ** -K * 64 * 2.0 ** -21 * np.abs(G).max() * amp
    for mode in modes:
        got = ctx.exp_bwd(torch.from_numpy(phi).cuda(), torch.from_numpy(G).cuda(), K, 1,
                          mode).cpu().numpy()
        err = np.abs(got - want).max()
        print(f"adjoint {shape} vmax {vmax} K {K} {mode}: {err:.2e} of {tol:.2e}", flush=True)
        assert err < tol


@pytest.mark.parametrize("vmax", [0.9, 1.4])
def test_chunks_of_eight_planes(ctx, vmax):
    """Large enough that both kernels take chunks of eight planes and a block of the far pass looks
    at more than one mark; the last chunk, rows and columns are cut short."""
    check(ctx, (110, 90, 255), vmax, 1, ("store",))


@pytest.mark.parametrize("shape", [(2, 7, 31), (3, 8, 32), (5, 9, 33), (4, 16, 64), (7, 17, 65),
                                   (8, 8, 63), (33, 7, 32)])
@pytest.mark.parametrize("vmax,K", [(0.9, 1), (1.3, 1), (4.0, 1), (1.2, 2)])
def test_edges_of_the_column_tiles(ctx, shape, vmax, K):
    check(ctx, shape, vmax, K, ("store", "recompute"))
