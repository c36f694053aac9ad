"""The marching kernels of the integration against the oracle where their
tiles, chunks and the limit of one voxel of displacement end: grids around
multiples of the 16 x 16 columns and of the point tiles, displacements on both
sides of one voxel (also exactly on it), from all near to all far, and the
clamp at every border."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import muster_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu

SHAPES = [(2, 15, 17), (3, 16, 16), (17, 33, 18), (9, 31, 47), (40, 17, 16)]


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
    phi = (u * 2.0 ** (K - (K - 1))).astype(np.float32)
    G = rng.standard_normal((3,) + shape).astype(np.float32)
    return phi, G


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("vmax,K", [(0.9, 1), (1.1, 1), (4.0, 1), (1.2, 2), (0.4, 3)])
def test_exp_adjoint_near_and_far(ctx, shape, vmax, K):
    phi, G = fields(shape, vmax, K, seed=sum(shape) + K)
    # far voxels are summed in fixed point with a quantum of at most the block's summed
    # magnitudes over 2^30 (1024 voxels), rounded to nearest: 2^-21 max|G| per contribution;
    # a rough field lays some tens of them on a voxel, and a squaring's Jacobian amplifies what
    # the steps before it left, by 1 + |du| below 1 + 2 vmax * 3
    amp = sum((1.0 + 6.0 * vmax) ** s for s in range(K))
    tol = 2.0 ** -K * 64 * 2.0 ** -21 * np.abs(G).max() * amp
    for sign in (1, -1):
        us = O.exp_fwd(sign * phi.astype(np.float64), K)
        want = sign * 2.0 ** -K * O.exp_bwd(us, G.astype(np.float64))
        for mode in ("store", "recompute"):
            got = ctx.exp_bwd(torch.from_numpy(phi).cuda(), torch.from_numpy(G).cuda(), K, sign,
                              mode).cpu().numpy()
            err = np.abs(got - want).max()
            print(f"exp adjoint {shape} vmax {vmax} K {K} sign {sign} {mode}: {err:.2e} of {tol:.2e}",
                  flush=True)
            assert err < tol


def test_exp_adjoint_writes_where_its_inputs_lie(ctx):
    """grad_svf may be the svf or, the gradient being read first, the incoming gradient."""
    import ctypes
    from paper_2412_14671_amd import _lib as L
    for K in (1, 3):
        phi, G = fields((18, 20, 35), 0.8, K, seed=K)
        want = ctx.exp_bwd(torch.from_numpy(phi).cuda(), torch.from_numpy(G).cuda(), K)
        for alias in (0, 1):
            p, g = torch.from_numpy(phi).cuda(), torch.from_numpy(G).cuda()
            out = (p, g)[alias]
            L.check(ctx.lib.muster_exp_bwd(ctx.h, None, L.DIMS(*phi.shape[1:]), K, 1,
                                           ctypes.c_void_p(p.data_ptr()),
                                           ctypes.c_void_p(g.data_ptr()),
                                           ctypes.c_void_p(out.data_ptr()), L.EXP_STORE))
            assert torch.equal(out, want)
