"""How far a value that is not finite reaches: no farther than the voxels that read it."""
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


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_exp_adjoint_spreads_a_gradient_over_its_cell_only(ctx, bad):
    """One squaring, every displacement below one voxel: a gradient that is not finite changes its
    own voxel (through the Jacobian, every component) and the corners of its cell (its own
    component); the other values are those without it."""
    shape, vmax = (9, 17, 66), 0.9
    rng = np.random.Generator(np.random.PCG64(17))
    u = vmax * (2.0 * rng.random((3,) + shape) - 1.0)
    phi = (2.0 * u).astype(np.float32)
    G = rng.standard_normal((3,) + shape).astype(np.float32)
    # the inside, a border, a corner of the grid and both sides of a column tile's edge
    sites = [(0, (4, 4, 10)), (1, (0, 9, 40)), (2, (8, 16, 65)), (0, (6, 7, 31)), (1, (2, 8, 32))]
    clean = G.astype(np.float64)
    reach = np.zeros((3,) + shape, bool)
    full = np.zeros((3,) + shape, bool)    # corners of positive weight: not finite
    u64 = 0.5 * phi.astype(np.float64)
    for c, p in sites:
        G[(c,) + p] = bad
        clean[(c,) + p] = 0.0
        reach[(slice(None),) + p] = True
        q = [min(max(p[d] + u64[(d,) + p], 0.0), shape[d] - 1.0) for d in range(3)]
        i0 = [min(int(np.floor(q[d])), shape[d] - 2) for d in range(3)]
        for k in range(8):
            v = tuple(i0[d] + (k >> d & 1) for d in range(3))
            w = np.prod([q[d] - i0[d] if k >> d & 1 else 1.0 - (q[d] - i0[d]) for d in range(3)])
            reach[(c,) + v] = True
            full[(c,) + v] |= w > 0.0
    want = 0.5 * O.exp_bwd(O.exp_fwd(phi.astype(np.float64), 1), clean)
    got = ctx.exp_bwd(torch.from_numpy(phi).cuda(), torch.from_numpy(G).cuda(), 1).cpu().numpy()
    print("not finite beyond the cells:", int((~np.isfinite(got) & ~reach).sum()), flush=True)
    assert np.isfinite(got[~reach]).all()
    assert not np.isfinite(got[full]).any()
    # as where far voxels meet: a quantum of at most 2^-21 max|G| per contribution, some tens of
    # them, and the Jacobian's 1 + 6 vmax
    tol = 0.5 * 64 * 2.0 ** -21 * np.abs(clean).max() * (1.0 + 6.0 * vmax)
    assert np.abs(got - want)[~reach].max() < tol
