"""Scratch of the adjoint of the integration against a context's budget."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 3, 4), (33, 40, 47)])
def test_flat_recompute_needs_five_fields(shape):
    """MUSTER_EXP_FLAT with recomputed steps runs in five fields of scratch, two of them for
    squaring steps, and gives what the other modes give."""
    from paper_2412_14671_amd import Context
    rng = np.random.Generator(np.random.PCG64(1))
    phi = torch.from_numpy(rng.standard_normal((3,) + shape).astype(np.float32)).cuda()
    G = torch.from_numpy(rng.standard_normal((3,) + shape).astype(np.float32)).cuda()
    wide = Context(0)
    try:
        base = wide.memory()["in_use"]
        want = wide.exp_bwd(phi, G, 7)
    finally:
        wide.close()
    field = 4 * phi.numel()
    c = Context(0, budget_bytes=base + 5 * field + 5 * 256)
    try:
        for K in (1, 2, 3, 7):
            got = c.exp_bwd(phi, G, K, mode="recompute", flat=True)
            assert torch.isfinite(got).all()
            # far voxels are added atomically, in any order
            if K == 7:
                assert (got - want).abs().max() <= 1e-4 * want.abs().max()
    finally:
        c.close()
