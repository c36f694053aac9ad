"""The window statistics and their adjoint against the oracle where the cuts along z end: depths
around multiples of the window (the parts of a chunk), grids around the tile widths, every tile
shape and window."""
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


@pytest.mark.parametrize("w", [3, 5, 7])
@pytest.mark.parametrize("shape", [0, 1, 2])
@pytest.mark.parametrize("dims", [(7, 9, 33), (8, 17, 31), (15, 16, 65), (29, 8, 64), (36, 18, 12)])
def test_parts_of_a_chunk(ctx, w, shape, dims):
    rng = np.random.Generator(np.random.PCG64(sum(dims) + w + shape))
    z, y, x = np.meshgrid(*[np.arange(n) for n in dims], indexing="ij")

    def image(p):
        return (0.5 + 0.3 * np.sin(0.31 * z + 0.23 * y + 0.19 * x + p)
                + 0.05 * rng.standard_normal(dims)).astype(np.float32)

    F, I = image(0.0), image(0.4)
    U = rng.uniform(-1.5, 1.5, (3,) + dims).astype(np.float32)
    for metric, m in (("lncc", O.LNCC), ("silncc", O.SILNCC)):
        s_ref, g_ref = O.pair_sim_grad([F.astype(np.float64), I.astype(np.float64)],
                                       U.astype(np.float64), 0, 1, O.Params(window=w, metric=m))
        for zchunk in (dims[0], 11):
            ctx.set_tiling("fixed", shape=shape, zchunk=zchunk)
            val, g = ctx.sim(*[torch.from_numpy(a).cuda() for a in (F, I, U)], w, metric, grad=True)
            g = g.cpu().numpy()
            # fp32 moments of shifted values of unit scale against variances above 2e-3: 2^-23 of
            # each, a few hundred terms summed: within 1e-4
            err = np.abs(g - g_ref).max() / np.abs(g_ref).max()
            print(f"sim {dims} w {w} shape {shape} {metric} chunk {zchunk}: {err:.1e}", flush=True)
            assert abs(val - s_ref) < 1e-4 * abs(s_ref) and err < 1e-4
