"""Deterministic mode with flows of several voxels: the fixed-point twins of the integration's
adjoint take what far voxels spread."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import muster_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_14671_amd import Context
    c = Context(0)
    c.set_tiling("default")
    yield c
    c.close()


def flows(shape, n, vmax, seed):
    """Smooth flows of up to vmax voxels."""
    rng = np.random.Generator(np.random.PCG64(seed))
    z, y, x = np.meshgrid(*[np.linspace(0, np.pi, k) for k in shape], indexing="ij")
    out = []
    for _ in range(n):
        a = rng.uniform(0.5, 1.0, 3) * rng.choice([-1, 1], 3)
        p = rng.uniform(0, 2, 3)
        f = np.stack([a[c] * np.sin(z + p[c]) * np.cos(y - p[c]) * np.sin(x + 2 * p[c])
                      for c in range(3)])
        out.append((f * (vmax / np.sqrt((f ** 2).sum(0)).max())).astype(np.float32))
    return np.stack(out)


def run(ctx, jobs, params):
    """One registration call over (series, initial flows) jobs; the flows and reports."""
    from paper_2412_14671_amd import _lib as L
    from paper_2412_14671_amd.api import _stream
    keep, outs = [], []
    arr = (L.Job * len(jobs))()
    for k, (s, init) in enumerate(jobs):
        imgs, phi = s.images.to(DEV), torch.from_numpy(init).to(DEV)
        out = torch.empty_like(phi)
        keep += [imgs, phi]
        outs.append(out)
        arr[k] = ctx._job(imgs, s.times, params, out, None, svf_init=phi, keep=keep)
    reps = (L.Report * len(jobs))()
    L.check(ctx.lib.muster_register_batch(ctx.h, _stream(), len(jobs), arr, reps))
    return outs, [r.as_dict() for r in reps]


@pytest.mark.parametrize("K,vmax", [(1, 5.0), (4, 6.0), (5, 1.5)])
@pytest.mark.parametrize("mode", ["store", "recompute"])
def test_gradient_of_large_flows(ctx, K, vmax, mode):
    """One Adam step with an eps far above the gradient moves the flows by -lr g / (|g| + eps): the
    step of a deterministic job is the oracle's gradient, has the same bits alone, again and in a
    batch, and agrees with the default mode."""
    from paper_2412_14671_amd import MusterParams, synth
    made = [((20, 24, 33), 3, 91), ((17, 30, 24), 2, 92)]
    jobs = [(synth.phantom_series(shape, N, seed=seed), flows(shape, N - 1, vmax, seed))
            for shape, N, seed in made]
    kw = dict(iters=[1], K=K, window=5, metric="silncc", alpha_ss=0.5, exp_mode=mode, eps=1.0)
    p = O.Params(K=K, window=5, metric=O.SILNCC, alpha_ss=0.5)
    wants = []
    for s, init in jobs:
        L_ref, g, _ = O.loss_and_grad([f.astype(np.float64) for f in init],
                                      [x.numpy().astype(np.float64) for x in s.images], p)
        wants.append((L_ref, np.stack(g)))
    top = max(np.abs(g).max() for _, g in wants)
    assert top < 1e-1
    kw["lr"] = float(1.0 / top)     # the largest step is about a voxel
    det = MusterParams(deterministic=True, **kw)
    both, reps = run(ctx, jobs, det)
    again, _ = run(ctx, jobs, det)
    free, _ = run(ctx, jobs, MusterParams(deterministic=False, **kw))
    for k, (s, init) in enumerate(jobs):
        (alone,), _ = run(ctx, [jobs[k]], det)
        assert torch.equal(both[k], again[k]) and torch.equal(both[k], alone)
        L_ref, g = wants[k]
        assert abs(reps[k]["loss_first"] - L_ref) < 1e-3 * abs(L_ref)
        want = -kw["lr"] * g / (np.abs(g) + 1.0)
        got = both[k].cpu().numpy().astype(np.float64) - init
        other = free[k].cpu().numpy().astype(np.float64) - init
        rel = np.linalg.norm(got - want) / np.linalg.norm(want)
        mx = np.abs(got - want).max() / np.abs(want).max()
        print(f"{made[k]} K {K} vmax {vmax} {mode}: rel {rel:.2e} max {mx:.2e} "
              f"default {np.abs(got - other).max():.2e}", flush=True)
        # a sample position within rounding (2^-21 of a voxel here) of a cell's face may take the
        # other cell's derivative: about one in a million of some million samples, each of which
        # moves a few values by at most their own size
        assert rel < 1e-2
        assert np.quantile(np.abs(got - want), 0.999) < 1e-3 * np.abs(want).max()
        # flows of a few voxels are held to 2^-22; twice that, and the accumulations' rounding
        assert np.abs(got - other).max() < 1e-4
