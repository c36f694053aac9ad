"""Levels that are long enough to be captured, replayed and compared with the oracle's loop."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import muster_oracle as O  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
RAGGED = [((24, 28, 32), 3, 81), ((16, 24, 20), 4, 82), ((20, 20, 24), 2, 83)]


@pytest.fixture(scope="module")
def ctx():
    from paper_2412_14671_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("steps", [3, 4, 6])
def test_replayed_levels_match_the_oracle(ctx, steps, det):
    """Ragged subjects in one batch, on both sides of the length from which a level is captured:
    the first and last losses are the oracle loop's, with graphs on and off; a deterministic run
    gives the same bits either way, also when it is run again."""
    from paper_2412_14671_amd import MusterParams, synth
    subjects = [synth.phantom_series(shape, N, seed=seed) for shape, N, seed in RAGGED]
    kw = dict(iters=[steps], K=6, window=5, metric="silncc", alpha_ss=0.5, lr=0.05,
              smooth_sigma=1.0, deterministic=det)
    imgs = [s.images.to(DEV) for s in subjects]
    times = [s.times for s in subjects]
    runs = [ctx.register_batch(imgs, times, MusterParams(use_graph=g, **kw))
            for g in (True, False, True)]
    for k, s in enumerate(subjects):
        p = O.Params(K=6, window=5, metric=O.SILNCC, alpha_ss=0.5, lr=0.05, smooth_sigma=1.0,
                     iters=(steps,))
        sm, _, hist = O.register([x.numpy() for x in s.images], p)
        for outs, reps in runs:
            r = reps[k]
            print(f"{RAGGED[k]} steps {steps} det {det}: {r['loss_first']:.8g} "
                  f"{r['loss_last']:.8g} oracle {hist[0]:.8g} {hist[-1]:.8g}", flush=True)
            assert r["status"] == 0 and r["iterations"] == steps
            assert abs(r["loss_first"] - hist[0]) < 1e-3 * abs(hist[0])
            assert abs(r["loss_last"] - hist[-1]) < 1e-3 * abs(hist[-1])
            got, want = outs[k].cpu().numpy().astype(np.float64), np.stack(sm)
            assert np.linalg.norm(got - want) < 2e-2 * np.linalg.norm(want)
            if det:
                assert torch.equal(outs[k], runs[0][0][k])
