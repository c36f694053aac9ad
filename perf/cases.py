"""Performance cases: the work that programs have this library do, through its public entry points.

Whole registrations and single differentiable losses carry the main path (Exp, compositions,
similarity, their adjoints, the optimiser); the single steps are the same layers as tools call them.
Sizes are those of the repository's workloads: 32^3 blob series, 64^3 for the gradient check, 96^3,
128^3 and 160x192x160 phantoms, and ragged grids between them.

listed() names the cases, draw() gives more of the same ranges, prepare() makes a case's inputs on the
GPU from a seed, run() is one pass, work() the bytes and operations it cannot do without, and exact()
the same result in 64 bits by plain torch.
"""
import math

import numpy as np
import torch

from paper_2412_14671_amd import Context, MusterLoss, MusterParams

_ctx = None


def context():
    """The one context a program keeps for its GPU. Its tiling of the window statistics is fixed, as
    a program does that wants the same rounding from one process to the next (the autotuner may choose
    differently each time); the tile is the one that the autotuner picks for the larger grids."""
    global _ctx
    if _ctx is None:
        _ctx = Context(0)
        _ctx.set_tiling("fixed", shape=1, zchunk=32)
    return _ctx


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------

def listed():
    return [
        # integration of one small field, as an interactive tool does: launches and latency
        dict(name="exp_32", op="exp", D=32, H=32, W=32, K=7, sign=1, vmax=1.0),
        # integration of one full-size field, both directions being equal work
        dict(name="exp_160x192x160", op="exp", D=160, H=192, W=160, K=7, sign=-1, vmax=1.5),
        # adjoint of the integration on a ragged grid, squaring steps recomputed to save memory
        dict(name="exp_bwd_ragged", op="exp_bwd", D=97, H=113, W=101, K=6, sign=1, vmax=1.0,
             mode="recompute"),
        # adjoint of the integration at full size, squaring steps stored: the largest single layer
        dict(name="exp_bwd_160x192x160", op="exp_bwd", D=160, H=192, W=160, K=7, sign=1, vmax=1.5,
             mode="store"),
        # one link of a composition chain over several intervals, forward and backward
        dict(name="compose_128", op="compose", D=128, H=128, W=128, vmax=2.0),
        # similarity of one small pair with its gradient
        dict(name="sim_lncc_32", op="sim", D=32, H=32, W=32, window=5, metric="lncc"),
        # similarity of one full-size pair with its gradient (the robust metric)
        dict(name="sim_silncc_160x192x160", op="sim", D=160, H=192, W=160, window=7,
             metric="silncc"),
        # the pyramid's and the outputs' tools on one field: smoothing, resampling, regulariser,
        # Jacobian determinants
        dict(name="tools_96x128x112", op="tools", D=96, H=128, W=112, sigma=3.0),
        # loss and gradient inside a training loop, the gradient check's size
        dict(name="loss_4x64", op="loss", N=4, D=64, H=64, W=64, K=6, window=7, metric="lncc",
             alpha=1.0, sigma=0.0, mode="store", factor=1, frac=0.5),
        # loss and gradient at full size with the robust metric
        dict(name="loss_4x160x192x160", op="loss", N=4, D=160, H=192, W=160, K=7, window=7,
             metric="silncc", alpha=1.0, sigma=0.0, mode="store", factor=1, frac=0.5),
        # a whole small registration with its pair fields. Registrations take two steps here: Adam
        # multiplies rounding from step to step, so longer ones cannot be compared between builds;
        # a step of any length of schedule is the same work
        dict(name="register_3x32", op="register", jobs=1, N=3, D=32, H=32, W=32, iters="2", K=7,
             window=5, metric="silncc", alpha=1.0, sigma=1.5, pairs=True),
        # several subjects of uneven size and session count in one batch, with smoothed flows
        dict(name="batch_4_subjects", op="register", jobs=4, N=4, D=128, H=128, W=128, iters="2",
             K=7, window=7, metric="silncc", alpha=0.1, sigma=3.0, pairs=False),
    ]


def _edge(rng, lo, hi):
    """A grid edge, spread over the logarithm of its range; every parity occurs."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo=24, hi=176, most=160 * 192 * 160, even=1):
    while True:
        e = [max(lo, _edge(rng, lo, hi) // even * even) for _ in range(3)]
        if e[0] * e[1] * e[2] <= most:
            return dict(D=e[0], H=e[1], W=e[2])


def draw(rng):
    op = rng.choice(["exp", "exp_bwd", "exp_bwd", "compose", "sim", "tools", "loss", "loss",
                     "register", "batch"])
    vmax = round(math.exp(rng.uniform(math.log(0.3), math.log(2.5))), 3)
    metric = rng.choice(["lncc", "silncc"])
    window = rng.choice([3, 5, 7])
    K = rng.choice([4, 5, 6, 7])
    if op == "exp":
        return dict(op="exp", K=K, sign=rng.choice([1, -1]), vmax=vmax, **_grid(rng))
    if op == "exp_bwd":
        return dict(op="exp_bwd", K=K, sign=rng.choice([1, -1]), vmax=vmax,
                    mode=rng.choice(["store", "store", "recompute"]), **_grid(rng))
    if op == "compose":
        return dict(op="compose", vmax=vmax, **_grid(rng))
    if op == "sim":
        return dict(op="sim", window=window, metric=metric, **_grid(rng))
    if op == "tools":
        return dict(op="tools", sigma=round(rng.uniform(1.5, 4.0), 2),
                    **_grid(rng, hi=128, most=96 * 128 * 112, even=2))
    if op == "loss":
        return dict(op="loss", N=rng.choice([2, 3, 4]), K=K, window=window, metric=metric,
                    alpha=rng.choice([0.1, 1.0]), sigma=0.0,
                    mode=rng.choice(["store", "store", "recompute"]), factor=1,
                    frac=round(rng.uniform(0.2, 0.9), 2),
                    **_grid(rng, hi=160, most=160 * 160 * 160, even=2))
    jobs = 1 if op == "register" else rng.choice([2, 3, 4])
    return dict(op="register", jobs=jobs, N=rng.choice([2, 3, 4]), iters="2", K=7, window=window,
                metric="silncc", alpha=rng.choice([0.1, 1.0]), sigma=rng.choice([1.5, 3.0]),
                pairs=jobs == 1, **_grid(rng, hi=128, most=128 * 128 * 128, even=4))


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------

def _dims(c):
    return c["D"], c["H"], c["W"]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _smooth_noise(shape, sigma, g):
    """White noise of the given shape, Gaussian-smoothed over its last three axes."""
    x = torch.randn(shape, device="cuda", generator=g)
    w = [2 * math.pi * torch.fft.fftfreq(n, device="cuda") for n in shape[-3:-1]]
    wx = 2 * math.pi * torch.fft.rfftfreq(shape[-1], device="cuda")
    tf = torch.exp(-0.5 * sigma ** 2 * (w[0][:, None, None] ** 2 + w[1][None, :, None] ** 2
                                        + wx[None, None, :] ** 2))
    return torch.fft.irfftn(torch.fft.rfftn(x, dim=(-3, -2, -1)) * tf, s=shape[-3:],
                            dim=(-3, -2, -1))


def _velocity(dims, vmax, g, sigma=6.0):
    """A smooth random vector field of the given largest vector norm (voxels)."""
    v = _smooth_noise((3,) + tuple(dims), sigma, g)
    return (v * (vmax / v.square().sum(0).sqrt().max())).contiguous()


def _series(dims, N, g, vmax=1.0):
    """N sessions of a textured head-like phantom drifting along smooth fields, with a
    session-wise intensity bias and noise, and the per-interval fields. Grids of at most 40^3
    voxels hold blobs that fill them, with less noise and no bias, as the small workload does."""
    D, H, W = dims
    small = D * H * W <= 40 ** 3
    p = torch.stack(torch.meshgrid(*[torch.arange(n, device="cuda", dtype=torch.float32)
                                     for n in dims], indexing="ij"))
    tex = _smooth_noise((1,) + tuple(dims), 3.0 if small else 2.0, g)
    tex = torch.tanh(tex / tex.std())
    vs = [_velocity(dims, vmax, g) for _ in range(N - 1)]
    half = torch.tensor([n / 2.0 for n in dims], device="cuda")[:, None, None, None]
    out = []
    q = p.clone()
    for k in range(N):
        if k:
            q = q + vs[k - 1]
        rho = ((q - half + 0.5) / half).square().sum(0).sqrt()
        img = sum(0.3 * torch.sigmoid((f - rho) * half.min() * 0.8) for f in (0.84, 0.64, 0.40))
        n = torch.stack([2 * q[2] / (W - 1) - 1, 2 * q[1] / (H - 1) - 1, 2 * q[0] / (D - 1) - 1], -1)
        t = torch.nn.functional.grid_sample(tex[None], n[None], align_corners=True,
                                            padding_mode="border")[0, 0]
        noise = torch.randn(dims, device="cuda", generator=g)
        if small:
            out.append(0.5 + 0.4 * t + 0.01 * noise)
            continue
        img = img + 0.15 * torch.sigmoid((0.84 - rho) * half.min() * 0.8) * t
        b = _smooth_noise((1,) + tuple(dims), 16.0, g)[0]
        img = img * (1 + 0.1 * b / b.abs().max())
        out.append((img + 0.02 * noise).abs())
    return torch.stack(out).contiguous(), vs


def _pair_gradient(dims, g):
    """The gradient that reaches an integration or a composition in a registration: that of one
    pair's similarity with respect to its deformation."""
    imgs, vs = _series(dims, 2, g)
    U = (-0.5 * vs[0]).double().requires_grad_(True)
    _sim64(imgs[0].double(), imgs[1].double(), U, 5, "lncc").backward()
    return U.grad.float().contiguous()


def _subjects(c):
    """(N, dims) of each subject of a registration case: the first as stated, the others with
    fewer voxels and one session more or less in turn."""
    subs = []
    lv = 2 ** (len(_iters(c)) - 1)
    for k in range(c["jobs"]):
        d = [max(16, int(n * (1 - 0.12 * k)) // (4 * lv) * (4 * lv)) if k else n for n in _dims(c)]
        subs.append((max(2, c["N"] + (0, 1, -1, 0)[k % 4]), tuple(d)))
    return subs


def _iters(c):
    return [int(t) for t in c["iters"].split(",")]


def _params(c):
    if c["op"] == "register":
        return MusterParams(iters=_iters(c), K=c["K"], window=c["window"], metric=c["metric"],
                            alpha_ss=c["alpha"], smooth_sigma=c["sigma"])
    return MusterParams(K=c["K"], window=c["window"], metric=c["metric"], alpha_ss=c["alpha"],
                        smooth_sigma=c["sigma"], exp_mode=c["mode"], flow_factor=c["factor"])


def _inputs(c, seed):
    """The tensors of a case, made from the seed alone."""
    g = _gen(seed)
    d = _dims(c)
    op = c["op"]
    if op == "exp":
        return dict(svf=_velocity(d, c["vmax"], g))
    if op == "exp_bwd":
        return dict(svf=_velocity(d, c["vmax"], g), G=_pair_gradient(d, g))
    if op == "compose":
        return dict(U=_velocity(d, c["vmax"], g), C=_velocity(d, 0.7 * c["vmax"], g),
                    G=_pair_gradient(d, g))
    if op == "sim":
        imgs, vs = _series(d, 2, g)
        return dict(F=imgs[0].contiguous(), I=imgs[1].contiguous(), U=(-0.5 * vs[0]).contiguous())
    if op == "tools":
        imgs, vs = _series(d, 2, g)
        return dict(img=imgs[0].contiguous(), v=vs[0],
                    fine=_smooth_noise((3, 2 * d[0], 2 * d[1], 2 * d[2]), 1.5, g).contiguous())
    if op == "loss":
        imgs, vs = _series(d, c["N"], g)
        f = c["factor"]
        flows = [-c["frac"] / f * v[:, ::f, ::f, ::f] for v in vs]
        return dict(images=imgs, svf=torch.stack(flows).contiguous())
    return dict(series=[_series(dd, n, g)[0] for n, dd in _subjects(c)])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["ctx"] = context()
    if case["op"] in ("loss", "register"):
        s["params"] = _params(case)
    if case["op"] == "loss":
        s["svf"].requires_grad_(True)
    return s


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------

def run(s):
    c, ctx = s["case"], s["ctx"]
    op = c["op"]
    if op == "exp":
        return ctx.exp(s["svf"], c["K"], sign=c["sign"])
    if op == "exp_bwd":
        return ctx.exp_bwd(s["svf"], s["G"], c["K"], sign=c["sign"], mode=c["mode"])
    if op == "compose":
        out = ctx.compose(s["U"], s["C"])
        gp, gc = torch.zeros_like(s["U"]), torch.zeros_like(s["U"])
        ctx.compose_bwd(s["U"], s["C"], s["G"], gp, gc)
        return dict(out=out, G_prev=gp, G_C=gc)
    if op == "sim":
        val, g = ctx.sim(s["F"], s["I"], s["U"], c["window"], c["metric"], grad=True)
        return dict(sim=val, grad=g)
    if op == "tools":
        reg, rg = ctx.reg(s["v"], grad=True)
        return dict(pool=ctx.pool2(s["img"]), smooth=ctx.smooth(s["v"], c["sigma"]),
                    up=ctx.upsample2(s["v"]), down=ctx.upsample2_adjoint(s["fine"]), reg=reg,
                    reg_grad=rg, jac=ctx.jacobian_det(s["v"]))
    if op == "loss":
        svf = s["svf"]
        svf.grad = None
        loss = MusterLoss.apply(svf, s["images"], s["params"], ctx)
        loss.backward()
        return dict(loss=float(loss.detach()), grad=svf.grad)
    if c["jobs"] == 1:
        svf, pairs, rep = ctx.register(s["series"][0], None, s["params"], pairs=c["pairs"])
        out = [dict(svf=svf, first=rep["loss_first"], last=rep["loss_last"])]
        if pairs is not None:
            out[0]["pairs"] = pairs
        return out
    svfs, reps = ctx.register_batch(s["series"], None, s["params"])
    return [dict(svf=v, first=r["loss_first"], last=r["loss_last"]) for v, r in zip(svfs, reps)]


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------

_SAMPLE = 3 * (7 * 3 + 6)     # three components: seven interpolations, and the position


def _iteration_work(N, Vi, Vf, K):
    """Bytes and operations of one loss and gradient. Between its layers everything has to go
    through memory: each layer's inputs read once and its outputs written once."""
    dirs, pairs, deep = 2 * (N - 1), N * (N - 1), (N - 1) * (N - 2)
    by = dirs * Vf * (24 * K + 36 * K) + deep * Vf * (36 + 60) + pairs * Vi * (20 + 32)
    fl = dirs * Vf * K * (_SAMPLE + 250) + deep * Vf * (_SAMPLE + 250) + pairs * Vi * 200
    return by, fl


def work(c):
    d = _dims(c)
    V = d[0] * d[1] * d[2]
    op = c["op"]
    if op == "exp":
        return {"bytes": 24 * V, "flops": c["K"] * _SAMPLE * V}
    if op == "exp_bwd":
        return {"bytes": 36 * V, "flops": c["K"] * (2 * _SAMPLE + 250) * V}
    if op == "compose":
        return {"bytes": (36 + 60) * V, "flops": (_SAMPLE + 250) * V}
    if op == "sim":
        return {"bytes": (8 + 12 + 12) * V, "flops": 200 * V}
    if op == "tools":
        return {"bytes": (4 + 0.5 + 24 + 108 + 108 + 24 + 16) * V, "flops": 600 * V}
    if op == "loss":
        f = c["factor"] ** 3
        by, fl = _iteration_work(c["N"], V, V // f, c["K"])
        return {"bytes": by, "flops": fl}
    by = fl = 0
    its = _iters(c)
    for N, dd in _subjects(c):
        V = dd[0] * dd[1] * dd[2]
        for lv, n in enumerate(its):
            b, f = _iteration_work(N, V // 8 ** (len(its) - 1 - lv), V // 8 ** (len(its) - 1 - lv),
                                   c["K"])
            by, fl = by + n * (b + (N - 1) * V * 84 // 8 ** (len(its) - 1 - lv)), fl + n * f
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ---------------------------------------------------------------------------------------------

def _axis(u, n, dim):
    """Cell, fraction along one axis of the displaced grid positions, clamped to the grid."""
    shape = [1, 1, 1]
    shape[dim] = -1
    p = torch.arange(n, device=u.device).view(shape)
    fl = torch.floor(u.detach())
    i = p + fl.long()
    t = u - fl
    low, high = i < 0, i >= n - 1
    exact_end = (i == n - 1) & (t.detach() == 0)
    t = torch.where(low, torch.zeros_like(t), t)
    t = torch.where(high & ~exact_end, torch.ones_like(t), t)
    t = torch.where(exact_end, t + 1, t)
    return i.clamp(0, n - 2), t


def _sample(f, u):
    """Trilinear values of f [C, D, H, W] at the grid displaced by u, border values outside."""
    C, D, H, W = f.shape
    (iz, tz), (iy, ty), (ix, tx) = _axis(u[0], D, 0), _axis(u[1], H, 1), _axis(u[2], W, 2)
    base = ((iz * H + iy) * W + ix).reshape(-1)
    flat = f.reshape(C, -1)
    at = lambda o: flat[:, base + o].reshape((C,) + u.shape[1:])  # noqa: E731
    mix = lambda a, b, t: a + t * (b - a)  # noqa: E731
    rows = [mix(at(o), at(o + 1), tx) for o in (0, W, H * W, H * W + W)]
    return mix(mix(rows[0], rows[1], ty), mix(rows[2], rows[3], ty), tz)


def _exp64(v, K, sign=1):
    u = sign * v / 2.0 ** K
    for _ in range(K):
        u = u + _sample(u, u)
    return u


def _box(x, w):
    return torch.nn.functional.avg_pool3d(x[None, None], w, stride=1)[0, 0]


def _sim64(F, I, U, w, metric):
    M = _sample(I[None], U)[0]
    F = F - F.mean()
    M = M - M.mean().detach()
    mF, mM = _box(F, w), _box(M, w)
    vF = (_box(F * F, w) - mF * mF).clamp_min(0)
    vM = (_box(M * M, w) - mM * mM).clamp_min(0)
    cv = _box(F * M, w) - mF * mM
    if metric == "lncc":
        return (1 - cv / (vF * vM).clamp_min(1e-10).sqrt()).mean()
    return (vM - cv * cv / vF.clamp_min(1e-6)).mean()


def _reg64(f):
    return sum(torch.diff(f, dim=1 + d).square().mean(dim=(1, 2, 3)).sum() for d in range(3))


def _smooth64(x, sigma):
    w = [2 * math.pi * torch.fft.fftfreq(n, device=x.device, dtype=torch.float64)
         for n in x.shape[-3:-1]]
    wx = 2 * math.pi * torch.fft.rfftfreq(x.shape[-1], device=x.device, dtype=torch.float64)
    tf = torch.exp(-0.5 * sigma ** 2 * (w[0][:, None, None] ** 2 + w[1][None, :, None] ** 2
                                        + wx[None, None, :] ** 2))
    return torch.fft.irfftn(torch.fft.rfftn(x, dim=(-3, -2, -1)) * tf, s=x.shape[-3:],
                            dim=(-3, -2, -1))


def _up64(v):
    """2 v((x - 0.5) / 2) on the grid twice as fine, border values outside."""
    for d in (1, 2, 3):
        n = v.shape[d]
        q = ((torch.arange(2 * n, device=v.device, dtype=torch.float64) - 0.5) / 2).clamp(0, n - 1)
        i = q.floor().long().clamp(0, n - 2)
        shape = [1, 1, 1, 1]
        shape[d] = -1
        t = (q - i).view(shape)
        a, b = v.index_select(d, i), v.index_select(d, i + 1)
        v = a + t * (b - a)
    return 2 * v


def _loss64(phis, images, K, w, metric, alpha, sigma, factor):
    N = images.shape[0]
    flows = [_smooth64(p, sigma) if sigma else p for p in phis]
    fw, bw = [_exp64(v, K) for v in flows], [_exp64(v, K, -1) for v in flows]
    loss = 0.0
    for i in range(N):
        for js, step in ((range(i + 1, N), lambda j: fw[j - 1]), (range(i - 1, -1, -1),
                                                                  lambda j: bw[j])):
            U = None
            for j in js:
                U = step(j) if U is None else U + _sample(step(j), U)
                loss = loss + _sim64(images[i], images[j], _up64(U) if factor == 2 else U, w, metric)
    return loss + alpha * sum(_reg64(f) for f in flows) / (N - 1)


def _register64(images, its, K, w, metric, alpha, sigma, pairs):
    """Adam with warm-up and cosine decay on each pyramid level, coarse to fine."""
    levels = [images]
    for _ in its[1:]:
        levels.insert(0, torch.nn.functional.avg_pool3d(levels[0][None], 2)[0])
    phi, losses = None, []
    for lv, (im, T) in enumerate(zip(levels, its)):
        N = im.shape[0]
        phi = torch.zeros((N - 1, 3) + im.shape[1:], dtype=torch.float64, device="cuda") \
            if phi is None else torch.stack([_up64(p) for p in phi])
        m, v = torch.zeros_like(phi), torch.zeros_like(phi)
        warm = max(1, math.ceil(float(np.float32(0.2)) * T))
        sg = sigma / 2 ** (len(its) - 1 - lv)
        for t in range(1, T + 1):
            x = phi.clone().requires_grad_(True)
            L = _loss64(list(x), im, K, w, metric, alpha, sg, 1)
            L.backward()
            losses.append(float(L.detach()))
            lr = 0.1 * t / warm if t <= warm else \
                0.1 * 0.5 * (1 + math.cos(math.pi * (t - warm) / (T - warm)))
            m = m + 0.1 * (x.grad - m)
            v = 0.999 * v + 0.001 * x.grad.square()
            phi = phi - lr / (1 - 0.9 ** t) * m / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
            del L, x
    flows = [_smooth64(p, sigma) if sigma else p for p in phi]
    out = dict(svf=torch.stack(flows), first=losses[0], last=losses[-1])
    if pairs:
        N = images.shape[0]
        fw, bw = [_exp64(f, K) for f in flows], [_exp64(f, K, -1) for f in flows]
        got = {}
        for i in range(N):
            for js, step in ((range(i + 1, N), lambda j: fw[j - 1]), (range(i - 1, -1, -1),
                                                                      lambda j: bw[j])):
                U = None
                for j in js:
                    U = step(j) if U is None else U + _sample(step(j), U)
                    got[i, j] = U
        out["pairs"] = torch.stack([got[i, j] for i in range(N) for j in range(N) if i != j])
    return out


def exact(c, seed):
    x = _inputs(c, seed)
    x = {k: v.double() for k, v in x.items()} if "series" not in x else x
    op = c["op"]
    if op == "exp":
        return _exp64(x["svf"], c["K"], c["sign"])
    if op == "exp_bwd":
        svf = x["svf"].requires_grad_(True)
        _exp64(svf, c["K"], c["sign"]).backward(x["G"])
        return svf.grad
    if op == "compose":
        U, C = x["U"].requires_grad_(True), x["C"].requires_grad_(True)
        out = U + _sample(C, U)
        out.backward(x["G"])
        return dict(out=out.detach(), G_prev=U.grad, G_C=C.grad)
    if op == "sim":
        U = x["U"].requires_grad_(True)
        val = _sim64(x["F"], x["I"], U, c["window"], c["metric"])
        val.backward()
        return dict(sim=float(val.detach()), grad=U.grad)
    if op == "tools":
        v = x["v"].clone().requires_grad_(True)
        reg = _reg64(v)
        reg.backward()
        z = torch.zeros_like(x["v"]).requires_grad_(True)
        (_up64(z) * x["fine"]).sum().backward()
        J = []
        for k in range(3):
            J.append([torch.gradient(x["v"][k], dim=d, edge_order=1)[0] + (1.0 if d == k else 0.0)
                      for d in range(3)])
        jac = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) \
            - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) \
            + J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0])
        return dict(pool=torch.nn.functional.avg_pool3d(x["img"][None], 2)[0],
                    smooth=_smooth64(x["v"], c["sigma"]), up=_up64(x["v"]), down=z.grad,
                    reg=float(reg.detach()), reg_grad=v.grad, jac=jac)
    if op == "loss":
        svf = x["svf"].requires_grad_(True)
        L = _loss64(list(svf), x["images"], c["K"], c["window"], c["metric"], c["alpha"],
                    c["sigma"], c["factor"])
        L.backward()
        return dict(loss=float(L.detach()), grad=svf.grad)
    # whole registrations: only where the loop in 64 bits ends in a few seconds
    its = _iters(c)
    cost = sum(its) * sum(n * n * d[0] * d[1] * d[2] for n, d in _subjects(c))
    if cost > 2.5e8:
        return None
    return [_register64(s.double(), its, c["K"], c["window"], c["metric"], c["alpha"], c["sigma"],
                        c["pairs"]) for s in x["series"]]
