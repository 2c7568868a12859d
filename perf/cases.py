"""Timed cases of the library's public entry points, over the sizes it is used at.

Each case is one call (or the short sequence of calls) that a program built
on the binding makes: a gradient evaluation, a differentiable loss, an
adjustment round, loading a problem, a whole solve, a batch of solves, and
the four stages before the adjustment.  The scenes are those of the synth
module (cameras on a noisy loop paired with their nearest neighbours, an
object-centric capture) with the matches drawn on the GPU, in random order
and orientation, with pixel noise and outliers.

Work-item sizes are fixed where the per-match kernel runs: the autotuner's
pick, and with it the rounding of the fp32 sums, may differ between
processes.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2605_18052_amd import autograd, fastea, learned, synth

DEV = "cuda:0"
WIDTH, HEIGHT = 640.0, 480.0
CHUNK = 4_000_000  # matches handled at once while inputs and references are made
TILE = 2048


def listed():
    return [
        # one objective and gradient at given poses on the 20-camera scene
        # (61k matches), as an outside optimiser calls it: latency
        dict(name="grad_sphere20_m61k", kind="grad", cams=20, nbrs=0, matches=60_857, outliers=0.1),
        # forward and backward of the differentiable loss on a training-size
        # scene, every camera sharing one focal length
        dict(name="autograd_traj500_m8M", kind="autograd", cams=500, nbrs=20, matches=8_000_011, outliers=0.2,
             shared=True),
        # one IRLS round (filter, compaction, 50 Adam steps over the matches)
        # on the largest scene
        dict(name="round_traj3000_m100M", kind="round", cams=3000, nbrs=30, matches=99_950_185, outliers=0.25),
        # a newly matched scene: loading (validate, canonicalise, sort by
        # pair), poses, first round and first gradient
        dict(name="load_traj1000_m30M", kind="load", cams=1000, nbrs=20, matches=30_050_151, outliers=0.3),
        # a whole adjustment from initial poses to final poses, quadratic form
        dict(name="solve_quad_traj1000_m30M", kind="solve", cams=1000, nbrs=20, matches=30_050_151, outliers=0.3),
        # a learned-weight round's start (network over every match, weighted
        # forms) and its gradient
        dict(name="learned_traj500_m20M", kind="learned", cams=500, nbrs=20, matches=19_987_074, outliers=0.2),
        # many small scenes solved together in one context, quadratic form
        dict(name="batch24_quad_m6M", kind="batch", scenes=24, cams=60, nbrs=20, matches=6_000_000, outliers=0.2),
        # relative-translation search, 2,048 directions, 8 px cap
        dict(name="search_traj1000_m30M", kind="search", cams=1000, nbrs=20, matches=30_050_151, outliers=0.3,
             cands=2048, cap=8.0),
        # camera centres of an object capture from two random starts
        dict(name="align_object500", kind="align", cams=500, angle=60.0, runs=2),
        # global rotations: initialisation and 1,000 Adam steps
        dict(name="rotation_traj1000", kind="rotation", cams=1000, nbrs=20),
        # focal-length vote, one intrinsics group per camera
        dict(name="focal_per_camera1000", kind="focal", cams=1000, nbrs=20, shared=False, cands=1024),
        # focal-length vote, one camera model for every image (the default)
        dict(name="focal_shared500", kind="focal", cams=500, nbrs=20, shared=True, cands=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grad", "autograd", "round", "load", "solve", "learned", "batch", "search", "align",
                       "rotation", "focal"])
    if kind == "grad":
        return dict(kind=kind, cams=_log(rng, 8, 200), nbrs=0, matches=_log(rng, 2e4, 1e6),
                    outliers=rng.choice([0.1, 0.2]))
    if kind == "align":
        return dict(kind=kind, cams=_log(rng, 60, 500), angle=rng.choice([60.0, 75.0]), runs=rng.randint(1, 4))
    if kind == "rotation":
        return dict(kind=kind, cams=_log(rng, 60, 2000), nbrs=rng.randint(8, 30))
    if kind == "focal":
        return dict(kind=kind, cams=_log(rng, 60, 1000), nbrs=rng.randint(8, 30), shared=rng.random() < 0.5,
                    cands=rng.randint(200, 1024))
    c = dict(kind=kind, cams=_log(rng, 60, 1500), nbrs=rng.randint(8, 30), matches=0,
             outliers=rng.choice([0.1, 0.2, 0.3]))
    if kind == "batch":
        c.update(scenes=rng.randint(4, 24), cams=_log(rng, 20, 120), matches=_log(rng, 2e5, 6e6))
        return c
    hi = {"autograd": 2e7, "round": 4e7, "load": 4e7, "solve": 2e7, "learned": 2e7, "search": 2e7}[kind]
    c["matches"] = _log(rng, hi / 100, hi)
    if kind == "autograd":
        c["shared"] = rng.random() < 0.5
    if kind == "search":
        c.update(cands=rng.randint(300, 2048), cap=rng.choice([8.0, 4.0, math.inf]))
    return c


# ---- inputs -----------------------------------------------------------------

def _pairs(centres, nbrs):
    """Pairs (i < j), lexicographic: each camera with its nbrs nearest (0: all)."""
    n = len(centres)
    if nbrs == 0 or nbrs >= n - 1:
        i, j = np.triu_indices(n, 1)
        return np.stack([i, j], 1).astype(np.int64)
    key = []
    for s in range(0, n, 512):
        d = np.linalg.norm(centres[s:s + 512, None, :] - centres[None, :, :], axis=2)
        d[np.arange(len(d)), np.arange(s, s + len(d))] = np.inf
        nn = np.argpartition(d, nbrs - 1, axis=1)[:, :nbrs]
        r = np.repeat(np.arange(s, s + len(d)), nbrs)
        key.append(np.minimum(r, nn.ravel()) * n + np.maximum(r, nn.ravel()))
    key = np.unique(np.concatenate(key))
    return np.stack([key // n, key % n], 1).astype(np.int64)


def _cameras(case, seed):
    """True cameras, pairs and starting values: the noisy loop, or (nbrs 0)
    the sphere looking at its centre, every pair matched."""
    rng = np.random.default_rng(seed)
    n = case["cams"]
    loop = case["nbrs"] > 0
    if loop:
        # the centres, and with them the pair graph and the outputs' sizes,
        # are the case's; all else is the seed's
        th = 2.0 * np.pi * np.arange(n) / n
        centres = np.stack([6.0 * np.cos(th), 6.0 * np.sin(th), np.sin(3.0 * th)], 1)
        centres = centres + np.random.default_rng(n).normal(0.0, 0.1, size=centres.shape)
        turn = synth.rotation_from_axis_angle(rng.normal(size=(n, 3)), np.deg2rad(rng.normal(0.0, 5.0, size=n)))
        R = turn @ synth.look_at(centres, np.zeros(3))
        f = rng.uniform(400.0, 1200.0, size=n)
        if case.get("shared"):
            f[:] = rng.uniform(500.0, 900.0)
        spread = 0.1
    else:
        centres = rng.normal(size=(n, 3))
        centres *= 4.0 / np.linalg.norm(centres, axis=1, keepdims=True)
        R = synth.look_at(centres, np.zeros(3))
        f = np.full(n, 500.0)
        spread = 0.0
    t = -np.einsum("nij,nj->ni", R, centres)
    pairs = _pairs(centres, case["nbrs"])
    f0 = f * np.exp(rng.uniform(-spread, spread, size=1 if case.get("shared") else n))
    ang = np.deg2rad(np.abs(rng.normal(0.0, 3.0, size=n)) + 2.0)
    R0 = synth.rotation_from_axis_angle(rng.normal(size=(n, 3)), ang) @ R
    base = np.median(np.linalg.norm(centres[pairs[:, 0]] - centres[pairs[:, 1]], axis=1))
    t0 = -np.einsum("nij,nj->ni", R0, centres + rng.normal(0.0, 0.05 * base, size=centres.shape))
    return SimpleNamespace(n=n, loop=loop, centres=centres, R=R, t=t, f=f, pairs=pairs, f0=f0, R0=R0, t0=t0,
                           cx=np.full(n, WIDTH / 2), cy=np.full(n, HEIGHT / 2), rng=rng)


def _matches(cam, case, seed):
    """x1, y1, x2, y2 (fp32), cam1, cam2 (int32) on the GPU: random pairs (of
    uneven size), points both cameras see where a few draws find one, pixel
    noise, outliers, random orientation."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    M = case["matches"]
    w = np.exp(cam.rng.normal(0.0, 0.3, size=len(cam.pairs)))
    edges = torch.tensor(np.cumsum(w) / w.sum(), dtype=torch.float32, device=DEV)
    pairs = torch.tensor(cam.pairs, device=DEV)
    R = torch.tensor(cam.R, dtype=torch.float32, device=DEV)
    t = torch.tensor(cam.t, dtype=torch.float32, device=DEV)
    f = torch.tensor(cam.f, dtype=torch.float32, device=DEV)
    size = torch.tensor([4.0, 4.0, 2.0] if cam.loop else [1.0, 1.0, 1.0], device=DEV)
    sigma = 1.0 if cam.loop else 0.5
    lim = torch.tensor([WIDTH, HEIGHT], device=DEV)
    out = [torch.empty(M, dtype=torch.float32, device=DEV) for _ in range(4)]
    ids = [torch.empty(M, dtype=torch.int32, device=DEV) for _ in range(2)]

    def rand(*s):
        return torch.rand(*s, generator=g, device=DEV)

    def project(c, X):
        Y = torch.bmm(R[c], X[:, :, None])[:, :, 0] + t[c]
        p = f[c, None] * Y[:, :2] / Y[:, 2:].clamp(min=1e-2) + lim / 2
        return p, (Y[:, 2] > 1e-2) & ((p >= 0) & (p < lim)).all(1)

    for lo in range(0, M, CHUNK):
        n = min(CHUNK, M - lo)
        q = pairs[torch.searchsorted(edges, rand(n)).clamp(max=len(pairs) - 1)]
        a, b = q[:, 0], q[:, 1]
        X = (rand(n, 3) - 0.5) * size
        for _ in range(2):
            ok = project(a, X)[1] & project(b, X)[1]
            X = torch.where(ok[:, None], X, (rand(n, 3) - 0.5) * size * 0.7)
        p, q = project(a, X)[0], project(b, X)[0]
        p = p + sigma * torch.randn(n, 2, generator=g, device=DEV)
        q = q + sigma * torch.randn(n, 2, generator=g, device=DEV)
        q = torch.where(rand(n, 1) < case["outliers"], rand(n, 2) * lim, q)
        flip = rand(n) < 0.5
        s = slice(lo, lo + n)
        for k in range(2):
            out[k][s] = torch.where(flip, q[:, k], p[:, k])
            out[2 + k][s] = torch.where(flip, p[:, k], q[:, k])
        ids[0][s] = torch.where(flip, b, a).int()
        ids[1][s] = torch.where(flip, a, b).int()
    return out + ids


def _context(cam, case, m=None, **opt):
    ctx = fastea.Context(0, fastea.default_options(**opt))
    ctx.load_intrinsics(cam.f0, cam.cx, cam.cy, np.zeros(cam.n, np.int32) if case.get("shared") else None)
    if m is not None:
        ctx.load_matches(*m)
    return ctx


def _moved(cam, seed):
    """Poses half a degree and a little translation away from the start."""
    rng = np.random.default_rng(seed + 77)
    R = synth.rotation_from_axis_angle(rng.normal(size=(cam.n, 3)), np.full(cam.n, np.deg2rad(0.5))) @ cam.R0
    return R, cam.t0 + rng.normal(0.0, 0.005, size=cam.t0.shape)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "align":
        pc, R, t, _ = synth.object_pair_graph(case["cams"], case["angle"], seed)
        rng = np.random.default_rng(seed)
        t = np.einsum("pij,pj->pi", synth.rotation_from_axis_angle(
            rng.normal(size=t.shape), np.deg2rad(rng.normal(0.0, 2.0, size=len(t)))), t)
        return dict(kind=kind, ctx=fastea.Context(0), pairs=pc, R=R, t=t,
                    o=synth.random_centres(seed, case["runs"], case["cams"]))
    if kind == "batch":
        return _prepare_batch(case, seed)
    cam = _cameras(case, seed)
    if kind == "rotation":
        i, j = cam.pairs[:, 0], cam.pairs[:, 1]
        noise = synth.rotation_from_axis_angle(cam.rng.normal(size=(len(i), 3)),
                                               np.deg2rad(np.abs(cam.rng.normal(0.0, 2.0, size=len(i)))))
        return dict(kind=kind, ctx=fastea.Context(0), n=cam.n, pairs=cam.pairs.astype(np.int32),
                    R=noise @ cam.R[j] @ cam.R[i].transpose(0, 2, 1), v0=cam.rng.normal(size=(2, cam.n, 3)))
    if kind == "focal":
        sc = SimpleNamespace(R_gt=cam.R, t_gt=cam.t, f_gt=cam.f)
        return dict(kind=kind, ctx=fastea.Context(0), n=cam.n, pairs=cam.pairs.astype(np.int32),
                    F=synth.fundamental_matrices(sc, cam.pairs, noise=0.01, seed=seed),
                    cand=synth.focal_candidates(case["cands"], 200.0, 3000.0),
                    group=None if case["shared"] else np.arange(cam.n, dtype=np.int32),
                    f_cur=None if case["shared"] else cam.f0, votes=case["shared"])
    m = _matches(cam, case, seed)
    if kind == "grad":
        ctx = _context(cam, case, m, tile_matches=TILE)
        ctx.init_poses(cam.R0, cam.t0)
        ctx.begin_round(128.0)
        return dict(kind=kind, ctx=ctx, poses=_moved(cam, seed))
    if kind == "autograd":
        ctx = _context(cam, case, m, tile_matches=TILE)
        ctx.init_poses(cam.R0, cam.t0)
        ctx.begin_round(128.0)
        ctx.set_poses(*_moved(cam, seed))
        return dict(kind=kind, ctx=ctx, params=[p.requires_grad_() for p in ctx.get_params()])
    if kind == "round":
        return dict(kind=kind, ctx=_context(cam, case, m, tile_matches=TILE), start=(cam.R0, cam.t0))
    if kind == "load":
        return dict(kind=kind, ctx=_context(cam, case, tile_matches=TILE), matches=m, start=(cam.R0, cam.t0))
    if kind == "solve":
        return dict(kind=kind, ctx=_context(cam, case, m, inner_loop=1), start=(cam.R0, cam.t0))
    if kind == "learned":
        ctx = _context(cam, case, m, inner_loop=1, weight_mode=1)
        ctx.set_mlp(learned.load_weights())
        return dict(kind=kind, ctx=ctx, start=(cam.R0, cam.t0))
    if kind == "search":
        cand = synth.sphere_candidates(case["cands"]).astype(np.float32).astype(np.float64)
        return dict(kind=kind, ctx=_context(cam, case, m), R=cam.R, f=cam.f, cand=cand, cap=case["cap"])
    raise ValueError(kind)


def _prepare_batch(case, seed):
    """Scenes of uneven size (camera counts and match counts spread around
    the case's means; the case's, not the seed's) in one context."""
    rng = np.random.default_rng(case["scenes"])
    S = case["scenes"]
    w = np.exp(rng.normal(0.0, 0.8, size=S))
    w /= w.sum()
    cams, parts, first = [], [], 0
    for s in range(S):
        n = max(8, int(case["cams"] * math.exp(rng.normal(0.0, 0.4))))
        c = dict(case, cams=n, nbrs=min(case["nbrs"], n - 2), matches=max(5000, int(w[s] * case["matches"])))
        cam = _cameras(c, seed * 100 + s)
        m = _matches(cam, c, seed * 100 + s)
        m[4] += first
        m[5] += first
        first += n
        cams.append(cam)
        parts.append(m)
    ctx = fastea.Context(0, fastea.default_options(inner_loop=1))
    ctx.load_intrinsics(*(np.concatenate([getattr(c, k) for c in cams]) for k in ("f0", "cx", "cy")))
    ctx.set_scenes(np.repeat(np.arange(S, dtype=np.int32), [c.n for c in cams]))
    ctx.load_matches(*(torch.cat(p) for p in zip(*parts)))
    return dict(kind="solve", ctx=ctx,
                start=(np.concatenate([c.R0 for c in cams]), np.concatenate([c.t0 for c in cams])))


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "grad":
        ctx.set_poses(*s["poses"])
        return ctx.residual_grad()
    if kind == "autograd":
        for p in s["params"]:
            p.grad = None
        loss = autograd.epipolar_loss(*s["params"], ctx)
        loss.backward()
        return [loss.detach()] + [p.grad for p in s["params"]]
    if kind == "round":
        ctx.init_poses(*s["start"])
        ctx.begin_round(128.0)
        ctx.step(50)
        return ctx.get_params()
    if kind == "load":
        ctx.load_matches(*s["matches"])
        ctx.init_poses(*s["start"])
        ctx.begin_round(128.0)
        return ctx.residual_grad()
    if kind == "solve":
        ctx.init_poses(*s["start"])
        rep = ctx.epipolar_adjust()
        return list(ctx.get_poses()) + [rep["loss"], rep["inliers"]]
    if kind == "learned":
        ctx.init_poses(*s["start"])
        ctx.begin_round(128.0)
        return ctx.residual_grad()
    if kind == "search":
        r = ctx.relative_translations(s["R"], s["cand"], f=s["f"], tau_px=s["cap"])
        return [r["t_rel"], r["best"], r["vote"], r["score_best"]]
    if kind == "align":
        r = ctx.translation_align(s["pairs"], s["R"], s["t"], s["o"])
        return [r["o"], r["run_of_cam"], r["run_loss"], r["final_loss"]]
    if kind == "rotation":
        r = ctx.rotation_averaging(s["n"], s["pairs"], s["R"], v0=s["v0"])
        return [r["R"], float(r["loss_init"]), float(r["loss"])]
    if kind == "focal":
        r = ctx.focal_vote(s["n"], s["pairs"], s["F"], s["cand"], 0.05, group=s["group"], f_cur=s["f_cur"],
                           votes=s["votes"])
        return [r["f_best"], r["k_best"]] + ([r["votes"]] if s["votes"] else [])
    raise ValueError(kind)


def work(case):
    """Bytes: match coordinates (16 B) once per pass that has to read them
    (24 B as loaded, with the camera ids), the sorted layout once where one
    is written, per-pair data per step.  Flops: the per-match residuals and
    gradient sums (~70 a pass), the network (9.3 k), the forms (~100), the
    candidate products (8), the per-pair work of a step (~800), one 3x3
    problem (~150)."""
    kind, n = case["kind"], case["cams"]
    nbrs = case.get("nbrs", 0)
    M = case.get("matches", 0)
    P = (n * min(n - 1, 1.05 * nbrs) / 2 * 1.2) if nbrs else n * (n - 1) / 2
    if kind in ("grad", "autograd", "learned"):
        passes = 2 if kind == "autograd" else 1
        extra = 9300 + 100 if kind == "learned" else 0
        return dict(bytes=16.0 * M * passes + 200.0 * n, flops=(70.0 * passes + extra) * M)
    if kind == "round":
        return dict(bytes=16.0 * M * 52, flops=70.0 * M * 51)
    if kind == "load":
        return dict(bytes=(24.0 + 16 + 16 + 16) * M, flops=110.0 * M)
    if kind in ("solve", "batch"):
        P *= case.get("scenes", 1)
        return dict(bytes=16.0 * M * 20 + 1000 * P * 360.0, flops=100.0 * M * 20 + 1000 * P * 800.0)
    if kind == "search":
        return dict(bytes=16.0 * M, flops=8.0 * M * case["cands"])
    if kind == "align":
        P = n * (n - 1) / 2 * (1 - math.cos(math.radians(case["angle"]))) / 2
        return dict(bytes=2000.0 * 24 * P, flops=(1500.0 * case["runs"] + 500) * P * 40)
    if kind == "rotation":
        return dict(bytes=1400.0 * 72 * P, flops=1000 * P * 250.0 + 400 * P * 60.0)
    if kind == "focal":
        return dict(bytes=72.0 * P, flops=150.0 * P * case["cands"] * (1 if case["shared"] else 2))
    raise ValueError(kind)


# ---- the same in 64 bits with plain torch ------------------------------------

def _fundamental(R, t, f, pairs):
    """F = D_j [u]x R_j R_i^T D_i of every pair, centred pixel coordinates."""
    i, j = pairs[:, 0], pairs[:, 1]
    Rij = R[j] @ R[i].transpose(1, 2).contiguous()
    tij = t[j] - (Rij @ t[i][:, :, None])[:, :, 0]
    u = tij / tij.norm(dim=1, keepdim=True)
    zero = torch.zeros_like(u[:, 0])
    ux = torch.stack([zero, -u[:, 2], u[:, 1], u[:, 2], zero, -u[:, 0], -u[:, 1], u[:, 0], zero], 1).reshape(-1, 3, 3)
    one = torch.ones_like(f)
    d = torch.stack([1 / f, 1 / f, one], 1)
    return d[j][:, :, None] * (ux @ Rij) * d[i][:, None, :]


def _chunks(m, cam):
    """(pair index, p1, p2) of the matches in the pairs' orientation, fp64, a chunk at a time."""
    code = cam.pairs[:, 0] * cam.n + cam.pairs[:, 1]
    code = torch.tensor(code, device=DEV)
    for lo in range(0, len(m[0]), CHUNK):
        x1, y1, x2, y2 = (a[lo:lo + CHUNK].double() for a in m[:4])
        a, b = (a[lo:lo + CHUNK].long() for a in m[4:])
        q = torch.searchsorted(code, torch.minimum(a, b) * cam.n + torch.maximum(a, b))
        one = torch.ones_like(x1)
        p1 = torch.stack([x1 - WIDTH / 2, y1 - HEIGHT / 2, one], 1)
        p2 = torch.stack([x2 - WIDTH / 2, y2 - HEIGHT / 2, one], 1)
        s = (a > b)[:, None]
        yield q, torch.where(s, p2, p1), torch.where(s, p1, p2)


def _median(v):
    return float(np.median(v))


def _present(cam, m):
    """The pairs that some match drew."""
    a, b = (c.long() for c in m[4:])
    code = torch.unique(torch.minimum(a, b) * cam.n + torch.maximum(a, b)).cpu().numpy()
    return np.stack([code // cam.n, code % cam.n], 1)


def _gauge(cam, R, t):
    """Translations in the solver's gauge of the starting poses: centres to
    mean 0, median matched-pair baseline 1."""
    o0 = -np.einsum("nji,nj->ni", cam.R0, cam.t0)
    c = o0.mean(0)
    s = _median(np.linalg.norm(o0[cam.pairs[:, 0]] - o0[cam.pairs[:, 1]], axis=1))
    o = -np.einsum("nji,nj->ni", R, t)
    return -np.einsum("nij,nj->ni", R, (o - c) / s)


def _eps(F, q, p1, p2):
    return (p2 * torch.bmm(F[q], p1[:, :, None])[:, :, 0]).sum(1)


def _network(feat):
    w = torch.tensor(learned.load_weights(), dtype=torch.float64, device=DEV)
    W1, b1, W2, b2, w3, b3 = torch.split(w, [512, 64, 4096, 64, 64, 1])
    h = torch.relu(feat @ W1.reshape(64, 8).T.contiguous() + b1)
    h = torch.relu(h @ W2.reshape(64, 64).T.contiguous() + b2)
    return torch.sigmoid(h @ w3 + b3)


def _objective(case, cam, m, R, t):
    """The round's objective at (R, t) with the snapshot at the starting
    poses, and each pair's dL/dF."""
    d = dict(dtype=torch.float64, device=DEV)
    pairs = torch.tensor(cam.pairs, device=DEV)
    f = np.exp(np.full(cam.n, np.log(cam.f0).mean())) if case.get("shared") else cam.f0
    f = torch.tensor(f, **d)
    Rt, tt = torch.tensor(R, **d), torch.tensor(_gauge(cam, R, t), **d)
    F = _fundamental(Rt, tt, f, pairs)
    R0, t0 = torch.tensor(cam.R0, **d), torch.tensor(_gauge(cam, cam.R0, cam.t0), **d)
    Fh = _fundamental(R0, t0, f, pairs)
    fm = _median(f.cpu().numpy())
    tau = 128.0 / fm
    net = case["kind"] == "learned"
    if net:
        z = R0[:, 2]
        ang = torch.arccos((z[pairs[:, 0]] * z[pairs[:, 1]]).sum(1).clamp(-1, 1)) / (math.pi / 2)
    G = torch.zeros(len(pairs), 9, **d)
    L, Z = torch.zeros((), **d), torch.zeros((), **d)
    for q, p1, p2 in _chunks(m, cam):
        e, eh = _eps(F, q, p1, p2), _eps(Fh, q, p1, p2).abs()
        w = (eh < tau).double()
        if net:
            r = torch.log1p(eh * fm) / math.log(257.0)
            k = torch.tensor([2 / WIDTH, 2 / HEIGHT], **d)
            w = w * _network(torch.cat([r[:, None].expand(-1, 3), p1[:, :2] * k, p2[:, :2] * k, ang[q][:, None]], 1))
        c = w / eh.clamp(min=1e-4)
        Z += w.sum()
        L += (c * e * e).sum()
        G.index_add_(0, q, ((2 * c * e)[:, None, None] * p2[:, :, None] * p1[:, None, :]).reshape(-1, 9))
    return L / Z, (G / Z).reshape(-1, 3, 3), pairs, Rt, tt, f


def _exact_objective(case, seed):
    cam = _cameras(case, seed)
    m = _matches(cam, case, seed)
    cam.pairs = _present(cam, m)
    kind = case["kind"]
    R, t = _moved(cam, seed) if kind in ("grad", "autograd") else (cam.R0, cam.t0)
    L, G, pairs, R, t, f = _objective(case, cam, m, R, t)
    if kind == "autograd":
        a6 = torch.cat([R[:, :, 0], R[:, :, 1]], 1).requires_grad_()
        b1 = a6[:, :3] / a6[:, :3].norm(dim=1, keepdim=True)
        v = a6[:, 3:] - (b1 * a6[:, 3:]).sum(1, keepdim=True) * b1
        b2 = v / v.norm(dim=1, keepdim=True)
        R = torch.stack([b1, b2, torch.linalg.cross(b1, b2)], 2)
        logf = (f[:1] if case.get("shared") else f).log().requires_grad_()
        f = logf.exp().expand(cam.n)
        leaves = [a6, t.requires_grad_(), logf]
    else:
        leaves = [R.requires_grad_(), t.requires_grad_(), f.requires_grad_()]
    (G * _fundamental(R, t, f, pairs)).sum().backward()
    loss = L if kind == "autograd" else L.reshape(1)
    return [loss] + [x.grad for x in leaves]


def _exact_search(case, seed):
    """Every candidate's mean capped error, the best (its sign by the
    matches' cheirality), by blocks of pairs."""
    d = dict(dtype=torch.float64, device=DEV)
    cam = _cameras(case, seed)
    m = _matches(cam, case, seed)
    cam.pairs = _present(cam, m)
    P, K = len(cam.pairs), case["cands"]
    pairs = torch.tensor(cam.pairs, device=DEV)
    cand = torch.tensor(synth.sphere_candidates(K).astype(np.float32), device=DEV).double()
    R, f = torch.tensor(cam.R, **d), torch.tensor(cam.f, **d)
    tau = case["cap"] / _median(cam.f)
    rays = []
    for q, p1, p2 in _chunks(m, cam):
        i, j = pairs[q, 0], pairs[q, 1]
        k1 = torch.cat([p1[:, :2] / f[i, None], p1[:, 2:]], 1)
        k2 = torch.cat([p2[:, :2] / f[j, None], p2[:, 2:]], 1)
        Rij = torch.bmm(R[j], R[i].transpose(1, 2).contiguous())
        rays.append((q, torch.bmm(Rij, k1[:, :, None])[:, :, 0], k2))
    q, a, b = (torch.cat(x) for x in zip(*rays))
    order = torch.argsort(q, stable=True)
    q, a, b = q[order], a[order], b[order]
    nrm = torch.linalg.cross(a, b)
    off = torch.searchsorted(q, torch.arange(P + 1, device=DEV)).cpu().numpy()
    best, val = torch.empty(P, dtype=torch.long, device=DEV), torch.empty(P, **d)
    for p in range(P):
        e = (nrm[off[p]:off[p + 1]] @ cand.T).abs()
        if math.isfinite(tau):
            e = e.clamp(max=tau)
        val[p], best[p] = e.mean(0).min(0)
    u = cand[best][q]
    s = lambda x, y: (x * y).sum(1)  # noqa: E731
    ab, aa, bb, au, bu = s(a, b), s(a, a), s(b, b), s(a, u), s(b, u)
    l1, l2 = ab * bu - au * bb, aa * bu - ab * au
    use = ((nrm * u).sum(1).abs() < tau) & (aa * bb - ab * ab > 0)
    v = (use & (l1 > 0) & (l2 > 0)).double() - (use & (l1 < 0) & (l2 < 0)).double()
    vote = torch.zeros(P, **d).index_add_(0, q, v)
    t = torch.where((vote >= 0)[:, None], cand[best], -cand[best])
    return [t, None, None, val]


def _ratio(E):
    """s1 / s2 of 3x3 matrices (last dimension 9) by one-sided Jacobi rotations of the columns."""
    c = [[E[..., 3 * r + k] for r in range(3)] for k in range(3)]
    dot = lambda x, y: x[0] * y[0] + x[1] * y[1] + x[2] * y[2]  # noqa: E731
    for _ in range(6):
        for i, j in ((0, 1), (0, 2), (1, 2)):
            x, y = c[i], c[j]
            g = dot(x, y)
            z = (dot(y, y) - dot(x, x)) / (2 * torch.where(g == 0, torch.ones_like(g), g))
            th = torch.where(z >= 0, 1.0, -1.0) / (z.abs() + torch.sqrt(1 + z * z))
            th = torch.where(g == 0, torch.zeros_like(th), th)
            cs = 1 / torch.sqrt(1 + th * th)
            sn = cs * th
            c[i] = [cs * u - sn * v for u, v in zip(x, y)]
            c[j] = [sn * u + cs * v for u, v in zip(x, y)]
    s = torch.stack([dot(v, v).sqrt() for v in c], -1).sort(-1, descending=True)[0]
    return s[..., 0] / s[..., 1]


def _exact_focal(case, seed):
    d = dict(dtype=torch.float64, device=DEV)
    s = prepare(case, seed)
    s["ctx"].close()
    K, G = case["cands"], 1 if case["shared"] else s["n"]
    pairs = torch.tensor(s["pairs"].astype(np.int64), device=DEV)
    F, cand = torch.tensor(s["F"], **d), torch.tensor(s["cand"], **d)
    cur = None if case["shared"] else torch.tensor(s["f_cur"], **d)
    votes = torch.zeros(G, K, **d)
    one = torch.ones((), **d)
    for lo in range(0, len(pairs), 2000):
        i, j, Fp = pairs[lo:lo + 2000, 0], pairs[lo:lo + 2000, 1], F[lo:lo + 2000]
        for side in ((0,) if case["shared"] else (0, 1)):
            fi = cand.expand(len(i), K) if case["shared"] or side == 0 else cur[i][:, None].expand(len(i), K)
            fj = cand.expand(len(i), K) if case["shared"] or side == 1 else cur[j][:, None].expand(len(i), K)
            di = torch.stack([fi, fi, one.expand_as(fi)], -1)
            dj = torch.stack([fj, fj, one.expand_as(fj)], -1)
            E = (dj[..., :, None] * Fp[:, None] * di[..., None, :]).reshape(len(i), K, 9)
            v = torch.exp((1 - _ratio(E)) / 0.05)
            votes.index_add_(0, torch.zeros_like(i) if case["shared"] else (i, j)[side], v)
    best = cand[votes.argmax(1)]
    return [best, None] + ([votes] if s["votes"] else [])


def exact(case, seed):
    """None where the result is the end of a long first-order iteration
    (whose digits the objective does not fix): solves, rounds, centres,
    rotations."""
    kind = case["kind"]
    if kind in ("grad", "autograd", "load", "learned"):
        return _exact_objective(case, seed)
    if kind == "search":
        return _exact_search(case, seed)
    if kind == "focal":
        return _exact_focal(case, seed)
    return None
