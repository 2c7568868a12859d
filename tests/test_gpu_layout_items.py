"""Work items and compaction at the edges of an item (1,024 matches) and of a
wavefront's 64 items, a pair that loses every match among them: the retained
set bit for bit, and the loss and gradient of the compacted layout, against
the oracle, over two rounds (the second compacts a compacted layout)."""
import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea

from gpu_helpers import per_camera_close, tau_in_gap

pytestmark = pytest.mark.gpu

TILE = 1024


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def _problem(lengths, drop, seed):
    """Matches of the pairs (0,1), (0,2), ... with the given run lengths, in
    shuffled order; the pairs in `drop` far from their epipolar lines."""
    rng = np.random.default_rng(seed)
    n = len(lengths) + 1
    R = np.tile(np.eye(3), (n, 1, 1))
    t = rng.normal(size=(n, 3))
    f = np.full(n, 500.0)
    cam1 = np.zeros(sum(lengths), np.int32)
    cam2 = np.repeat(np.arange(1, n, dtype=np.int32), lengths)
    X = rng.uniform(-1, 1, (len(cam1), 3)) + [0, 0, 6]
    def see(c):
        Y = np.einsum("mij,mj->mi", R[c], X) + t[c]
        return 500.0 * Y[:, :2] / Y[:, 2:]
    p1, p2 = see(cam1), see(cam2)
    p2 += rng.normal(size=p2.shape) * np.where(np.isin(cam2, drop), 4e4, 1.0)[:, None]
    o = rng.permutation(len(cam1))
    m = [a[o] for a in (*p1.T.astype(np.float32), *p2.T.astype(np.float32), cam1, cam2)]
    return n, R, t, f, m


@pytest.mark.parametrize("lengths,drop", [
    ([70 * TILE + 5, TILE + 1, 1, TILE, 37, TILE - 1], [5]),
    ([64 * TILE, 64 * TILE + 1, 3], []),
    ([33], []),
])
def test_compaction_matches_oracle(lengths, drop):
    n, R, t, f, m = _problem(lengths, drop, seed=len(lengths))
    pb = oracle.OracleProblem(*m, np.zeros(n), np.zeros(n))
    eps = np.abs(oracle.residuals(pb, R, t, f))
    with fastea.Context(0, fastea.default_options(gauge_normalize=0, tile_matches=TILE)) as ctx:
        ctx.load_intrinsics(f, f * 0, f * 0)
        ctx.load_matches(*m)
        ctx.init_poses(R, t)
        mask = np.ones(len(eps), np.uint8)
        kept = ~np.isin(m[5], drop)
        for q in (0.9, 0.5):
            tau = tau_in_gap(eps, np.quantile(eps[kept], q))
            ctx.begin_round(tau * 500.0)
            mask &= (eps < tau).astype(np.uint8)
            got, z = ctx.get_mask()
            assert z == mask.sum() and 0 < z < len(eps)
            np.testing.assert_array_equal(got.astype(np.uint8), mask)
            assert not got[np.isin(m[5], drop)].any()
            l, gR, gt, gf = (x.cpu().numpy() for x in ctx.residual_grad())
            lr, gRr, gtr, gfr = oracle.loss_grad(pb, R, t, f, R, t, f, mask)
            assert abs(l[0] - lr) <= 1e-5 * lr
            for a, b in ((gR, gRr), (gt, gtr), (gf[:, None], gfr[:, None])):
                ok, worst = per_camera_close(a, b)
                assert ok, worst


@pytest.mark.parametrize("lengths,drop", [
    ([1, 3, 4, 63, 64, 65, 127, 129], [3]),
    ([191, 192, 193, 255, 256, 257, 384], []),
    ([8192 + 1, 8191, 8192 + 191], []),
    ([2], []),
])
def test_quadratic_form_matches_oracle(lengths, drop):
    """The same with the quadratic form, whose pass keeps the layout and marks
    the retained matches, at run lengths around its trips of 64 matches, the
    three in flight and an item of 8,192."""
    n, R, t, f, m = _problem(lengths, drop, seed=10 + len(lengths))
    pb = oracle.OracleProblem(*m, np.zeros(n), np.zeros(n))
    eps = np.abs(oracle.residuals(pb, R, t, f))
    with fastea.Context(0, fastea.default_options(gauge_normalize=0, inner_loop=1)) as ctx:
        ctx.load_intrinsics(f, f * 0, f * 0)
        ctx.load_matches(*m)
        ctx.init_poses(R, t)
        mask = np.ones(len(eps), np.uint8)
        kept = ~np.isin(m[5], drop)
        for q in (1.0, 0.7):
            tau = tau_in_gap(eps, np.quantile(eps[kept], q)) if q < 1.0 else float(np.inf)
            ctx.begin_round(tau * 500.0)
            mask &= (eps < tau).astype(np.uint8)
            got, z = ctx.get_mask()
            assert z == mask.sum()
            np.testing.assert_array_equal(got.astype(np.uint8), mask)
            if mask.sum() == 0:
                break
            l, gR, gt, gf = (x.cpu().numpy() for x in ctx.residual_grad())
            lr, gRr, gtr, gfr = oracle.loss_grad(pb, R, t, f, R, t, f, mask)
            assert abs(l[0] - lr) <= 1e-5 * lr
            for a, b in ((gR, gRr), (gt, gtr), (gf[:, None], gfr[:, None])):
                ok, worst = per_camera_close(a, b)
                assert ok, worst
