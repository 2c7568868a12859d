"""The candidate search at the edges of its work items, blocks and candidate
groups, and with candidates that cannot be told apart, against the oracle,
through the C-ABI."""
import math

import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea, synth

from gpu_helpers import check_search, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def _cand32(k):
    return synth.sphere_candidates(k).astype(np.float32).astype(np.float64)


def _scene(counts, seed):
    """A scene whose pair k holds counts[k] matches."""
    sc = synth.sphere_scene(n_cams=8, n_pts=3000, p_det=1.0, sigma=0.5, outlier_frac=0.1, seed=seed, name="edges")
    key = np.minimum(sc.cam1, sc.cam2) * 8 + np.maximum(sc.cam1, sc.cam2)
    rng = np.random.default_rng(seed)
    keep = []
    for code, n in zip(np.unique(key), counts):
        keep.append(rng.permutation(np.flatnonzero(key == code))[:1] if n == 1 else
                    rng.choice(np.flatnonzero(key == code), n, replace=True))
    keep = rng.permutation(np.concatenate(keep))
    for name in ("x1", "y1", "x2", "y2", "cam1", "cam2", "inlier"):
        setattr(sc, name, np.ascontiguousarray(getattr(sc, name)[keep]))
    return sc


def _context(sc):
    ctx = fastea.Context(0, fastea.default_options())
    ctx.load_intrinsics(sc.f_init, sc.cx, sc.cy)
    ctx.load_matches(sc.x1, sc.y1, sc.x2, sc.y2, sc.cam1, sc.cam2)
    return ctx


# blocks of 16 and 32 matches, segments of 512, runs of 2,048, two and three items
COUNTS = (1, 15, 16, 17, 31, 32, 33, 511, 512, 513, 2047, 2048, 2049, 2560, 4095, 4096, 4097, 6145)


@pytest.mark.parametrize("tau_px", [math.inf, 8.0])
@pytest.mark.parametrize("K", [1, 31, 128, 129, 512, 513, 1025])
def test_search_at_the_edges(K, tau_px):
    sc = _scene(COUNTS, seed=5)
    with _context(sc) as ctx:
        got = ctx.relative_translations(sc.R_init, _cand32(K), f=sc.f_gt, tau_px=tau_px, scores=True)
        quiet = ctx.relative_translations(sc.R_init, _cand32(K), f=sc.f_gt, tau_px=tau_px)
    ref = oracle.rel_trans(oracle_problem(sc), sc.R_init, sc.f_gt, _cand32(K), scores=True,
                           tau=tau_px / np.median(sc.f_gt))
    check_search(got, ref, K)
    P = len(got["best"])
    # the chosen candidate's score is the one returned beside the others
    np.testing.assert_array_equal(got["scores"][np.arange(P), got["best"]], got["score_best"].astype(np.float32))
    for k in ("best", "vote", "t_rel", "score_best"):
        np.testing.assert_array_equal(got[k], quiet[k])


def test_equal_candidates_take_the_lower_index():
    """Every direction twice and more: each copy scores the same bits, so the
    lowest index of the best direction is chosen, over several batches of
    candidates scored again and several chunks of candidates."""
    sc = _scene(COUNTS, seed=6)
    base = _cand32(40)
    with _context(sc) as ctx:
        one = ctx.relative_translations(sc.R_init, base, f=sc.f_gt, tau_px=8.0)
        many = ctx.relative_translations(sc.R_init, np.tile(base, (60, 1)), f=sc.f_gt, tau_px=8.0)
    for k in ("best", "vote", "t_rel", "score_best"):
        np.testing.assert_array_equal(one[k], many[k])


def test_matches_without_parallax_score_zero_everywhere():
    """Identical rays (n = 0): every candidate scores zero up to rounding, none
    can be ruled out, and all are scored again."""
    n = 700
    rng = np.random.default_rng(0)
    x, y = (rng.uniform(0, 640, n).astype(np.float32) for _ in range(2))
    f = np.full(2, 500.0)
    with fastea.Context(0) as ctx:
        ctx.load_intrinsics(f, f * 0 + 320, f * 0 + 240)
        ctx.load_matches(x, y, x, y, np.zeros(n, np.int32), np.ones(n, np.int32))
        got = ctx.relative_translations(np.tile(np.eye(3), (2, 1, 1)), _cand32(1500), scores=True)
    # fp32 rounding of the cross product of equal rays: a few 2^-24 of |x~|^2 < 1.5
    assert got["scores"].max() < 1e-6
    assert np.float32(got["score_best"][0]) == got["scores"].min()
