"""The candidate search's two ways of scoring, products of split bf16 parts and
fp32 products: which one a call takes follows from its sizes and cap, and the
chosen direction, its score and its vote are the same bits either way.  Small
sets of matches with edges of every block, segment, run and item size are
searched beside one long pair (fp32) and amid millions of matches in pairs like
them (split), against the oracle, through the C-ABI."""
import math
import time

import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea, synth

from gpu_helpers import check_search, oracle_problem

pytestmark = pytest.mark.gpu

COUNTS = (1, 15, 16, 17, 31, 32, 33, 511, 512, 513, 2047, 2048, 2049, 2560, 4095, 4096, 4097, 6145)
FILL_CAMS, FILL = 52, 4000  # 1,326 pairs of 4,000 matches
LONG = 400_000              # matches of one more pair


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def _cand32(k):
    return synth.sphere_candidates(k).astype(np.float32).astype(np.float64)


def _edges():
    """A scene of 8 cameras whose pair k holds COUNTS[k] matches."""
    sc = synth.sphere_scene(n_cams=8, n_pts=3000, p_det=1.0, sigma=0.5, outlier_frac=0.1, seed=5, name="routes")
    key = np.minimum(sc.cam1, sc.cam2) * 8 + np.maximum(sc.cam1, sc.cam2)
    rng = np.random.default_rng(5)
    keep = [rng.choice(np.flatnonzero(key == code), n, replace=True) for code, n in zip(np.unique(key), COUNTS)]
    keep = rng.permutation(np.concatenate(keep))
    for name in ("x1", "y1", "x2", "y2", "cam1", "cam2", "inlier"):
        setattr(sc, name, np.ascontiguousarray(getattr(sc, name)[keep]))
    sc.f_gt = np.full(8, 500.0)
    return sc


def _with(sc, i, j, per):
    """A context of the scene and of `per` random matches in each pair (i + 8,
    j + 8), with the rotations and focal lengths of its cameras."""
    rng = np.random.default_rng(6)
    n, m = 9 + int(j.max()), len(i) * per
    xy = [np.concatenate([a, rng.uniform(0, 480, m).astype(np.float32)]) for a in (sc.x1, sc.y1, sc.x2, sc.y2)]
    c1 = np.concatenate([sc.cam1, np.repeat(i + 8, per)]).astype(np.int32)
    c2 = np.concatenate([sc.cam2, np.repeat(j + 8, per)]).astype(np.int32)
    f = np.full(n, 500.0)
    ctx = fastea.Context(0)
    ctx.load_intrinsics(f, np.resize(sc.cx, n), np.resize(sc.cy, n))
    ctx.load_matches(*xy, c1, c2)
    R = np.concatenate([sc.R_init, synth.rotation_from_axis_angle(rng.normal(size=(n - 8, 3)),
                                                                  rng.uniform(0, 0.5, n - 8))])
    return ctx, R, f


@pytest.fixture(scope="module")
def both():
    sc = _edges()
    split = _with(sc, *np.triu_indices(FILL_CAMS, 1), FILL)
    fp32 = _with(sc, np.array([0]), np.array([1]), LONG)
    yield sc, fp32, split
    split[0].close()
    fp32[0].close()


def _search(side, K, tau_px, **kw):
    ctx, R, f = side
    return ctx.relative_translations(R, _cand32(K), f=f, tau_px=tau_px, **kw)


@pytest.mark.parametrize("tau_px", [math.inf, 8.0, 1.5])
@pytest.mark.parametrize("K", [1, 31, 128, 129, 512, 513, 1025])
def test_same_choice_by_both(both, K, tau_px):
    sc, fp32, split = both
    a, b = (_search(side, K, tau_px, scores=True) for side in (fp32, split))
    P = len(COUNTS)
    ref = oracle.rel_trans(oracle_problem(sc), sc.R_init, sc.f_gt, _cand32(K), scores=True, tau=tau_px / 500.0)
    for r in (a, b):
        check_search({k: r[k][:P] for k in r}, ref, K)
        np.testing.assert_array_equal(r["scores"][np.arange(P), r["best"][:P]], r["score_best"][:P].astype(np.float32))
    for k in ("best", "vote", "t_rel", "score_best"):
        np.testing.assert_array_equal(a[k][:P], b[k][:P])


@pytest.mark.parametrize("tau_px", [0.9, 0.05, 1e-4])
@pytest.mark.parametrize("K", [1, 257, 1025])
def test_tight_caps(both, K, tau_px):
    """Caps below 2e-3 in normalised units take fp32 products at any size."""
    sc, fp32, split = both
    a, b = (_search(side, K, tau_px, scores=True) for side in (fp32, split))
    P = len(COUNTS)
    ref = oracle.rel_trans(oracle_problem(sc), sc.R_init, sc.f_gt, _cand32(K), scores=True, tau=tau_px / 500.0)
    check_search({k: a[k][:P] for k in a}, ref, K)
    for k in ("best", "vote", "t_rel", "score_best", "scores"):
        np.testing.assert_array_equal(a[k][:P], b[k][:P])


def _best_of(f, n=5):
    f()
    t = []
    for _ in range(n):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return min(t)


def test_a_tight_cap_does_not_score_every_candidate_twice(both):
    _, _, split = both
    wide = _best_of(lambda: _search(split, 2048, 8.0))
    tight = _best_of(lambda: _search(split, 2048, 0.3))
    assert tight < 2.5 * wide, (tight, wide)  # 1.5 with one scoring, 3.6 with two
