"""The focal vote's forms of a pair (rank 2 with one or both sides taking the
candidate, full rank) and the cutting of a group's pairs into runs, against
the numpy oracle's singular values, through the C-ABI."""
import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea, synth

from gpu_helpers import vote_tol

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _pairs(n_cams, n_pairs, seed):
    """Random distinct pairs in both orientations and random F of rank 2."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(n_cams, 1)
    pick = rng.permutation(len(i))[:n_pairs]
    pc = np.stack([i[pick], j[pick]], 1)
    pc = np.where(rng.random((len(pc), 1)) < 0.5, pc, pc[:, ::-1]).astype(np.int32)
    E = rng.normal(size=(len(pc), 3, 3))
    U, _, Vt = np.linalg.svd(E)
    s = np.stack([1 + rng.uniform(0, 0.5, len(pc)), np.ones(len(pc)), np.zeros(len(pc))], 1)
    E = U @ (s[:, :, None] * Vt)
    f = rng.uniform(400, 1200, size=n_cams)
    d = np.stack([1 / f, 1 / f, np.ones(n_cams)], 1)
    F = d[pc[:, 1]][:, :, None] * E * d[pc[:, 0]][:, None, :]
    return pc, F / np.linalg.norm(F, axis=(1, 2), keepdims=True), f, rng


# (cameras, pairs, candidates, groups): one group whose pairs are cut into
# many runs; a candidate count below, at and past a wave; groups of one
# camera; a few uneven groups and one without pairs
CASES = [(40, 700, 130, "one"), (12, 60, 1, "one"), (12, 17, 64, "one"), (30, 300, 65, "each"),
         (25, 200, 200, "few")]


@pytest.mark.parametrize("full", ["none", "some", "all"])
@pytest.mark.parametrize("n_cams,n_pairs,K,groups", CASES)
def test_vote_forms_match_singular_values(n_cams, n_pairs, K, groups, full):
    pc, F, f, rng = _pairs(n_cams, n_pairs, seed=n_pairs + K)
    # full rank: a third singular value of 1e-6 to 1e-2 of the others
    if full != "none":
        E = F * np.array([800.0, 800.0, 1.0])[:, None] * np.array([800.0, 800.0, 1.0])
        add = 10.0 ** rng.uniform(-6, -2, size=(len(F), 1, 1)) * rng.normal(size=F.shape) * \
            np.linalg.norm(E, axis=(1, 2), keepdims=True)
        add /= np.array([800.0, 800.0, 1.0])[:, None] * np.array([800.0, 800.0, 1.0])
        F = F + (add if full == "all" else add * (rng.random((len(F), 1, 1)) < 0.3))
    tau = 0.05
    if groups == "one":
        grp, fcur, arg = np.zeros(n_cams, np.int32), [0.0], None
    elif groups == "each":
        grp, fcur = np.arange(n_cams, dtype=np.int32), f * rng.uniform(0.9, 1.1, n_cams)
        arg = grp
    else:  # ids 0, 1, 3: group 2 has no camera, hence no pair
        grp = np.array([0, 1, 3], np.int32)[np.minimum(rng.integers(0, 6, n_cams), 2)]
        fcur = np.array([700.0, 650.0, 800.0, 720.0])
        arg = grp
    cand = synth.focal_candidates(K, 200.0, 3000.0) if K > 1 else np.array([700.0])
    with fastea.Context(0) as ctx:
        got = ctx.focal_vote(n_cams, pc, F, cand, tau, group=arg, f_cur=None if arg is None else fcur, votes=True)
    ref, _ = oracle.focal_vote(pc, F, grp, fcur, cand, tau)
    tol = vote_tol(ref, tau, n_pairs)
    bad = np.abs(got["votes"] - ref) > tol
    assert not bad.any(), (np.argwhere(bad)[:5], got["votes"][bad][:5], ref[bad][:5])
    chosen = ref[np.arange(len(ref)), got["k_best"]]
    assert np.all(chosen >= ref.max(1) - 2 * vote_tol(ref.max(1), tau, n_pairs))
    np.testing.assert_array_equal(got["f_best"], cand[got["k_best"]])


@pytest.mark.parametrize("scale", [1e-90, 1e90])
def test_vote_does_not_depend_on_the_scale_of_F(scale):
    """F has any scale: the reduced forms normalise it, so the votes agree to
    rounding."""
    pc, F, f, _ = _pairs(15, 50, seed=3)
    cand = synth.focal_candidates(70, 200.0, 3000.0)
    with fastea.Context(0) as ctx:
        a = ctx.focal_vote(15, pc, F, cand, 0.05, votes=True)["votes"]
        b = ctx.focal_vote(15, pc, F * scale, cand, 0.05, votes=True)["votes"]
    np.testing.assert_allclose(b, a, rtol=1e-9, atol=1e-12)
