"""Stage calls whose work does not fit one launch (a grid dimension takes fewer
than 2^32 threads), through the C-ABI."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _scores64(x1, y1, x2, y2, cx, cy, f, cand):
    """Mean |u . (x~1 x x~2)| of one pair at R_ij = I, in fp64 on the GPU."""
    import torch
    d = [torch.tensor(v, dtype=torch.float64, device="cuda") for v in (x1, y1, x2, y2)]
    one = torch.ones_like(d[0])
    a = torch.stack([(d[0] - cx) / f, (d[1] - cy) / f, one], 1)
    b = torch.stack([(d[2] - cx) / f, (d[3] - cy) / f, one], 1)
    n = torch.linalg.cross(a, b)
    out = [(n @ c.T).abs().mean(0) for c in cand.split(1 << 16)]
    return torch.cat(out)


def test_search_over_more_candidates_and_items_than_one_launch_takes():
    """2,100 pairs by 2^22 candidates (the documented most): 2,100 items by
    8,192 groups of 512 candidates by 256 threads."""
    import torch
    n_cams, n_pairs, per, K = 66, 2100, 400, 1 << 22
    free, _ = torch.cuda.mem_get_info()
    if free < 60e9:
        pytest.skip("needs 60 GB of free device memory")
    rng = np.random.default_rng(0)
    i, j = (v[:n_pairs].astype(np.int32) for v in np.triu_indices(n_cams, 1))
    m = n_pairs * per
    x1, x2 = (rng.uniform(0, 640, m).astype(np.float32) for _ in range(2))
    y1, y2 = (rng.uniform(0, 480, m).astype(np.float32) for _ in range(2))
    f = np.full(n_cams, 500.0)
    cand = synth.sphere_candidates(K).astype(np.float32).astype(np.float64)
    with fastea.Context(0) as ctx:
        ctx.load_intrinsics(f, f * 0 + 320, f * 0 + 240)
        ctx.load_matches(x1, y1, x2, y2, np.repeat(i, per), np.repeat(j, per))
        R = np.tile(np.eye(3), (n_cams, 1, 1))
        got = ctx.relative_translations(R, cand, timing=True)
        quarter = ctx.relative_translations(R, cand[::4], timing=True)
    # every workgroup ran: what a cut launch leaves out is scored a second time
    # by the selection where its scratch happens to hold zeros
    assert got["score_ms"] > 2 * quarter["score_ms"]
    cd = torch.tensor(cand, device="cuda")
    for p in (0, 1, 1023, 1024, 2046, 2047, 2048, 2099):
        s = slice(p * per, (p + 1) * per)
        ref = _scores64(x1[s], y1[s], x2[s], y2[s], 320.0, 240.0, 500.0, cd)
        lo = float(ref.min())
        tol = 1e-6 + 1e-5 * lo  # of fp32 scores, as in gpu_helpers.score_tol
        assert abs(got["score_best"][p] - lo) <= tol
        assert float(ref[int(got["best"][p])]) <= lo + 2 * tol


def test_vote_over_more_groups_and_candidates_than_one_launch_takes():
    """16,384 groups by 16,384 candidates with one group's pairs cut into runs:
    4.2 million blocks of 64 candidates, whose sums take 1,024 threads each."""
    G, K, shared = 16384, 16384, 40
    rng = np.random.default_rng(1)
    n = G - 1 + shared
    grp = np.concatenate([np.zeros(shared, np.int32), np.arange(1, G, dtype=np.int32)])
    a, b = np.triu_indices(shared, 1)
    far = np.arange(n - 50, n)  # 25 pairs among the last groups
    pc = np.concatenate([np.stack([a, b], 1), far.reshape(25, 2)]).astype(np.int32)
    F = rng.normal(size=(len(pc), 3, 3))
    U, _, Vt = np.linalg.svd(F)
    F = (U * np.stack([1 + rng.uniform(0, 0.5, len(F)), np.ones(len(F)), np.zeros(len(F))], 1)[:, None, :]) @ Vt
    d = np.array([1 / 700.0, 1 / 700.0, 1.0])
    F = d[:, None] * F * d
    cand = synth.focal_candidates(K, 200.0, 3000.0)
    fcur = rng.uniform(400, 1200, G)
    with fastea.Context(0) as ctx:
        got = ctx.focal_vote(n, pc, F, cand, 0.05, group=grp, f_cur=fcur)
        # the same votes in calls of few groups
        one = ctx.focal_vote(shared, pc[:len(a)], F[:len(a)], cand, 0.05, votes=True)
        last = ctx.focal_vote(50, far.reshape(25, 2) - (n - 50), F[len(a):], cand, 0.05,
                              group=np.arange(50, dtype=np.int32), f_cur=fcur[G - 50:], votes=True)
    # the runs are cut elsewhere: the sums agree to rounding, the choice to a tie of it
    v = one["votes"][0]
    assert v[got["k_best"][0]] >= v.max() * (1 - 1e-12)
    np.testing.assert_array_equal(got["k_best"][G - 50:], last["k_best"])
    np.testing.assert_array_equal(got["k_best"][1:G - 50], 0)  # no pairs: every vote zero, the first candidate
    np.testing.assert_array_equal(got["f_best"], cand[got["k_best"]])
