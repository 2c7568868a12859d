"""One context's stage calls one after another, in sizes that share, outgrow
and exceed the scratch it keeps between calls and the staging of its copies,
against the same calls on fresh contexts, bit for bit."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _vote(ctx, n, cands, seed):
    rng = np.random.default_rng(seed)
    pairs = np.stack([np.arange(n), (np.arange(n) + 1) % n], 1).astype(np.int32)
    F = rng.normal(size=(n, 3, 3)) * 1e-3
    r = ctx.focal_vote(n, pairs, F, np.geomspace(300, 1500, cands), 0.05, group=np.arange(n, dtype=np.int32),
                       f_cur=rng.uniform(400, 900, n), votes=True)
    return [np.asarray(r[k]) for k in sorted(r) if k != "ms" and r[k] is not None]


def _align(ctx, n, runs, seed):
    rng = np.random.default_rng(seed)
    pairs = np.stack([np.arange(n - 1), np.arange(1, n)], 1).astype(np.int32)
    R = np.tile(np.eye(3), (n, 1, 1))
    r = ctx.translation_align(pairs, R, rng.normal(size=(n - 1, 3)), rng.normal(size=(runs, n, 3)),
                              fastea.ta_default_options(iters_run=20, iters_final=5), details=True)
    r = r if isinstance(r, dict) else {"o": r}
    return [np.asarray(r[k]) for k in sorted(r) if k != "ms" and r[k] is not None]


# votes of 1,000 groups by 4,096 candidates: 33 MB, past the 16 MiB ring;
# 3,000 by 16,384: 393 MB, past what is kept
CALLS = [(_vote, 5, 8, 1), (_vote, 1000, 4096, 2), (_align, 40, 3, 3), (_vote, 5, 8, 4), (_vote, 3000, 16384, 5),
         (_align, 500, 64, 6), (_vote, 300, 64, 7), (_vote, 5, 8, 1)]


def test_calls_share_a_context():
    with fastea.Context(0) as ctx:
        got = [f(ctx, *a) for f, *a in CALLS]
    for (f, *a), g in zip(CALLS, got):
        with fastea.Context(0) as fresh:
            want = f(fresh, *a)
        assert len(g) == len(want) > 0
        for x, y in zip(g, want):
            np.testing.assert_array_equal(x, y)
    for x, y in zip(got[0], got[-1]):
        np.testing.assert_array_equal(x, y)
