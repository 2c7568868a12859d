"""The focal vote of fundamental matrices at any scale, of rank 2 and of full
rank: multiplying them by a power of two changes no bit of a vote."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("rank", [2, 3])
@pytest.mark.parametrize("exponent", [-960, -500, -300, -100, 100, 300, 500, 1000])
def test_scale(exponent, rank, shared):
    n, P = 15, 50
    rng = np.random.default_rng(4)
    i, j = np.triu_indices(n, 1)
    pick = rng.permutation(len(i))[:P]
    pc = np.stack([i[pick], j[pick]], 1).astype(np.int32)
    U, _, Vt = np.linalg.svd(rng.normal(size=(P, 3, 3)))
    s = np.stack([1 + rng.uniform(0, 0.5, P), np.ones(P), np.full(P, 0.01 if rank == 3 else 0.0)], 1)
    d = np.array([1 / 700.0, 1 / 700.0, 1.0])
    F = d[:, None] * ((U * s[:, None, :]) @ Vt) * d
    F /= np.linalg.norm(F, axis=(1, 2), keepdims=True)
    cand = synth.focal_candidates(70, 200.0, 3000.0)
    kw = {} if shared else dict(group=np.arange(n, dtype=np.int32), f_cur=rng.uniform(500, 900, n))
    with fastea.Context(0) as ctx:
        a = ctx.focal_vote(n, pc, F, cand, 0.05, votes=True, **kw)["votes"]
        b = ctx.focal_vote(n, pc, np.ldexp(F, exponent), cand, 0.05, votes=True, **kw)["votes"]
    assert np.isfinite(a).all() and a.max() > 0
    np.testing.assert_array_equal(a, b)
