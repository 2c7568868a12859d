"""Votes of fundamental matrices of rank 2, whose reduced forms lose nothing to
cancellation: against singular values, to fp64 rounding."""
import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(200.0, 3000.0), (50.0, 20000.0)])
@pytest.mark.parametrize("groups", ["one", "each"])
def test_rank2_votes_to_rounding(groups, lo, hi):
    """s1/s2 comes out of some hundred fp64 operations, and of numpy's
    decomposition, to about 1e-14 of itself; terms that count have s1/s2 below
    30, so a term is within 3e-13/tau of itself.  Some of the essential matrices
    have s1/s2 = 1 + 1e-9, where a closed form of the cubic is off by 1e-8."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, P, tau = 30, 300, 0.05
    rng = np.random.default_rng(8)
    i, j = np.triu_indices(n, 1)
    pick = rng.permutation(len(i))[:P]
    pc = np.stack([i[pick], j[pick]], 1).astype(np.int32)
    U, _, Vt = np.linalg.svd(rng.normal(size=(P, 3, 3)))
    s1 = 1.0 + np.where(rng.random(P) < 0.5, 1e-9, rng.uniform(0, 0.5, P))
    E = (U * np.stack([s1, np.ones(P), np.zeros(P)], 1)[:, None, :]) @ Vt
    f = np.full(n, 640.0) if groups == "one" else rng.uniform(400, 1200, n)
    d = np.stack([1 / f, 1 / f, np.ones(n)], 1)
    F = d[pc[:, 1]][:, :, None] * E * d[pc[:, 0]][:, None, :]
    F /= np.linalg.norm(F, axis=(1, 2), keepdims=True)
    cand = np.append(synth.focal_candidates(127, lo, hi), 640.0)
    grp = np.zeros(n, np.int32) if groups == "one" else np.arange(n, dtype=np.int32)
    kw = {} if groups == "one" else dict(group=grp, f_cur=f)
    with fastea.Context(0) as ctx:
        got = ctx.focal_vote(n, pc, F, cand, tau, votes=True, **kw)["votes"]
    ref, _ = oracle.focal_vote(pc, F, grp, f if groups == "each" else [0.0], cand, tau)
    bad = np.abs(got - ref) > 1e-11 / tau * ref + 1e-14 * P
    assert not bad.any(), (np.argwhere(bad)[:5], got[bad][:5], ref[bad][:5])
