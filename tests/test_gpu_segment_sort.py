"""The pair sort at the edges of its tiles, digits and passes, bit for bit
against the oracle's segmenting, through the C-ABI."""
import numpy as np
import pytest

import oracle
from paper_2605_18052_amd import fastea

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def _matches(n_cams, M, order, seed):
    rng = np.random.default_rng(seed)
    if order == "one pair":
        c1, c2 = np.zeros(M, np.int32), np.full(M, n_cams - 1, np.int32)
    elif order == "few pairs":  # long runs, ends of the key range among them
        a = rng.integers(0, 3, M)
        c1 = np.array([0, n_cams - 2, min(1, n_cams - 2)])[a].astype(np.int32)
        c2 = np.array([1, n_cams - 1, n_cams - 1])[a].astype(np.int32)
        if n_cams == 2:
            c1[:], c2[:] = 0, 1
    else:
        c1 = rng.integers(0, n_cams, M).astype(np.int32)
        c2 = ((c1 + rng.integers(1, n_cams, M)) % n_cams).astype(np.int32)
    flip = rng.random(M) < 0.5
    c1, c2 = np.where(flip, c2, c1).astype(np.int32), np.where(flip, c1, c2).astype(np.int32)
    if order == "sorted":
        o = np.lexsort((np.maximum(c1, c2), np.minimum(c1, c2)))
        c1, c2 = c1[o], c2[o]
    return [rng.random(M).astype(np.float32) * 640 for _ in range(4)] + [c1, c2]


# cameras: 2 to 32 bits of key, one to four passes; matches around one and
# two tiles of 4,096 and a wave's 1,024
@pytest.mark.parametrize("order", ["random", "sorted", "few pairs", "one pair"])
@pytest.mark.parametrize("n_cams,M", [(2, 1), (2, 4096), (3, 4097), (16, 1024), (17, 4095), (300, 8193),
                                      (5000, 20_011), (65535, 9001)])
def test_sort_matches_oracle(n_cams, M, order):
    m = _matches(n_cams, M, order, seed=n_cams + M)
    f = np.full(n_cams, 500.0)
    with fastea.Context(0) as ctx:
        ctx.load_intrinsics(f, f * 0 + 320, f * 0 + 240)
        ctx.load_matches(*m)
        perm, sw, pc, so = ctx.get_segments()
        # the layout: a round that keeps everything returns every match
        if n_cams <= 300:
            rng = np.random.default_rng(1)
            R = np.tile(np.eye(3), (n_cams, 1, 1))
            ctx.init_poses(R, rng.normal(size=(n_cams, 3)))
            ctx.begin_round(float("inf"))
            mask, z = ctx.get_mask()
            assert z == M and mask.all()
    operm, osw, opc, oso = oracle.segment(m[4], m[5], n_cams)
    np.testing.assert_array_equal(perm, operm)
    np.testing.assert_array_equal(sw, osw)
    np.testing.assert_array_equal(pc, opc)
    np.testing.assert_array_equal(so, oso)


def test_reload_smaller_larger_and_bad():
    """One context loads problems of other sizes in turn (its buffers hold
    the sort of the next); a refused load leaves it loadable."""
    f = np.full(300, 500.0)
    with fastea.Context(0) as ctx:
        ctx.load_intrinsics(f, f * 0 + 320, f * 0 + 240)
        for M in (9000, 10, 30_000):
            m = _matches(300, M, "random", seed=M)
            bad = [a.copy() for a in m]
            bad[0][M // 2] = np.nan
            with pytest.raises(fastea.FeaError):
                ctx.load_matches(*bad)
            bad = [a.copy() for a in m]
            bad[4][M - 1] = 300
            with pytest.raises(fastea.FeaError):
                ctx.load_matches(*bad)
            ctx.load_matches(*m)
            perm, sw, pc, so = ctx.get_segments()
            operm, osw, opc, oso = oracle.segment(m[4], m[5], 300)
            np.testing.assert_array_equal(perm, operm)
            np.testing.assert_array_equal(sw, osw)
            np.testing.assert_array_equal(so, oso)
