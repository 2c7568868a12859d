"""The round's threshold from the median focal length, selected on the device,
against the sorted median: bit for bit, at the edges of the selection (odd,
even, repeated and nearly equal values, one to several values per thread, one
wavefront of candidates)."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _focals(kind, n, rng):
    if kind == "equal":
        return np.full(n, 640.0)
    if kind == "repeated":
        return rng.choice([500.0, 600.0, 700.0], n)
    if kind == "neighbours":  # consecutive doubles around one value
        return (np.float64(800.0).view(np.int64) + rng.integers(-3, 4, n)).view(np.float64)
    if kind == "wide":
        return np.exp(rng.uniform(-200, 200, n))
    return rng.uniform(400, 1200, n)


def _median(f):
    s = np.sort(f)
    n = len(s)
    return s[n // 2] if n % 2 else 0.5 * (s[n // 2 - 1] + s[n // 2])


@pytest.mark.parametrize("kind", ["uniform", "equal", "repeated", "neighbours", "wide"])
@pytest.mark.parametrize("n", [2, 3, 64, 65, 128, 1000, 1024, 1025, 8191, 8192])
def test_threshold(n, kind):
    rng = np.random.default_rng(n)
    f = _focals(kind, n, rng)
    with fastea.Context(0, fastea.default_options(gauge_normalize=0)) as ctx:
        ctx.load_intrinsics(f, f * 0, f * 0)
        x = rng.uniform(-100, 100, (4, 8)).astype(np.float32)
        ctx.load_matches(*x, np.zeros(8, np.int32), np.ones(8, np.int32))
        ctx.init_poses(np.tile(np.eye(3), (n, 1, 1)), rng.normal(size=(n, 3)))
        # the focal lengths the context works with: exp(log f) per camera
        fc = ctx.get_poses()[2]
        for tau_px in (128.0, 4.0):
            ctx.begin_round(tau_px)
            assert ctx.info()["tau"] == tau_px / _median(fc)
