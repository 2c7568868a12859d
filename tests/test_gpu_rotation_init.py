"""The Lanczos initialisation at the ends of its looks and restarts: any bound
on the products, basis exhaustion, more cameras than a wave adds up by
itself, against numpy's eigenvectors, through the C-ABI."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _ring(n, reach, seed, noise_deg):
    """Cameras paired with the next `reach` on a ring, relative rotations with noise."""
    rng = np.random.default_rng(seed)
    R = synth.rotation_from_axis_angle(rng.normal(size=(n, 3)), rng.uniform(0, np.pi, n))
    i = np.repeat(np.arange(n), reach)
    j = (i + np.tile(np.arange(1, reach + 1), n)) % n
    N = synth.rotation_from_axis_angle(rng.normal(size=(len(i), 3)),
                                       np.deg2rad(np.abs(rng.normal(0, noise_deg, len(i))) if noise_deg else
                                                  np.zeros(len(i))))
    return R, np.stack([i, j], 1).astype(np.int32), N @ R[j] @ R[i].transpose(0, 2, 1), rng.normal(size=(2, n, 3))


def _lanczos_first_column(n, pc, Rr, v0, steps):
    """The Ritz vector of the smallest Ritz value after `steps` steps, per
    camera normalised (the first columns), in numpy."""
    M = np.zeros((3 * n, 3 * n))
    for (i, j), R in zip(pc, Rr):
        a, b = slice(3 * i, 3 * i + 3), slice(3 * j, 3 * j + 3)
        M[b, b] += np.eye(3)
        M[a, a] += R.T @ R
        M[b, a] -= R
        M[a, b] -= R.T
    V = [v0.ravel() / np.linalg.norm(v0)]
    for _ in range(steps):
        w = M @ V[-1]
        for _ in range(2):
            w = w - np.array(V).T @ (np.array(V) @ w)
        V.append(w / np.linalg.norm(w))
    Q = np.array(V[:steps])
    val, vec = np.linalg.eigh(Q @ M @ Q.T)
    c = (vec[:, 0] @ Q).reshape(n, 3)
    return c / np.linalg.norm(c, axis=1, keepdims=True)


# one step to just past the second look; the steps queued past a look are not used
@pytest.mark.parametrize("steps", [1, 2, 15, 16, 17, 20, 21, 32, 33])
def test_first_columns_after_a_bounded_number_of_products(steps):
    n = 40
    R, pc, Rr, v0 = _ring(n, 4, seed=3, noise_deg=30.0)
    with fastea.Context(0) as ctx:
        got = ctx.rotation_averaging(n, pc, Rr, v0=v0,
                                     options=fastea.ra_default_options(iters=0, init_iters=steps))
    ref = _lanczos_first_column(n, pc, Rr, v0[0], steps)
    c = got["R_init"][:, :, 0]
    c = c * np.sign((c * ref).sum())
    # a Ritz vector of a well-separated value: both sides to rounding, which
    # the tridiagonal's eigenvector solve amplifies by 1 / (gap ~ 1e-3)
    np.testing.assert_allclose(c, ref, atol=1e-9)


@pytest.mark.parametrize("n,reach", [(2, 1), (3, 1), (22, 3), (6000, 3)])
def test_noiseless_rotations_are_recovered(n, reach):
    """Krylov spaces that run out before the first look (n small), and more
    norm parts than a wave adds up by itself (6,000 cameras: 282 parts)."""
    R, pc, Rr, v0 = _ring(n, reach, seed=n, noise_deg=0.0)
    if n == 2:
        pc, Rr = pc[:1], Rr[:1]
    if n == 6000:  # long rings converge slowly: chords across it
        rng = np.random.default_rng(0)
        extra = rng.integers(0, n, size=(6 * n, 2))
        extra = extra[extra[:, 0] != extra[:, 1]].astype(np.int32)
        pc = np.concatenate([pc, extra])
        Rr = R[pc[:, 1]] @ R[pc[:, 0]].transpose(0, 2, 1)
    with fastea.Context(0) as ctx:
        got = ctx.rotation_averaging(n, pc, Rr, v0=v0, options=fastea.ra_default_options(iters=0))
    G = got["R_init"].transpose(0, 2, 1) @ R  # one rotation for all cameras
    # the stopping test leaves the Ritz value within 3e-5 of itself: near zero
    # that is 1e-12 of the spectrum's scale, its vector off by its square root
    np.testing.assert_allclose(G, np.broadcast_to(G[0], G.shape), atol=2e-4)
