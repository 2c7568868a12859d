"""The quadratic forms in a checkpoint: 45 entries per pair (the upper triangle
of a symmetric 9x9 matrix, row by row), of which those that are the same
product of monomials are equal; they come back as they were written."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

from gpu_helpers import make_context

pytestmark = pytest.mark.gpu


def _section(state, P, M, S=1):
    """Bytes of the forms in a state: their offset from the end is fixed."""
    after = 4 * S + 8 * S + 24 * S + 4 * S + 4 * S + 24 * S + 8 * S + 4 * ((M + 31) // 32) + 4 * S
    end = len(state) - after
    return slice(end - 8 * 45 * P, end)


@pytest.mark.parametrize("n_cams", [2, 3, 12])
def test_forms_of_a_state(n_cams):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = synth.sphere_scene(n_cams=n_cams, n_pts=300, p_det=1.0, sigma=1.0, outlier_frac=0.2, seed=2, name="forms")
    mk = lambda: make_context(sc, gauge=1, inner_loop=1, tile_matches=2048)
    with mk() as a, mk() as b:
        a.init_poses(sc.R_init, sc.t_init)
        a.begin_round(64.0)
        a.step(5)
        P = a.info()["n_pairs"]
        state = a.get_state()
        s = _section(state, P, len(sc.x1))
        W = np.frombuffer(state[s], np.float64).reshape(P, 45)
        i, j = np.triu_indices(9)
        sym = np.array([[0, 1, 2], [1, 3, 4], [2, 4, 5]])
        value = 6 * sym[i // 3, j // 3] + sym[i % 3, j % 3]
        assert len(np.unique(value)) == 36 and np.isfinite(W).all() and (W[:, 0] > 0).all()
        for v in range(36):
            assert (W[:, value == v] == W[:, value == v][:, :1]).all()
        b.set_state(state)
        assert b.get_state() == state
        loss = a.residual_grad()[0].item()
        assert b.residual_grad()[0].item() == loss
        # the forms are what the gradient reads: doubled, the loss doubles
        b.set_state(state[:s.start] + (2.0 * W).tobytes() + state[s.stop:])
        assert b.residual_grad()[0].item() == 2.0 * loss
