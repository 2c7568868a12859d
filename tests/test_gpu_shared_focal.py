"""Intrinsics groups of every size around a wavefront's 64 cameras: the log
focal gradient of a group and the solver's Adam step on it, against the same
sums formed from the per-camera gradients on the host."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

from gpu_helpers import make_context

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _scene(n):
    return synth.trajectory_scene(n_cams=n, n_pts=3000, knn=4, target_matches=20_000, seed=12, name="groups",
                                  calib_sample=2000)


def _groups(sizes):
    """Cameras dealt to groups in a shuffled order, so a group's are scattered."""
    g = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    return np.random.default_rng(3).permutation(g)


def _group_sums(groups, gf, f):
    """Per group: sum of f_c dL/df_c and the sum of its terms' sizes."""
    s, size = np.zeros(groups.max() + 1), np.zeros(groups.max() + 1)
    np.add.at(s, groups, gf * f)
    np.add.at(size, groups, np.abs(gf * f))
    return s, size


@pytest.mark.parametrize("sizes", [[1, 63, 64, 65, 7], [129, 2, 69], [200]])
def test_group_gradient_and_step(sizes):
    import torch

    from paper_2605_18052_amd.autograd import epipolar_loss
    n = sum(sizes)
    sc = _scene(n)
    groups = _groups(sizes)
    # one starting focal length per group
    f0 = np.array([sc.f_init[groups == k].mean() for k in range(len(sizes))])[groups]
    ctx = make_context(sc, f=f0, groups=groups, lr_decay=1.0)
    ctx.init_poses(sc.R_init, sc.t_init)
    ctx.begin_round(64.0)
    o = fastea.default_options()

    # the adjoint behind autograd, at the current parameters
    a6, t, logf = (x.clone() for x in ctx.get_params())
    logf.requires_grad_(True)
    epipolar_loss(a6, t, logf, ctx).backward()
    s, size = _group_sums(groups, ctx.residual_grad()[3].cpu().numpy(), ctx.get_poses()[2])
    # the same terms added in another order, n roundings of 2^-53 each
    np.testing.assert_allclose(logf.grad.cpu().numpy(), s, rtol=0, atol=float((n * 2.0**-52 * size).max()))

    # Adam on log f: the same recurrence from the per-camera gradients
    p = logf.detach().cpu().numpy().copy()
    m, v = np.zeros_like(p), np.zeros_like(p)
    for k in range(1, 5):
        s, _ = _group_sums(groups, ctx.residual_grad()[3].cpu().numpy(), ctx.get_poses()[2])
        m = o.beta1 * m + (1 - o.beta1) * s
        v = o.beta2 * v + (1 - o.beta2) * s * s
        p = p - o.lr_logf * (m / (1 - o.beta1**k)) / (np.sqrt(v / (1 - o.beta2**k)) + o.adam_eps)
        ctx.step(1)
        torch.cuda.synchronize()
        # the sums' roundings enter relative to s, which a step scales to lr_logf
        np.testing.assert_allclose(ctx.get_params()[2].cpu().numpy(), p, rtol=1e-12, atol=1e-10)
        f = ctx.get_poses()[2]
        for q in range(len(sizes)):
            assert np.ptp(f[groups == q]) == 0.0
        np.testing.assert_allclose(f, np.exp(p)[groups], rtol=1e-9)
    ctx.close()
