"""fea_init_poses on a stream under capture is refused and leaves the poses,
the round and the gauge as they were."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gauge", [0, 1])
def test_refused_init_poses_changes_nothing(gauge):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = synth.tiny_scene(n_cams=6, n_pts=70, seed=5, sigma=1.0, outlier_frac=0.2)
    stream = torch.cuda.Stream()
    with fastea.Context(0, fastea.default_options(gauge_normalize=gauge), stream=stream.cuda_stream) as ctx:
        ctx.load_intrinsics(sc.f_init, sc.cx, sc.cy)
        ctx.load_matches(sc.x1, sc.y1, sc.x2, sc.y2, sc.cam1, sc.cam2)
        ctx.init_poses(sc.R_init, sc.t_init)
        ctx.begin_round(64.0)
        ctx.step(3)
        before, info = ctx.get_poses(), ctx.info()
        x = torch.zeros(4, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
            x += 1
            with pytest.raises(fastea.FeaError) as e:
                ctx.init_poses(sc.R_gt, 3.0 * sc.t_gt + 1.0)
        assert e.value.status == fastea.FEA_EDEVICE
        torch.cuda.synchronize()
        assert ctx.info() == info
        for a, b in zip(before, ctx.get_poses()):
            np.testing.assert_array_equal(a, b)
        ctx.step(2)  # the solver goes on from them
        ctx.init_poses(sc.R_gt, sc.t_gt)
        np.testing.assert_allclose(ctx.get_poses()[0], sc.R_gt, atol=1e-12)
