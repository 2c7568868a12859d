"""Poses are read from staging memory when their launch runs, so setting them
on a stream under capture is refused, and works again once the capture is
over."""
import numpy as np
import pytest

from paper_2605_18052_amd import fastea, synth

pytestmark = pytest.mark.gpu


def test_poses_refused_under_capture():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sc = synth.tiny_scene(n_cams=6, n_pts=70, seed=5, sigma=1.0, outlier_frac=0.2)
    stream = torch.cuda.Stream()
    ctx = fastea.Context(0, fastea.default_options(gauge_normalize=0), stream=stream.cuda_stream)
    ctx.load_intrinsics(sc.f_init, sc.cx, sc.cy)
    ctx.load_matches(sc.x1, sc.y1, sc.x2, sc.y2, sc.cam1, sc.cam2)
    ctx.init_poses(sc.R_init, sc.t_init)
    before = ctx.get_poses()
    x = torch.zeros(4, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
        x += 1
        with pytest.raises(fastea.FeaError) as e:
            ctx.set_poses(sc.R_gt, sc.t_gt, sc.f_gt)
    assert e.value.status == fastea.FEA_EDEVICE
    torch.cuda.synchronize()
    for a, b in zip(before, ctx.get_poses()):
        np.testing.assert_array_equal(a, b)
    ctx.set_poses(sc.R_gt, sc.t_gt, sc.f_gt)
    np.testing.assert_allclose(ctx.get_poses()[2], sc.f_gt, rtol=1e-12)
    ctx.close()
