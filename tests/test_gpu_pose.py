"""The backward that forms only the pose gradient's sums, the zeroing of the
rows in view, and the tracking loss's depth count."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import np_, rel_l2, require_gpu, run_render

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


@pytest.mark.parametrize("n,c_sem,stride", [(1, 0, 1), (17, 3, 1), (300, 8, 2), (2000, 16, 1), (900, 54, 3)])
def test_pose_rows_equal_the_full_backward(xgs, n, c_sem, stride):
    """dL/dxi from XGS_BWD_POSE (d_out of four channels, no gradient arrays) and
    from the full backward with zero semantic channels: the same sums in another
    order (relative 1e-5: some hundred FP32 terms), into a workspace that held
    NaN before."""
    scene = synth.tiny_scene(seed=n, n=n, c_sem=c_sem)
    cam = synth.tiny_camera().with_grid(stride, stride - 1, 0)
    r = run_render(xgs, scene, cam)
    hs, ws, _, _ = oracle.grid_info(cam)
    d = np.zeros((4 + c_sem, hs, ws), np.float32)
    d[:4] = synth.upstream_grad(4, hs, ws, seed=3)
    d = torch.from_numpy(d).cuda()
    got = []
    for flags, up in ((xgs.BWD_ALL, d), (xgs.BWD_POSE, d[:4].clone())):
        w = torch.full((int(xgs.lib.xgs_render_bwd_workspace(n)) // 4,), float("nan"), device="cuda").view(torch.uint8)
        xgs.xgs_render_bwd(r["g"], r["p"], r["b"], r["cam"], up, r["final_T"], r["n_last"], flags=flags, workspace=w)
        got.append(np_(xgs.xgs_pose_grad(r["g"], r["p"], r["cam"], w)))
    assert np.isfinite(got[0]).all()
    assert rel_l2(got[1], got[0]) < 1e-5


@pytest.mark.parametrize("hs,ws", [(1, 1), (1, 3), (1, 4), (1, 5), (7, 9), (33, 31), (256, 257), (300, 301)])
@pytest.mark.parametrize("offset", [0, 1])
def test_depth_count(xgs, hs, ws, offset):
    """Counts at the ends of the groups of four, at any 4-byte alignment."""
    rng = np.random.default_rng(hs * ws)
    out, img = rng.random((5, hs, ws)).astype(np.float32), rng.random((3, hs, ws)).astype(np.float32)
    dep = rng.random((hs, ws)).astype(np.float32)
    dep[rng.random((hs, ws)) < 0.4] = 0.0
    flat = torch.zeros(hs * ws + 1, device="cuda")
    d = flat[offset:offset + hs * ws].view(hs, ws)
    d.copy_(torch.from_numpy(dep))
    loss, g = xgs.xgs_tracking_loss(torch.from_numpy(out).cuda(), torch.from_numpy(img).cuda(), d, 0.7)
    ref, dref = oracle.track_loss(out, img, dep, 0.7)
    assert abs(float(np_(loss)[0]) - ref) <= 1e-5 * ref
    np.testing.assert_allclose(np_(g), dref, rtol=1e-6, atol=1e-12)
