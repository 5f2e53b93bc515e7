"""Infinities and NaN in the backward: what one splat or pixel holds stays out of
the geometry gradients of splats that do not blend there."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import np_, require_gpu, run_render
from test_gpu_render import GROUPS

pytestmark = pytest.mark.gpu

CAM = synth.Camera(width=8, height=8, fx=20.0, fy=20.0, cx=4.0, cy=4.0)
ROW = 16  # words of a splat's workspace row, the first ten used


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def corners(infinite_behind, value):
    """Two splats on opposite corners of one quadrant of 8 x 8 pixels, no pixel
    in common; splat 0 has `value` as a feature and as a colour."""
    s = synth.tiny_scene(seed=1, n=2, c_sem=8)
    z = (2.2, 2.0) if infinite_behind else (2.0, 2.2)
    s.means[:] = [[-0.3, -0.3, z[0]], [0.3, 0.3, z[1]]]
    s.log_scales[:] = -4.0
    s.opacity[:] = 0.8
    s.features[0, 3] = value
    s.colors[0, 1] = value
    return s


def backward(xgs, scene, d, flags):
    """Gradients of splat 1 and its workspace row."""
    r = run_render(xgs, scene, CAM)
    ws = torch.zeros(int(xgs.lib.xgs_render_bwd_workspace(2)), dtype=torch.uint8, device="cuda")
    gr = xgs.xgs_render_bwd(r["g"], r["p"], r["b"], r["cam"], d, r["final_T"], r["n_last"], flags=flags, workspace=ws)
    torch.cuda.synchronize()
    row = np_(ws.view(torch.float32))[ROW:ROW + 10]
    return row, [] if gr is None else [np_(getattr(gr, k))[1] for k in GROUPS]


@pytest.mark.parametrize("infinite_behind", [False, True])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("pose", [False, True])
def test_infinite_channel_in_either_depth_order(xgs, infinite_behind, value, pose):
    """The other splat's gradients are the bits that they are with finite channels."""
    d = torch.from_numpy(synth.upstream_grad(12, 8, 8, seed=2)).cuda()
    flags = xgs.BWD_POSE if pose else xgs.BWD_ALL
    got = backward(xgs, corners(infinite_behind, value), d, flags)
    want = backward(xgs, corners(infinite_behind, 1.0), d, flags)
    np.testing.assert_array_equal(got[0], want[0])
    for a, b in zip(got[1], want[1]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("pose", [False, True])
def test_infinite_upstream_gradient_of_one_pixel(xgs, behind, value, pose):
    """A colour gradient that is not finite at a pixel that only splat 0 covers:
    the geometry gradients of splat 1 are what they are without it."""
    d = torch.from_numpy(synth.upstream_grad(12, 8, 8, seed=2)).cuda()
    flags = xgs.BWD_POSE if pose else xgs.BWD_ALL
    want = backward(xgs, corners(behind, 1.0), d, flags)
    d[0, 1, 1] = value
    got = backward(xgs, corners(behind, 1.0), d, flags)
    np.testing.assert_array_equal(got[0][:7], want[0][:7])
    for name, a, b in zip(GROUPS, got[1], want[1]):
        if name in ("means", "log_scales", "quats", "opacity"):
            np.testing.assert_array_equal(a, b)
