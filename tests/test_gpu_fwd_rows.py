"""The forward's output rows and its separate colour product: image widths that
cut the groups of four pixels, and infinite channels."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import np_, require_gpu, run_render
from test_gpu_render import check_forward, staged

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


@pytest.mark.parametrize("c_sem", [0, 5, 16, 32])
@pytest.mark.parametrize("w,h", [(1, 1), (2, 9), (3, 8), (4, 4), (5, 3), (7, 17), (9, 2), (14, 16), (15, 15), (17, 1),
                                 (18, 33), (31, 5)])
def test_row_ends(xgs, c_sem, w, h):
    scene = synth.tiny_scene(seed=w + 40 * h, n=300, c_sem=c_sem)
    cam = synth.Camera(width=w, height=h, fx=20.0, fy=20.0, cx=w / 2, cy=h / 2)
    r, ref, amb = staged(xgs, scene, cam)
    check_forward(r, ref, amb, 1.0)
    np.testing.assert_array_equal(np_(r["n_last"])[~amb], ref.n_last[~amb])


@pytest.mark.parametrize("where", ["feature", "colour", "two"])
@pytest.mark.parametrize("c_sem", [8, 16, 33])
def test_infinite_channel_stays_with_its_pixels(xgs, c_sem, where):
    """Pixels whose weight for the splat is zero get what they get with a finite
    value; the others, infinity of its sign (NaN where two meet)."""
    def image(value, other):
        s = synth.tiny_scene(seed=4, n=60, c_sem=c_sem)
        s.log_scales[:] -= 1.0
        if where == "colour":
            s.colors[7, 1] = value
        else:
            s.features[7, c_sem - 1] = value
        if where == "two":
            s.features[9, c_sem - 1] = other
        r = run_render(xgs, s, synth.tiny_camera())
        return np_(r["out"]), s
    finite, s = image(0.0, 0.0)
    w7 = (image(1.0, 0.0)[0] - finite)
    w9 = (image(0.0, 1.0)[0] - finite)
    got = image(np.inf, -np.inf)[0]
    c = 1 if where == "colour" else 4 + c_sem - 1
    other = np.arange(4 + c_sem) != c
    np.testing.assert_array_equal(got[other], finite[other])
    a, b = w7[c] != 0, w9[c] != 0
    assert a.any() and not a.all()
    want = np.where(a & b, np.nan, np.where(a, np.inf, np.where(b, -np.inf, finite[c])))
    if where != "two":
        want = np.where(a, np.inf, finite[c])
    bad = np.isfinite(want) & (got[c] != want) | (np.isinf(want) & (got[c] != want)) | (np.isnan(want) != np.isnan(got[c]))
    # a weight too small to move the sum cannot be told from none
    assert bad.mean() < 1e-3, bad.mean()
    assert np.isfinite(got[c][~(a | b)]).mean() > 0.999
