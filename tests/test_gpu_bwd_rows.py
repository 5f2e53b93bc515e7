"""The backward's per-Gaussian rows: every way that its channel rows are read
and its gradients added, lists at the edges of its batches, rows past 4 GiB,
and an infinite feature beside pixels that it does not reach."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import gaussians, np_, rel_l2, require_gpu, run_render
from test_gpu_render import GROUPS, backward_errors, check_forward, staged

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


@pytest.mark.parametrize("c_sem", [2, 4, 7, 8, 12, 13, 16, 17, 24, 25, 28, 29, 31, 32, 33, 48])
def test_channel_counts_of_the_rows(xgs, c_sem):
    """Widths that are whole groups of four features (one to three groups a
    lane, the last group partial), pairs of whole tiles, and the widths that
    run masked on the next wider one."""
    scene = synth.tiny_scene(seed=20 + c_sem, n=700, c_sem=c_sem)
    r, ref, amb = staged(xgs, scene, synth.tiny_camera())
    assert check_forward(r, ref, amb, 0.01) < 0.01
    errs = backward_errors(xgs, r, ref, amb, scene, synth.tiny_camera(), seed=12)
    assert all(v <= 1e-3 for v in errs.values()), errs


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 97, 130])
def test_list_lengths(xgs, n):
    """n faint splats over one tile: lists that end inside, at and past the
    batches of 16 and the candidate groups of 64."""
    rng = np.random.default_rng(n)
    scene = synth.tiny_scene(seed=n, n=n, c_sem=8)
    scene.means[:, :2] = rng.uniform(-0.05, 0.05, (n, 2))
    scene.log_scales[:] = rng.uniform(-2.2, -1.5, (n, 3))
    scene.opacity[:] = rng.uniform(0.02, 0.06, n)
    cam = synth.Camera(width=16, height=16, fx=20.0, fy=20.0, cx=8.0, cy=8.0)
    r, ref, amb = staged(xgs, scene, cam)
    assert int(r["n_last"].max().item()) == n  # every pixel's walk takes the whole list
    errs = backward_errors(xgs, r, ref, amb, scene, cam, seed=3)
    assert all(v <= 1e-3 for v in errs.values()), errs


def test_rows_past_4_gib(xgs):
    """A small scene as the last rows of 2^26 Gaussians (the others culled):
    the workspace rows lie past 4 GiB.  Same gradients as the scene alone, up to
    the order of the atomic sums (a few hundred terms of 2^-24 each)."""
    scene, cam = synth.tiny_scene(seed=3), xgs.camera_from(synth.tiny_camera())
    small = run_render(xgs, scene, synth.tiny_camera())
    hs, ws, _, _ = xgs.grid_dims(cam)
    d_out = torch.from_numpy(synth.upstream_grad(4 + scene.c_sem, hs, ws, seed=5)).cuda()
    want = xgs.xgs_render_bwd(small["g"], small["p"], small["b"], cam, d_out, small["final_T"], small["n_last"])
    n, k = (1 << 26) + 512, scene.n
    big = []
    for t in (getattr(small["g"], name) for name in GROUPS):
        b = torch.zeros((n, *t.shape[1:]), device="cuda")
        b[n - k:] = t
        big.append(b)
    g = xgs.Gaussians(*big)
    p = xgs.xgs_project(g, cam)
    b = xgs.alloc_binning(n, small["m"], cam)
    xgs.xgs_tile_sort(p, cam, n, b)
    out, fT, nl = xgs.xgs_render_fwd(g, p, b, cam)
    got = xgs.xgs_render_bwd(g, p, b, cam, d_out, fT, nl)
    torch.cuda.synchronize()
    assert torch.equal(out, small["out"]) and torch.equal(nl, small["n_last"])
    for name in GROUPS:
        x = getattr(got, name)
        assert not bool(x[:n - k].any()), name
        assert rel_l2(np_(x[n - k:]), np_(getattr(want, name))) < 1e-5, name


def test_infinite_feature_stays_with_its_pixels(xgs):
    """Two splats on opposite corners of one quadrant of 8 x 8 pixels, no pixel
    in common, and an infinite feature on one of them: the gradients of the
    other are what they are with a finite one."""
    def grads(value):
        s = synth.tiny_scene(seed=1, n=2, c_sem=8)
        s.means[:] = [[-0.3, -0.3, 2.0], [0.3, 0.3, 2.2]]
        s.log_scales[:] = -4.0
        s.opacity[:] = 0.8
        s.features[0, 3] = value
        cam = synth.Camera(width=8, height=8, fx=20.0, fy=20.0, cx=4.0, cy=4.0)
        r = run_render(xgs, s, cam)
        d = torch.from_numpy(synth.upstream_grad(12, 8, 8, seed=2)).cuda()
        gr = xgs.xgs_render_bwd(r["g"], r["p"], r["b"], r["cam"], d, r["final_T"], r["n_last"])
        torch.cuda.synchronize()
        return [np_(getattr(gr, k))[1] for k in GROUPS]
    for a, b in zip(grads(np.inf), grads(1.0)):
        np.testing.assert_array_equal(a, b)
