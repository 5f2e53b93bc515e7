"""The binning form of the tile sort at the edges of its list sorts, bit for
bit against the oracle's instance list, and against the radix form."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import np_, require_gpu
from test_gpu_render import check_sort, projected_from_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def lists(lengths, cam, depths, seed):
    """One-tile Gaussians, lengths[k] of them on tile k, in random order, and a
    few rectangles on both sides of the 32 tiles that a lane walks itself."""
    rng = np.random.default_rng(seed)
    _, _, ty, tx = oracle.grid_info(cam)
    tile = np.repeat(np.arange(len(lengths)), lengths)
    rect = np.stack([tile % tx, tile // tx, tile % tx + 1, tile // tx + 1], 1)
    wide = np.array([[0, ty - 2, min(tx, w), ty] for w in (1, 15, 16, 17)])
    rect = rng.permutation(np.concatenate([rect, wide])).astype(np.int32)
    n = len(rect)
    depth = rng.uniform(0.5, 9.0, n) if depths == 0 else rng.choice(np.linspace(0.5, 9.0, depths), n)
    touched = ((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).astype(np.int64)
    return oracle.Projection(None, None, depth, None, None, rect, touched, np.ones(n, np.int32)), n


LENGTHS = (0, 1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1024, 1025, 2047, 2048, 2049, 4096, 4097,
           6145)


@pytest.mark.parametrize("depths", [0, 1, 40])
@pytest.mark.parametrize("ordered", [True, False])
def test_list_lengths_at_the_edges(xgs, depths, ordered):
    """Lists at the edges of the wavefront, workgroup and merged sorts, with
    distinct, equal and tied depths, with and without the tile order."""
    cam = synth.Camera(width=300, height=100, fx=200.0, fy=200.0, cx=150.0, cy=50.0)
    pr, n = lists(LENGTHS, cam, depths, 3 + depths)
    c = xgs.camera_from(cam)
    if ordered:
        check_sort(xgs, pr, cam, n, extra_cap=5)
        return
    _, _, ty, tx = oracle.grid_info(cam)
    keys, vals, ranges = oracle.bin_instances(pr.rect, oracle.depth_bits(pr.depth), tx, ty)
    b = xgs.alloc_binning(n, len(keys), c)
    b.tile_order = None
    xgs.xgs_tile_sort(projected_from_oracle(xgs, pr, n), c, n, b)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np_(b.keys).view(np.uint64), keys)
    np.testing.assert_array_equal(np_(b.vals).view(np.uint32), vals)
    np.testing.assert_array_equal(np_(b.ranges).view(np.uint32), ranges)


@pytest.mark.parametrize("n", [1, 64, 257, 70_001])
def test_bins_equal_the_radix_form(xgs, n):
    """The same instances with a capacity that keeps the radix form (above
    8,192 per tile): every array is the same; the overflow report too."""
    cam = synth.Camera(width=130, height=100, fx=200.0, fy=200.0, cx=65.0, cy=50.0)
    c = xgs.camera_from(cam)
    _, _, ty, tx = oracle.grid_info(cam)
    rng = np.random.default_rng(n)
    x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
    rect = np.stack([x0, y0, np.minimum(x0 + rng.integers(1, 4, n), tx), np.minimum(y0 + rng.integers(1, 4, n), ty)],
                    1).astype(np.int32)
    depth = rng.choice(np.linspace(0.5, 9.0, 1000), n)
    touched = ((rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])).astype(np.int64)
    touched[rng.random(n) < 0.3] = 0  # culled: the rectangle is not read
    p = projected_from_oracle(xgs, oracle.Projection(None, None, depth, None, None, rect, touched,
                                                     (touched > 0).astype(np.int32)), n)
    m = int(touched.sum())
    got = []
    for cap in (max(m, 1), 8193 * tx * ty):
        b = xgs.alloc_binning(n, cap, c)
        xgs.xgs_tile_sort(p, c, n, b)
        torch.cuda.synchronize()
        assert int(b.status.item()) == 0 and int(b.num_instances.item()) == m
        got.append([np_(b.keys)[:m], np_(b.vals)[:m], np_(b.ranges), np_(b.tile_order)])
    for x, y in zip(*got):
        np.testing.assert_array_equal(x, y)
    if m > 1:
        b = xgs.alloc_binning(n, m - 1, c)
        xgs.xgs_tile_sort(p, c, n, b)
        torch.cuda.synchronize()
        assert int(b.status.item()) == 1 and int(b.num_instances.item()) == 0
        assert not np_(b.ranges).any()
        np.testing.assert_array_equal(np_(b.tile_order), np.arange(tx * ty))
