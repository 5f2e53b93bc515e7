"""The radix form of the tile sort, which serves more than 16,384 tiles, more than
8,192 instances of capacity a tile, and workspaces that hold only it: its
boundaries, long lists, overflow report and the fall back to it."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import np_, require_gpu
from test_gpu_render import check_sort, projected_from_oracle

pytestmark = pytest.mark.gpu

SMALL = synth.Camera(width=64, height=48, fx=50.0, fy=50.0, cx=32.0, cy=24.0)         # 12 tiles
LARGE = synth.Camera(width=2100, height=2100, fx=900.0, fy=900.0, cx=1050.0, cy=1050.0)  # 17,424 tiles


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def one_tile(n, cam, seed, depths=40):
    rng = np.random.default_rng(seed)
    _, _, ty, tx = oracle.grid_info(cam)
    x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
    rect = np.stack([x0, y0, x0 + 1, y0 + 1], 1).astype(np.int32)
    return oracle.Projection(None, None, rng.choice(np.linspace(0.5, 9.0, depths), n), None, None, rect,
                             np.ones(n, np.int64), np.ones(n, np.int32))


@pytest.mark.parametrize("n", [1, 63, 64, 2048, 4097, 70_000])
@pytest.mark.parametrize("cam", [SMALL, LARGE])
def test_scatter_boundaries(xgs, n, cam):
    """A lone key, a partial and a full wavefront, one full block of 2,048 keys and
    one more by a key; depths with exact ties.  Few tiles: a capacity above
    8,192 a tile."""
    _, _, ty, tx = oracle.grid_info(cam)
    assert check_sort(xgs, one_tile(n, cam, n), cam, n, extra_cap=8193 * tx * ty if cam is SMALL else 100) == n


@pytest.mark.parametrize("cam", [SMALL, LARGE])
@pytest.mark.parametrize("ordered", [True, False])
def test_overflow(xgs, cam, ordered):
    """More instances than the capacity: status 1, no instances, empty lists, and
    the order of equal lists."""
    _, _, ty, tx = oracle.grid_info(cam)
    T = tx * ty
    # the few tiles need a capacity above 8,192 each to come here
    n = 8193 * T + 1 if cam is SMALL else 5000
    pr = one_tile(n, cam, 3)
    c = xgs.camera_from(cam)
    p = projected_from_oracle(xgs, pr, n)
    b = xgs.alloc_binning(n, n - 1, c)
    if not ordered:
        b.tile_order = None
    b.ranges.fill_(7)
    xgs.xgs_tile_sort(p, c, n, b)
    torch.cuda.synchronize()
    assert int(b.status.item()) == 1 and int(b.num_instances.item()) == 0
    assert not np_(b.ranges).any()
    if ordered:
        np.testing.assert_array_equal(np_(b.tile_order), np.arange(T))


@pytest.mark.parametrize("n", [300, 70_000])
def test_workspace_of_the_radix_form_only(xgs, n):
    """Sizes at which the binning form needs more: a workspace that holds only the
    radix form takes it, with the same arrays; one byte less than it is refused."""
    cam = synth.Camera(width=2048, height=2048, fx=900.0, fy=900.0, cx=1024.0, cy=1024.0)  # 16,384 tiles
    c = xgs.camera_from(cam)
    p = projected_from_oracle(xgs, one_tile(n, cam, n), n)
    got = []
    small = int(xgs.lib.xgs_tile_sort_workspace(n, n, 20_000))  # past 16,384 tiles: the radix form's alone
    both = int(xgs.lib.xgs_tile_sort_workspace(n, n, 16_384))
    assert small < both
    for nbytes in (both, small):
        b = xgs.alloc_binning(n, n, c)
        b.workspace = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        xgs.xgs_tile_sort(p, c, n, b)
        torch.cuda.synchronize()
        assert int(b.status.item()) == 0 and int(b.num_instances.item()) == n
        got.append([np_(t) for t in (b.keys, b.vals, b.ranges, b.tile_order)])
    for x, y in zip(*got):
        np.testing.assert_array_equal(x, y)
    b.workspace = torch.empty(small - 1, dtype=torch.uint8, device="cuda")
    with pytest.raises(xgs.XgsError):
        xgs.xgs_tile_sort(p, c, n, b)


def test_long_lists(xgs):
    """Four tiles with 10,500 instances each beside scattered rectangles."""
    rng = np.random.default_rng(6)
    _, _, ty, tx = oracle.grid_info(LARGE)
    n = 14_000
    x0, y0 = rng.integers(0, tx, n), rng.integers(0, ty, n)
    x1, y1 = np.minimum(x0 + rng.integers(1, 4, n), tx), np.minimum(y0 + rng.integers(1, 4, n), ty)
    big = np.arange(n) < 10_500
    x0[big], y0[big], x1[big], y1[big] = 3, 2, 5, 4
    rect = np.stack([x0, y0, x1, y1], 1).astype(np.int32)
    pr = oracle.Projection(None, None, rng.choice(np.linspace(0.5, 9.0, 300), n), None, None, rect,
                           ((x1 - x0) * (y1 - y0)).astype(np.int64), np.ones(n, np.int32))
    check_sort(xgs, pr, LARGE, n)
