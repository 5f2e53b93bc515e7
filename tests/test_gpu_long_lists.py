"""The binning form's merge of lists above 2,048 instances, bit for bit against a
sort of the instances: every number of passes, the ends of the runs and groups,
depths that interleave the runs, that split them and that are all equal."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu

BLOCK, RANKS, FAN = 2048, 8 * 2048, 1024 * 2048  # a run, the longest list merged by ranks, and of the first pass


@pytest.fixture(scope="module")
def xgs():
    return require_gpu()


def sort_and_check(xgs, cam, tile, depth, extra_cap):
    """One-tile Gaussians; the oracle is NumPy's stable sort by (tile, depth)."""
    n = len(tile)
    _, _, ty, tx = oracle.grid_info(cam)
    rect = np.stack([tile % tx, tile // tx, tile % tx + 1, tile // tx + 1], 1)
    p = xgs.Projected.alloc(n)
    sp = np.zeros((n, 8), np.float32)
    sp[:, 6] = depth
    p.splat.copy_(torch.from_numpy(sp))
    p.tile_rect.copy_(torch.from_numpy(rect.astype(np.uint16).view(np.int16)))
    p.tiles_touched.fill_(1)
    p.radius.fill_(1)
    c = xgs.camera_from(cam)
    b = xgs.alloc_binning(n, n + extra_cap, c)
    b.keys.fill_(-1)
    b.vals.fill_(-1)
    xgs.xgs_tile_sort(p, c, n, b)
    torch.cuda.synchronize()
    assert int(b.status.item()) == 0 and int(b.num_instances.item()) == n
    key = tile.astype(np.uint64) << np.uint64(32) | np.ascontiguousarray(sp[:, 6]).view(np.uint32).astype(np.uint64)
    order = np.argsort(key, kind="stable")
    np.testing.assert_array_equal(np_(b.vals)[:n].view(np.uint32), order.astype(np.uint32))
    np.testing.assert_array_equal(np_(b.keys)[:n].view(np.uint64), key[order])


def depths(kind, m, rng):
    if kind == "random":
        return rng.uniform(0.5, 9.0, m)
    if kind == "ascending":   # each run is a range of its own
        return np.linspace(0.5, 9.0, m)
    if kind == "profile":     # every 2,048 Gaussians have the same depths, as on a regular grid
        return 0.5 + 8.0 * (np.arange(m) % BLOCK) / BLOCK
    if kind == "tied":        # some hundred Gaussians to a depth, the order is the index
        return rng.choice(np.linspace(0.5, 9.0, 1 + m // 300), m)
    if kind == "equal":
        return np.full(m, 3.0)
    # clumped: half of the list at one depth, within a wide range
    d = rng.uniform(0.5, 9.0, m)
    d[rng.random(m) < 0.5] = 4.0
    d[rng.random(m) < 0.01] = 1e-30
    d[rng.random(m) < 0.001] = 1e30
    return d


KINDS = ["random", "ascending", "profile", "tied", "equal", "clumped"]
CAM = synth.Camera(width=320, height=240, fx=200.0, fy=200.0, cx=160.0, cy=120.0)  # 300 tiles


@pytest.mark.parametrize("m", [BLOCK + 1, 2 * BLOCK - 1, 2 * BLOCK, 3 * BLOCK + 5, 4 * BLOCK + 1, RANKS - 1, RANKS, RANKS + 1,
                               RANKS + 255, 9 * BLOCK, 100_000, 128 * BLOCK + 1, 256 * BLOCK, 256 * BLOCK + 1,
                               512 * BLOCK, 512 * BLOCK + 1, FAN - 1, FAN, FAN + 1])
@pytest.mark.parametrize("kind", KINDS)
def test_one_long_list(xgs, m, kind):
    """Ends of the runs, of the lists merged by ranks, of the sample sort's widths, of
    the two sizes of a range and of the first pass."""
    rng = np.random.default_rng(m)
    sort_and_check(xgs, CAM, np.full(m, 17), depths(kind, m, rng), 5)


@pytest.mark.parametrize("kind", KINDS)
def test_more_runs_than_workgroups(xgs, kind):
    """2,500 runs, more than the merge's 256 workgroups, and than the sort's on a
    grid of 1,200 tiles; lists of both passes beside shorter ones."""
    rng = np.random.default_rng(5)
    cam = synth.Camera(width=640, height=480, fx=200.0, fy=200.0, cx=320.0, cy=240.0)
    lengths = {3: 2_500_000, 4: 300_000, 5: 1_000_000, 6: FAN + 1, 7: 9_000, 8: 2_049, 9: 700, 1199: 120_000}
    tile = rng.permutation(np.repeat(list(lengths), list(lengths.values())))
    sort_and_check(xgs, cam, tile, depths(kind, len(tile), rng), 1000)


def interleaved(m, offsets):
    """Depths whose runs all have their samples in the same places of the order."""
    run, at = np.arange(m) // BLOCK, np.arange(m) % BLOCK
    return at + offsets[run]


@pytest.mark.parametrize("m", [100 * BLOCK, 489 * BLOCK])
def test_ranges_that_do_not_fit(xgs, m):
    """Runs shifted against each other as their samples are: all samples of a
    round are neighbours, and what lies between the rounds is one range of up to
    a quarter of a million pairs, which is taken in parts."""
    offsets = (np.arange(m // BLOCK, dtype=np.uint64) * 0x9E3779B1 % (1 << 32)).astype(np.int64) >> (32 - 8)
    d = 10_000.0 + interleaved(m, -offsets)
    # in list order of the Gaussians' blocks: the index order is the order of the runs
    sort_and_check(xgs, CAM, np.full(m, 17), d, 0)


def test_a_last_pass_of_many_runs(xgs):
    """Five runs of the first pass's longest, with ranges that do not fit."""
    rng = np.random.default_rng(6)
    m = 4 * FAN + 4097
    sort_and_check(xgs, synth.Camera(width=640, height=480, fx=200.0, fy=200.0, cx=320.0, cy=240.0), np.full(m, 1199),
                   depths("clumped", m, rng), 0)
