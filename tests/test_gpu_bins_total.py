"""The binning form's capacity check past 2^32 instances."""
import pytest
import torch

import synth
from gpu_util import np_, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 1000])
def test_total_past_2_32_is_reported(extra):
    """2^26 Gaussians over all 64 tiles of an image are 2^32 instances (and 64,000
    more): far above the capacity, whatever they are modulo 2^32.  The lists are
    empty and status says why, as for any overflow."""
    xgs = require_gpu()
    n = (1 << 26) + extra
    cam = xgs.camera_from(synth.Camera(width=128, height=128, fx=100.0, fy=100.0, cx=64.0, cy=64.0))
    p = xgs.Projected.alloc(n)
    p.tile_rect[:] = torch.tensor([0, 0, 8, 8], dtype=torch.int16, device="cuda")
    p.tiles_touched.fill_(64)
    p.splat.fill_(1.0)
    b = xgs.alloc_binning(n, 70_000, cam)
    b.status.fill_(7)
    b.ranges.fill_(9)
    xgs.xgs_tile_sort(p, cam, n, b)
    torch.cuda.synchronize()
    assert int(b.status.item()) == 1 and int(b.num_instances.item()) == 0
    assert not np_(b.ranges).any()
